"""GPU parity of the CPU-forwarding stream where messages are staged in pieces: either side of the sizes and windows that
change their number, packed buffers with a hole behind a short last chunk, against the oracle."""
import pytest
import torch

from tests.cases import Case, contig, make_storages
from tests.test_gpu_parity import run_exchange, run_exchange_tagged, say

pytestmark = pytest.mark.gpu
MiB = 1 << 20


@pytest.mark.parametrize("nbytes,messages,how", [
    (10 * MiB - 256, 3, {}), (10 * MiB, 3, {}), (14 * MiB, 3, {}),                    # 1, 2 and 3 pieces (the planner's tests count them)
    (25 * MiB + 300, 5, {"drain_every": 2}),                                          # 3 pieces, 4 copies: one piece lies in both ranges
    (10 * MiB, 9, {"drain_every": 4}), (10 * MiB, 9, {}),                             # 2 pieces, and 1 in a window that is too long
    (24 * MiB, 9, {"drain_every": 8}),                                                # 2 pieces, 16 copies a window
])
@pytest.mark.parametrize("n_buffers", [1, 2])
def test_messages_staged_in_pieces(nbytes, messages, how, n_buffers):
    case = Case("contig_%d" % nbytes, (contig((nbytes // 4,), 4),), 3, 640 << 10)
    say("pieces", nbytes, messages, how, n_buffers)
    streams = [torch.cuda.Stream() for _ in range(3)]
    run_exchange(case, [make_storages(case, 40 + i) for i in range(messages)], "cpu_forward", n_buffers, streams, **how)


def test_a_tagged_message_staged_in_pieces():
    case = Case("contig", (contig((25 * MiB // 4 + 75,), 4),), 3, 640 << 10)
    run_exchange_tagged(case, [make_storages(case, 60 + i) for i in range(3)], "cpu_forward", 2, [torch.cuda.Stream() for _ in range(3)])
