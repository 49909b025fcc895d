"""The surrogate's inference over more queries than one step of the whole grid takes
(1024 blocks of four waves, 64 queries each): the later steps' queries, their inputs
loaded ahead, and the ragged last one give the bits that the same rows give alone."""
import pytest
import torch

from oracle import surrogate as S
from tests.test_gpu_mlp import _batch

pytestmark = pytest.mark.gpu

STEP = 1024 * 4 * 64


@pytest.mark.parametrize("n", [STEP + 1, 600_001])
def test_forward_over_several_steps(n):
    from paper_2512_11800_amd import surrogate as G
    packed = G.mlp_pack(torch.tensor(S.init_params(6).astype("float32"), device="cuda"))
    x = torch.tensor(_batch(n, 12)[0], device="cuda")
    full = G.mlp_forward(packed, x)
    for q0, q1 in ((0, 300), (STEP - 70, min(STEP + 300, n)), (2 * STEP - 33, 2 * STEP + 95), (n - 130, n)):
        rows = x[q0:q1].contiguous()
        if rows.shape[0]:
            assert torch.equal(G.mlp_forward(packed, rows), full[q0:q1]), (q0, q1)
