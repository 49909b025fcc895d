"""The surrogate's kernels over batch sizes at the edges of their tiles and of
the partial sums' split, against the float64 reference that reproduces their
rounding points (oracle.surrogate)."""
import numpy as np
import pytest
import torch

from oracle import surrogate as S
from tests.gpu_helpers import log
from tests.test_gpu_mlp import _batch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 31, 33, 64, 65, 1000, 8193, 65536])
def test_loss_grad_over_batch_sizes(n):
    """Few, odd and many rows of partial sums. A bf16 rounding tie that falls the
    other way moves one activation of one query by 2^-8 of itself, hence its
    gradients by up to about that; averaged over more queries the share falls."""
    from paper_2512_11800_amd import surrogate as G
    theta = S.init_params(5).astype(np.float32)
    x, t = _batch(n, 10 + n)
    packed = G.mlp_pack(torch.tensor(theta, device="cuda"))
    loss, grad = G.mlp_loss_grad(packed, torch.tensor(x, device="cuda"), torch.tensor(t, device="cuda"))
    loss, grad = float(loss.item()), grad.cpu().numpy().astype(np.float64)
    lref, gref = S.loss_grad(theta.astype(np.float64), x.astype(np.float64), t.astype(np.float64))
    tol = 2e-2 if n < 100 else 3e-3
    o, worst = 0, 0.0
    for k, s in S.SIZES.items():
        m = int(np.prod(s))
        a, b = grad[o:o + m], gref[o:o + m]
        worst = max(worst, np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))
        o += m
    log(f"[mlp] n={n} loss gpu={loss:.6e} ref={lref:.6e} worst grad rel={worst:.2e}")
    assert loss == pytest.approx(lref, rel=1e-3 if n < 100 else 1e-4)
    assert worst < tol


@pytest.mark.parametrize("n", [1, 31, 32, 33, 63, 64, 65, 255, 257, 4097])
def test_forward_does_not_depend_on_the_place(n):
    """A query's output is the same bits in whichever tile, half and step of a
    wave it falls: the first n of a long list, alone, and in reverse order."""
    from paper_2512_11800_amd import surrogate as G
    theta = torch.tensor(S.init_params(6).astype(np.float32), device="cuda")
    x = torch.tensor(_batch(200_000, 11)[0], device="cuda")
    packed = G.mlp_pack(theta)
    full = G.mlp_forward(packed, x)
    assert torch.equal(G.mlp_forward(packed, x[:n].contiguous()), full[:n])
    assert torch.equal(G.mlp_forward(packed, x[:n].flip(0).contiguous()), full[:n].flip(0))
