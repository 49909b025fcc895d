"""The block list of the render kernels over tiles of every kind: heavy ones (more
than 512 entries, four blocks of a quadrant each), light and empty ones, for the
single-block order (up to 16384 tiles), the radix passes beyond, and the lists that a
single block builds."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


def _block_list(st, n_keys):
    """(lengths of the tiles' lists, block codes) from the pair workspace: six arrays of
    the entries, the sort's counts, the tiles' ranges, the list; each 256-byte aligned."""
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    e = st.n_entries
    off = 6 * up(4 * e) + up(4 * (256 * ((e + 4095) // 4096) + 1))
    ranges = st.ws.pws[off:off + 8 * n_keys].view(torch.int32).reshape(-1, 2).cpu().numpy()
    off += up(8 * n_keys)
    return ranges[:, 1] - ranges[:, 0], st.ws.pws[off:off + 16 * n_keys].view(torch.int32).cpu().numpy()


@pytest.mark.parametrize("n,w,h,extent", [(3000, 2048, 2048, 0.05), (3000, 2064, 2048, 0.05), (900, 96, 80, 0.05),
                                          (1500, 1040, 1024, 0.03)])
def test_each_tile_or_quadrant_is_listed_once(n, w, h, extent):
    import paper_2512_11800_amd as M
    g = M.Gaussians.from_scene(W.uniform_scene(n, seed=n, extent=extent, log_scale_mean=-3.5))
    _, _, st = M.render_forward(g, [W.camera_on_axis(2.0, w, h)], W.Options())
    n_keys = ((w + 15) // 16) * ((h + 15) // 16)
    length, codes = _block_list(st, n_keys)
    log(f"[order] {w}x{h}: {st.n_entries} entries, {int((length > 512).sum())} heavy, "
        f"{int((length == 0).sum())} empty of {n_keys} tiles")
    assert length.sum() == st.n_entries and (length > 512).any() and (length <= 512).any()
    part, whole = -codes[codes < 0] - 1, codes[(codes >= 0) & (codes < n_keys)]
    assert np.array_equal(np.sort(whole), np.flatnonzero(length <= 512))
    heavy = np.flatnonzero(length > 512)
    assert np.array_equal(np.sort(part), (4 * heavy[:, None] + np.arange(4)).reshape(-1))


def test_heavy_tiles_alike_on_both_sides_of_the_limit():
    """16384 tiles (one block orders them) and 16512 (radix passes), the same rays: the
    common pixels' image, state and, through them, gradients are the same bits."""
    import paper_2512_11800_amd as M
    g = M.Gaussians.from_scene(W.uniform_scene(2000, seed=4, extent=0.05, log_scale_mean=-3.5))
    cam = W.camera_on_axis(2.0, 2048, 2048)
    out = []
    up = torch.randn(2048, 2048, 3, generator=torch.Generator().manual_seed(1)).cuda()
    for width in (2048, 2064):
        img, saved, st = M.render_forward(g, [dataclasses.replace(cam, width=width)], W.Options())
        gi = torch.zeros_like(img)
        gi[0, :, :2048] = up
        grads = M.render_backward(g, [dataclasses.replace(cam, width=width)], W.Options(), st, saved, gi)
        out.append([img[:, :, :2048], saved[:, :, :2048]] + [grads[k] for k in sorted(grads)])
    assert all(torch.equal(x, y) for x, y in zip(*out))
