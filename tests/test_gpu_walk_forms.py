"""The walks of the render kernels' forms that the tests on small images do not reach,
with list lengths at the edges of their 64-pair windows, 256-entry batches and the
heavy-tile split (512), against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests.gpu_helpers import compare, gpu_render, log, proxy_error, tolerances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,full", [(1, True), (63, True), (64, True), (65, True), (130, True), (257, True)]
                         + [(n, False) for n in (63, 64, 65, 130, 255, 256, 257, 513, 700)])
def test_trig_k6_list_lengths_match_oracle(n, full):
    """The trigonometric K = 6 quadrature pass walks its lists entry by entry. The
    bar of the trigonometric forward tests; excluded are the oracle's ambiguous pixels
    (an atom at the cut, the coverage band) and at most 1% with another degeneracy flag."""
    scene = W.uniform_scene(n, seed=n, extent=0.25, log_scale_mean=-2.5)
    cam = W.camera_on_axis(2.0, 21, 18)
    opts = W.Options(n_moments=6, full_coverage=full, basis="trigonometric")
    img, saved, st = gpu_render(scene, [cam], opts)
    tol_m, tol_o = (0.0, 0.0) if full else tolerances(proxy_error(scene, cam, opts))
    ref = oracle.render_image(scene, cam, opts, margin_tol=tol_m, orient_eps=tol_o)
    log(f"[walk trig] n {n} full {full}: {st.n_entries} entries, {ref['n_pairs']} pairs")
    mx, _ = compare(img[0].reshape(-1, 3), ref, f"walk trig n={n}", gpu_saved=saved[0].reshape(-1, 8),
                    max_excluded=ref["ambiguous"].mean() + 0.01)
    assert mx <= 1e-4
    c = saved[0].reshape(-1, 8)[:, 7]
    if full:
        assert np.all(np.where(c < 0, -c - 1, c) == n)
