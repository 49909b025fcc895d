"""The walks of the render kernels' forms that the tests on small images do not reach,
with list lengths at the edges of their 64-pair windows, 256-entry batches and the
heavy-tile split (512), against the oracle."""
import numpy as np
import pytest

import oracle
import workloads as W
from tests.gpu_helpers import compare, gpu_render, log, proxy_error, tolerances
from tests.test_gpu_backward import _check, _gpu_grads

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


def _crowd():
    """Sixteen cameras of 80 tiles: beyond the 1200 tiles up to which frames take the
    wide form. All alike, so that one stands for the batch; the pixels compared are 150
    about the scene and 50 anywhere."""
    cam = W.camera_on_axis(2.0, 80, 250)
    rng = np.random.default_rng(8)
    pix = np.concatenate([rng.integers(85, 165, 150) * 80 + rng.integers(0, 80, 150),
                          rng.integers(0, 80 * 250, 50)])
    return cam, [cam] * 16, np.unique(pix)


@pytest.mark.parametrize("k_mom,n,full", [(4, n, True) for n in (1, 63, 64, 65, 255, 256, 257, 512, 513, 700)]
                         + [(k, n, True) for k in (6, 8) for n in (64, 257, 513)]
                         + [(k, n, False) for k in (4, 6, 8) for n in (65, 700, 5000)])
def test_ordinary_form_list_lengths_match_oracle(k_mom, n, full):
    scene = W.uniform_scene(n, seed=n, extent=0.25, log_scale_mean=-2.5)
    cam, cams, pix = _crowd()
    opts = W.Options(n_moments=k_mom, full_coverage=full)
    img, saved, st = gpu_render(scene, cams, opts)
    assert np.array_equal(img[0], img[15]) and np.array_equal(saved[0], saved[15])
    tol_m, tol_o = (0.0, 0.0) if full else tolerances(proxy_error(scene, cam, opts))
    ref = oracle.render_image(scene, cam, opts, pixels=pix, margin_tol=tol_m, orient_eps=tol_o)
    log(f"[walk] ordinary n {n} full {full} K {k_mom}: {st.n_entries} entries, {ref['n_pairs']} pairs")
    mx, _ = compare(img[0].reshape(-1, 3)[pix], ref, f"walk ordinary n={n}", gpu_saved=saved[0].reshape(-1, 8)[pix],
                    max_excluded=ref["ambiguous"].mean() + 0.01)
    assert mx <= 1e-4
    if full:
        c = saved[0].reshape(-1, 8)[:, 7]
        assert np.all(np.where(c < 0, -c - 1, c) == n)


@pytest.mark.parametrize("n,full", [(n, True) for n in (63, 64, 65, 130, 257, 520)] + [(65, False), (700, False)])
def test_ordinary_form_list_lengths_gradients_match_oracle(n, full):
    """To the backward tests' bar of 1e-3 per parameter group; no upstream gradient
    where the coverage or the degeneracy flag is undecided."""
    scene = W.uniform_scene(n, seed=n, extent=0.25, log_scale_mean=-2.5)
    cam, cams, pix = _crowd()
    opts = W.Options(full_coverage=full)
    _, saved, _ = gpu_render(scene, cams, opts)
    tol_m, tol_o = (0.0, 0.0) if full else tolerances(proxy_error(scene, cam, opts))
    ref = oracle.render_image(scene, cam, opts, pixels=pix, margin_tol=tol_m, orient_eps=tol_o)
    up = np.random.default_rng(n).normal(size=(len(pix), 3))
    up[ref["ambiguous"] | ((saved[0].reshape(-1, 8)[pix, 7] < 0) != ref["fallback"])] = 0.0
    g_img = np.zeros((16, cam.width * cam.height, 3))
    g_img[0, pix] = up
    gpu, _ = _gpu_grads(scene, cams, opts, g_img)
    assert _check(gpu, oracle.render_backward(scene, cam, opts, up, pixels=pix), f"walk ordinary n={n} full={full}")
