"""The surrogate's render and a frame without Gaussians captured in a HIP graph: their
counters are cleared by kernels, so that every replay, with eager frames and
synchronisations between the replays, equals the eager frame."""
import ctypes

import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def _capture(frame):
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        frame()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = frame()
    return graph, out


def test_surrogate_replays_equal_the_eager_frame():
    import paper_2512_11800_amd as M
    from paper_2512_11800_amd import _lib as L
    from paper_2512_11800_amd import surrogate as G
    from paper_2512_11800_amd.render import _Frame, _ptr, _stream
    scene, cams, opts = W.w1_small()
    opts.n_moments = 6
    g = M.Gaussians.from_scene(scene)
    packed = G.mlp_pack(G.init_params(3))
    ws = M.Workspace()
    img, saved, st = M.render_forward_surrogate(g, cams, opts, packed, ws=ws)
    torch.cuda.synchronize()
    n_queries = int(ws.qws[:8].view(torch.int64).item())
    assert 0 < n_queries <= st.q_cap
    f = _Frame(g, cams, opts, ws)
    lib = L.load()

    def frame():  # the list count is known: nothing waits
        L.check(lib.mb_prepare(ctypes.byref(f.gs), f.cam_arr, f.n_cams, ctypes.byref(f.o), _ptr(ws.gws),
                               ws.gws.numel(), None, _stream()))
        L.check(lib.mb_render_forward_surrogate(*f.head(), _ptr(packed), _ptr(ws.qws), ws.qws.numel(), st.q_cap,
                                                _ptr(f.image), _ptr(f.saved), _stream()))
        return f.image, f.saved

    graph, _ = _capture(frame)
    for r in range(3):
        f.image.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(f.image, img) and torch.equal(f.saved, saved), r
        assert int(ws.qws[:8].view(torch.int64).item()) == n_queries
        frame()  # the program's own eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(f.image, img), r


def test_empty_frame_replays():
    import paper_2512_11800_amd as M
    scene, cams, opts = W.w1_small()
    g = M.Gaussians.from_scene(scene.subset([]))
    ws = M.Workspace()
    ref = M.render_forward(g, cams, opts, ws=ws, on_device=True)[0].clone()
    graph, out = _capture(lambda: M.render_forward(g, cams, opts, ws=ws, on_device=True))
    for r in range(3):
        graph.replay()
        torch.cuda.synchronize()
        out[2].check()
        assert torch.equal(out[0], ref) and out[2].entry_count() == 0, r
        assert torch.equal(M.render_forward(g, cams, opts, ws=ws, on_device=True)[0], ref), r
