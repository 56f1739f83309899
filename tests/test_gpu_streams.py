"""Frames that share a stream's launch-order and occupancy buffers: several threads
on one stream, one stream per thread, and captured frames replayed beside others."""
import ctypes as C
import threading

import pytest
import torch

import paper_1801_01155_amd as L
from paper_1801_01155_amd import synth

pytestmark = pytest.mark.gpu

PER_THREAD = 2          # hipStreamPerThread


def _views(mode, w, h):
    """Two sets of different grids and their transparent views (the second grid's
    buffers are larger), each with its image rendered alone."""
    views = []
    for grid, n in (((40, 44, 36), 300), ((96, 100, 92), 1500)):
        ls = synth.abc_lineset(n, 50, 5 + n)
        s = L.lineset_voxelize(ls.curve_off, grid, 32, xyz=ls.xyz, attr=ls.attr)
        lut = torch.as_tensor(synth.lut_importance_alpha()).cuda()
        cam = synth.orbit_cameras(grid, 1, n, w, h)[0]
        kw = dict(radius=0.4, mode=mode, opaque=False, shading=1)
        ref = L.lineset_render(s, cam, lut, **kw)
        views.append((s, cam, lut, kw, ref))
    torch.cuda.synchronize()
    return views


def _differs(a, b):
    d = (a - b).abs().amax(-1)
    return f"{int((d > 0).sum())} pixels differ by up to {float(d.max()):.3g}, " \
           f"{int((a[..., 3] < 0).sum())} not written"


def _render(view, out, stream):
    s, cam, lut, kw, _ = view
    c, p = L.camera_struct(cam), L.render_params(lut, **kw)
    rc = L.lib().lineset_render(s.handle, C.byref(c), C.byref(p), C.c_void_p(out.data_ptr()),
                                C.c_void_p(stream))
    assert rc == L.LS_OK, L.lib().ls_last_error()


# 200 x 150: below the device's resident workgroups; 900 x 700: ordered frames
@pytest.mark.parametrize("mode,w,h", [(1, 200, 150), (1, 900, 700), (0, 900, 700)])
@pytest.mark.parametrize("stream", ["shared", "per_thread"])
def test_threads_render_their_own_images(mode, w, h, stream):
    views = _views(mode, w, h)
    st = PER_THREAD if stream == "per_thread" else torch.cuda.Stream().cuda_stream
    frames = 12
    outs = [[torch.full((h, w, 4), -1.0, device="cuda") for _ in range(frames)] for _ in views]
    torch.cuda.synchronize()
    errors = []

    def work(k):
        try:
            torch.cuda.set_device(0)
            for out in outs[k]:
                _render(views[k], out, st)
            torch.cuda.ExternalStream(st).synchronize()   # a thread's stream ends with it
        except BaseException as e:   # noqa: B036 (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for view, imgs in zip(views, outs):
        for img in imgs:
            assert torch.equal(img, view[4]), _differs(img, view[4])


@pytest.mark.parametrize("mode,w,h", [(1, 200, 150), (1, 900, 700), (0, 900, 700)])
def test_captured_frame_beside_others(mode, w, h):
    small, large = _views(mode, w, h)
    out = torch.empty((h, w, 4), device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        _render(small, out, side.cuda_stream)       # the stream has buffers
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        _render(small, out, side.cuda_stream)
    for k in range(4):
        # eager frames of a larger set replace the stream's buffers
        with torch.cuda.stream(side):
            img = torch.empty((h, w, 4), device="cuda")
            _render(large, img, side.cuda_stream)
        torch.cuda.synchronize()
        assert torch.equal(img, large[4]), _differs(img, large[4])
        out.fill_(-1.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, small[4]), (k, _differs(out, small[4]))
