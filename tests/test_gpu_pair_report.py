"""The pair count a frame reports to the host before its render has finished:
equal to the device's count for every route of the binning, grown frames
render the same image, and the cases without a report (no entries, recorded
renders, another stream, frames made without auto_grow) read the count back."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2605_06876_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2605_06876_amd import api  # noqa: E402


def scene(n, seed=1):
    rng = np.random.default_rng(seed)
    g = api.Gaussians.empty(n, 0)
    g.means.copy_(torch.from_numpy(rng.uniform(-1.0, 1.0, (3, n)).astype(np.float32)))
    g.log_scales.fill_(-4.0)
    g.quats[0] = 1.0
    g.sh.copy_(torch.from_numpy(rng.uniform(-1, 1, tuple(g.sh.shape)).astype(np.float32)))
    return g


def wait(frame):
    count = ctypes.c_uint32()
    rc = api.lib().as_frame_wait_pairs(frame.handle, ctypes.byref(count), api._stream(None))
    return rc, count.value


CAM = synth.look_at((0.0, 0.0, -4.0), (0.0, 0.0, 0.0), 320, 256, 50.0)


# one block, sample sort, radix sort, two-level binning
@pytest.mark.parametrize("n,key_cap", [(1, 64), (4000, 1 << 17), (60_000, 1 << 20), (60_000, 1 << 22), (1_400_000, 1 << 24)])
def test_report_is_the_device_count(n, key_cap):
    frame = api.Frame(api.Context(0), n, 320, 256, key_cap=key_cap)
    for seed in range(3):
        api.render(frame.ctx, scene(n, seed), CAM, frame)
        assert wait(frame) == (api.AS_OK, frame.n_keys())


def test_a_growing_frame_renders_the_same_image():
    ctx, g = api.Context(0), scene(30_000)
    want = api.render(ctx, g, CAM, api.Frame(ctx, g.n, 320, 256, key_cap=1 << 20))
    frame = api.Frame(ctx, g.n, 320, 256, key_cap=100)
    assert torch.equal(api.render(ctx, g, CAM, frame), want) and frame.key_cap >= frame.n_keys()


def test_renders_without_a_report_read_the_count_back():
    ctx, g = api.Context(0), scene(5000)
    want = api.render(ctx, g, CAM, api.Frame(ctx, g.n, 320, 256))
    frame = api.Frame(ctx, g.n, 320, 256, key_cap=100, auto_grow=False)
    frame.auto_grow = True
    assert torch.equal(api.render(ctx, g, CAM, frame), want) and wait(frame)[0] == api.AS_ERR_STATE
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    frame = api.Frame(ctx, g.n, 320, 256, key_cap=100)
    assert torch.equal(api.render(ctx, g, CAM, frame, stream=side), want)
    frame = api.Frame(ctx, g.n, 320, 256, key_cap=1 << 17)
    image = api.render(ctx, g, CAM, frame)
    frame.auto_grow = False
    graph = api.Graph.capture(ctx, lambda: api.render(ctx, g, CAM, frame, image=image), side)
    assert wait(frame)[0] == api.AS_ERR_STATE
    for _ in range(3):
        image.zero_()
        torch.cuda.synchronize()
        graph.launch(side)
        torch.cuda.synchronize()
        assert torch.equal(image, want)
    frame.auto_grow = True
    assert torch.equal(api.render(ctx, g, CAM, frame), want) and wait(frame) == (api.AS_OK, frame.n_keys())


def test_threads_wait_for_their_own_frames():
    scenes = [scene(2000 + 7000 * k, k) for k in range(4)]
    bad = []

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            ctx = api.Context(0)
            frame = api.Frame(ctx, scenes[k].n, 320, 256)
            for _ in range(20):
                api.render(ctx, scenes[k], CAM, frame)
                if wait(frame) != (api.AS_OK, frame.n_keys()):
                    bad.append(k)

    torch.cuda.synchronize()
    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad
