"""What a render leaves for its backward and for inspection, and the calls after which it is
gone: they are refused on the host, before anything is launched."""
import pytest

from gpu_common import gpu_map, torch_mod
from paper_2404_06926_amd import gslic, scenes

pytestmark = pytest.mark.gpu


def _scene(n=4000, width=160, height=120):
    cam = scenes.pinhole(width, height, 130.0)
    return cam, scenes.frustum_gaussians(n, 1, cam, seed=n + width)


def _refused(call, code=gslic.GS_ERR_STATE):
    with pytest.raises(gslic.GsError) as e:
        call()
    assert e.value.code == code


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("width", [160, 4192])  # the lists by counting, and by sorting
def test_growing_the_instance_buffers_ends_the_render(width, deterministic):
    torch = torch_mod()
    cam, params = _scene(width=width, height=120 if width == 160 else 3200)
    m = gpu_map(params, 1)
    m.set_deterministic(deterministic)
    g = [torch.ones(3, cam.height, cam.width, device="cuda")]
    held = 1 << 22
    m.set_instance_policy(True, held)
    m.render([cam])
    m.set_instance_policy(True, held // 2)  # nothing grows: the render stays
    m.render_backward(g)
    torch.cuda.synchronize()
    want = m.grads().clone()
    m.adam_step()
    m.render([cam])
    m.set_instance_policy(True, 2 * held)
    print(f"grown after a render, width {width}, deterministic {deterministic}", flush=True)
    _refused(lambda: m.render_backward(g))
    _refused(m.debug_last_render)
    m = gpu_map(params, 1)
    m.set_deterministic(deterministic)
    m.render([cam])
    m.render_backward(g)
    torch.cuda.synchronize()
    if deterministic:
        assert torch.equal(m.grads(), want)


# A render that fails for memory: with its first buffer, which leaves the render before it as
# it was, and after some were replaced (a larger view, on a map of one small render)
@pytest.mark.parametrize("granted", [0, 1, 3])
@pytest.mark.parametrize("deterministic", [False, True])
def test_a_render_that_fails_for_memory_ends_the_one_before(granted, deterministic, monkeypatch):
    torch = torch_mod()
    left = [1 << 30]
    alloc = gslic.TorchAllocator._do_alloc

    def rationed(self, nbytes, stream, ctx):
        left[0] -= 1
        return alloc(self, nbytes, stream, ctx) if left[0] >= 0 else None

    monkeypatch.setattr(gslic.TorchAllocator, "_do_alloc", rationed)
    cam, params = _scene()
    views = [cam, scenes.pinhole(320, 240, 260.0), scenes.pinhole(300, 200, 260.0)]
    m = gpu_map(params, 1)
    m.set_deterministic(deterministic)
    g = [torch.ones(3, cam.height, cam.width, device="cuda")]
    m.render([cam])
    m.render_backward(g)
    torch.cuda.synchronize()
    want = m.grads().clone()
    m.adam_step()
    torch.cuda.synchronize()
    m = gpu_map(params, 1)
    m.set_deterministic(deterministic)
    m.render([cam])
    left[0] = granted
    print(f"{granted} buffers granted, deterministic {deterministic}", flush=True)
    _refused(lambda: m.render(views), gslic.GS_ERR_OOM)
    left[0] = 1 << 30
    if granted:
        _refused(lambda: m.render_backward(g))
        _refused(m.debug_last_render)
        m.render([cam])
    m.render_backward(g)
    torch.cuda.synchronize()
    if deterministic:
        assert torch.equal(m.grads(), want)


def _step_buffers(cam):
    torch = torch_mod()
    h, w = cam.height, cam.width
    fr = [gslic.Frame(torch.empty(3, h, w, device="cuda"), torch.empty(h, w, device="cuda"),
                      torch.empty(h, w, device="cuda", dtype=torch.int32))]
    target = torch.from_numpy(scenes.smooth_image(7, h, w)).float().cuda()
    return fr, [target], [gslic.identity_exposure_state()], [torch.empty(3, h, w, device="cuda")], torch.empty(
        1, device="cuda")


# An eager step, a larger capacity, a capture: by counting, and by sorting (more Gaussians than
# the counting lists take for so few cells). The replays give what eager steps give.
@pytest.mark.parametrize("n", [5000, 70_000])
@pytest.mark.parametrize("deterministic", [False, True])
def test_a_capacity_set_before_a_capture_holds_for_both_lists(n, deterministic):
    torch = torch_mod()
    cam = scenes.pinhole(30, 28, 25.0)
    params = scenes.frustum_gaussians(n, 0, cam, seed=n)
    out = []
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        for captured in (False, True):
            m = gpu_map(params, 0)
            m.set_deterministic(deterministic)
            b = _step_buffers(cam)
            m.step([cam], *b)
            m.set_instance_policy(False, 4 * m.debug_last_render()["n_inst"])
            print(f"{n} Gaussians, deterministic {deterministic}, captured {captured}", flush=True)
            if captured:
                g = m.capture_step([cam], *b)
                for _ in range(3):
                    g.launch()
                    stream.synchronize()
                g.close()
            else:
                for _ in range(3):
                    m.step([cam], *b)
            stream.synchronize()
            assert not m.check_overflow()
            out.append((b[0][0].rgb.clone(), m.params().clone()))
    if deterministic:
        assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    else:
        # atomic sums of another order: an ulp of a gradient is at most a few ulps of an Adam step
        assert torch.allclose(out[0][0], out[1][0], rtol=0, atol=1e-3)


@pytest.mark.parametrize("n", [5000, 70_000])  # by counting, by sorting
def test_instance_buffers_are_shared_by_both_lists(n):
    cam = scenes.pinhole(30, 28, 25.0)
    m = gpu_map(scenes.frustum_gaussians(n, 0, cam, seed=n), 0)
    m.render([cam])
    held = []
    for capacity in (1 << 22, 1 << 23):
        m.set_instance_policy(True, capacity)
        m.render([cam])
        held.append(m.info()[2])
    # 20 B per instance and a word per 512 of them
    assert held[1] - held[0] <= (20 + 0.01) * (1 << 22)
