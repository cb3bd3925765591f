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
