"""The blend backward's sums of four list entries at a time (blend.hip) at list lengths around
its group, mask and batch sizes, with and without the maps' gradients and the deterministic
records, against the oracle's adjoint at the parity tests' bar."""
import numpy as np
import pytest

import oracle
from gpu_common import TIE_ALPHA, TIE_T, exposures, gpu_map, grad_close, oracle_forward, torch_mod
from paper_2404_06926_amd import scenes

pytestmark = pytest.mark.gpu

# one entry, a partial, full and overfull group of four, and both sides of the 64-entry masks
# and of one and two batches of 64 and 128
LENGTHS = [1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 257]


@pytest.mark.parametrize("maps", [False, True])
@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("n", LENGTHS)
def test_backward_at_group_and_batch_edges(n, deterministic, maps):
    torch = torch_mod()
    # a single tile and three pixels of its neighbours: most Gaussians reach every quadrant;
    # faint ones, so that no pixel stops and the whole list is walked
    cam = scenes.pinhole(19, 17, 20.0)
    cam.bg = np.array([0.2, 0.3, 0.1], np.float32)
    params = scenes.frustum_gaussians(n, 1, cam, seed=100 + n, log_scale_mean=-1.0)
    params[:, 10] = -3.0 + 0.2 * params[:, 10]
    print(f"{n} Gaussians, deterministic {deterministic}, maps {maps}", flush=True)
    m = gpu_map(params, 1)
    m.set_deterministic(deterministic)
    e = exposures([cam])
    m.render([cam], e, depth=maps, opacity=maps)
    r = np.random.default_rng(n)
    g = r.normal(size=(3, cam.height, cam.width)).astype(np.float32)
    gd, go = (r.normal(size=(cam.height, cam.width)).astype(np.float32) for _ in range(2))
    dev = lambda a: torch.tensor(a, device="cuda")
    gexp = torch.zeros(12, device="cuda")
    m.render_backward([dev(g)], [gexp], dl_ddepth=[dev(gd)] if maps else None, dl_dopacity=[dev(go)] if maps else None)
    torch.cuda.synchronize()
    views, projs, bins, rend = oracle_forward(params, 1, [cam])
    extra = dict(gdepths=[gd.astype(np.float64)], gopacs=[go.astype(np.float64)]) if maps else {}
    gp, gE, tie = oracle.backward(params, 1, views, projs, bins, [g.astype(np.float64)], TIE_ALPHA, TIE_T, **extra)
    sel = (projs[0]["count"] > 0) & (tie == 0)
    assert sel.sum() >= 0.8 * (projs[0]["count"] > 0).sum() and sel.any()
    ok, err = grad_close(m.grads().cpu().numpy().T[sel], gp[sel])
    print(f"compared {sel.sum()} of {n}, worst {err.max():.2e}", flush=True)
    assert ok.all(), err.max()
    if not (tie > 0).any():
        np.testing.assert_allclose(gexp.cpu().numpy(), gE[0], rtol=1e-3, atol=1e-3 * np.abs(gE[0]).max())


# every pixel of a lane's four: the mean 2^-16 pixels from its centre, and the only gradient
# there, so that the position moments are small against the distance to the four's first pixel
@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("column", range(8))
def test_moments_of_a_pixel_at_the_mean(column, deterministic):
    torch = torch_mod()
    cam = scenes.pinhole(48, 48, 64.0)
    x, y = 16 + column, 16 + column
    params = scenes.frustum_gaussians(1, 0, cam, seed=1)
    off = 0.5 + 2.0 ** -16
    params[0, 0:3] = (2.0 * (x + off - 24.0) / 64.0, 2.0 * (y + off - 24.0) / 64.0, 2.0)
    params[0, 3:6] = np.log(0.1)
    params[0, 6:10] = (1.0, 0.0, 0.0, 0.0)
    g = np.zeros((3, 48, 48), np.float32)
    g[:, y, x] = (1.0, -2.0, 0.5)
    m = gpu_map(params, 0)
    m.set_deterministic(deterministic)
    m.render([cam])
    m.render_backward([torch.tensor(g, device="cuda")])
    torch.cuda.synchronize()
    views, projs, bins, rend = oracle_forward(params, 0, [cam])
    off_centre = np.array([x, y]) + 0.5 - projs[0]["mean2d"][0]
    assert (np.abs(off_centre) < 2e-5).all()
    gp, gE, tie = oracle.backward(params, 0, views, projs, bins, [g.astype(np.float64)], TIE_ALPHA, TIE_T)
    cols = [0, 1, 3, 4]  # mean x and y, scales x and y: products of the moments without cancellation
    got, want = m.grads().cpu().numpy()[cols, 0].astype(np.float64), gp[0, cols]
    print(f"column {column}: {got} against {want}", flush=True)
    assert (want != 0).all()
    np.testing.assert_allclose(got, want, rtol=1e-3)
