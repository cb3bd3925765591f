"""Tile lists (tilelist.hip, and the radix path for images of more tiles) at the sizes where
their branches change, against the oracle's keys, order and ranges bit for bit: cells of more
entries than the small and the large sorting block hold (chunks and their merge), depths too
clustered for the bins (bitonic order, ties by index), images past the counters' LDS, and the
deterministic render's emission indices."""
import numpy as np
import pytest

from gpu_common import exposures, gpu_map, torch_mod
from helpers import oview
import oracle
from paper_2404_06926_amd import scenes

pytestmark = pytest.mark.gpu


def _check_lists(params, deg, cams, deterministic=False):
    torch = torch_mod()
    m = gpu_map(params, deg)
    m.set_deterministic(deterministic)
    m.render(cams, exposures(cams))
    torch.cuda.synchronize()
    dbg = m.debug_last_render()
    views = [oview(c) for c in cams]
    projs = [oracle.project(params, deg, v) for v in views]
    bins = oracle.bin_views(projs, views)
    assert dbg["n_inst"] == bins["key"].shape[0]
    np.testing.assert_array_equal(dbg["ranges"].cpu().numpy().astype(np.int64), bins["ranges"])
    np.testing.assert_array_equal(dbg["vals"].cpu().numpy().view(np.uint32), bins["local_val"])
    np.testing.assert_array_equal(dbg["tiles"].cpu().numpy().view(np.uint32).astype(np.uint64),
                                  bins["key"] >> np.uint64(32))
    return m, bins


def _cell_sizes(bins, cams):
    """Entries per cell of 2x2 tiles of the first view."""
    tx, ty = -(-cams[0].width // 16), -(-cams[0].height // 16)
    tiles = (bins["key"] >> np.uint64(32)).astype(np.int64)
    first = tiles < tx * ty
    t, g = tiles[first], bins["local_val"][first].astype(np.int64)
    cell = (t // tx // 2) * ((tx + 1) // 2) + (t % tx) // 2
    return np.bincount(np.unique(cell << 32 | g) >> 32)


# (Gaussians, entries the largest cell must exceed, at most): one block's small size, its
# large size, chunks with a merge
@pytest.mark.parametrize("n,over,most", [(300, 0, 4096), (12_000, 4096, 16384), (60_000, 16384, 1 << 30)])
@pytest.mark.parametrize("deterministic", [False, True])
def test_lists_of_small_large_and_chunked_cells(n, over, most, deterministic):
    cams = [scenes.pinhole(70, 45, 50.0), scenes.pinhole(33, 31, 30.0)]
    cams[1].t = np.array([0.1, 0.05, 0.2], np.float32)
    params = scenes.frustum_gaussians(n, 0, cams[0], seed=n)
    print(f"{n} Gaussians over two small views, deterministic {deterministic}", flush=True)
    _, bins = _check_lists(params, 0, cams, deterministic)
    largest = _cell_sizes(bins, cams).max()
    print(f"largest cell: {largest} entries", flush=True)
    assert over < largest <= most


# one cell: the most Gaussians that it takes in chunks, and past them (radix path); and a few
# entries either side of what one wave-wide comparison ranks
@pytest.mark.parametrize("n", [65_536, 65_600, 100, 128, 129, 260])
@pytest.mark.parametrize("deterministic", [False, True])
def test_lists_of_one_cell(n, deterministic):
    cam = scenes.pinhole(24, 20, 20.0)
    params = scenes.frustum_gaussians(n, 0, cam, seed=n)
    print(f"{n} Gaussians over one cell, deterministic {deterministic}", flush=True)
    _check_lists(params, 0, [cam], deterministic)


# all depths equal (order by index alone), a few distinct depths, and a tight cluster with one
# far outlier: more entries per bin than the bins take
@pytest.mark.parametrize("shape", ["equal", "steps", "cluster"])
@pytest.mark.parametrize("n", [700, 5000, 40_000])
def test_lists_of_clustered_depths(shape, n):
    cam = scenes.pinhole(48, 40, 40.0)
    params = scenes.frustum_gaussians(n, 0, cam, seed=3 * n)
    r = np.random.default_rng(n)
    z = {"equal": np.full(n, 5.0), "steps": 5.0 + 0.25 * r.integers(0, 3, n),
         "cluster": 5.0 + 1e-6 * r.random(n)}[shape].astype(np.float32)
    if shape == "cluster":
        z[n // 2] = 400.0
    params[:, 0:2] *= (z / params[:, 2])[:, None]
    params[:, 2] = z
    print(f"{n} Gaussians, depths: {shape}", flush=True)
    _check_lists(params, 0, [cam])


# the last image whose cells fit the counters and one past it (radix path), the latter also
# among two views and deterministic
@pytest.mark.parametrize("width,height,views,deterministic",
                         [(4160, 3200, 1, False), (4192, 3200, 1, False), (4192, 3200, 2, True)])
def test_lists_of_large_images(width, height, views, deterministic):
    cams = [scenes.pinhole(width, height, 3000.0), scenes.pinhole(90, 50, 60.0)][:views]
    params = scenes.frustum_gaussians(3000, 0, cams[0], seed=9, log_scale_mean=-2.5)
    print(f"{width}x{height}, {views} views, deterministic {deterministic}", flush=True)
    _check_lists(params, 0, cams, deterministic)


# Gaussians whose rectangles have more than 64 tiles, walked by all waves of a block: a run of
# them among small ones, and more in a block than its list of them holds
@pytest.mark.parametrize("n,first,large", [(900, 100, 40), (1500, 0, 1500)])
@pytest.mark.parametrize("deterministic", [False, True])
def test_lists_of_runs_of_large_gaussians(n, first, large, deterministic):
    cams = [scenes.pinhole(333, 250, 250.0), scenes.pinhole(260, 205, 180.0)]
    params = scenes.frustum_gaussians(n, 0, cams[0], seed=n + large)
    params[first:first + large, 3:6] = 1.0  # several metres across
    print(f"{large} large of {n} Gaussians, deterministic {deterministic}", flush=True)
    m, _ = _check_lists(params, 0, cams, deterministic)
    counts = m.debug_last_render()["counts"][0].cpu().numpy()
    assert (counts[first:first + large] > 64).sum() > 0.6 * large


def test_deterministic_gradients_do_not_depend_on_the_lists_path():
    """The per-instance records (emission indices) of the lists by counting and of the radix
    path sum to the same gradients: one view alone, and beside a large image that sends the
    batch through the radix path and gets no gradient."""
    torch = torch_mod()
    cam, big = scenes.pinhole(100, 75, 80.0), scenes.pinhole(4192, 3200, 3000.0)
    params = scenes.frustum_gaussians(3000, 1, cam, seed=77, log_scale_mean=-2.0)
    params[::50, 3:6] += 2.0  # some rectangles of more than 64 tiles in the large view
    g = torch.randn(3, 75, 100, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = []
    for cams in ([cam], [cam, big]):
        m = gpu_map(params, 1)
        m.set_deterministic(True)
        m.render(cams)
        m.render_backward([g] + [torch.zeros(3, c.height, c.width, device="cuda") for c in cams[1:]])
        torch.cuda.synchronize()
        out.append(m.grads().double().cpu().numpy())
    # the sums run over the same records in another order: a few roundings of FP32 sums of at
    # most ~50 terms, 50 x 2^-24 of the column's largest entry
    scale = np.abs(out[0]).max(axis=1, keepdims=True)
    assert (np.abs(out[0] - out[1]) <= 3e-6 * scale + 3e-6 * np.abs(out[0])).all()


def _one_cell(n, depths, seed):
    """n small Gaussians of the given depths, all inside one cell of 2x2 tiles of the view."""
    cam = scenes.pinhole(320, 240, 400.0)
    params = scenes.frustum_gaussians(n, 0, cam, seed=seed)
    r = np.random.default_rng(seed)
    z = np.asarray(depths, np.float32)
    params[:, 0] = (128 + 10 + 12 * r.random(n) - cam.cx) / cam.fx * z
    params[:, 1] = (96 + 10 + 12 * r.random(n) - cam.cy) / cam.fy * z
    params[:, 2] = z
    params[:, 3:6] = np.log(2e-4 * z)[:, None]
    return cam, params


# 8 chunks, which are ranked, and 9 and more, which are merged in segments; depths at random, in
# order of the map (no chunk is a sample of the others), equal, and in a tight cluster
@pytest.mark.parametrize("n,depths,deterministic", [
    (131_072, "random", False), (131_073, "random", True), (131_073, "ordered", False), (200_000, "equal", False),
    (300_000, "random", False), (300_000, "ordered", True), (300_000, "cluster", False), (300_000, "equal", True)])
def test_lists_of_a_cell_of_many_chunks(n, depths, deterministic):
    r = np.random.default_rng(n)
    z = {"random": 5.0 + 20.0 * r.random(n), "ordered": 5.0 + 20.0 * np.arange(n) / n, "equal": np.full(n, 5.0),
         "cluster": np.where(np.arange(n) == n // 3, 400.0, 5.0 + 1e-6 * r.random(n))}[depths]
    cam, params = _one_cell(n, z, n)
    print(f"{n} Gaussians in one cell, depths {depths}, deterministic {deterministic}", flush=True)
    _, bins = _check_lists(params, 0, [cam], deterministic)
    assert _cell_sizes(bins, [cam]).max() == n


def test_time_of_a_crowded_cell_grows_with_its_entries():
    # a far view puts a map into one cell: four times the Gaussians may take four times as long
    # (about 2 measured; 10 with a search in every other chunk per entry)
    torch = torch_mod()
    times = []
    for n in (500_000, 2_000_000):
        cam, params = _one_cell(n, 5.0 + 20.0 * np.random.default_rng(n).random(n), n)
        m = gpu_map(params, 0)
        m.render([cam])
        m.set_stage_timing(True)
        best = np.inf
        for _ in range(5):
            m.stage_times()
            m.render([cam])
            torch.cuda.synchronize()
            best = min(best, m.stage_times()["duplicate"][0])
        times.append(best)
        print(f"{n} in one cell: lists {1e3 * best:.0f} us", flush=True)
        m.close()
    assert times[1] < 6 * times[0]


# chunks past a quarter and a half of a merge block's lanes, and more than it has
@pytest.mark.parametrize("n", [4_300_000, 8_500_000, 17_000_000])
def test_lists_of_a_cell_of_hundreds_of_chunks(n):
    # checked without the oracle: each tile's list is in strict order of (depth, index), and each
    # Gaussian is listed once per tile that it reaches
    torch = torch_mod()
    cam, rows = _one_cell(1000, 5.0 + 20.0 * np.random.default_rng(1).random(1000), 1)
    params = torch.from_numpy(rows).cuda().repeat(n // 1000, 1)
    scale = 1.0 + 0.2 * torch.rand(n, 1, device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    params[:, 0:3] *= scale  # along the rays of the thousand
    from paper_2404_06926_amd import gslic
    m = gslic.GaussianMap(sh_degree=0, capacity=n)
    m.add_gaussians(params)
    print(f"{n} Gaussians in one cell", flush=True)
    m.render([cam])
    torch.cuda.synchronize()
    dbg = m.debug_last_render()
    counts, vals, tiles = dbg["counts"][0].long(), dbg["vals"].long(), dbg["tiles"].long()
    assert dbg["n_inst"] == int(counts.sum()) > n
    assert torch.equal(torch.bincount(vals, minlength=n), counts)
    assert (tiles[1:] >= tiles[:-1]).all() and torch.unique(tiles).numel() <= 4
    depth = dbg["proj"][0, :, 9].contiguous().view(torch.int32).long()[vals]
    key = depth << 32 | vals
    assert ((key[1:] > key[:-1]) | (tiles[1:] > tiles[:-1])).all()


def test_renders_of_other_sizes_on_other_threads():
    # maps on different host threads are independent: an image whose counters take most of a
    # CU's LDS beside one whose counters take little, each equal to its render alone
    from concurrent.futures import ThreadPoolExecutor
    torch = torch_mod()
    cams = [scenes.pinhole(4160, 3200, 3000.0), scenes.pinhole(64, 48, 50.0)]
    maps = [gpu_map(scenes.frustum_gaussians(3000, 0, c, seed=k, log_scale_mean=-2.5), 0) for k, c in enumerate(cams)]
    alone = [m.render([c])[0].rgb.clone() for m, c in zip(maps, cams)]
    torch.cuda.synchronize()

    def renders(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            out = [maps[k].render([cams[k]])[0].rgb for _ in range(10 if k == 0 else 100)]
            stream.synchronize()
        return out

    with ThreadPoolExecutor(2) as ex:
        for k, out in enumerate(ex.map(renders, range(2))):
            assert all(torch.equal(o, alone[k]) for o in out)


# the most Gaussians whose merge holds a chunk per lane, and the most that the counting lists
# take, each and one more behind the camera: equal lists
@pytest.mark.parametrize("n", [1 << 24, 1 << 26])
def test_lists_at_the_largest_maps(n):
    torch = torch_mod()
    from paper_2404_06926_amd import gslic
    cam = scenes.pinhole(1920, 1080, 1200.0)
    rows = torch.from_numpy(scenes.frustum_gaussians(1 << 14, 0, cam, seed=6, log_scale_mean=-5.0)).cuda()
    params = rows.repeat(n >> 14, 1)
    gen = torch.Generator("cuda").manual_seed(6)
    params[:, 0:3] += 0.05 * torch.randn(n, 3, device="cuda", generator=gen)
    m = gslic.GaussianMap(sh_degree=0, capacity=n + 1)
    m.add_gaussians(params)
    out = []
    for past in (False, True):
        if past:
            behind = rows[:1].clone()
            behind[0, 2] = -5.0
            m.add_gaussians(behind)
        print(f"{m.n} Gaussians", flush=True)
        m.set_stage_timing(True)
        m.stage_times()
        f = m.render([cam])[0]
        torch.cuda.synchronize()
        assert m.stage_times()["depth_sort"][1] == (1 if m.n > 1 << 26 else 0)
        dbg = m.debug_last_render()
        out.append((f.rgb, dbg["ranges"], dbg["vals"]))
    assert all(torch.equal(a, b) for a, b in zip(*out))
