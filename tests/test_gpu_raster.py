"""GPU parity of the raster-only entry (gsc_render_gaussians) against the
FP64 oracle: closed-form image, random anisotropic scenes with ragged tiles,
tile lists and their order, empty and fully culled inputs, and the
full-64-bit-key sort mode."""
import math

import numpy as np
import pytest

import oracle
import synth
from parity import assert_image, assert_pairs, assert_ranges_from_keys, mask_tiles

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gs():
    import paper_2502_14938_amd as gs
    gs.lib()
    assert torch.cuda.is_available()
    return gs


def run(gs, mu, cov, rgb, al, cam, full_key=False):
    W, H = cam["width"], cam["height"]
    r = gs.Renderer(max_width=W, max_height=H, full_key_sort=full_key)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()
    out = torch.zeros(3, H, W, device="cuda")
    T = torch.zeros(H, W, device="cuda")
    nc = torch.zeros(H, W, dtype=torch.int32, device="cuda")
    r.render_gaussians(dev(mu), dev(cov), dev(rgb), dev(al), cam, out, T, nc)
    torch.cuda.synchronize()
    r.sync()
    pairs = r.debug("pairs") if len(al) else np.zeros((0, 2), np.int32)
    return out.cpu().numpy(), T.cpu().numpy(), nc.cpu().numpy(), pairs, r


def test_single_gaussian_closed_form(gs):
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), 64, 64, math.radians(60), math.radians(60))
    mu = np.array([[0.0, 0.0, 5.0]]); cov = np.array([[0.01, 0, 0, 0.01, 0, 0.01]])
    rgb = np.array([[0.2, 0.5, 0.9]]); al = np.array([0.8])
    img, T, nc, pairs, _ = run(gs, mu, cov, rgb, al, cam)
    ref = oracle.render_gaussians(mu, cov, rgb, al, cam)
    assert np.abs(img - ref["image"]).max() < 1e-5
    assert np.abs(T - ref["T"]).max() < 1e-5


@pytest.mark.parametrize("n,seed,W,H", [(300, 1, 72, 56), (2000, 2, 130, 97), (5000, 3, 256, 256), (1, 4, 17, 9)])
def test_random_scene_matches_oracle(gs, n, seed, W, H):
    mu, cov, rgb, al = synth.random_gaussians(n, seed=seed, box=3.0, zc=8.0)
    cam = synth.look_camera((0.1, -0.2, 0), (0.05, 0.02, 1), (0, -1, 0), W, H, math.radians(60))
    img, T, nc, pairs, _ = run(gs, mu, cov, rgb, al, cam)
    ref = oracle.render_gaussians(mu, cov, rgb, al, cam, debug=True)
    rep = assert_image(img, ref)
    ok = ref["band"] == 0
    assert np.abs(T - ref["T"])[ok].max() <= 1e-4
    assert np.array_equal(nc[ok], ref["n_contrib"][ok])
    assert_pairs(pairs, ref, ref["pre"]["depth"])
    print(rep)


def test_empty_and_culled(gs):
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), 40, 24, math.radians(60))
    img, T, nc, pairs, _ = run(gs, np.zeros((0, 3)), np.zeros((0, 6)), np.zeros((0, 3)), np.zeros(0), cam)
    assert np.all(img == 0) and np.all(T == 1) and np.all(nc == 0)
    mu, cov, rgb, al = synth.random_gaussians(100, seed=9, box=1.0, zc=-5.0)  # all behind the camera
    img, T, nc, pairs, _ = run(gs, mu, cov, rgb, al, cam)
    assert np.all(img == 0) and np.all(T == 1) and len(pairs) == 0


def test_full_key_sort_gives_same_order(gs):
    mu, cov, rgb, al = synth.random_gaussians(3000, seed=5, box=3.0, zc=8.0)
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), 200, 150, math.radians(60))
    a = run(gs, mu, cov, rgb, al, cam, full_key=False)
    b = run(gs, mu, cov, rgb, al, cam, full_key=True)
    assert np.array_equal(a[3], b[3])
    assert np.array_equal(a[0], b[0])


@pytest.mark.parametrize("seed", [21, 22])
def test_large_footprints_match_oracle(gs, seed):
    # Gaussians 0.3-3 m in front of the camera with metre-scale covariances:
    # footprints span tens of tiles, many cross the image border, the image
    # is 200x120 so the last tile column and row are clipped.
    mu, cov, rgb, al = synth.random_gaussians(400, seed=seed, box=2.5, zc=1.8, s_lo=0.05, s_hi=1.2)
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), 200, 120, math.radians(90))
    img, T, nc, pairs, _ = run(gs, mu, cov, rgb, al, cam)
    ref = oracle.render_gaussians(mu, cov, rgb, al, cam, debug=True)
    assert ref["n_pairs"] > 20 * 400 * 0.2
    assert_image(img, ref)
    assert_pairs(pairs, ref, ref["pre"]["depth"])


def test_many_tiles_two_pass_sort_and_ranges(gs):
    # 1000x560: 63 x 35 tiles, 32 x 18 = 576 super tiles, so the sort takes
    # two radix passes (8 + 2 bits); the item count is not a multiple of
    # 1024, so the ranges see both their full 1024-key steps and the ragged
    # tail; the odd tile counts leave a half-filled super tile at the right
    # and bottom edges
    mu, cov, rgb, al = synth.random_gaussians(40000, seed=6, box=6.0, zc=12.0, s_hi=0.25)
    cam = synth.look_camera((0.1, -0.2, 0), (0.05, 0.02, 1), (0, -1, 0), 1000, 560, math.radians(70))
    img, T, nc, pairs, r = run(gs, mu, cov, rgb, al, cam)
    keys = r.debug("sort_keys")
    vals = r.debug("sort_vals")
    ranges = r.debug("raw_ranges")
    ref = oracle.render_gaussians(mu, cov, rgb, al, cam, debug=True)
    assert len(ranges) == 32 * 18 and keys.max() >= 256
    assert len(vals) == len(keys) and mask_tiles(vals) == len(pairs)
    assert len(keys) % 1024 != 0 and len(pairs) > 100000, (len(keys), len(pairs))
    assert_ranges_from_keys(keys, ranges)
    assert_pairs(pairs, ref, ref["pre"]["depth"])
    assert_image(img, ref)
    r.close()


@pytest.mark.parametrize("n,W,H", [(2000, 2050, 1585), (2000, 2561, 2449), (700, 1, 1), (900, 17, 33), (1500, 250, 9)])
def test_halves_and_whole_tiles_match_oracle(gs, n, W, H):
    """The blend takes quarters of tiles up to 12,288 tiles, halves up to
    20,480 and whole tiles above: one size of each of the larger two (ragged
    right and bottom edges), and the smallest ones, where a part of a tile
    has no pixel at all.  Thin footprints among them, whose exponents are
    differences of large terms (few enough of them to fit the context's
    tall footprints and their rows)."""
    mu, cov, rgb, al = synth.random_gaussians(n, seed=n + W, box=3.0, zc=8.0, s_lo=0.002, s_hi=0.02)
    cov[::31] = 0.0
    cov[::31, 0], cov[::31, 3], cov[::31, 5] = 0.09, 1e-6, 1e-6   # needles along x ...
    cov[::62, 1], cov[::62, 3] = 0.0899, 0.09                  # ... and along the diagonal
    cam = synth.look_camera((0.1, -0.2, 0), (0.05, 0.02, 1), (0, -1, 0), W, H, math.radians(60), math.radians(60))
    img, T, nc, pairs, _ = run(gs, mu, cov, rgb, al, cam)
    ref = oracle.render_gaussians(mu, cov, rgb, al, cam, debug=True)
    assert_image(img, ref)
    ok = ref["band"] == 0
    assert np.abs(T - ref["T"])[ok].max() <= 1e-4
    assert np.array_equal(nc[ok], ref["n_contrib"][ok])


def depths(kind, n, rng):
    if kind == "spread":
        return rng.uniform(4.0, 12.0, n)
    if kind == "equal":                       # one depth: the order is the entries'
        return np.full(n, 8.0)
    if kind == "planes":                      # two planes far apart: two buckets hold everything
        return np.where(rng.uniform(size=n) < 0.5, 1.0, 4000.0)
    z = rng.uniform(7.9999, 8.0001, n)        # a crowd at 8 among a few from 0.3 to 10,000
    far = rng.uniform(size=n) < 0.01
    z[far] = np.exp(rng.uniform(np.log(0.3), np.log(1e4), int(far.sum())))
    return z


@pytest.mark.parametrize("kind", ["spread", "equal", "planes", "crowd"])
@pytest.mark.parametrize("n", [1, 2, 47, 512, 2048, 4096, 4097, 8192, 9000, 40000])
def test_lists_of_every_length_and_depth_equal_full_key_sort(gs, n, kind):
    """Every list in the order of the whole (super tile, depth) key with ties
    by entry, against the radix sort of exactly that key: lists that fit one
    block and ones that do not (2,048 items), divided by depth or, where the
    depths crowd, merged; small and large footprints (tall ones among them)
    over four super tiles."""
    rng = np.random.default_rng(n + len(kind))
    W, H = 64, 50
    z = depths(kind, n, rng)
    px, py = rng.uniform(-4, W + 4, n), rng.uniform(-4, H + 4, n)
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), W, H, math.radians(60), math.radians(60))
    fx, fy = W / (2 * math.tan(math.radians(30))), H / (2 * math.tan(math.radians(30)))
    mu = np.stack([(px - W / 2) * z / fx, (py - H / 2) * z / fy, z], 1)
    if not np.allclose(cam["R"], np.eye(3)):
        mu = mu @ cam["R"]                    # camera axes to world
    sig = np.exp(rng.uniform(np.log(0.5), np.log(30.0), n)) * z / fx
    sig[rng.uniform(size=n) > 0.2] *= 0.05    # at most a fifth large
    cov = np.zeros((n, 6)); cov[:, 0] = cov[:, 3] = cov[:, 5] = sig ** 2
    rgb, al = rng.uniform(0, 1, (n, 3)), rng.uniform(0.01, 0.6, n)
    a = run(gs, mu, cov, rgb, al, cam)
    b = run(gs, mu, cov, rgb, al, cam, full_key=True)
    assert np.array_equal(a[3], b[3])
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[4].debug("raw_ranges"), b[4].debug("raw_ranges"))
    assert np.array_equal(a[4].debug("sort_vals"), b[4].debug("sort_vals"))


@pytest.mark.parametrize("W,H", [(4096, 2048), (4096, 2049), (16384, 31), (33, 16384)])
def test_batches_around_the_most_lists_binned_equal_full_key_sort(gs, W, H):
    """8,192 super tiles of 32x32 pixels are still binned, 8,320 radix-sorted:
    the same lists and images as the sort of the whole key either way."""
    n = 20000
    rng = np.random.default_rng(W + H)
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), W, H, math.radians(60), math.radians(60))
    fx, fy = W / (2 * math.tan(math.radians(30))), H / (2 * math.tan(math.radians(30)))
    z = rng.uniform(4.0, 12.0, n)
    mu = np.stack([rng.uniform(-0.5, 0.5, n) * W * z / fx, rng.uniform(-0.5, 0.5, n) * H * z / fy, z], 1)
    if not np.allclose(cam["R"], np.eye(3)):
        mu = mu @ cam["R"]
    sig = np.exp(rng.uniform(np.log(0.5), np.log(40.0), n)) * z / max(fx, fy)
    cov = np.zeros((n, 6)); cov[:, 0] = cov[:, 3] = cov[:, 5] = sig ** 2
    rgb, al = rng.uniform(0, 1, (n, 3)), rng.uniform(0.01, 0.6, n)
    a = run(gs, mu, cov, rgb, al, cam)
    b = run(gs, mu, cov, rgb, al, cam, full_key=True)
    for x, y in zip(a[:4], b[:4]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[4].debug("raw_ranges"), b[4].debug("raw_ranges"))
    assert np.array_equal(a[4].debug("sort_vals"), b[4].debug("sort_vals"))


def render_capped(gs, g, cam, max_pairs):
    """Image, transmittance, ranges and sorted items of two renders with a
    pair capacity (0: the default one), and whether it was exceeded."""
    W, H = cam["width"], cam["height"]
    r = gs.Renderer(max_width=W, max_height=H, max_pairs=max_pairs)
    out = []
    for _ in range(2):
        img, T = torch.zeros(3, H, W, device="cuda"), torch.zeros(H, W, device="cuda")
        r.render_gaussians(*g, cam, img, T)
        torch.cuda.synchronize()
        over = False
        try:
            r.sync()
        except gs.GscError as e:
            assert e.code == gs.GSC_E_CAPACITY
            over = True
        out.append((img.cpu().numpy(), T.cpu().numpy(), r.debug("raw_ranges").reshape(-1, 2), r.debug("sort_vals")))
    r.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    return out[0] + (over,)


def capped_lists(ranges, vals, z, cap):
    """The lists that remain of the whole ones where only the first `cap`
    items fit, entries in the order (float32 depth, entry), each entry's items
    by super tile: ranges and items."""
    sup = np.repeat(np.arange(len(ranges)), ranges[:, 1] - ranges[:, 0])
    entry = (vals & 0x0fffffff).astype(np.int64)
    order = np.lexsort((sup, entry, z.astype(np.float32)[entry]))
    keep = np.zeros(len(vals), bool)
    keep[order[:cap]] = True
    count = np.bincount(sup[keep], minlength=len(ranges))
    end = np.cumsum(count)
    rg = np.stack([end - count, end], 1)
    rg[count == 0] = 0
    return rg, vals[keep]


# 3,000 short and tall footprints on 35 super tiles; more entries than one
# run of them; all at one depth; as many super tiles as are binned, and more
# (radix sorts)
@pytest.mark.parametrize("n,W,H,kind,caps", [(3000, 200, 150, "spread", (1, 77, 0.3, -1, 0)), (70000, 250, 190, "crowd", (4099, 0.7)),
                                             (2500, 130, 97, "equal", (500, 0.5)), (30000, 4096, 2048, "planes", (1000, 0.5)),
                                             (3000, 4096, 2049, "spread", (1000, 0.5))])
def test_pair_capacity_keeps_the_nearest(gs, n, W, H, kind, caps):
    """An image that needs more (super tile, entry) pairs than the capacity
    keeps those of the nearest entries, whichever way its lists are made, the
    same ones every time, and reports GSC_E_CAPACITY."""
    rng = np.random.default_rng(n + W)
    z = depths(kind, n, rng).astype(np.float32).astype(np.float64)
    fx, fy = W / (2 * math.tan(math.radians(30))), H / (2 * math.tan(math.radians(30)))
    cam = {"R": np.eye(3), "pos": np.zeros(3), "fovx": math.radians(60), "fovy": math.radians(60), "width": W,
           "height": H, "znear": 0.01}   # (depth = z, bit for bit)
    mu = np.stack([rng.uniform(-0.5, 0.5, n) * W * z / fx, rng.uniform(-0.5, 0.5, n) * H * z / fy, z], 1)
    sig = np.exp(rng.uniform(np.log(0.5), np.log(30.0), n)) * z / max(fx, fy)
    sig[rng.uniform(size=n) > 0.2] *= 0.1
    cov = np.zeros((n, 6)); cov[:, 0] = cov[:, 3] = cov[:, 5] = sig ** 2
    rgb, al = rng.uniform(0, 1, (n, 3)), rng.uniform(0.01, 0.6, n)
    g = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in (mu, cov, rgb, al)]
    _, _, ranges, vals, over = render_capped(gs, g, cam, 0)
    assert not over
    total = len(vals)
    for c in caps:
        cap = total + c if c <= 0 else int(c * total) if c < 1 else c
        img, T, rg, v, over = render_capped(gs, g, cam, cap)
        assert over == (cap < total) and len(v) == min(cap, total)
        want_rg, want_v = capped_lists(ranges, vals, z, cap)
        assert np.array_equal(rg, want_rg), cap
        assert np.array_equal(v, want_v), cap


def test_pair_capacity_of_the_allocation_free_entry(gs):
    """The allocation-free entry's 2,097,152 pairs, exceeded: status bit 0, and
    the image of a context with that capacity."""
    n, W, H = 60000, 1024, 96
    mu, _, rgb, al = synth.random_gaussians(n, seed=4, box=0.4, zc=8.0)
    cov = np.zeros((n, 6))
    cov[:, 0], cov[:, 3], cov[:, 5] = 4.0, 1e-4, 1e-4      # needles across the whole image
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), W, H, math.radians(50), math.radians(6))
    g = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in (mu, cov, rgb, al)]
    img, T, _, v, over = render_capped(gs, g, cam, gs.NOALLOC_MAX_PAIRS)
    assert over and len(v) == gs.NOALLOC_MAX_PAIRS
    out, T2 = torch.zeros(3, H, W, device="cuda"), torch.zeros(H, W, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    for _ in range(2):
        gs.render_gaussians_noalloc(*g, cam, out, T2, status)
        torch.cuda.synchronize()
        assert int(status) & 1
        assert np.array_equal(out.cpu().numpy(), img) and np.array_equal(T2.cpu().numpy(), T)


def thumbnail(n, W, H, kind, box=None):
    """n small Gaussians all over a W x H image, or on the `box` (w, h) pixels
    at its middle's super tile, and its camera."""
    rng = np.random.default_rng(n + W)
    z = depths(kind, n, rng)
    cam = synth.look_camera((0, 0, 0), (0, 0, 1), (0, -1, 0), W, H, math.radians(60), math.radians(60))
    fx, fy = W / (2 * math.tan(math.radians(30))), H / (2 * math.tan(math.radians(30)))
    px, py = rng.uniform(0, 1, n) * (box[0] if box else W), rng.uniform(0, 1, n) * (box[1] if box else H)
    if box:
        px, py = px + W // 64 * 32, py + H // 64 * 32
    mu = np.stack([(px - W / 2) * z / fx, (py - H / 2) * z / fy, z], 1) @ cam["R"]
    sig = np.exp(rng.uniform(np.log(0.3), np.log(3.0), n)) * z / fx
    cov = np.zeros((n, 6)); cov[:, 0] = cov[:, 3] = cov[:, 5] = sig ** 2
    return mu, cov, rng.uniform(0, 1, (n, 3)), rng.uniform(0.01, 0.6, n), cam


@pytest.mark.parametrize("kind", ["spread", "equal", "planes", "crowd"])
@pytest.mark.parametrize("n,W,H,box", [(65536, 96, 96, (29, 29)), (65537, 96, 96, (29, 29)), (69632, 96, 96, (29, 29)),
                                       (69633, 96, 96, (32, 32)), (300001, 130, 97, (30, 32)), (180000, 250, 90, (70, 30)),
                                       (1200000, 512, 512, (64, 32)), (65536, 32, 32, None), (65537, 32, 32, None),
                                       (300001, 32, 32, None)])
def test_lists_of_many_blocks_equal_full_key_sort(gs, n, W, H, box, kind):
    """Lists that one block divides (65,536 items) and ones that many sort by
    chunks (4,096 items) and groups of chunks, one or several of them beside
    shorter lists; and images with so many entries to every list that they are
    radix-sorted: the order of the whole key with ties by entry."""
    g = thumbnail(n, W, H, kind, box)
    a = run(gs, *g)
    b = run(gs, *g, full_key=True)
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
    assert np.array_equal(a[4].debug("raw_ranges"), b[4].debug("raw_ranges"))
    assert np.array_equal(a[4].debug("sort_vals"), b[4].debug("sort_vals"))


@pytest.mark.parametrize("kind", ["spread", "equal"])
def test_many_items_in_few_lists_are_not_slower_than_sorted(gs, kind):
    """2,000,000 Gaussians on one super tile: no slower than with the radix
    sort of the whole key (0.40 and 0.34 ms measured, 0.37 and 0.36 with that;
    20 and 17 when one block divided the list)."""
    n, W, H = 2_000_000, 32, 32
    *arrays, cam = thumbnail(n, W, H, kind)
    g = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in arrays]
    out = torch.zeros(3, H, W, device="cuda")
    best = []
    for full_key in (False, True):
        r = gs.Renderer(max_width=W, max_height=H, full_key_sort=full_key)
        times = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            r.render_gaussians(*g, cam, out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        r.close()
        best.append(min(times))
    print("binned %.3f ms, sorted by the whole key %.3f ms" % tuple(best))
    assert best[0] <= 1.5 * best[1]


@pytest.mark.parametrize("n,W,H", [(300_000, 64, 64), (20000, 4096, 2049), (20000, 16384, 4128)])
def test_radix_sorted_keys_and_ranges(gs, n, W, H):
    """Batches that are radix-sorted: more than 65,536 entries to every super
    tile, 8,320 super tiles (16-bit keys, two passes) and 66,048 (32-bit keys,
    three).  The sorted keys as the device holds them against the runs that
    k_ranges found in them, and key for key against the sort of the whole key."""
    mu, cov, rgb, al, cam = thumbnail(n, W, H, "spread")
    g = [torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda() for a in (mu, cov, rgb, al)]
    out = torch.zeros(3, H, W, device="cuda")
    keys, vals = [], []
    for full_key in (False, True):
        r = gs.Renderer(max_width=W, max_height=H, full_key_sort=full_key)
        r.render_gaussians(*g, cam, out)
        torch.cuda.synchronize()
        r.sync()
        keys.append(r.debug("sort_keys"))
        vals.append(r.debug("sort_vals"))
        assert assert_ranges_from_keys(keys[-1], r.debug("raw_ranges")) > 1
        r.close()
    assert np.array_equal(keys[0], keys[1]) and np.array_equal(vals[0], vals[1])


@pytest.mark.parametrize("W,H,n,s_lo,s_hi,bound", [
    # counted over uncounted 1.13; 1.24 when the kernel took a branch around every composite step
    (4096, 2160, 400000, 0.004, 0.02, 1.19),
    # 1.16; 1.225 when its registers spilled
    (8192, 8192, 100000, 0.004, 0.01, 1.195),
])
def test_counting_work_costs_a_few_instructions(gs, W, H, n, s_lo, s_hi, bound):
    """Counting the blend's work costs a big image a fraction of its time, at
    most halfway between what it does and what it once did, and the image is
    the same."""
    g = [torch.from_numpy(x).cuda() for x in synth.random_gaussians(n, seed=1, box=3.0, zc=8.0, s_lo=s_lo, s_hi=s_hi)]
    cam = synth.look_camera((0.1, -0.2, 0), (0.05, 0.02, 1), (0, -1, 0), W, H, math.radians(60), math.radians(60))
    r = gs.Renderer(max_width=W, max_height=H)
    out = [torch.zeros(3, H, W, device="cuda") for _ in range(2)]
    ms = [[], []]
    for _ in range(40):
        for count in (0, 1):
            r.count_work(bool(count))
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            r.render_gaussians(*g, cam, out[count])
            b.record()
            r.sync()  # raises if a capacity was exceeded
            b.synchronize()
            ms[count].append(a.elapsed_time(b))
    r.close()
    assert torch.equal(out[0], out[1])
    plain, counted = (float(np.median(x)) for x in ms)
    print("%.3f ms, counted %.3f" % (plain, counted))
    assert counted <= bound * plain
