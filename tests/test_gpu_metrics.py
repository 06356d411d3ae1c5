"""GPU parity of the device SSIM (gsc_ssim) with the FP64 oracle: seeded
random images of several sizes, from the 11 x 11 minimum to sizes that leave
ragged 16 x 16 tiles of window positions; identical images; constant images
against the closed form; two rendered frames; the size limit."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gs():
    import paper_2502_14938_amd as gs
    gs.lib()
    return gs


@pytest.fixture(scope="module")
def r(gs):
    rr = gs.Renderer(k=10, max_width=64, max_height=64)
    yield rr
    rr.close()


@pytest.mark.parametrize("shape", [(3, 11, 11), (1, 12, 27), (3, 37, 53), (1, 64, 64), (3, 100, 129)])
def test_ssim_matches_oracle(r, shape):
    rng = np.random.default_rng(sum(shape))
    x = rng.random(shape, dtype=np.float32)
    # a correlated second image (SSIM well inside (0, 1))
    y = np.clip(x + 0.1 * rng.standard_normal(shape).astype(np.float32), 0, 1).astype(np.float32)
    got = r.ssim(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    want = oracle.ssim(x, y)
    assert abs(got - want) < 1e-9, (shape, got, want)
    assert 0.0 < want < 1.0


def test_ssim_identical_and_constant(r):
    rng = np.random.default_rng(9)
    x = torch.from_numpy(rng.random((3, 40, 50), dtype=np.float32)).cuda()
    assert abs(r.ssim(x, x) - 1.0) < 1e-12
    a, b = float(np.float32(0.3)), float(np.float32(0.7))  # the values the float32 images hold
    want = (2 * a * b + 1e-4) / (a * a + b * b + 1e-4)
    ca = torch.full((2, 20, 30), a, device="cuda")
    cb = torch.full((2, 20, 30), b, device="cuda")
    assert abs(r.ssim(ca, cb) - want) < 1e-9


def test_ssim_of_rendered_frames(gs, tiny, tiny_cams):
    L, R = tiny_cams
    W, H = L["width"], L["height"]
    rr = gs.Renderer(k=tiny.k, max_width=W, max_height=H)
    rr.load(tiny)
    oL = torch.zeros(3, H, W, device="cuda"); oR = torch.zeros(3, H, W, device="cuda")
    rr.frame(L, R, oL, oR)
    rr.sync()
    torch.cuda.synchronize()
    got = rr.ssim(oL, oR)
    want = oracle.ssim(oL.cpu().numpy(), oR.cpu().numpy())
    assert abs(got - want) < 1e-9, (got, want)
    rr.close()


def test_ssim_size_limit(gs, r):
    x = torch.zeros(3, 10, 20, device="cuda")
    with pytest.raises(gs.GscError):
        r.ssim(x, x)


@pytest.mark.parametrize("shape", [(1, 11, 74), (2, 12, 75), (1, 13, 76), (3, 24, 138), (1, 300, 11), (1, 400, 651),
                                   (1100, 12, 14), (4200, 11, 12)])
def test_ssim_at_strip_edges(r, shape):
    """Maps of one row or column, columns on either side of a strip's 64 (and
    of the pixels it may read past them), long and short strips, and more
    planes than the slots that are kept; the bound of the test above."""
    rng = np.random.default_rng(sum(shape))
    x = rng.random(shape, dtype=np.float32)
    y = np.clip(x + 0.1 * rng.standard_normal(shape).astype(np.float32), 0, 1).astype(np.float32)
    X, Y = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    want = oracle.ssim(x, y)
    for _ in range(2):
        assert abs(r.ssim(X, Y) - want) < 1e-9


@pytest.mark.parametrize("shape", [(511, 13, 12), (512, 13, 12), (514, 14, 26), (513, 12, 27), (600, 30, 42), (601, 12, 43),
                                   (2051, 21, 11)])
def test_ssim_of_many_narrow_planes(r, shape):
    """Planes that share a strip by four (up to 16 window columns) and by two
    (up to 32), the last group of them not full, and ones that do not; the
    bound of the first test."""
    rng = np.random.default_rng(sum(shape))
    x = rng.random(shape, dtype=np.float32)
    y = np.clip(x + 0.1 * rng.standard_normal(shape).astype(np.float32), 0, 1).astype(np.float32)
    want = oracle.ssim(x, y)
    assert abs(r.ssim(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()) - want) < 1e-9


def test_many_narrow_planes_take_less_than_wide_ones(r):
    """65,535 planes of one window each share a strip of 64 columns by four;
    33 columns wide, each has a strip of its own.  A quarter of the strips, so
    at most 0.6 of the time (0.18 ms a call; 0.55 when they had a strip each)."""
    def best(shape):
        x, y = torch.rand(shape, device="cuda"), torch.rand(shape, device="cuda")
        times = []
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            r.ssim(x, y)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    narrow, wide = best((65535, 11, 11)), best((65535, 11, 43))
    print("%.3f ms, %.3f" % (narrow, wide))
    assert narrow <= 0.6 * wide
