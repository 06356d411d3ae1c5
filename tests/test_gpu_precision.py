"""GPU parity of the derivation precision forms.

BF16 (weights and activations rounded to bfloat16, FP32 accumulate) and
FP8 (e4m3fn weights with per-row scales, BF16 activations) are checked two
ways: against the oracle's emulation of the same rounding (isolates kernel
error from quantisation error), and against the exact FP64 oracle, where
the per-image PSNR must clear 40 dB.  The plain FP32 form (FP32 MFMA) is
checked against the exact oracle to the FP32 tolerance."""
import numpy as np
import pytest

import oracle
import synth
from parity import assert_image

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gs():
    import paper_2502_14938_amd as gs
    gs.lib()
    return gs


def frame(gs, scene, L, R, prec):
    W, H = L["width"], L["height"]
    r = gs.Renderer(k=scene.k, precision=prec, max_width=W, max_height=H)
    r.load(scene)
    oL = torch.zeros(3, H, W, device="cuda"); oR = torch.zeros(3, H, W, device="cuda")
    r.frame(L, R, oL, oR)
    torch.cuda.synchronize()
    r.sync()
    return oL.cpu().numpy(), oR.cpu().numpy(), r.debug("derived"), r.debug("gauss")


@pytest.mark.parametrize("prec,emu", [("f32", 0), ("bf16", 1), ("fp8", 2)])
def test_derived_parameters_vs_emulation(gs, tiny, tiny_cams, prec, emu):
    L, R = tiny_cams
    iL, iR, der, G = frame(gs, tiny, L, R, prec)
    U = oracle.unified_camera(L, R)
    ids, _ = oracle.select(tiny, U)
    ref = oracle.derive(tiny, ids, U["pos"], emu)
    # compare on the Gaussians both sides kept
    ora_keep = np.nonzero(ref["alpha"] > 0)[0]
    common, gi, oi = np.intersect1d(G, ora_keep, return_indices=True)
    assert len(common) >= 0.99 * max(len(G), len(ora_keep))
    d_alpha = np.abs(der[gi, 12] - ref["alpha"][common])
    d_rgb = np.abs(der[gi, 9:12] - ref["rgb"][common]).max(1)
    cov = ref["cov"][common]
    d_cov = np.abs(der[gi, 3:9] - cov).max(1) / np.abs(cov).max(1)
    d_mu = np.abs(der[gi, 0:3] - ref["mu"][common]).max(1)
    print(prec, "alpha max %.3g p99 %.3g | rgb max %.3g | cov rel max %.3g | mu max %.3g" % (
        d_alpha.max(), np.percentile(d_alpha, 99), d_rgb.max(), d_cov.max(), d_mu.max()))
    if prec == "f32":
        assert d_alpha.max() < 2e-6 and d_rgb.max() < 2e-6 and d_cov.max() < 2e-5 and d_mu.max() < 2e-6
        assert np.array_equal(G, np.nonzero(ref["alpha"] > 0)[0]) or (np.abs(ref["alpha_pre"]) < 1e-6).any()
    else:
        # FP32 accumulation order and rare bf16 rounding flips of activations
        assert np.percentile(d_alpha, 99) < 2e-3 and d_alpha.max() < 3e-2
        assert np.percentile(d_rgb, 99) < 2e-3 and d_rgb.max() < 3e-2
        assert np.percentile(d_cov, 99) < 5e-3
        assert d_mu.max() < 2e-6  # means do not pass through the MLP


@pytest.mark.parametrize("prec", ["f32", "bf16", "fp8"])
def test_images_vs_exact_oracle(gs, tiny, tiny_cams, prec):
    L, R = tiny_cams
    iL, iR, _, _ = frame(gs, tiny, L, R, prec)
    ref = oracle.render_frame(tiny, L, R)
    for img, eye in ((iL, "left"), (iR, "right")):
        p = oracle.psnr(img, ref[eye]["image"])
        print(prec, eye, "PSNR vs exact oracle %.2f dB, max-abs %.3g" % (p, oracle.max_abs(img, ref[eye]["image"])))
        if prec == "f32":
            assert_image(img, ref[eye])
        else:
            assert p >= 40.0


@pytest.mark.parametrize("prec,emu", [("f32", 0), ("bf16", 1), ("fp8", 2)])
@pytest.mark.parametrize("n,k", [(1, 10), (17, 3), (500, 1), (700, 5), (333, 16), (9000, 2)])
def test_derived_parameters_at_tile_edges(gs, n, k, prec, emu):
    """Every k from one to the most (its outputs fill whole and partial matrix
    tiles), counts of anchors that leave a tile ragged, and more tiles than
    waves; the bounds of the test above."""
    scene = synth.tiny_scene(n=n, k=k, seed=n + k)
    L, R = synth.tiny_pair(64, 48)
    _, _, der, G = frame(gs, scene, L, R, prec)
    U = oracle.unified_camera(L, R)
    ids, _ = oracle.select(scene, U)
    ref = oracle.derive(scene, ids, U["pos"], emu)
    keep = np.nonzero(ref["alpha"] > 0)[0]
    common, gi, _ = np.intersect1d(G, keep, return_indices=True)
    assert len(common) >= 0.99 * max(len(G), len(keep))
    if not len(common):
        return
    d_alpha = np.abs(der[gi, 12] - ref["alpha"][common])
    d_rgb = np.abs(der[gi, 9:12] - ref["rgb"][common]).max(1)
    cov = ref["cov"][common]
    d_cov = np.abs(der[gi, 3:9] - cov).max(1) / np.abs(cov).max(1)
    d_mu = np.abs(der[gi, 0:3] - ref["mu"][common]).max(1)
    assert d_mu.max() < 2e-6
    if prec == "f32":
        assert d_alpha.max() < 2e-6 and d_rgb.max() < 2e-6 and d_cov.max() < 2e-5
    else:
        assert d_alpha.max() < 3e-2 and d_rgb.max() < 3e-2 and np.median(d_cov) < 5e-3


@pytest.mark.parametrize("prec,emu", [("f32", 0), ("bf16", 1), ("fp8", 2)])
def test_derived_parameters_of_more_tiles_than_waves(gs, prec, emu):
    """70,001 misses are 4,376 tiles of 16 anchors, more than the 4,096 waves
    of the decoding: some waves take a second tile, whose inputs they loaded
    while the first was computed.  Every anchor's parameters against the
    oracle.  A 32-term FP32 dot product of terms adding up to about 8 is off
    by sqrt(32) 6e-8 8 = 2.7e-6 where the roundings don't all have one sign:
    4e-6; a rounding flip of a BF16 activation (2^-8 of about 2) moves an
    output by at most 2e-3 a weight of 0.3, of which a few may meet: 3e-2."""
    n = 70001
    scene = synth.tiny_scene(n=n, k=2, seed=70)
    L, R = synth.tiny_pair(64, 48)
    _, _, der, G = frame(gs, scene, L, R, prec)
    U = oracle.unified_camera(L, R)
    ids, _ = oracle.select(scene, U)
    assert len(ids) > 65536
    ref = oracle.derive(scene, ids, U["pos"], emu)
    keep = np.nonzero(ref["alpha"] > 0)[0]
    common, gi, _ = np.intersect1d(G, keep, return_indices=True)
    assert len(common) >= 0.99 * max(len(G), len(keep))
    d_alpha = np.abs(der[gi, 12] - ref["alpha"][common])
    d_rgb = np.abs(der[gi, 9:12] - ref["rgb"][common]).max(1)
    cov = ref["cov"][common]
    d_cov = np.abs(der[gi, 3:9] - cov).max(1) / np.abs(cov).max(1)
    assert np.abs(der[gi, 0:3] - ref["mu"][common]).max() < 2e-6
    if prec == "f32":
        assert d_alpha.max() < 4e-6 and d_rgb.max() < 4e-6 and d_cov.max() < 4e-5
    else:
        assert d_alpha.max() < 3e-2 and d_rgb.max() < 3e-2 and np.median(d_cov) < 5e-3
