"""GPU parity of the fused training loss (gs_loss: Eq. 1 and Eq. 3 of
VastGaussian, (1 - lambda) L1 + lambda D-SSIM) against the FP64 oracle.

Every test calls the HIP kernels through the C ABI and compares with the
oracle on the same seeded image pairs.  Tolerances:
  loss value     |L_gpu - L_ref| <= 2e-5 for the total, the L1 mean and the
                 SSIM mean (quantities of order 0.01..1; the kernel sums
                 FP32 terms per 32 x 32 tile and the tiles in FP64, and the
                 SSIM terms carry FP32 rounding of sigma^2 = E[x^2] - mu^2,
                 about 1e-7 absolute against C2 = 9e-4);
  d_image        the gradient bar of gpu_util (elementwise 1e-3 of |g_ref|
                 plus 1e-2 of the largest, and 1e-3 in norm);
  d_image_l1     bit-exact: sign(I^a - I) is decided on the same FP32
                 values on both sides and the oracle is given lambda as
                 the FP32 value the kernel uses.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from gen import images
from oracle import loss as orc
from paper_2402_17427_amd import loss as gl

from gpu_util import grad_close

pytestmark = pytest.mark.gpu

LOSS_ATOL = 2e-5


def _case(name):
    print(f"\n[case] {name}", flush=True)


def _f32(x):
    return float(np.float32(x))


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a, np.float32)).cuda()


def _run(r, t, lam, ra=None):
    out, d, d1 = gl.image_loss(_dev(r), _dev(t), lam, None if ra is None else _dev(ra))
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64), d.cpu().numpy(), None if d1 is None else d1.cpu().numpy()


def _appearance(r, seed):
    """An appearance-adjusted image: a smooth per-pixel gain of the render."""
    rng = np.random.default_rng(seed)
    C, H, W = r.shape
    gain = 1.0 + 0.1 * np.sin(np.arange(W)[None, None, :] / 17.0 + rng.uniform(0, 6, (C, 1, 1)))
    return (r * gain * rng.uniform(0.95, 1.05, (C, H, 1))).astype(np.float32)


@pytest.mark.parametrize("C,H,W,lam,eq3,seed", [
    (3, 70, 97, 0.2, False, 1),     # several tiles, ragged in both directions
    (3, 70, 97, 0.2, True, 2),      # Eq. 3: L1 on the adjusted image
    (3, 64, 64, 0.2, False, 3),     # exact multiple of the 32 x 32 tile
    (1, 33, 31, 1.0, False, 4),     # D-SSIM only
    (2, 45, 40, 0.0, True, 5),      # L1 only, Eq. 3 form
    (2, 5, 3, 0.2, False, 6),       # image smaller than the window
    (1, 1, 1, 0.2, False, 7),       # a single pixel
    (3, 1, 130, 0.2, False, 8),     # a single row across five tiles
])
def test_loss_matches_the_oracle(C, H, W, lam, eq3, seed):
    _case(f"loss C={C} H={H} W={W} lam={lam} eq3={eq3}")
    r, t = images.image_pair(seed, W, H, channels=C)
    ra = _appearance(r, seed) if eq3 else None
    lam32 = _f32(lam)
    out, d, d1 = _run(r, t, lam, ra)
    ref = orc.loss(r, t, lam32, ra)
    print("loss err", [abs(out[k] - ref[n]) for k, n in enumerate(("loss", "l1", "ssim"))], flush=True)
    for k, name in enumerate(("loss", "l1", "ssim")):
        assert abs(out[k] - ref[name]) <= LOSS_ATOL, (name, out[k], ref[name])
    rd, rd1 = orc.loss_grad(r, t, lam32, ra)
    if lam > 0:
        print("d_image norm rel", grad_close("d_image", d, rd), flush=True)
    if eq3:
        np.testing.assert_array_equal(d1, rd1.astype(np.float32))
        if lam == 0:
            assert np.all(d == 0)
    elif lam == 0:
        np.testing.assert_array_equal(d, rd.astype(np.float32))


def test_identical_images_give_zero_loss_and_gradient():
    """SSIM(x, x) = 1 and L1 = 0: the loss and the gradient vanish (up to
    FP32 rounding of the SSIM terms) at a ragged full-HD-width shape."""
    _case("loss identical images")
    r, _ = images.image_pair(11, 1000, 77)
    out, d, _ = _run(r, r, 0.2)
    assert abs(out[0]) < 1e-6 and out[1] == 0.0 and abs(out[2] - 1.0) < 1e-6
    n = r.size
    assert np.abs(d).max() < 1e-2 * 0.2 / n


def test_loss_is_deterministic():
    _case("loss determinism")
    r, t = images.image_pair(12, 300, 200)
    rd, td = _dev(r), _dev(t)
    L = gl.ImageLoss(3, 200, 300)
    o1, d1, _ = L(rd, td)
    a = (o1.clone(), d1.clone())
    o2, d2, _ = L(rd, td)
    torch.cuda.synchronize()
    assert torch.equal(a[0], o2) and torch.equal(a[1], d2)


def test_full_hd_loss_and_sampled_gradient_windows():
    """1920 x 1080 x 3, the shape the benchmark times: the loss value
    against the oracle on the whole image, the gradient on windows at the
    corners, an edge and the centre (the oracle runs on each window plus
    the 10-pixel margin that determines it, clipped to the image, so its
    values inside the window are those of the whole image)."""
    _case("loss 1920x1080x3")
    W, H = 1920, 1080
    r, t = images.image_pair(5, W, H)
    lam = 0.2
    out, d, _ = _run(r, t, lam)
    n = r.size
    ref = orc.loss(r, t, _f32(lam))
    print("loss err", [abs(out[k] - ref[n]) for k, n in enumerate(("loss", "l1", "ssim"))], flush=True)
    for k, name in enumerate(("loss", "l1", "ssim")):
        assert abs(out[k] - ref[name]) <= LOSS_ATOL, (name, out[k], ref[name])
    win = 48
    for (y, x) in [(0, 0), (0, W - win), (H - win, 0), (H - win, W - win), (0, 931), (517, 1003), (700, 1888)]:
        ya, yb = max(0, y - 10), min(H, y + win + 10)
        xa, xb = max(0, x - 10), min(W, x + win + 10)
        # the oracle normalises by its own pixel count: rescale to the full image's
        rc, tc = r[:, ya:yb, xa:xb], t[:, ya:yb, xa:xb]
        g, _ = orc.loss_grad(rc, tc, _f32(lam))
        g *= rc.size / n
        sub = g[:, y - ya:y - ya + win, x - xa:x - xa + win]
        rel = grad_close(f"d_image window ({y},{x})", d[:, y:y + win, x:x + win], sub)
        print(f"window ({y},{x}) norm rel {rel:.3e}", flush=True)


@pytest.mark.parametrize("C,H,W,eq3", [
    # more than 1536 tiles of 32 x 32: the strips (236 columns, four-row
    # groups); their segments and waves at the edges
    (97, 100, 119, False),   # 97 x 16 tiles; one strip of three waves, ragged segment
    (64, 129, 149, True),    # 64 x 25: one row over a segment of 128
    (40, 193, 236, False),   # 40 x 56: one strip of 236 columns exactly
    (40, 190, 237, True),    # one column in the second strip
    (1600, 3, 44, False),    # image lower than the window, one wave
    (800, 33, 45, False),    # one column of the second wave
    (48, 32, 1056, False),   # 48 x 33 tiles = 1584: five strips
    (48, 32, 1024, False),   # 48 x 32 tiles = 1536: the tile kernel's last size
])
def test_loss_at_the_edges_of_strips_and_of_the_rule(C, H, W, eq3):
    """The strip kernel at the edges of its strips, waves, row groups and
    segments and on both sides of the rule that takes it: the same gradient
    bits as channel by channel (few tiles: the tile kernel, which sums in
    the same order), scaled by the channel count's power of two or within
    an FP32 rounding of each factor; the loss against the oracle."""
    _case(f"loss edges C={C} H={H} W={W} eq3={eq3}")
    few = min(C, 4)
    r, t = images.image_pair(21, W, H, channels=few)
    r, t = np.concatenate([r] * (C // few) + [r[:C % few]]), np.concatenate([t] * (C // few) + [t[:C % few]])
    ra = _appearance(r, 21) if eq3 else None
    out, d, d1 = _run(r, t, 0.2, ra)
    one, dd, dd1 = _run(r[:few], t[:few], 0.2, None if ra is None else ra[:few])
    ref = orc.loss(r, t, _f32(0.2), ra)
    for k, name in enumerate(("loss", "l1", "ssim")):
        assert abs(out[k] - ref[name]) <= LOSS_ATOL, (name, out[k], ref[name])
    rd, rd1 = orc.loss_grad(r, t, _f32(0.2), ra)
    grad_close("d_image", d, rd)
    if eq3:
        np.testing.assert_array_equal(d1, rd1.astype(np.float32))
    if C == few * (C // few) and (C // few) & (C // few - 1) == 0:   # 1 / n scales by a power of two: the same bits
        np.testing.assert_array_equal(d[:few] * (C // few), dd)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("C,y,x", [(1, 0, 0), (1, 20, 113), (80, 37, 235), (80, 0, 0), (80, 19, 236), (80, 39, 299)])
def test_values_that_are_not_finite_reach_their_windows_only(C, y, x, value):
    """A pixel that is NaN or infinite makes the gradient NaN exactly where
    the oracle has it NaN (the two windows' reach of 10 pixels), and leaves
    it within tolerance elsewhere: 1 channel (20 tiles of 32 x 32) and 80
    (1600, the strips)."""
    _case(f"loss {value} at ({y},{x}) of {C}")
    r, t = images.image_pair(22, 300, 40, channels=1)
    r, t = np.concatenate([r] * C), np.concatenate([t] * C)
    c = C // 2
    r[c, y, x] = value
    out, d, _ = _run(r, t, 0.2)
    lo, hi = max(0, c - 1), min(C, c + 2)
    with np.errstate(all="ignore"):
        rd, _ = orc.loss_grad(r[lo:hi], t[lo:hi], _f32(0.2))
    rd *= (hi - lo) / C
    assert not np.isfinite(out[0])
    np.testing.assert_array_equal(np.isnan(d[lo:hi]), np.isnan(rd))
    assert np.isnan(d).sum() == np.isnan(rd).sum()
    ok = ~np.isnan(rd)
    grad_close("d_image", d[lo:hi][ok], rd[ok])


@pytest.mark.parametrize("C,H,W", [(3, 2160, 3840), (600, 130, 44)])
@pytest.mark.parametrize("x,y", [(0.7, 0.4), (0.3, 0.17), (0.8, 0.13)])
def test_mean_of_a_uniform_difference_over_long_segments(C, H, W, x, y):
    """Segments of 216 and 132 rows whose every L1 term is the same number: a
    lane that adds them one by one in FP32 drifts by some 1e-6 of the sum.
    At most four terms are added in FP32, then FP64 sums are rounded once a
    segment and once at the end: 2 + 1 + 1 roundings of 2^-24."""
    _case(f"uniform |{x} - {y}| C={C} H={H} W={W}")
    r, t = (torch.full((C, H, W), v, dtype=torch.float32, device="cuda") for v in (x, y))
    out, _, _ = gl.image_loss(r, t, 0.2)
    want = float(np.float32(x) - np.float32(y))
    assert abs(float(out[1]) / want - 1.0) <= 4 * 2.0 ** -24
