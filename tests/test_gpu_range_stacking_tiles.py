"""Range stacking at the edges of its tiles: 64 x 16 pixel tiles, 64-column and 64-row groups of a tile's window,
bands of rows when the slice bitmaps exceed their workspace, and non-finite shades.

Tolerance: FP32 sums of KW + KH terms, each with a relative rounding error of 2^-24, against the oracle's FP64
correlations: under 2e-5 of a pixel's largest correlation for every kernel here (2 x 255 terms)."""
import numpy as np
import pytest

import scenes
from oracle import range_stacking as RS
from oracle import surrogate as SUR

pytestmark = pytest.mark.gpu
TOL = 2e-5


@pytest.fixture(scope="module")
def lidar():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    lidar.load()
    return lidar


def _run(lidar, gb, n_bins, Hk, Vk, rho):
    import torch
    p = scenes.SensorParams(n_bins=n_bins, bin_ns=1.0, max_echoes=3, threshold=1e-6, emit_power=1.0, pulse_fwhm_ns=4.0)
    h, w = gb.depth.shape
    s = torch.full((h, w), -5, dtype=torch.int32, device="cuda")
    x = torch.full((h, w), -1.0, dtype=torch.float32, device="cuda")
    sim = lidar.LidarSim(p, stream=torch.cuda.current_stream())
    try:
        sim.set_gbuffer(gb.raster, lidar.upload_gbuffer(gb, "cuda"))
        sim.range_stacking(Hk, Vk, rho, s, x)
        torch.cuda.synchronize()
    finally:
        sim.close()
    return s.cpu().numpy(), x.cpu().numpy(), p


def _factor(half):
    x = np.arange(-half, half + 1)
    return np.exp(-0.5 * ((x - 0.3 * half) / (0.5 * max(half, 1))) ** 2).astype(np.float32)


def _image(width, height, seed, near, far):
    r = scenes.Raster(width, height, -0.05 * width, 0.05 * width, -0.05 * height, 0.05 * height)
    gb = scenes.random_gbuffer(r, np.random.default_rng(seed), depth_range=(near, far), retro_frac=0.05)
    gb.depth[np.random.default_rng(seed + 1).uniform(size=gb.depth.shape) < 0.2] = np.inf
    return gb


@pytest.mark.parametrize("width,height,M,N", [(1, 1, 0, 0), (63, 15, 3, 2), (64, 16, 32, 24), (65, 17, 33, 25),
                                              (129, 33, 64, 57), (130, 31, 5, 127), (200, 18, 127, 1)])
def test_window_groups_and_tile_remainders(lidar, oracle_mod, width, height, M, N):
    gb = _image(width, height, width + height, 3.0, 6.0)
    Hk, Vk = _factor(M), _factor(N)
    p = scenes.SensorParams(n_bins=64, bin_ns=1.0, max_echoes=3, threshold=1e-6, emit_power=1.0, pulse_fwhm_ns=4.0)
    t = SUR.pixel_terms(gb, p, lambda v: oracle_mod.row_solid_angle(gb.raster, v))
    inten, bins = t["shade"], t["kbin"].astype(np.int64)
    corr = RS.slice_correlations(inten, bins, np.outer(Vk.astype(np.float64), Hk.astype(np.float64)), 64)
    if not corr:
        corr = {0: np.zeros_like(inten)}
    stack = np.stack([corr[k] for k in sorted(corr)])
    top = stack.max(axis=0)
    rho = 0.4 * float(np.median(top[top > 0])) if (top > 0).any() else 1.0
    s, x, _ = _run(lidar, gb, 64, Hk, Vk, rho)
    hit = stack >= rho
    s_ref = np.where(hit.any(0), np.array(sorted(corr))[hit.argmax(0)], 64)
    x_ref = np.where(hit.any(0), np.take_along_axis(stack, hit.argmax(0)[None], 0)[0], 0.0)
    ok = ~(np.abs(stack - rho) <= TOL * top).any(0)
    np.testing.assert_array_equal(s[ok], s_ref[ok])
    np.testing.assert_allclose(x[ok], x_ref[ok], rtol=TOL, atol=0)


def test_bands_of_rows(lidar):
    """One column block of 70003 rows and 8000 bins: the bitmaps of all rows exceed their 64 MB.  A centred unit
    kernel leaves every pixel its own slice."""
    h = 70003
    r = scenes.Raster(9, h, -0.5, 0.5, -85.0, 85.0)
    rng = np.random.default_rng(8)
    gb = scenes.shell_gbuffer(r, 10.0, 0.5)
    gb.depth[:] = rng.uniform(1.0, 1150.0, gb.depth.shape)
    gb.depth[rng.uniform(size=gb.depth.shape) < 0.1] = np.inf
    V = np.zeros(5, np.float32)
    V[2] = 1.0
    s, x, p = _run(lidar, gb, 8000, np.ones(1, np.float32), V, 1e-30)
    d = gb.depth.astype(np.float64)
    with np.errstate(invalid="ignore"):
        k = np.floor(d * (2.0 / (scenes.C_LIGHT * 1e-9)))
    want = np.where(np.isfinite(d) & (k < 8000), k, 8000)
    np.testing.assert_array_equal(s, want.astype(np.int32))
    assert np.all((x > 0) == (want < 8000))


def test_infinite_shade_stays_inside_its_kernel(lidar):
    """A pixel at a vanishing range has an infinite shade: pixels that its kernel does not reach are as without it."""
    M, N, at = 6, 4, (20, 70)
    gb = _image(140, 40, 3, 3.0, 6.0)
    Hk, Vk = _factor(M), _factor(N)
    gb.depth[at] = np.inf
    rho = 1e-6
    s0, x0, _ = _run(lidar, gb, 64, Hk, Vk, rho)
    gb.depth[at], gb.reflectance[at] = 1e-25, 0.5
    s1, x1, _ = _run(lidar, gb, 64, Hk, Vk, rho)
    vv, uu = np.mgrid[0:40, 0:140]
    near = (np.abs(vv - at[0]) <= N) & (np.abs(uu - at[1]) <= M)
    np.testing.assert_array_equal(s1[~near], s0[~near])
    np.testing.assert_array_equal(x1[~near], x0[~near])
    assert (s1[near] == 0).all() and np.isinf(x1[near]).all()
