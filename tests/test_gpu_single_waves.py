"""Single frames of many narrow beams (a wave per group of beams) against the same beams in frames of fewer than 2048
beams (a workgroup per group): every echo selection, waveform lengths around the passes of 512 bins, range intervals,
sun, supplied floors and kept waveforms; beam counts that leave waves and groups partly empty, beams off the image.

The two routes add the same FP32 products in different orders: n terms of one sign differ by at most
n 2^-24 relative, n the kernel's cells (1e-5 at least); what is decided from bins is the same."""
from dataclasses import replace

import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu

# half extents in pixels
KERNELS = {"narrow": (4, 3), "wide": (6, 5)}


@pytest.fixture(scope="module")
def lidar():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    lidar.load()
    return lidar


def _run(lidar, w, params, idx, kernel, keep):
    import torch
    az, el = w.pattern.beam_az[idx], w.pattern.beam_el[idx]
    sd = w.gbuffer.raster.dphi, w.gbuffer.raster.de
    if kernel == "table":
        k = np.outer([1, 2, 1], [1, 3, 5, 3, 1]).astype(np.float32)
        pat = scenes.Pattern(scenes.PATTERN_TABLE, az, el, table=k, half_deg=(2.5 * sd[0], 1.5 * sd[1]),
                             rx_table=np.ones_like(k))
    else:
        m, n = KERNELS[kernel]
        pat = scenes.Pattern(scenes.PATTERN_GAUSS, az, el, sigma_deg=((m + 0.2) / 3 * sd[0], (n + 0.2) / 3 * sd[1]),
                             trunc_sigmas=3.0)
    sim = lidar.LidarSim(params, stream=torch.cuda.current_stream(), keep_waveforms=keep)
    try:
        sim.set_pattern(pat)
        sim.set_gbuffer(w.gbuffer.raster, lidar.upload_gbuffer(w.gbuffer, "cuda"))
        sim.simulate_frame()
        return sim.read(waveforms=keep)
    finally:
        sim.close()


@pytest.mark.parametrize("n_beams,bins,select,range_mode,sun,kernel,keep", [
    (2048, 512, 0, 0, 0.0, "narrow", False),
    (2049, 513, 1, 0, 0.03, "narrow", False),
    (2050, 1200, 2, 0, 0.0, "narrow", True),
    (2051, 2048, 3, 0, 0.03, "table", True),
    (4099, 2048, 0, 0, 0.03, "narrow", False),
    (4099, 511, 4, 0, 0.0, "narrow", True),
    (4100, 1025, 5, 0, 0.03, "narrow", False),
    (4101, 1024, 0, 2, 0.0, "narrow", False),
    (9001, 2048, 0, 0, 0.0, "table", False),
    (4801, 512, 0, 0, 0.03, "wide", True),
    (4803, 2048, 1, 0, 0.0, "wide", False),
])
def test_same_as_small_frames(lidar, n_beams, bins, select, range_mode, sun, kernel, keep):
    w = scenes.iid_frame(3)
    r = w.gbuffer.raster
    rng = np.random.default_rng(n_beams)
    az = rng.uniform(r.az_min - 4 * r.dphi, r.az_max + 4 * r.dphi, n_beams)   # some beyond the image
    el = rng.uniform(r.el_min - 4 * r.de, r.el_max + 4 * r.de, n_beams)
    w = replace(w, pattern=replace(w.pattern, beam_az=az, beam_el=el))
    params = replace(w.params, n_bins=bins, bin_ns=512.0 / bins, echo_select=select, range_mode=range_mode,
                     sun_irradiance=sun, sun_dir=(0.6, 0.0, 0.8))
    m, n = KERNELS.get(kernel, (2, 1))
    tol = max(1e-5, (2 * m + 1) * (2 * n + 1) * 2.0 ** -24)
    whole = _run(lidar, w, params, np.arange(n_beams), kernel, keep)
    for part in np.array_split(np.arange(n_beams), n_beams // 2047 + 1):
        ref = _run(lidar, w, params, part, kernel, keep)
        count = whole["n_echoes"][part]
        np.testing.assert_array_equal(count, ref["n_echoes"])
        live = np.arange(ref["echoes"].shape[1])[None] < count[:, None]
        for k in ("bin_peak", "bin_first", "bin_last", "flags", "range_m"):
            np.testing.assert_array_equal(whole["echoes"][k][part][live], ref["echoes"][k][live])
        np.testing.assert_allclose(whole["echoes"]["intensity"][part][live], ref["echoes"]["intensity"][live], rtol=tol)
        np.testing.assert_allclose(whole["beams"]["floor"][part], ref["beams"]["floor"], rtol=tol)
        if keep:
            top = ref["waveforms"].max(axis=1, keepdims=True)
            assert np.all(np.abs(whole["waveforms"][part] - ref["waveforms"]) <= tol * top)
