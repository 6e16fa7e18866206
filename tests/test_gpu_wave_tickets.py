"""Batches in the wave schedule whose tickets are fewer than, as many as and more than the waves' own: every frame gives
the echoes of the same frame simulated alone.

Both routes bin and detect alike; sums differ in order or are truncated to one unit per add, each under 1e-6 of the
waveform's maximum, so 1e-5 for intensities; what is decided from bins is the same."""
from dataclasses import replace

import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bins", [512, 1200])
@pytest.mark.parametrize("counts", [(1,), (3,), (4,), (5, 1), (17, 64, 2), (2500, 1, 9000), (9000, 9000, 9000, 9000)])
def test_tickets(counts, bins):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    w = scenes.iid_frame(5)
    r = w.gbuffer.raster
    params = replace(w.params, n_bins=bins, bin_ns=512.0 / bins)
    planes = lidar.upload_gbuffer(w.gbuffer, "cuda")
    rng = np.random.default_rng(len(counts) + bins)
    pats = [replace(w.pattern, beam_az=rng.uniform(r.az_min, r.az_max, n), beam_el=rng.uniform(r.el_min, r.el_max, n),
                    sigma_deg=(1.4 * r.dphi, 1.4 * r.de)) for n in counts]
    sim = lidar.LidarSim(params, stream=torch.cuda.current_stream())
    one = lidar.LidarSim(params, stream=torch.cuda.current_stream())
    try:
        sim.simulate_batch(lidar.Batch([(r, planes)] * len(counts), pats))
        assert sim.batch_info()["wave_items"] > 0
        one.set_gbuffer(r, planes)
        for i, p in enumerate(pats):
            got = sim.read_batch(i)
            one.set_pattern(p)
            one.simulate_frame()
            ref = one.read()
            np.testing.assert_array_equal(got["n_echoes"], ref["n_echoes"])
            live = np.arange(ref["echoes"].shape[1])[None] < ref["n_echoes"][:, None]
            for k in ("bin_peak", "bin_first", "bin_last", "flags", "range_m"):
                np.testing.assert_array_equal(got["echoes"][k][live], ref["echoes"][k][live])
            np.testing.assert_allclose(got["echoes"]["intensity"][live], ref["echoes"]["intensity"][live], rtol=1e-5)
    finally:
        sim.close()
        one.close()
