"""Single frames that the wave-per-group route takes, against the FP64 oracle: every instance (one or four output
passes, with and without sun and kept waveforms), supplied floors, the selections it takes, single beams and groups of
four, on surfaces of one-pixel runs, on a road with sky and long runs, and on a wall of one range.

The route is asserted by the engine's own rule on the frame's group count (a one-frame batch reports it)."""
from dataclasses import replace

import numpy as np
import pytest

import scenes

from . import routes
from .parity import compare, compare_selection

pytestmark = pytest.mark.gpu

# half extents in pixels
KERNELS = {"narrow": (4, 3), "wide": (6, 5), "long": (20, 1), "table": (2, 1)}


@pytest.fixture(scope="module")
def lidar():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    lidar.load()
    return lidar


def _scene(name):
    if name == "iid":
        return scenes.iid_frame(3)
    w = scenes.road_scan(0, width=2048, height=128, n_lines=4, n_cols=10)
    if name == "wall":
        w = replace(w, gbuffer=scenes.shell_gbuffer(w.gbuffer.raster, 9.7, 0.4))
    return w


def _beams(r, n, kernel, per_group):
    """n beams in pixel columns so that a group holds per_group of them: runs of neighbouring columns, a kernel's width
    between the runs; some beyond the image's sides."""
    gap = per_group + 2 * KERNELS[kernel][0] + 1
    runs = (r.width + 6 * gap) // gap
    i = np.arange(n)
    run, row = i // per_group % runs, i // per_group // runs
    assert row.max() < r.height
    u, v = run * gap - 3 * gap + i % per_group, row
    return r.az_min + (u + 0.37) * r.dphi, r.el_max - (v + 0.41) * r.de


@pytest.mark.parametrize("scene,n,per_group,bins,select,sun,kernel,keep", [
    ("iid", 4603, 1, 512, 0, 0.0, "narrow", False),
    ("road", 4603, 1, 512, 2, 0.03, "wide", True),
    ("wall", 4603, 1, 511, 0, 0.03, "narrow", False),
    ("road", 6601, 1, 512, 4, 0.0, "long", True),
    ("road", 9201, 1, 513, 0, 0.0, "narrow", False),
    ("road", 9201, 1, 1200, 0, 0.03, "wide", True),
    ("wall", 9201, 1, 1025, 2, 0.03, "narrow", False),
    ("iid", 9201, 1, 2048, 5, 0.0, "wide", True),
    ("road", 60404, 4, 2048, 0, 0.0, "narrow", False),
    ("road", 9201, 1, 2048, 0, 0.03, "table", True),
    ("iid", 30404, 4, 400, 0, 0.03, "table", False),
])
def test_wave_route(lidar, oracle_mod, scene, n, per_group, bins, select, sun, kernel, keep, range_mode=0):
    import torch
    w = _scene(scene)
    r = w.gbuffer.raster
    az, el = _beams(r, n, kernel, per_group)
    m, k = KERNELS[kernel]
    if kernel == "table":
        t = np.outer([1, 2, 1], [1, 3, 5, 3, 1]).astype(np.float32)
        pat = scenes.Pattern(scenes.PATTERN_TABLE, az, el, table=t, half_deg=(2.5 * r.dphi, 1.5 * r.de),
                             rx_table=np.sqrt(t))
    else:
        pat = scenes.Pattern(scenes.PATTERN_GAUSS, az, el, sigma_deg=((m + 0.2) / 3 * r.dphi, (k + 0.2) / 3 * r.de),
                             trunc_sigmas=3.0)
    span = w.params.n_bins * w.params.bin_ns
    params = replace(w.params, n_bins=bins, bin_ns=span / bins, echo_select=select, sun_irradiance=sun,
                     sun_dir=(0.6, 0.0, 0.8), range_mode=range_mode)
    planes = lidar.upload_gbuffer(w.gbuffer, "cuda")
    sim = lidar.LidarSim(params, stream=torch.cuda.current_stream(), keep_waveforms=keep)
    try:
        sim.simulate_batch(lidar.Batch([(r, planes)], [pat]))
        info = sim.batch_info()
        assert info["group_size"] == 4 and info["n_items"] == n // per_group + (n % per_group > 0)
        sim.set_pattern(pat)
        sim.set_gbuffer(r, planes)
        sim.simulate_frame()
        got = sim.read(waveforms=keep)
        st = sim.stats()
    finally:
        sim.close()
    assert (st["kernel_w"], st["kernel_h"]) == (2 * m + 1, 2 * k + 1)
    # (eight groups resident per CU at most: the strictest line)
    assert routes.in_waves(n, info["n_items"], 2 * m + 1, 2 * k + 1, select, range_mode, 8, 8 if bins <= 512 else 4)
    idx = np.unique(np.concatenate([np.arange(0, n, max(1, n // 1200)), np.arange(n - 40, n)]))
    part = replace(pat, beam_az=az[idx], beam_el=el[idx])
    ref = oracle_mod.simulate(w.gbuffer, part, params)
    got = {key: v[idx] if v is not None else None for key, v in got.items()}
    rep = (compare if select == 0 else compare_selection)(got, ref, params)
    assert rep.echoes_compared > 300 and rep.ambiguous < len(idx) // 4


@pytest.mark.parametrize("scene,n,per_group,bins,select,sun,kernel,keep", [
    ("road", 3103, 1, 512, 0, 0.0, "narrow", False),
    ("iid", 3103, 1, 400, 2, 0.03, "wide", True),
    ("wall", 13103, 2, 512, 0, 0.03, "narrow", False),
    ("road", 3103, 1, 511, 4, 0.0, "narrow", True),
])
def test_wave_route_of_range_intervals(lidar, oracle_mod, scene, n, per_group, bins, select, sun, kernel, keep):
    test_wave_route(lidar, oracle_mod, scene, n, per_group, bins, select, sun, kernel, keep, range_mode=2)
