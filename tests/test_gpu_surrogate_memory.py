"""The surrogate's calls at what a caller may rely on besides the values: the deterministic mode's loss repeats bit for
bit where one workgroup sums it, and inference allocates nothing that only training uses."""
import numpy as np
import pytest

import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lidar():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    lidar.load()
    return lidar


@pytest.mark.parametrize("n", [129, 200, 256])
def test_deterministic_loss_repeats(lidar, n):
    import torch
    sim = lidar.LidarSim(scenes.iid_frame(0).params, stream=torch.cuda.current_stream(), deterministic=True)
    try:
        sim.set_weights(scenes.surrogate_init(3))
        x = torch.from_numpy(scenes.random_bf16_bits(n, n, scale=1.0).view(np.int16)).cuda()
        lab = torch.from_numpy(scenes.random_surrogate_labels(n + 1, n)).cuda()
        g = torch.empty(lidar._binding.SUR_PARAMS, device="cuda")
        losses = torch.empty(400, device="cuda")
        for i in range(len(losses)):
            sim.surrogate_gradients(x, lab, g, losses[i:i + 1])
        got = losses.cpu().numpy()
        assert (got == got[0]).all(), np.unique(got)
    finally:
        sim.close()


@pytest.mark.parametrize("frame", [False, True])
def test_inference_allocates_no_training_workspace(lidar, frame):
    """The activations and gradients of a training step take 7.2 KB a row.  A forward pass writes the caller's outputs;
    a surrogate frame holds its inputs and outputs (2.2 KB a beam), its results and its records (less than 1 KB)."""
    import torch
    if frame:
        w = scenes.road_scan(0, width=2048, height=128, n_lines=40, n_cols=400)
        n, most = w.pattern.n_beams, 3200
        planes = lidar.upload_gbuffer(w.gbuffer, "cuda")
    else:
        w, n, most = scenes.iid_frame(0), 40000, 100
        x = torch.zeros((n, 1056), dtype=torch.int16, device="cuda")
        y = torch.zeros((n, 16), device="cuda")
    sim = lidar.LidarSim(w.params, stream=torch.cuda.current_stream())
    try:
        sim.set_weights(scenes.surrogate_init(3))
        if frame:
            sim.set_pattern(w.pattern)
            sim.set_gbuffer(w.gbuffer.raster, planes)
            sim.simulate_frame()
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        if frame:
            sim.simulate_frame(mode=lidar.LIDAR_MODE_SURROGATE)
        else:
            sim.surrogate_forward(x, y)
        torch.cuda.synchronize()
        used = before - torch.cuda.mem_get_info()[0]
        assert used < most * n + (24 << 20), (used, n)
    finally:
        sim.close()
