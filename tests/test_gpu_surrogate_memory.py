"""The surrogate's calls at what a caller may rely on besides the values: the deterministic mode's loss repeats bit for
bit where one workgroup sums it."""
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
