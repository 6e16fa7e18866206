"""The fused inference kernel at the edges of its row tiles, against the FP64
oracle that mirrors the BF16 roundings of operands and activations.

Tolerance: the FP32 accumulations and the BF16 activation that a rounding
boundary moves by one ulp agree to 3e-3 of the largest output, as for whole
batches.  A row's output does not depend on the rows beside it, so it is the
same bits as in the largest batch, and rows behind the last one stay as they
were."""
import numpy as np
import pytest

import scenes
from oracle import surrogate as S

pytestmark = pytest.mark.gpu

N = 321


@pytest.fixture(scope="module")
def net():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    sim = lidar.LidarSim(scenes.iid_frame(0).params, stream=torch.cuda.current_stream())
    flat = scenes.surrogate_init(11)
    p = S.unpack(flat)
    rng = np.random.default_rng(12)
    for b in ("b1", "b2", "b3", "b4"):
        p[b][:] = rng.standard_normal(p[b].shape).astype(np.float32) * np.float32(0.1)
    sim.set_weights(flat)
    bits = scenes.random_bf16_bits(13, N, scale=1.0)
    x = torch.from_numpy(bits.view(np.int16).copy()).cuda()
    ref = S.forward(scenes.bf16_bits_to_float(bits), flat, rounded=True).Y
    yield sim, x, ref
    sim.close()


def _run(sim, x, n):
    import torch
    y = torch.full((N + 64, 16), 7.0, dtype=torch.float32, device="cuda")
    sim.surrogate_forward(x[:n], y[:n])
    return y.cpu().numpy()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 192, 255, 257, N])
def test_row_tiles(net, n):
    sim, x, ref = net
    got = _run(sim, x, n)
    err = np.abs(got[:n] - ref[:n]).max()
    assert err <= 3e-3 * np.abs(ref).max(), (n, err)
    assert np.all(got[n:] == 7.0)
    np.testing.assert_array_equal(got[:n], _run(sim, x, N)[:n])
