"""Weight and bias gradients at row counts around the kernel's steps and shares (64 rows a step, shares of 256 rows
added with atomics), against the FP64 oracle with the same BF16 roundings.

Tolerance, of a tensor's largest magnitude: an element may meet one operand re-rounded across a BF16 boundary, at most
2^-7 of its value (seven explicit mantissa bits); FP32 accumulation adds less than 1e-3."""
import numpy as np
import pytest

import scenes
from oracle import surrogate as S

pytestmark = pytest.mark.gpu
TOL = 2.0 ** -7 + 1e-3


def _case(n, seed):
    """n rows whose loss decisions lie clear of their boundaries, and the oracle's loss and gradients on them."""
    flat = scenes.surrogate_init(seed)
    bits = scenes.random_bf16_bits(seed + 1, 2 * n + 64, scale=1.0)
    lab = scenes.random_surrogate_labels(seed + 2, 2 * n + 64)
    Y = S.forward(scenes.bf16_bits_to_float(bits), flat).Y
    keep = np.ones(len(Y), bool)
    for e in range(3):
        keep &= np.abs(Y[:, e]) > 0.05
        keep &= (lab[:, e] < 0.5) | (np.abs(np.abs(Y[:, 3 + e] - lab[:, 3 + e]) * 16.0 - 0.5) > 0.05)
    bits, lab = bits[keep][:n], lab[keep][:n]
    assert len(bits) == n
    c = S.forward(scenes.bf16_bits_to_float(bits), flat)
    L, dY = S.loss_and_grad(c.Y, lab)
    return flat, bits, lab, L, S.backward(c, dY, flat)


@pytest.mark.parametrize("n", [1, 7, 63, 64, 65, 255, 256, 257, 320, 511, 513, 1025])
@pytest.mark.parametrize("deterministic", [False, True])
def test_row_counts(n, deterministic):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    flat, bits, lab, L, ref = _case(n, n)
    sim = lidar.LidarSim(scenes.iid_frame(0).params, stream=torch.cuda.current_stream(), deterministic=deterministic)
    try:
        sim.set_weights(flat)
        # one element past an aligned address, and gradients one float past one, too
        room = torch.zeros(n * 1056 + 8, dtype=torch.int16, device="cuda")
        labd = torch.from_numpy(lab).cuda()
        for shift in (0, 1):
            x = room[shift:shift + n * 1056].view(n, 1056)
            x.copy_(torch.from_numpy(bits.view(np.int16).copy()))
            g = torch.full((S.N_PARAMS + 8,), 7.0, dtype=torch.float32, device="cuda")
            loss = torch.full((3,), 7.0, dtype=torch.float32, device="cuda")
            sim.surrogate_gradients(x, labd, g[shift:shift + S.N_PARAMS], loss[1:2])
            got = g.cpu().numpy()
            assert (got[:shift] == 7.0).all() and (got[shift + S.N_PARAMS:] == 7.0).all()
            assert loss[0].item() == 7.0 and loss[2].item() == 7.0
            assert loss[1].item() == pytest.approx(L, rel=1e-3)
            for name, _ in S.SHAPES:
                a, b = S.unpack(got[shift:shift + S.N_PARAMS].astype(np.float64))[name], S.unpack(ref)[name]
                assert np.abs(a - b).max() <= TOL * np.abs(b).max() + 1e-12, (name, shift)
    finally:
        sim.close()
