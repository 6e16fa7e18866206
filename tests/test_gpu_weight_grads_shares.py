"""Weight and bias gradients above 64 shares of 256 rows, where a share grows and the last one is short: the last row,
or the first of the last share, has a label so far off that its gradient outweighs all others together, so that the
gradients lose nearly everything if it is left out.  Tolerance as for fewer rows: 2^-7 of a tensor's largest element
for an operand re-rounded across a BF16 boundary, 1e-3 for FP32 sums."""
import numpy as np
import pytest

import scenes
from oracle import surrogate as S

pytestmark = pytest.mark.gpu
TOL = 2.0 ** -7 + 1e-3


@pytest.mark.parametrize("n,row", [(16385, 16384), (16385, 16320), (20001, 20000), (20001, 19840), (20480, 20479)])
def test_rows_of_the_last_share(n, row):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_05932_amd as lidar
    span = (-(-n // 64) + 63) // 64 * 64
    assert n > 64 * 256 and (row == n - 1 or row == (n - 1) // span * span)
    flat = scenes.surrogate_init(5)
    bits, lab = scenes.random_bf16_bits(6, n, scale=1.0), scenes.random_surrogate_labels(7, n)
    lab[row, 0], lab[row, 3] = 1.0, 1e6
    c = S.forward(scenes.bf16_bits_to_float(bits), flat)
    L, dY = S.loss_and_grad(c.Y, lab)
    ref = S.backward(c, dY, flat)
    one = np.zeros_like(dY)
    one[row] = dY[row]
    alone = S.backward(c, one, flat)
    sim = lidar.LidarSim(scenes.iid_frame(0).params, stream=torch.cuda.current_stream())
    try:
        sim.set_weights(flat)
        g, loss = torch.full((S.N_PARAMS,), 7.0, device="cuda"), torch.full((1,), 7.0, device="cuda")
        x = torch.from_numpy(bits.view(np.int16).copy()).cuda()
        sim.surrogate_gradients(x, torch.from_numpy(lab).cuda(), g, loss)
        got = g.cpu().numpy().astype(np.float64)
    finally:
        sim.close()
    assert loss.item() == pytest.approx(L, rel=1e-3)
    for name, _ in S.SHAPES:
        a, b, o = (S.unpack(v)[name] for v in (got, ref, alone))
        assert np.abs(o - b).max() <= 0.05 * np.abs(b).max(), name      # nearly all of it is that row's
        assert np.abs(a - b).max() <= TOL * np.abs(b).max(), name
