"""One training step of the peak filter at the sizes where its split over
windows can go wrong: a single window, a tile less and more one, one tile for
every workgroup of the backward pass, and several tiles with a ragged tail."""
import numpy as np
import pytest

from oracle import cnn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 16 * 128, 16 * 128 + 33])
def test_train_step_sizes(n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1309_6275_amd import houghtrig as ht
    rng = np.random.default_rng(100 + n)
    x = np.zeros((n, ht.CNN_WINDOW), np.float32)
    x[:, :125] = rng.integers(0, 40, (n, 125)) / 16.0  # exact in bfloat16
    labels = (rng.uniform(size=n) < 0.3).astype(np.float32)
    params = cnn.init_params(7)
    mom = rng.normal(0, 1e-3, cnn.N_PARAMS).astype(np.float32)
    lr, mu, pw = 0.05, 0.9, 3.0
    loss_w, g_w, _ = cnn.loss_and_grad(params, x[:, :125].reshape(-1, 5, 5, 5), labels, pw)
    win = torch.from_numpy(x).to(torch.bfloat16).cuda()
    lab = torch.from_numpy(labels).cuda()
    ws = ht.cnn_workspace(n, training=True)
    for _ in range(2):  # the workspace of the first step carries nothing into the second
        p = torch.from_numpy(params).cuda()
        m = torch.from_numpy(mom).cuda()
        loss = torch.full((1,), 5.0, dtype=torch.float32, device="cuda")
        ht.cnn_train_step(p, m, win, lab, lr, mu, pw, loss, ws)
        torch.cuda.synchronize()
        assert abs(loss.item() - loss_w) <= 1e-3 * abs(loss_w) + 1e-6
        g_got = m.cpu().numpy().astype(np.float64) - mu * mom
        scale = np.abs(g_w).max()
        # bfloat16 activations and signals, rounded from float32 here and from
        # float64 there: a step of 2^-8 in single terms of a sum
        assert np.abs(g_got - g_w).max() <= 2e-2 * scale
