"""Scores at the sizes where the forward pass's split can go wrong: a window, a
tile less and more one, one and two tiles for every workgroup; peaks on the phi0
seam, on the outer q/pT and d0 planes, and cells outside the grid."""
import numpy as np
import pytest

from oracle import cnn
from paper_1309_6275_amd import configs as CF

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1024 * 16, 1024 * 16 + 1, 3 * 1024 * 16 + 7])
def test_score_sizes(T, n):
    from paper_1309_6275_amd import houghtrig as ht
    rng = np.random.default_rng(n)
    plan = ht.Plan(CF.WORKLOADS[2]["grid"], max_peaks=1 << 16, max_member_cap=128, max_tracks=4096)
    nd, nq, nphi = plan.acc_shape
    acc = rng.integers(0, 60, plan.acc_shape).astype(np.int32)
    edge = lambda m, k: np.where(rng.uniform(size=n) < 0.3, rng.choice([0, 1, m - 2, m - 1], n),
                                 rng.integers(0, m, n)) if k else rng.integers(0, m, n)
    lin = (edge(nd, True) * nq + edge(nq, True)) * nphi + edge(nphi, n % 2)
    out = rng.uniform(size=n) < (0.01 if n > 100 else 0.0)
    lin = np.where(out, rng.choice([-1, nd * nq * nphi], n), lin).astype(np.int32)
    peaks = np.zeros((n, 2), np.int32)
    peaks[:, 0] = lin
    params = cnn.init_params(5)
    params[cnn.N_PARAMS - 1] = 0.25
    d = lambda a: T.from_numpy(a).cuda()
    acc_d, peaks_d, p = d(acc), d(peaks), d(params)
    nf = T.tensor([n], dtype=T.int32, device="cuda")
    win = T.empty((n, ht.CNN_WINDOW), dtype=T.bfloat16, device="cuda")
    ht.cnn_windows(plan, acc_d, peaks_d, nf, win)
    ws = ht.cnn_workspace(n)
    fwd = T.full((n,), np.nan, dtype=T.float32, device="cuda")
    ht.cnn_forward(p, win, fwd, ws)
    score = T.full((n,), np.nan, dtype=T.float32, device="cuda")
    ht.cnn_score(plan, p, acc_d, peaks_d, nf, score, ws)
    fwd, score = fwd.cpu().numpy(), score.cpu().numpy()
    assert np.array_equal(fwd, score)
    x = win[:4096].float().cpu().numpy()[:, :125].reshape(-1, 5, 5, 5)
    ok = ~out[:4096]
    assert np.array_equal(x[ok], cnn.windows(acc, lin[:4096][ok]))
    assert not np.any(x[~ok])
    want, _ = cnn.forward(params, x)
    # bfloat16 activations rounded from float32 here and from float64 there
    assert np.all(np.abs(score[:4096] - want) <= 2e-2 + 2e-2 * np.abs(want))


def test_forward_keeps_windows_apart(T):
    """A window that holds infinities changes no other window's logit."""
    from paper_1309_6275_amd import houghtrig as ht
    rng = np.random.default_rng(3)
    x = T.from_numpy((rng.integers(0, 40, (40, ht.CNN_WINDOW)) / 16.0).astype(np.float32))
    p = T.from_numpy(cnn.init_params(6)).cuda()
    got = []
    for bad in (False, True):
        w = x.clone()
        if bad:
            w[7, 10:20] = float("inf")
            w[16, 124:] = float("nan")
            w[31, 0] = float("-inf")
        logits = T.zeros(40, dtype=T.float32, device="cuda")
        ht.cnn_forward(p, w.to(T.bfloat16).cuda(), logits, ht.cnn_workspace(40))
        got.append(logits.cpu().numpy())
    keep = np.setdiff1d(np.arange(40), [7, 16, 31])
    assert np.array_equal(got[0][keep], got[1][keep])
