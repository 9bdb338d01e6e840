"""Peaks where a workgroup walks its rows along d0 and a wave emits a tile: one,
two, four and eight planes a workgroup with a ragged last group, rows of one,
two and four waves, plateaus and negative counts, against the oracle."""
import numpy as np
import pytest

from test_gpu_vote_peaks import gpu_peaks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def T():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("n_phi,n_qpt,n_d0", [(512, 64, 1), (512, 64, 2), (1024, 40, 67),
                                              (256, 256, 75), (512, 128, 131), (1024, 3, 5)])
@pytest.mark.parametrize("lo,hi,thr", [(0, 7, 1), (0, 3, 2), (-6, 2, -5)])
def test_peaks_walk(T, oracle, n_phi, n_qpt, n_d0, lo, hi, thr):
    from paper_1309_6275_amd import houghtrig as ht
    g = dict(n_phi=n_phi, n_qpt=n_qpt, n_d0=n_d0, qpt_lo=-1.0, qpt_hi=1.0, d0_lo=-20.0,
             d0_hi=20.0, bfield=3.8)
    rng = np.random.default_rng(n_phi + n_d0 + hi)
    acc = rng.integers(lo, hi, (n_d0, n_qpt, n_phi)).astype(np.int32)
    want, n_w = oracle.hough_peaks(g, acc, thr)
    for cap in (n_w + 3, n_w // 2):
        pk, n = gpu_peaks(T, ht, g, T.from_numpy(acc).cuda(), thr, cap)
        assert n == n_w
        m = min(cap, n_w)
        assert np.array_equal(pk[:m, 0], want["lin"][:m])
        assert np.array_equal(pk[:m, 1], want["votes"][:m])
