"""GPU parity of the seed search on the layer runs at its edges: hits at the edge
of the road.

Every result is compared with the oracle as in test_gpu_assoc (bit-exact, the
refit to rounding)."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from test_gpu_assoc import compare, ht, run_oracle, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def event(r, phi, layer):
    r = np.concatenate(r).astype(np.float32)
    return SimpleNamespace(r=r, phi=np.concatenate(phi).astype(np.float32),
                           layer=np.concatenate(layer).astype(np.uint8), n_hits=int(r.size))


def run_small(torch, ht, grid, ev, cfg, min_votes=8):  # noqa: F811
    """Vote, peaks and assoc_cluster with a plan of a few thousand peaks; returns the
    results and the list."""
    plan = ht.Plan(grid, max_hits=8192, max_peaks=4096, max_member_cap=1024, max_tracks=4096)
    d = lambda a: torch.from_numpy(a).cuda()
    r, phi, layer = d(ev.r), d(ev.phi), d(ev.layer)
    peaks = torch.full((4096, 2), -1, dtype=torch.int32, device="cuda")
    nf = torch.zeros(1, dtype=torch.int32, device="cuda")
    acc = torch.empty(plan.acc_shape, dtype=torch.int32, device="cuda")
    ht.hough_vote(plan, r, phi, acc)
    ht.hough_peaks(plan, acc, min_votes, peaks, nf)
    bufs = ht.ClusterBuffers(ev.n_hits, 4096, 512, 1 << 15, cfg["n_rho"], cfg["n_theta"])
    ht.assoc_cluster(plan, r, phi, layer, peaks, nf, cfg, bufs, with_vacc=True)
    torch.cuda.synchronize()
    n = int(nf.item())
    assert n <= 4096
    return bufs.to_host(ev.n_hits), peaks[:n].cpu().numpy()


@pytest.mark.parametrize("part", range(4))
def test_runs_hits_at_the_roads_edge(torch, ht, oracle, part):  # noqa: F811
    """Straight tracks through the beam line with nine hits on them and one, on the
    innermost layer, at the road's edge: within it by a few millionths of the road
    up to 7e-5, or just outside.  Roads of 0.3 to 2.5 cm, wide for the layer."""
    rng = np.random.default_rng(40 + part)
    for road in np.float32(10.0 ** rng.uniform(np.log10(0.3), np.log10(2.5), 8)):
        scale = float(road) / 0.4  # the innermost layer at ten times the road
        n = 20
        phi0 = np.float32(-3.0 + 0.3 * np.arange(n) + rng.uniform(0, 0.01, n))
        inside = 4e-6 * (np.arange(n) - 2)
        phi = np.repeat(phi0[:, None], 10, axis=1)
        r = np.float32(np.array(G.RADII) * scale)
        dphi = np.arcsin(float(road) * (1.0 - inside) / float(r[0]))
        phi[:, 0] = np.float32(phi0.astype(np.float64) + dphi * rng.choice([-1.0, 1.0], n))
        ev = event([np.tile(r, n)], [phi.ravel()], [np.tile(np.arange(10), n)])
        grid = dict(CF.GRID_3D, n_phi=128, n_qpt=33, n_d0=3, d0_lo=-3.0 * scale, d0_hi=3.0 * scale)
        cfg = dict(CF.CLUSTER_3D, member_cap=1024, win_bins=6, road_sigmas=1.0,
                   sigma_rphi=float(road))
        print(f"road {road!r}", flush=True)
        got, pk = run_small(torch, ht, grid, ev, cfg)
        want = run_oracle(oracle, grid, ev, None, pk, cfg)
        compare(got, want, f"road {road!r}")
        assert np.sum(want["tracks"]["n_inliers"] == 10) >= n // 2
