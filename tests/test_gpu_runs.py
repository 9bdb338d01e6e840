"""GPU parity of the seed search on the layer runs, at the sizes where its paths
meet: candidate lists around the size that skips the float32 rejection, layers
whose radii spread up to and beyond what the runs take, runs across +-pi, runs
longer than one stage and than the member bits, and hits that tie.

Every result is compared with the oracle as in test_gpu_assoc (bit-exact, the
refit to rounding)."""
import numpy as np
import pytest

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from test_gpu_assoc import compare, ht, run_gpu, run_oracle, torch  # noqa: F401

pytestmark = pytest.mark.gpu


def check(torch, ht, oracle, grid, ev, cfg, label, min_votes=7, **kw):  # noqa: F811
    print(f"{label}: {ev.n_hits} hits", flush=True)
    got, acc, pk = run_gpu(torch, ht, grid, ev, min_votes, cfg, **kw)
    want = run_oracle(oracle, grid, ev, acc, pk, cfg)
    compare(got, want, label)
    return want, pk


def merge(ev, r, phi, layer):
    """ev with the hits (r, phi, layer) appended."""
    ev.r = np.concatenate([ev.r, np.asarray(r, np.float32)])
    ev.phi = np.concatenate([ev.phi, np.asarray(phi, np.float32)])
    ev.layer = np.concatenate([ev.layer, np.asarray(layer, np.uint8)])
    return ev


@pytest.mark.parametrize("n_peaks", [1, 63, 4095, 4096, 4097, 70001])
def test_runs_candidate_counts(torch, ht, oracle, n_peaks):  # noqa: F811
    W = CF.WORKLOADS[2]
    ev = G.make_event(2, W["seed0"] + 31)
    check(torch, ht, oracle, W["grid"], ev, W["cluster"], f"{n_peaks} peaks", peak_cap=n_peaks)


@pytest.mark.parametrize("spread", [1e-7, 0.02, 0.11, 0.24, 0.26])
def test_runs_radius_spread(torch, ht, oracle, spread):  # noqa: F811
    """Each layer's radii between r and r (1 + spread): the last one's layers are
    too wide for the runs."""
    W = CF.WORKLOADS[2]
    ev = G.make_event(2, W["seed0"] + 32, n_prompt=100, n_noise=150)
    rng = np.random.default_rng(int(spread * 1e7))
    ev.r = (ev.r.astype(np.float64) * (1.0 + spread * rng.random(ev.n_hits))).astype(np.float32)
    cfg = dict(W["cluster"], road_sigmas=60.0, min_layers=5)
    want, _ = check(torch, ht, oracle, W["grid"], ev, cfg, f"spread {spread}", peak_stride=9)
    assert want["counts"][0] > 0


@pytest.mark.parametrize("cap", [128, 1024])
def test_runs_across_pi(torch, ht, oracle, cap):  # noqa: F811
    """Tracks that leave along phi = +-pi, with hits at float(pi) and -float(pi)
    and azimuths written one turn apart."""
    rng = np.random.default_rng(7)
    tracks = [(np.pi + rng.normal(0, 0.02), rng.uniform(-0.6, 0.6), rng.uniform(-3, 3))
              for _ in range(60)]
    ev = G.make_tracks_event(tracks, n_noise=400, seed=8)
    n = len(G.RADII)
    pi = np.float32(np.pi)
    ev = merge(ev, list(G.RADII) * 2, [pi] * n + [-pi] * n, list(range(n)) * 2)
    far = np.flatnonzero(ev.phi < -2.6)[::3]
    ev.phi[far] = (ev.phi[far].astype(np.float64) + 2 * np.pi).astype(np.float32)
    W = CF.WORKLOADS[2]
    cfg = dict(W["cluster"], member_cap=cap)
    want, _ = check(torch, ht, oracle, W["grid"], ev, cfg, f"pi {cap}")
    assert want["counts"][1] > 5


@pytest.mark.parametrize("n", [60, 130, 250, 270, 600])
def test_runs_long_and_tied(torch, ht, oracle, n):  # noqa: F811
    """n hits of one layer inside the windows of a group of tracks, a third of
    them at one azimuth: runs beyond the two hits per lane of the ranking, the
    staged hits and the list of a short candidate, with ties of every kind."""
    rng = np.random.default_rng(n)
    tracks = [(0.3 + rng.normal(0, 0.004), rng.uniform(-0.05, 0.05), rng.normal(0, 0.3))
              for _ in range(12)]
    ev = G.make_tracks_event(tracks, n_noise=200, seed=n)
    for li in (2, 7):
        r = G.RADII[li]
        phi = 0.3 + rng.uniform(-0.02, 0.02, n)
        phi[:n // 3] = np.float32(0.3)
        ev = merge(ev, [r] * n, phi, [li] * n)
    W = CF.WORKLOADS[2]
    cfg = dict(W["cluster"], member_cap=1024, seed_k=4)
    want, pk = check(torch, ht, oracle, W["grid"], ev, cfg, f"pile {n}", peak_stride=5)
    assert want["counts"][0] > 0


def test_runs_beyond_the_member_bits(torch, ht, oracle):  # noqa: F811
    """Layers of several radii whose cells reach |u| = 1: the interval is the whole
    circle, more hits than the member bits hold, few of them members."""
    rng = np.random.default_rng(12)
    ev = G.make_event(2, 2_000_333, n_prompt=60, n_noise=200)
    n = 4500
    ev = merge(ev, rng.uniform(11.0, 12.0, n), rng.uniform(-np.pi, np.pi, n), [2] * n)
    W = CF.WORKLOADS[2]
    cfg = dict(W["cluster"], member_cap=1024, min_layers=4)
    grid = dict(W["grid"], n_phi=256, n_qpt=64, n_d0=32)
    check(torch, ht, oracle, grid, ev, cfg, "whole circle", min_votes=9, peak_stride=37)
