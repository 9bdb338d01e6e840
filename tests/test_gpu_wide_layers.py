"""Events with a layer of widely spread radii: member lists by radius class (at most 16
distinct radii among the member-eligible hits) and the sweep (more), beside events
on the layer runs, against the oracle as in test_gpu_assoc."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from test_gpu_assoc import compare, ht, run_gpu, run_oracle, torch  # noqa: F401

pytestmark = pytest.mark.gpu

SHELLS = np.array([0, 0, 1, 2, 2, 3, 4, 5, 6, 7], np.uint8)  # 4 and 7 cm, 22 and 30 cm share a number


def widen(ev, kind, seed):
    rng = np.random.default_rng(seed)
    r, phi, layer = ev.r.copy(), ev.phi.copy(), ev.layer.copy()
    if kind == "stray":
        layer[rng.integers(0, r.size)] = 0
        layer[rng.integers(0, r.size)] = 9
    elif kind == "shells":
        layer = SHELLS[layer]
    elif kind in ("16 radii", "17 radii", "16 radii and voters"):
        n = 7 if kind == "17 radii" else 6
        new = np.float32(rng.uniform(12.0, 100.0, n))
        r = np.concatenate([r, new, new])
        phi = np.concatenate([phi, rng.uniform(-np.pi, np.pi, 2 * n)])
        layer = np.concatenate([layer, np.zeros(n), np.full(n, 9)])
        if kind == "16 radii and voters":  # valid hits beyond the layer range: no members
            r = np.concatenate([r, rng.uniform(5.0, 90.0, 40)])
            phi = np.concatenate([phi, rng.uniform(-np.pi, np.pi, 40)])
            layer = np.concatenate([layer, rng.integers(16, 256, 40)])
    elif kind == "smeared":
        r = r.astype(np.float64) * (1.0 + 1e-3 * rng.random(r.size))
        layer[rng.integers(0, r.size)] = 0
    return SimpleNamespace(r=r.astype(np.float32), phi=phi.astype(np.float32),
                           layer=layer.astype(np.uint8), n_hits=int(r.size))


KINDS = ("stray", "shells", "16 radii", "16 radii and voters", "17 radii", "smeared")


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n_prompt,cap", [(100, 128), (320, 128), (320, 1024)])
def test_wide_layers(torch, ht, oracle, kind, n_prompt, cap):  # noqa: F811
    """Below and above the hit count of the one-launch sort, on the displaced grid."""
    W = CF.WORKLOADS[2]
    cfg = dict(W["cluster"], member_cap=cap, min_layers=6 if kind == "shells" else 7)
    ev = widen(G.make_event(2, W["seed0"] + 80, n_prompt=n_prompt, n_noise=n_prompt), kind, n_prompt)
    print(f"{kind}: {ev.n_hits} hits", flush=True)
    got, acc, pk = run_gpu(torch, ht, W["grid"], ev, 7, cfg, use_acc=kind != "stray")
    want = run_oracle(oracle, W["grid"], ev, acc, pk, cfg)
    compare(got, want, kind)
    assert want["counts"][1] > 50


@pytest.mark.parametrize("kind", KINDS)
def test_wide_layers_over_the_cap(torch, ht, oracle, kind):  # noqa: F811
    """Lists that end at the cap, candidates beyond it, and runs across +-pi."""
    W = CF.WORKLOADS[2]
    base = G.make_event(2, W["seed0"] + 81, n_prompt=500, n_noise=1500)
    base = SimpleNamespace(r=base.r, phi=base.phi, layer=base.layer, n_hits=base.n_hits)
    far = np.flatnonzero(base.phi < -2.6)[::3]
    base.phi[far] = (base.phi[far].astype(np.float64) + 2 * np.pi).astype(np.float32)
    ev = widen(base, kind, 5)
    cfg = dict(W["cluster"], member_cap=96, min_layers=6 if kind == "shells" else 7)
    print(f"{kind}: {ev.n_hits} hits", flush=True)
    got, acc, pk = run_gpu(torch, ht, W["grid"], ev, 7, cfg, peak_stride=3)
    want = run_oracle(oracle, W["grid"], ev, acc, pk, cfg)
    compare(got, want, kind)
    assert want["counts"][4] > 100 and want["counts"][1] > 5


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n_prompt", [20, 400])
def test_wide_layers_prompt_grid(torch, ht, oracle, kind, n_prompt):  # noqa: F811
    """The prompt grid: few column tiles, the hits in slices, the beam-line seed."""
    W = CF.WORKLOADS[1]
    cfg = dict(W["cluster"], min_layers=6 if kind == "shells" else 8)
    ev = widen(G.make_event(1, W["seed0"] + 80, n_prompt=n_prompt, n_noise=2 * n_prompt), kind, 7)
    print(f"{kind}: {ev.n_hits} hits", flush=True)
    got, acc, pk = run_gpu(torch, ht, W["grid"], ev, W["min_votes"], cfg)
    want = run_oracle(oracle, W["grid"], ev, acc, pk, cfg)
    compare(got, want, kind)
    assert want["counts"][1] >= 15


@pytest.mark.parametrize("n_prompt", [60, 250])
def test_wide_layers_in_a_batch(torch, ht, oracle, n_prompt):  # noqa: F811
    """Events of every way in one batch."""
    W = CF.WORKLOADS[2]
    cfg = W["cluster"]
    cap = 1 << 18
    evs = [widen(G.make_event(2, W["seed0"] + 82 + b, n_prompt=n_prompt, n_noise=n_prompt), kind, b)
           for b, kind in enumerate(("narrow", "stray", "smeared", "16 radii"))]
    n_max = max(e.n_hits for e in evs)
    pad = lambda a: np.concatenate([a, np.zeros(n_max - a.size, a.dtype)])
    d = lambda a: torch.from_numpy(a).cuda()
    events = []
    for e in evs:
        plan = ht.Plan(W["grid"], max_hits=n_max, max_peaks=cap, max_member_cap=128, max_tracks=4096)
        events.append(dict(plan=plan, r=d(pad(e.r)), phi=d(pad(e.phi)), layer=d(pad(e.layer)),
                           n_dev=torch.tensor([e.n_hits], dtype=torch.int32, device="cuda"),
                           acc=torch.zeros(plan.acc_shape, dtype=torch.int32, device="cuda"),
                           peaks=torch.zeros((cap, 2), dtype=torch.int32, device="cuda"),
                           nf=torch.zeros(1, dtype=torch.int32, device="cuda"),
                           bufs=ht.ClusterBuffers(n_max, 4096, 512, 1 << 15, cfg["n_rho"],
                                                  cfg["n_theta"])))
    ht.hough_batch(events, n_max, 7, cfg, with_vacc=True)
    torch.cuda.synchronize()
    for b, (e, ev) in enumerate(zip(events, evs)):
        n = int(e["nf"].item())
        assert n <= cap
        want = run_oracle(oracle, W["grid"], ev, None, e["peaks"][:n].cpu().numpy(), cfg)
        compare(e["bufs"].to_host(ev.n_hits), want, f"event {b}")
        assert want["counts"][1] > 20
