"""The line between the events whose candidates are first rejected in float32 and those
that are not (12288 candidates): lists at it, the list's capacity above it with
fewer candidates, the two passes of the queue behind it, and a batch with events on
both sides, against the oracle as in test_gpu_assoc."""
import numpy as np
import pytest

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from test_gpu_assoc import compare, ht, plan_for, run_gpu, run_oracle, torch  # noqa: F401

pytestmark = pytest.mark.gpu

LINE = 12288


def spread(pk, n):
    """n entries spread over a list (still in cell order)."""
    return np.ascontiguousarray(pk[np.linspace(0, pk.shape[0] - 1, n).astype(int)])


@pytest.fixture(scope="module")
def event(torch, ht):  # noqa: F811
    W = CF.WORKLOADS[2]
    ev = G.make_event(2, W["seed0"] + 95, n_prompt=150, n_noise=300)
    _, acc, pk = run_gpu(torch, ht, W["grid"], ev, W["min_votes"], W["cluster"])
    assert pk.shape[0] > 2 * LINE
    return ev, acc, pk


@pytest.mark.parametrize("n", [LINE - 1, LINE, LINE + 1, 2 * LINE])
@pytest.mark.parametrize("room", [0, 1, 30000])
def test_at_the_line(torch, ht, oracle, event, n, room):  # noqa: F811
    W = CF.WORKLOADS[2]
    cfg = W["cluster"]
    ev, acc, full = event
    pk = spread(full, n)
    d = lambda a: torch.from_numpy(a).cuda()
    peaks = torch.full((n + room, 2), -1, dtype=torch.int32, device="cuda")
    peaks[:n] = d(pk)
    # a count beyond the capacity, and one within it
    nf = torch.tensor([n if room else n + 5], dtype=torch.int32, device="cuda")
    bufs = ht.ClusterBuffers(ev.n_hits, 4096, 512, 1 << 15, cfg["n_rho"], cfg["n_theta"])
    ht.assoc_cluster(plan_for(ht, W["grid"]), d(ev.r), d(ev.phi), d(ev.layer), peaks, nf, cfg, bufs,
                     with_vacc=True)
    torch.cuda.synchronize()
    want = run_oracle(oracle, W["grid"], ev, acc, pk, cfg)
    compare(bufs.to_host(ev.n_hits), want, f"{n} + {room}")
    assert want["counts"][1] > 20


@pytest.mark.parametrize("min_votes", [7, 8])
def test_batch_on_both_sides(torch, ht, oracle, min_votes):  # noqa: F811
    W = CF.WORKLOADS[2]
    cfg = W["cluster"]
    cap = 1 << 18
    evs = [G.make_event(2, W["seed0"] + 96 + b, n_prompt=n, n_noise=n) for b, n in
           enumerate((20, 150, 60, 240))]
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
    ht.hough_batch(events, n_max, min_votes, cfg, with_vacc=True)
    torch.cuda.synchronize()
    counts = [int(e["nf"].item()) for e in events]
    assert min(counts) < LINE <= max(counts) <= cap, counts
    for b, (e, ev) in enumerate(zip(events, evs)):
        want = run_oracle(oracle, W["grid"], ev, None, e["peaks"][:counts[b]].cpu().numpy(), cfg)
        compare(e["bufs"].to_host(ev.n_hits), want, f"event {b}: {counts[b]}")
