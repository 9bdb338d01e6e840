"""assoc_cluster on peak lists some of whose entries lie outside the grid (a caller
that strikes candidates out in place): those are no candidates, the others keep
their indices and results, whichever way the event's members are found."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from test_gpu_assoc import compare, ht, plan_for, run_gpu, run_oracle, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["narrow", "wide_few_radii", "wide_many_radii"])
@pytest.mark.parametrize("n_prompt", [120, 350])
def test_struck_out_entries(torch, ht, oracle, kind, n_prompt):  # noqa: F811
    W = CF.WORKLOADS[2]
    cfg = W["cluster"]
    ev = G.make_event(2, W["seed0"] + 70, n_prompt=n_prompt, n_noise=2 * n_prompt)
    rng = np.random.default_rng(70 + n_prompt)
    r, layer = ev.r.copy(), ev.layer.copy()
    if kind != "narrow":
        layer[rng.integers(0, r.size, 3)] = 0  # a few hits with another layer's number
    if kind == "wide_many_radii":
        r = (r.astype(np.float64) * (1.0 + 1e-3 * rng.random(r.size))).astype(np.float32)
    ev = SimpleNamespace(r=r, phi=ev.phi, layer=layer, n_hits=ev.n_hits)
    grid = W["grid"]
    print(f"{kind}: {ev.n_hits} hits", flush=True)
    _, acc, pk = run_gpu(torch, ht, grid, ev, W["min_votes"], cfg)
    cells = grid["n_phi"] * grid["n_qpt"] * grid["n_d0"]
    pk = pk.copy()
    out = rng.random(pk.shape[0]) < 0.05
    out[[0, -1]] = True
    pk[out, 0] = rng.choice([-1, -7, cells, 2**31 - 1], int(out.sum()))
    d = lambda a: torch.from_numpy(a).cuda()
    nf = torch.tensor([pk.shape[0]], dtype=torch.int32, device="cuda")
    bufs = ht.ClusterBuffers(ev.n_hits, 4096, 512, 1 << 15, cfg["n_rho"], cfg["n_theta"])
    ht.assoc_cluster(plan_for(ht, grid), d(ev.r), d(ev.phi), d(ev.layer), d(pk), nf, cfg, bufs,
                     with_vacc=True)
    torch.cuda.synchronize()
    want = run_oracle(oracle, grid, ev, acc, pk, cfg)
    compare(bufs.to_host(ev.n_hits), want, kind)
    assert want["counts"][1] > 50
