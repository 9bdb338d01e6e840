"""Performance cases of the trigger path: what a user of this package has it do,
called through the package's public entry points.

Families (a case names one under ``"family"``):

* ``event``    one event through hough_vote, hough_peaks and assoc_cluster, the
               path every program of this package runs, on the 2D prompt grid,
               the 3D displaced grid or any other grid;
* ``two_pass`` iterative hit removal (prompt pass, hits removed, displaced pass);
* ``batch``    up to four small events in one launch per kernel (hough_batch);
* ``band``     the band vote and the peaks of its accumulator;
* ``filter``   the learned peak filter: scores of a peak list and the kept list;
* ``train``    one training step of that filter;
* ``server``   the serving loop: host events submitted, results collected.

Sizes follow the package's workload definitions, its tests' grids and its
benchmark; events come from its generator.
"""
import math

import numpy as np
import torch

from paper_1309_6275_amd import configs as CF
from paper_1309_6275_amd import eventgen as G
from paper_1309_6275_amd import houghtrig as H
from paper_1309_6275_amd import iterative

GRIDS = {"2d": CF.GRID_2D, "3d": CF.GRID_3D}
# clustering settings by name: the workloads' own, the serving loop's 3D kind
# (a cap of 256 members) and the paper's toy detector (many tracks: cap 1024)
CLUSTERS = {"2d": CF.CLUSTER_2D, "3d": CF.CLUSTER_3D, "3d_dense": CF.CLUSTER_3D_DENSE,
            "3d_serving": dict(CF.CLUSTER_3D, member_cap=256),
            "toy": CF.CLUSTER_PAPER, "toy_dense": dict(CF.CLUSTER_PAPER, member_cap=1024)}
MIN_VOTES = {"2d": 8, "3d": 7}


def listed():
    return [
        # the smallest call: one prompt event of 20 tracks on the 2D grid, where
        # launches and host work are what a trigger waits for
        dict(name="prompt_2d_250", family="event", grid="2d", cluster="2d", events="prompt",
             hits=250, log2_peaks=16),
        # the displaced-jet workload, the ordinary event (benchmark, smoke tests)
        dict(name="jets_3d_3600", family="event", grid="3d", cluster="3d", events="jets", hits=3600,
             log2_peaks=19),
        # the high-pileup workload, the benchmark's default and the largest event
        dict(name="pileup_3d_55k", family="event", grid="3d", cluster="3d_dense", events="pileup",
             hits=55000, log2_peaks=21),
        # a large trigger event at the serving loop's member cap: most candidates
        # hold more members than the cap and the accumulator says so beforehand
        dict(name="trigger_3d_31k", family="event", grid="3d", cluster="3d_serving", events="jets",
             hits=31000, log2_peaks=21, with_acc=True),
        # the paper's toy detector with 3000 tracks of ten hits: every hit has
        # its own radius (x and y are smeared), as in its third efficiency study
        dict(name="toy_3d_3000_tracks", family="event", grid="3d", cluster="toy_dense", events="toy",
             hits=30000, log2_peaks=21),
        # another detector's grid (no power of two) with the other options: Kalman
        # refit and vertex votes on both branches
        dict(name="kalman_500x120x24", family="event", grid="500x120x24", cluster="3d", events="jets",
             hits=1500, log2_peaks=19, fit_kind=1, two_branch=1),
        # iterative hit removal on the displaced-jet workload
        dict(name="two_pass_3600", family="two_pass", hits=3600),
        # a full batch of small 3D events, as the serving loop forms under load
        dict(name="batch4_3d_2500", family="batch", grid="3d", events=4, hits=2500),
        # the band vote on the displaced-jet event
        dict(name="band_3d_3600", family="band", grid="3d", hits=3600),
        # the learned filter on a peak list the size of the displaced-jet event's
        dict(name="filter_3d", family="filter", grid="3d", mean_votes=5.6, min_votes=7),
        # one step of the filter's training at its default batch
        dict(name="filter_train_4096", family="train", windows=4096),
        # a burst of mixed events through the serving loop, from host memory
        dict(name="server_6_mixed", family="server", events=6, lo=2000, hi=16000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same families and ranges."""
    family = rng.choice(["event"] * 7 + ["two_pass", "batch", "band", "filter", "train", "server"])
    if family == "event":
        kind = rng.choice(["2d", "jets", "pileup", "trigger", "toy", "grid"])
        if kind == "2d":
            return dict(family=family, grid="2d", cluster="2d", events="prompt",
                        hits=_log(rng, 60, 55000), log2_peaks=16, fit_kind=rng.randrange(2))
        if kind == "jets":
            return dict(family=family, grid="3d", cluster="3d", events="jets",
                        hits=_log(rng, 500, 5000), log2_peaks=19, with_acc=rng.random() < 0.5)
        if kind == "pileup":
            return dict(family=family, grid="3d", cluster="3d_dense", events="pileup",
                        hits=_log(rng, 5000, 50000), log2_peaks=21)
        if kind == "trigger":
            return dict(family=family, grid="3d", cluster="3d_serving", events="jets",
                        hits=_log(rng, 2000, 55000), log2_peaks=21, with_acc=True)
        if kind == "toy":
            n = _log(rng, 300, 25000)
            return dict(family=family, grid="3d", cluster="toy_dense" if n > 4000 else "toy",
                        events="toy", hits=n, log2_peaks=21)
        grid = "%dx%dx%d" % (rng.choice([200, 243, 250, 256, 384, 500, 512]), rng.randint(40, 256),
                             rng.choice([1, 3, 8, 24, 33, 64]))
        return dict(family=family, grid=grid, cluster="3d", events="jets", hits=_log(rng, 300, 3600),
                    log2_peaks=19, fit_kind=rng.randrange(2), two_branch=rng.randrange(2))
    if family == "two_pass":
        return dict(family=family, hits=_log(rng, 400, 12000))
    if family == "batch":
        return dict(family=family, grid=rng.choice(["2d", "3d"]), events=rng.randint(2, 4),
                    hits=_log(rng, 250, 8000))
    if family == "band":
        return dict(family=family, grid=rng.choice(["2d", "3d", "500x120x24", "243x77x9"]),
                    hits=_log(rng, 250, 20000))
    if family == "filter":
        return dict(family=family, grid=rng.choice(["2d", "3d", "250x130x24"]),
                    mean_votes=round(rng.uniform(3.0, 9.0), 2), min_votes=rng.randint(6, 9))
    if family == "train":
        return dict(family=family, windows=_log(rng, 100, 8192))
    lo = _log(rng, 500, 8000)
    return dict(family=family, events=rng.randint(2, 6), lo=lo, hi=lo * 2)


# ---- inputs -------------------------------------------------------------------

def _grid(name):
    if name in GRIDS:
        return dict(GRIDS[name])
    n_phi, n_qpt, n_d0 = (int(v) for v in name.split("x"))
    d = 0.0 if n_d0 == 1 else 20.0
    return dict(CF.GRID_3D, n_phi=n_phi, n_qpt=n_qpt, n_d0=n_d0, d0_lo=-d, d0_hi=d)


def _min_votes(grid):
    return MIN_VOTES["2d" if grid["n_d0"] == 1 else "3d"]


def _event(kind, hits, seed):
    """A generated event of about `hits` hits: the compositions of the
    package's workloads, scaled by their prompt tracks and noise hits."""
    if kind == "prompt":
        noise = int(0.2 * hits)
        return G.make_event(1, seed, n_prompt=max(1, round((hits - noise) / 10.0)), n_noise=noise)
    if kind == "jets":
        noise = int(0.14 * hits)
        return G.make_event(2, seed, n_prompt=max(1, round((hits - noise - 160) / 9.7)), n_noise=noise)
    if kind == "pileup":
        noise = int(0.09 * hits)
        return G.make_event(3, seed, n_prompt=max(1, round((hits - noise - 900) / 9.7)), n_noise=noise)
    if kind == "toy":
        return G.make_paper_event(seed, n_prompt=max(0, hits // 10 - 20), n_jets=2, jet_ntrk=10)
    raise ValueError(kind)


def _upload(ev):
    return dict(r=torch.from_numpy(ev.r).cuda(), phi=torch.from_numpy(ev.phi).cuda(),
                layer=torch.from_numpy(ev.layer).cuda())


def _room(hits):
    """Hits that an event generated for about `hits` of them is given room for."""
    return min(65535, hits + hits // 8 + 512)


def _buffers(n_hits, cl, track_cap=1 << 14, object_cap=1024, member_cap=1 << 16):
    bufs = H.ClusterBuffers(n_hits, track_cap, object_cap, member_cap, cl["n_rho"], cl["n_theta"])
    bufs.hit_owner.fill_(-1)
    return bufs


def _cluster_outputs(b):
    """A ClusterBuffers' tensors, the track and object records split into
    their integer and floating fields (views).  The seed search's count of the
    distances it happened to compute (``work``, which the roofline figures
    read) is a measurement of the search and no result: it is left out."""
    ft, fo = b.tracks.view(torch.float32), b.objects.view(torch.float32)
    return dict(counts=b.counts, owner=b.hit_owner, members=b.members, vacc=b.vacc,
                track_head=b.tracks[:, :7], track_fit=ft[:, 7:13], track_hits=b.tracks[:, 13:],
                object_head=b.objects[:, :4], object_place=fo[:, 4:7], object_begin=b.objects[:, 7:])


def _record_views(o):
    """The same split of host results (structured records)."""
    t, b = (o[k].view(np.int32).reshape(o[k].size, -1) for k in ("tracks", "objects"))
    return dict(counts=o["counts"], owner=o["owner"], members=o["members"], track_head=t[:, :7],
                track_fit=t[:, 7:13].view(np.float32), track_hits=t[:, 13:], object_head=b[:, :4],
                object_place=b[:, 4:7].view(np.float32), object_begin=b[:, 7:])


def _filter_params(rng):
    """He-scaled normal weights and small biases in the flat layout of the
    filter's parameters."""
    parts = []
    for n, fan_in in ((16 * 27, 27), (16, 0), (16 * 16 * 27, 432), (16, 0), (64 * 16, 16), (64, 0),
                      (64, 64), (1, 0)):
        s = math.sqrt(2.0 / fan_in) if fan_in else 0.05
        parts.append(rng.normal(0.0, s, n))
    return np.concatenate(parts).astype(np.float32)


def _filter_inputs(case, seed):
    """Parameters, an accumulator of Poisson votes and the list of its local
    maxima at or above the threshold (cell order)."""
    rng = np.random.default_rng([seed, 41])
    g = _grid(case["grid"])
    params = _filter_params(rng)
    acc = rng.poisson(case["mean_votes"], (g["n_d0"], g["n_qpt"], g["n_phi"])).astype(np.int32)
    a = torch.from_numpy(acc).float()[None]
    a = torch.nn.functional.pad(a, (1, 1, 0, 0, 0, 0), mode="circular")
    top = torch.nn.functional.max_pool3d(a, 3, stride=1, padding=(1, 1, 0))[0].numpy()
    lin = np.flatnonzero((acc >= case["min_votes"]) & (acc >= top)).astype(np.int32)
    peaks = np.stack([lin, acc.reshape(-1)[lin]], axis=1).astype(np.int32)
    return g, params, acc, peaks


def _train_inputs(case, seed):
    """Parameters, momentum and labelled windows: Poisson votes around a peak
    cell, a ridge through the centre of the positive ones."""
    rng = np.random.default_rng([seed, 43])
    n = case["windows"]
    params = _filter_params(rng)
    mom = rng.normal(0.0, 1e-3, params.size).astype(np.float32)
    labels = (rng.random(n) < 0.08).astype(np.float32)
    labels[0] = 1.0
    votes = rng.poisson(5.6, (n, 5, 5, 5))
    votes[:, 2, 2, 2] = 7 + rng.poisson(1.0, n)
    for d in range(5):  # (dk, dj, di): d0 and q/pT trade against phi0 along a track's ridge
        votes[:, d, 2, d] += (labels * rng.poisson(3.0, n)).astype(votes.dtype)
    win = np.zeros((n, H.CNN_WINDOW), np.float32)
    win[:, :125] = votes.reshape(n, 125) / 16.0
    return params, mom, labels, torch.from_numpy(win).to(torch.bfloat16)


def _server_events(case, seed):
    rng = np.random.default_rng([seed, 47])
    out = []
    for e in range(case["events"]):
        n = int(rng.integers(case["lo"], case["hi"] + 1))
        out.append((e % 2, _event("jets" if e % 2 else "prompt", n, seed * 64 + e)))
    return out


# ---- cases --------------------------------------------------------------------

def prepare(case, seed):
    family = case["family"]
    if family == "event":
        g = _grid(case["grid"])
        cl = dict(CLUSTERS[case["cluster"]], fit_kind=case.get("fit_kind", 0),
                  vtx_two_branch=case.get("two_branch", 0))
        cap = 1 << case["log2_peaks"]
        ev = _event(case["events"], case["hits"], seed)
        plan = H.Plan(g, max_hits=65535, max_peaks=cap, max_member_cap=cl["member_cap"],
                      max_tracks=1 << 14)
        s = dict(_upload(ev), plan=plan, cl=cl, min_votes=_min_votes(g),
                 acc=torch.zeros(plan.acc_shape, dtype=torch.int32, device="cuda"),
                 peaks=torch.zeros((cap, 2), dtype=torch.int32, device="cuda"),
                 nf=torch.zeros(1, dtype=torch.int32, device="cuda"),
                 bufs=_buffers(_room(case["hits"]), cl))
        s["given_acc"] = s["acc"] if case.get("with_acc") else None
        s["out"] = dict(_cluster_outputs(s["bufs"]), acc=s["acc"], peaks=s["peaks"], n_peaks=s["nf"])
    elif family == "two_pass":
        ev = _event("jets", case["hits"], seed)
        tp = iterative.TwoPass(max_hits=_room(case["hits"]))
        for t in (tp.pk_p, tp.pk_d, tp.keep):
            t.zero_()
        tp.bufs_p.hit_owner.fill_(-1)
        tp.bufs_d.hit_owner.fill_(-1)
        s = dict(_upload(ev), tp=tp)
        s["out"] = dict(first=_cluster_outputs(tp.bufs_p), second=_cluster_outputs(tp.bufs_d),
                        keep=tp.keep, n_keep=tp.n_keep, n_peaks=tp.nf, first_peaks=tp.pk_p,
                        second_peaks=tp.pk_d, first_acc=tp.acc_p, second_acc=tp.acc_d)
    elif family == "batch":
        g = _grid(case["grid"])
        cl = CLUSTERS["2d" if case["grid"] == "2d" else "3d_serving"]
        cap = 1 << (16 if case["grid"] == "2d" else 19)
        evs = [_event("prompt" if case["grid"] == "2d" else "jets", max(60, case["hits"] * (8 - e) // 8),
                      seed * 8 + e) for e in range(case["events"])]
        n_max = _room(case["hits"])
        events, outs = [], []
        for ev in evs:
            n = ev.n_hits
            plan = H.Plan(g, max_hits=n_max, max_peaks=cap, max_member_cap=cl["member_cap"],
                          max_tracks=4096)
            d = {k: torch.zeros(n_max, dtype=t.dtype, device="cuda") for k, t in _upload(ev).items()}
            for k, t in _upload(ev).items():
                d[k][:n] = t
            e = dict(d, plan=plan, n_dev=torch.tensor([n], dtype=torch.int32, device="cuda"),
                     acc=torch.zeros(plan.acc_shape, dtype=torch.int32, device="cuda"),
                     peaks=torch.zeros((cap, 2), dtype=torch.int32, device="cuda"),
                     nf=torch.zeros(1, dtype=torch.int32, device="cuda"),
                     bufs=_buffers(n_max, cl, 4096, 256, 4096))
            events.append(e)
            outs.append(dict(_cluster_outputs(e["bufs"]), acc=e["acc"], peaks=e["peaks"],
                             n_peaks=e["nf"]))
        s = dict(events=events, n_max=n_max, cl=cl, min_votes=_min_votes(g), out=outs)
    elif family == "band":
        g = _grid(case["grid"])
        ev = _event("prompt" if g["n_d0"] == 1 else "jets", case["hits"], seed)
        cap = 1 << 20
        plan = H.Plan(g, max_hits=65535, max_peaks=16, max_member_cap=16, max_tracks=16)
        s = dict(_upload(ev), plan=plan, min_votes=_min_votes(g),
                 acc=torch.zeros(plan.acc_shape, dtype=torch.int32, device="cuda"),
                 peaks=torch.zeros((cap, 2), dtype=torch.int32, device="cuda"),
                 nf=torch.zeros(1, dtype=torch.int32, device="cuda"),
                 nv=torch.zeros(1, dtype=torch.int64, device="cuda"))
        s["out"] = dict(acc=s["acc"], peaks=s["peaks"], n_peaks=s["nf"], n_votes=s["nv"])
    elif family == "filter":
        g, params, acc, peaks = _filter_inputs(case, seed)
        cap = 1 << 19
        n = min(cap, peaks.shape[0])
        pk = np.zeros((cap, 2), np.int32)
        pk[:n] = peaks[:n]
        plan = H.Plan(g, max_hits=16, max_peaks=cap, max_member_cap=16, max_tracks=16)
        s = dict(plan=plan, params=torch.from_numpy(params).cuda(), acc=torch.from_numpy(acc).cuda(),
                 peaks=torch.from_numpy(pk).cuda(),
                 nf=torch.tensor([n], dtype=torch.int32, device="cuda"),
                 logits=torch.zeros(cap, dtype=torch.float32, device="cuda"),
                 kept=torch.zeros((cap, 2), dtype=torch.int32, device="cuda"),
                 nk=torch.zeros(1, dtype=torch.int32, device="cuda"), ws=H.cnn_workspace(cap))
        s["out"] = dict(logits=s["logits"], kept=s["kept"], n_kept=s["nk"])
    elif family == "train":
        params, mom, labels, win = _train_inputs(case, seed)
        s = dict(params=torch.from_numpy(params).cuda(), mom=torch.from_numpy(mom).cuda(),
                 labels=torch.from_numpy(labels).cuda(), win=win.cuda(),
                 pos_weight=float((labels.size - labels.sum()) / labels.sum()),
                 loss=torch.zeros(1, dtype=torch.float32, device="cuda"),
                 ws=H.cnn_workspace(labels.size, training=True))
        s["out"] = dict(params=s["params"], mom=s["mom"], loss=s["loss"])
    else:
        kinds = [dict(grid=CF.GRID_2D, cluster=CLUSTERS["2d"], min_votes=8, peak_cap=1 << 16),
                 dict(grid=CF.GRID_3D, cluster=CLUSTERS["3d_serving"], min_votes=7, peak_cap=1 << 19)]
        s = dict(events=_server_events(case, seed),
                 server=H.Server(kinds, max_hits=65535, track_cap=4096, object_cap=256,
                                 member_cap=4096, max_slots=3, queue_cap=64, batch_max=4,
                                 batch_max_hits=16384))
        # what the program collects: room for each event's results
        s["out"] = [dict(counts=np.zeros(8, np.int32), owner=np.full(_room(case["hi"]), -1, np.int32),
                         members=np.zeros(4096, np.int32), tracks=np.zeros(4096, H.TRACK_DTYPE),
                         objects=np.zeros(256, H.OBJECT_DTYPE)) for _ in s["events"]]
    s["family"] = family
    return s


def run(s):
    family = s["family"]
    if family == "event":
        H.hough_vote(s["plan"], s["r"], s["phi"], s["acc"])
        H.hough_peaks(s["plan"], s["acc"], s["min_votes"], s["peaks"], s["nf"])
        H.assoc_cluster(s["plan"], s["r"], s["phi"], s["layer"], s["peaks"], s["nf"], s["cl"],
                        s["bufs"], acc=s["given_acc"])
    elif family == "two_pass":
        s["tp"].run(s["r"], s["phi"], s["layer"])
    elif family == "batch":
        H.hough_batch(s["events"], s["n_max"], s["min_votes"], s["cl"])
    elif family == "band":
        H.hough_vote_cell(s["plan"], s["r"], s["phi"], s["acc"], s["nv"])
        H.hough_peaks(s["plan"], s["acc"], s["min_votes"], s["peaks"], s["nf"])
    elif family == "filter":
        H.cnn_score(s["plan"], s["params"], s["acc"], s["peaks"], s["nf"], s["logits"], s["ws"])
        H.cnn_keep(s["plan"], s["logits"], s["peaks"], s["nf"], 0.0, s["kept"], s["nk"])
    elif family == "train":
        H.cnn_train_step(s["params"], s["mom"], s["win"], s["labels"], 0.05, 0.9, s["pos_weight"],
                         s["loss"], s["ws"])
    else:
        srv, got = s["server"], []
        for tag, (kind, ev) in enumerate(s["events"]):
            while not srv.submit(kind, ev.r, ev.phi, ev.layer, tag):
                got += srv.poll(wait=True)
        got += srv.drain()
        for d in got:
            o = s["out"][d["tag"]]
            for key, v in (("counts", d["counts"]), ("owner", d["hit_owner"]),
                           ("members", d["members"]), ("tracks", d["tracks"]),
                           ("objects", d["objects"])):
                o[key][:v.size] = v
        return [_record_views(o) for o in s["out"]]
    return s["out"]


def _path_work(g, hits):
    """The path's own least: the hits read, the accumulator written and read
    once by the peak finder, a peak list of a fortieth of the cells; per hit
    and column the four operations that turn an arcsine per radius into a bin."""
    cells, cols = g["n_phi"] * g["n_qpt"] * g["n_d0"], g["n_qpt"] * g["n_d0"]
    return np.array([9.0 * hits + 8.0 * cells + 8.0 * cells / 40, 4.0 * hits * cols])


def work(case):
    family = case["family"]
    if family == "event":
        w = _path_work(_grid(case["grid"]), case["hits"])
    elif family == "two_pass":
        w = _path_work(CF.GRID_2D, case["hits"]) + _path_work(CF.GRID_3D, 0.3 * case["hits"])
    elif family == "batch":
        w = sum(_path_work(_grid(case["grid"]), case["hits"] * (8 - e) / 8)
                for e in range(case["events"]))
    elif family == "band":
        w = _path_work(_grid(case["grid"]), case["hits"]) * np.array([1.0, 4.0])  # two corners
    elif family == "filter":
        g = _grid(case["grid"])
        cells = g["n_phi"] * g["n_qpt"] * g["n_d0"]
        n = min(1 << 19, cells / 40)
        # multiply-adds of a window: 27 x 16 x 27, 27 x 16 x 16, 16 x 64, 64
        w = np.array([4.0 * cells + 12.0 * n + 8.0 * n / 2, 2.0 * n * (11664 + 6912 + 1024 + 64)])
    elif family == "train":
        n = case["windows"]
        w = np.array([n * 260.0 + 4 * 4 * 8529, 3 * 2.0 * n * (11664 + 6912 + 1024 + 64)])
    else:
        n = 0.5 * (case["lo"] + case["hi"])
        w = sum(_path_work(CF.GRID_3D if e % 2 else CF.GRID_2D, n) for e in range(case["events"]))
    return {"bytes": float(w[0]), "flops": float(w[1])}


# ---- 64-bit values --------------------------------------------------------------

def _split(p):
    sizes = (16 * 27, 16, 16 * 16 * 27, 16, 64 * 16, 64, 64, 1)
    out, o = [], 0
    for n in sizes:
        out.append(p[o:o + n])
        o += n
    return out


def _network(p, x):
    """Logits of windows x [n, 5, 5, 5] with flat parameters p, in their type."""
    w1, b1, w2, b2, w3, b3, w4, b4 = _split(p)
    f = torch.nn.functional
    h = torch.relu(f.conv3d(x[:, None], w1.reshape(16, 1, 3, 3, 3), b1))
    h = torch.relu((h.reshape(x.shape[0], 16 * 27) @ w2.reshape(16, 16 * 27).T) + b2)
    h = torch.relu(h @ w3.reshape(64, 16).T + b3)
    return h @ w4 + b4


def exact(case, seed):
    """Logits, or updated weights, momentum and loss, in float64.  The other
    families' results are integers decided by float32 arithmetic, and refits of
    the tracks those decisions select: they have no 64-bit value of their own."""
    if case["family"] == "filter":
        g, params, acc, peaks = _filter_inputs(case, seed)
        n = min(1 << 19, peaks.shape[0])
        k, j, i = np.unravel_index(peaks[:n, 0], acc.shape)
        padded = np.pad(acc, ((2, 2), (2, 2), (0, 0)))
        padded = np.pad(padded, ((0, 0), (0, 0), (2, 2)), mode="wrap")
        p = torch.from_numpy(params).double()
        logits = np.zeros(1 << 19)
        d = np.arange(5)
        for a in range(0, n, 1 << 15):
            sl = slice(a, min(n, a + (1 << 15)))
            x = padded[(k[sl, None, None, None] + d[:, None, None]),
                       (j[sl, None, None, None] + d[:, None]), (i[sl, None, None, None] + d)]
            logits[sl] = _network(p, torch.from_numpy(x / 16.0)).numpy()
        return dict(logits=logits, kept=None, n_kept=None)
    if case["family"] == "train":
        params, mom, labels, win = _train_inputs(case, seed)
        p = torch.from_numpy(params).double().requires_grad_()
        y = torch.from_numpy(labels).double()
        z = _network(p, win.double()[:, :125].reshape(-1, 5, 5, 5))
        pos = float((labels.size - labels.sum()) / labels.sum())
        wgt = torch.where(y > 0.5, pos, 1.0)
        loss = (wgt * (torch.nn.functional.softplus(z) - y * z)).mean()
        loss.backward()
        m = 0.9 * torch.from_numpy(mom).double() + p.grad
        return dict(params=(p - 0.05 * m).detach(), mom=m, loss=loss.detach().reshape(1))
    return None
