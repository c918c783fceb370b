"""Performance cases of the pixel-track library: what its users have it do.

Each case is one pass through public entry points of `paper_2008_13461_amd` on
seeded synthetic inputs (`synth`): whole reconstructions event by event
(`api.Pipeline`) and batched (`api.Plan`), and single stages (doublets with the
Fishbone, the broken-line fit and its adjoint, the autograd function, the
allocation-free fit).  The kinds of a case (its "kind"):

  event     one event through Pipeline.reconstruct, then Pipeline.backward
            when "adjoint" is set: the event loop of an online program
  plan      a batch of events as one pt_plan step ("stages": forward, adjoint,
            or workflow = covariance, ambiguity resolution and vertices)
  doublets  pt_build_doublets alone on a batch, with or without the Fishbone
  fit       pt_fit_broken_line, then its adjoint when "adjoint" is set, on
            tracks whose hits are given in track order: alignment passes
  autograd  broken_line_fit and its gradient: a training step
  noalloc   pt_fit_broken_line_noalloc: fits in a serving loop

Output buffers are cleared when they are made, because the library writes only
the entries it counts; every buffer is then returned whole.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2008_13461_amd import _abi as A
from paper_2008_13461_amd import api
from paper_2008_13461_amd import autograd as AG
from synth import config as C
from synth import events as E

DEVICE = "cuda"
PRECISION = {"f64": A.PT_FIT_F64, "f32": A.PT_FIT_F32, "f32+f64": A.PT_FIT_F32_F64SOLVE}
# the settings the autotuner picks for pileup-200 batches; 0: the defaults
TUNED = {"n_phi_bins": 512, "block_doublets": 128, "block_links": 64}
MAX_VERTICES = 64 * 200     # events x pileup of the largest batch
UNIQUE_TRACKS = 100_000     # generated tracks of a fit workload; more are rotated copies


def listed():
    return [
        # the smallest call: one vertex with 20 tracks in the barrel, double hits and
        # double fit with its adjoint (a smoke run, a unit test, a calibration sample)
        dict(name="event_one_vertex_f64", kind="event", pileup=1, tracks=20, noise=0.0, barrel=True, hits="f64",
             precision="f64", adjoint=True, tuned=False),
        # an ordinary event of the paper's data taking (pileup 50), event by event
        dict(name="event_pu50", kind="event", pileup=50, tracks=0, noise=0.10, barrel=False, hits="f32",
             precision="f32+f64", adjoint=False, tuned=False),
        # an event at the high-luminosity pileup, with the gradient for alignment
        dict(name="event_pu200_adjoint", kind="event", pileup=200, tracks=0, noise=0.15, barrel=False, hits="f32",
             precision="f32+f64", adjoint=True, tuned=True),
        # the benchmark's batch: 64 events at pileup 200, forward and adjoint, one graph
        dict(name="plan_pu200_adjoint", kind="plan", events=64, lo=200, hi=200, noise=0.15, overlap=0.0, min_hits=4,
             fishbone=0.0, stages="adjoint", tuned=True),
        # an uneven batch (pileup 20 to 200), forward only, default settings
        dict(name="plan_mixed", kind="plan", events=48, lo=20, hi=200, noise=0.10, overlap=0.0, min_hits=4,
             fishbone=0.0, stages="forward", tuned=False),
        # the paper's quadruplet workflow to vertices
        dict(name="plan_quadruplets", kind="plan", events=16, lo=200, hi=200, noise=0.15, overlap=0.0, min_hits=4,
             fishbone=0.0, stages="workflow", tuned=True),
        # the paper's triplet workflow to vertices, about 15 times as many tracks
        dict(name="plan_triplets", kind="plan", events=16, lo=200, hi=200, noise=0.15, overlap=0.0, min_hits=3,
             fishbone=0.0, stages="workflow", tuned=True),
        # doublets with the Fishbone on overlapping modules
        dict(name="doublets_fishbone", kind="doublets", events=16, pileup=200, noise=0.10, overlap=0.25,
             fishbone=0.01, hits="f32", tuned=True),
        # the fit and its adjoint on a million tracks with alignment offsets
        dict(name="fit_million", kind="fit", tracks=1_000_000, min_hits=4, hits="f32", precision="f32+f64",
             adjoint=True, cov=False),
        # fits with covariances of an odd number of triplets and longer
        dict(name="fit_cov_triplets", kind="fit", tracks=77_777, min_hits=3, hits="f32", precision="f32+f64",
             adjoint=False, cov=True),
        # a training step in double precision
        dict(name="autograd_f64", kind="autograd", tracks=20_000, min_hits=4, hits="f64"),
        # a serving loop that fits what one event gives
        dict(name="noalloc_event", kind="noalloc", tracks=1_500, min_hits=4, hits="f32", precision="f32+f64"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("event", "event", "event", "plan", "plan", "plan", "doublets", "fit", "fit", "autograd",
                       "noalloc"))
    if kind == "event":
        f64 = rng.random() < 0.25
        return dict(kind=kind, pileup=_log_int(rng, 1, 200), tracks=0, noise=rng.choice((0.0, 0.10, 0.15)),
                    barrel=rng.random() < 0.2, hits="f64" if f64 else "f32", precision="f64" if f64 else "f32+f64",
                    adjoint=rng.random() < 0.5, tuned=rng.random() < 0.5)
    if kind == "plan":
        events = _log_int(rng, 2, 64)
        stages = rng.choice(("adjoint", "forward", "workflow"))
        min_hits = 3 if stages == "workflow" and rng.random() < 0.5 else 4
        hi = _log_int(rng, 10, 200)
        overlap = rng.choice((0.0, 0.0, 0.0, 0.25))
        if overlap or min_hits == 3:       # these take several times as long an event
            hi = min(hi, MAX_VERTICES // ((3 if min_hits == 3 else 1) * (4 if overlap else 1) * events))
        hi = max(10, hi)
        lo = hi if rng.random() < 0.5 else max(1, hi // 10)
        return dict(kind=kind, events=events, lo=lo, hi=hi, noise=rng.choice((0.10, 0.15)), overlap=overlap,
                    min_hits=min_hits, fishbone=0.01 if overlap else 0.0, stages=stages,
                    tuned=rng.random() < 0.5)
    if kind == "doublets":
        events = _log_int(rng, 1, 16)
        overlap = rng.choice((0.0, 0.25))
        return dict(kind=kind, events=events, pileup=_log_int(rng, 10, 200), noise=0.10, overlap=overlap,
                    fishbone=0.01 if overlap or rng.random() < 0.5 else 0.0, hits=rng.choice(("f32", "f32", "f64")),
                    tuned=rng.random() < 0.5)
    if kind == "autograd":
        return dict(kind=kind, tracks=_log_int(rng, 100, 200_000), min_hits=rng.choice((3, 4)),
                    hits=rng.choice(("f32", "f64")))
    if kind == "noalloc":
        return dict(kind=kind, tracks=_log_int(rng, 50, 100_000), min_hits=rng.choice((3, 4)), hits="f32",
                    precision=rng.choice(("f32", "f32+f64", "f64")))
    return dict(kind=kind, tracks=_log_int(rng, 1000, 1_000_000), min_hits=rng.choice((3, 4)), hits="f32",
                precision=rng.choice(("f32", "f32+f64", "f32+f64", "f64")), adjoint=rng.random() < 0.5,
                cov=rng.random() < 0.3)


# ---------------------------------------------------------------------------
# inputs

def _dtype(case):
    return np.float64 if case.get("hits") == "f64" else np.float32


def _event(rng, case, vertices):
    """One event of `vertices` vertices with a fixed number of hits: the tracks'
    (4 a track, 5 with overlaps), filled up with noise."""
    per = case.get("tracks") or (35 if case.get("lo", case.get("pileup")) > 100 else 30)
    kw = dict(disks=False, eta_max=1.5, pt="loguniform", eff=1.0) if case.get("barrel") else {}
    h = E.make_event(rng, n_vertices=vertices, fixed_tracks=per, noise_frac=case["noise"] + 0.5,
                     overlap=case.get("overlap", 0.0), dtype=_dtype(case), **kw)
    want = int(round(vertices * per * (5.0 if case.get("overlap") else 4.0) * (1.0 + case["noise"])))
    keep = np.sort(np.argsort(h.track < 0, kind="stable")[:want])    # tracks' hits first, then noise
    return E.Hits(h.x[keep], h.y[keep], h.z[keep], h.layer[keep], h.module[keep], h.track[keep],
                  np.array([0, len(keep)], dtype=np.int32))


def _batch(case, seed):
    """Host hits of the case's events (numpy)."""
    rng = np.random.Generator(np.random.PCG64(seed))
    if case["kind"] == "plan":      # pileups spread evenly over lo .. hi, in any order
        pileups = rng.permutation(np.linspace(case["lo"], case["hi"], case["events"]).round().astype(int))
    else:
        pileups = [case["pileup"]] * case.get("events", 1)
    return E.concat([_event(rng, case, int(p)) for p in pileups])


def _caps(n_hits, n_events, min_hits=4):
    """The benchmark's capacities: 128 cells a hit, a quarter as many links."""
    cells = max(4096, 128 * n_hits)
    return dict(n_hits=n_hits, n_events=n_events, cells_cap=cells, links_cap=cells // 4,
                tuplets_cap=max(1024, (24 if min_hits == 3 else 1) * n_hits))


def _cleared(buffers):
    """A product's buffers with every entry zero."""
    for t in vars(buffers).values():
        if isinstance(t, torch.Tensor):
            t.zero_()
    return buffers


def _normal(seed, stream, *shape, dtype=torch.float32):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000 * int(seed) + stream)
    return torch.randn(*shape, dtype=dtype, device=DEVICE, generator=g)


def _offsets(seed):
    """Alignment translations of the modules, 10 um each way."""
    return 10e-4 * _normal(seed, 1, C.N_MODULES, 3)


def _tracks(case, seed):
    """Hits in track order and their rows: (x, y, z, layer, module, rows [n, 8], nhits [n]) on the GPU.

    Tracks of min_hits to 8 hits as they cross the detector (a tenth of the
    crossings on overlapping modules); beyond UNIQUE_TRACKS of them, copies turned by
    a random azimuth each.
    """
    n = case["tracks"]
    rng = np.random.Generator(np.random.PCG64([seed, 3]))
    copies = -(-n // UNIQUE_TRACKS)
    base = -(-n // copies)
    parts, have, first = [], 0, 0
    while have < base:
        m = int(1.5 * (base - have)) + 64
        trk = E.draw_tracks(rng, m)
        ti, li, x, y, z, _ = E.track_hits(rng, trk, eff=0.99, overlap=0.1)
        cnt = np.bincount(ti, minlength=m)
        good = np.flatnonzero((cnt >= case["min_hits"]) & (cnt <= A.PT_MAX_HITS))[: base - have]
        take = np.zeros(m, bool)
        take[good] = True
        sel = take[ti]
        parts.append((li[sel], x[sel], y[sel], z[sel], cnt[good]))
        have += len(good)
    li, x, y, z, cnt = (np.concatenate([p[i] for p in parts]) for i in range(5))
    module = E.module_id(li, x, y, z)
    dt = torch.float64 if case["hits"] == "f64" else torch.float32
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEVICE)
    x, y, z, li, module = up(x), up(y), up(z), up(li.astype(np.uint8)), up(module.astype(np.int16))
    cnt = up(cnt.astype(np.int64))
    # hits of no track behind the tracks', to a fixed number (5 a track)
    spare = torch.arange(max(0, 5 * base + 64 - x.numel()), device=DEVICE) % x.numel()
    x, y, z, li, module = (torch.cat([t, t[spare]]) for t in (x, y, z, li, module))
    start = torch.cumsum(cnt, 0) - cnt
    track = torch.repeat_interleave(torch.arange(base, device=DEVICE), cnt)
    track = torch.cat([track, track[spare]])
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1000 * int(seed) + 2)
    turn = 2.0 * math.pi * torch.rand(copies, base, dtype=torch.float64, device=DEVICE, generator=g)
    turn[0] = 0.0
    a = turn[:, track]
    X = (x * torch.cos(a) - y * torch.sin(a)).reshape(-1)
    Y = (x * torch.sin(a) + y * torch.cos(a)).reshape(-1)
    k = torch.arange(A.PT_MAX_HITS, device=DEVICE)
    rows = torch.where(k < cnt[:, None], start[:, None] + k, -1)
    shift = (torch.arange(copies, device=DEVICE) * x.numel())[:, None, None]
    rows = torch.where(rows[None] >= 0, rows[None] + shift, -1).reshape(-1, A.PT_MAX_HITS)[:n]
    tile = lambda t: t.repeat(copies).contiguous()
    return (X.to(dt), Y.to(dt), tile(z).to(dt), tile(li), tile(module), rows.to(torch.int32).contiguous(),
            tile(cnt)[:n].to(torch.uint8))


def _fit_offsets(case, seed):
    return None if case["kind"] == "noalloc" else _offsets(seed)


def _cotangents(case, seed):
    dt = torch.float64 if case.get("precision", "f64" if case["hits"] == "f64" else "") == "f64" else torch.float32
    return _normal(seed, 4, case["tracks"], 5, dtype=dt), _normal(seed, 5, case["tracks"], dtype=dt)


def _prepare_tracks(case, seed):
    s = {"case": case}
    x, y, z, layer, module, rows, nhits = _tracks(case, seed)
    s["offsets"] = _fit_offsets(case, seed)
    n = case["tracks"]
    if case["kind"] == "autograd":
        s["leaves"] = [t.requires_grad_() for t in (x, y, z, s["offsets"])]
        s["fixed"] = (layer, module, rows, nhits)
        s["cfg"] = AG.FitConfig(C.default_config())
        s["cot"] = _cotangents(case, seed)
        return s
    s["cfg"] = A.make_config(C.default_config(exclusive_hits=1))
    s["hits"] = api.Hits(x, y, z, layer, module, torch.tensor([0, x.numel()], dtype=torch.int32, device=DEVICE))
    s["rows"] = api.Tuplets.from_rows(rows, nhits)
    prec = PRECISION[case["precision"]]
    s["tracks"] = _cleared(api.Tracks.empty(n, prec, with_cov=bool(case.get("cov"))))
    s["status"] = api.new_status()
    if case["kind"] == "fit":
        s["ws"] = api.new_workspace(api.workspace_size(s["cfg"], x.numel(), 1, 0, 0, n))
        if case["adjoint"]:
            s["cot"] = _cotangents(case, seed)
            s["grad_hits"] = torch.zeros((x.numel(), 3), dtype=s["cot"][0].dtype, device=DEVICE)
            s["grad_offsets"] = torch.zeros((C.N_MODULES, 3), dtype=torch.float64, device=DEVICE)
    return s


def prepare(case, seed):
    if case["kind"] in ("fit", "autograd", "noalloc"):
        return _prepare_tracks(case, seed)
    h = _batch(case, seed)
    perf = TUNED if case["tuned"] else {}
    s = {"case": case, "hits": api.Hits.from_host(h)}
    cp = _caps(h.n_hits, h.n_events, case.get("min_hits", 4))
    if case["kind"] == "doublets":
        s["cfg"] = A.make_config(C.default_config(fishbone_theta=case["fishbone"]), **perf)
        s["cells"] = _cleared(api.Cells.empty(cp["cells_cap"], h.n_hits))
        s["status"] = api.new_status()
        s["ws"] = api.new_workspace(api.workspace_size(s["cfg"], h.n_hits, h.n_events, cp["cells_cap"], 0, 0))
        return s
    if case["kind"] == "event":
        prec, adjoint, workflow = PRECISION[case["precision"]], case["adjoint"], False
        s["pipe"] = p = api.Pipeline(C.default_config(), precision=prec, **cp, **perf)
        s["products"] = (p.cells, p.links, p.tuplets, p.tracks)
        s["status"] = p.status
    else:
        prec, adjoint, workflow = A.PT_FIT_F32_F64SOLVE, case["stages"] == "adjoint", case["stages"] == "workflow"
        cfg = A.make_config(C.default_config(min_hits=case["min_hits"], fishbone_theta=case["fishbone"]), **perf)
        s["products"] = (api.Cells.empty(cp["cells_cap"], h.n_hits), api.Links.empty(cp["links_cap"], cp["cells_cap"]),
                         api.Tuplets.empty(cp["tuplets_cap"]),
                         api.Tracks.empty(cp["tuplets_cap"], prec, with_cov=workflow))
        s["status"] = api.new_status()
        s["plan"] = api.Plan(cfg, precision=prec, with_adjoint=adjoint,
                             stages=A.PT_STAGE_AMBIGUITY | A.PT_STAGE_VERTICES if workflow else 0, **cp)
    for p in s["products"]:
        _cleared(p)
    n = cp["tuplets_cap"]
    s["args"] = {}
    if adjoint:
        dt = torch.float64 if prec == A.PT_FIT_F64 else torch.float32
        s["args"] = dict(offsets=_offsets(seed), g_params=_normal(seed, 4, n, 5, dtype=dt),
                         g_chi2=_normal(seed, 5, n, dtype=dt),
                         grad_hits=torch.zeros((h.n_hits, 3), dtype=dt, device=DEVICE),
                         grad_offsets=torch.zeros((C.N_MODULES, 3), dtype=torch.float64, device=DEVICE))
    if workflow:
        s["args"] = dict(selected=torch.zeros(n, dtype=torch.int32, device=DEVICE),
                         n_selected=torch.zeros(1, dtype=torch.int32, device=DEVICE),
                         vertices=_cleared(api.Vertices.empty(n, h.n_events, n)))
    return s


# ---------------------------------------------------------------------------
# one pass

def _tensors(products):
    return {f"{type(p).__name__}.{k}": t for p in products for k, t in vars(p).items() if isinstance(t, torch.Tensor)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "autograd":
        x, y, z, off = state["leaves"]
        layer, module, rows, nhits = state["fixed"]
        params, chi2, status = AG.broken_line_fit(x, y, z, layer, module, rows, nhits, off, state["cfg"])
        grads = torch.autograd.grad((params, chi2), (x, y, z, off), state["cot"])
        return {"params": params.detach(), "chi2": chi2.detach(), "status": status, "grads": list(grads)}
    status = state["status"]
    status.zero_()          # flags and counters of this pass alone
    hits = state["hits"]
    if kind == "doublets":
        api.build_doublets(hits, state["cfg"], state["cells"], status, state["ws"])
        return {**_tensors([state["cells"]]), "status": status}
    if kind in ("fit", "noalloc"):
        prec, tracks = PRECISION[case["precision"]], state["tracks"]
        if kind == "noalloc":
            api.fit_broken_line_noalloc(hits, state["cfg"], state["rows"], None, prec, tracks, status)
            return {"params": tracks.params, "chi2": tracks.chi2, "track_status": tracks.status, "status": status}
        api.fit_broken_line(hits, state["cfg"], state["rows"], state["offsets"], prec, tracks, status, state["ws"])
        out = {"params": tracks.params, "chi2": tracks.chi2, "track_status": tracks.status, "status": status}
        if case["cov"]:
            out["cov"] = tracks.cov
        if case["adjoint"]:
            state["grad_hits"].zero_()      # the adjoint adds into its outputs
            state["grad_offsets"].zero_()
            api.fit_broken_line_bwd(hits, state["cfg"], state["rows"], state["offsets"], prec, *state["cot"],
                                    state["grad_hits"], state["grad_offsets"], status, state["ws"])
            out.update(grad_hits=state["grad_hits"], grad_offsets=state["grad_offsets"])
        return out
    args = state["args"]
    for k in ("grad_hits", "grad_offsets"):
        if k in args:
            args[k].zero_()
    if kind == "event":
        state["pipe"].reconstruct(hits, offsets=args.get("offsets"))
        if case["adjoint"]:
            state["pipe"].backward(hits, args["g_params"], args["g_chi2"], args["grad_hits"], args["grad_offsets"],
                                   offsets=args["offsets"])
    else:
        state["plan"].run(hits, *state["products"], status, **args)
    out = {**_tensors(state["products"]), "status": status}
    for k in ("grad_hits", "grad_offsets", "selected", "n_selected"):
        if k in args:
            out[k] = args[k]
    if "vertices" in args:
        out.update(_tensors([args["vertices"]]))
    return out


# ---------------------------------------------------------------------------
# the bytes and operations a pass cannot do without

def _sizes(case):
    """(hits, doublets, links, rows) of the case's events: the hits as they are
    made, doublets in proportion to the hits of an event (93 a hit at 32 000)."""
    events = case.get("events", 1)
    lo, hi = (case["lo"], case["hi"]) if case["kind"] == "plan" else (case["pileup"], case["pileup"])
    per = case.get("tracks") or (35 if lo > 100 else 30)
    per *= (5.0 if case.get("overlap") else 4.0) * (1.0 + case["noise"])
    mean = 0.5 * (lo + hi)
    hits = events * mean * per
    cells = events * (mean * mean + (hi - lo) ** 2 / 12.0) * per * per * 93.0 / 32000.0
    return hits, cells, 0.2 * cells, hits * (18.0 if case.get("min_hits") == 3 else 0.5)


def _fit_work(n, hit_bytes, value, adjoint, cov, mean=4.5):
    """Bytes and operations of n fits: 4.5 hits a track with layer, module and
    row entry; about 400 operations a hit each way."""
    b = n * mean * (3 * hit_bytes + 1 + 2 + 4) + n * (6 * value + 2)
    if cov:
        b += n * 15 * value
    if adjoint:
        b += n * mean * (3 * hit_bytes + 1 + 2 + 4) + n * (6 * value + 1) + n * mean * 3 * value
    return b, n * mean * 400.0 * (3 if adjoint else 1)


def work(case):
    kind = case["kind"]
    if kind in ("fit", "autograd", "noalloc"):
        value = 8 if (case.get("precision") or case["hits"]) == "f64" else 4
        b, f = _fit_work(case["tracks"], 8 if case["hits"] == "f64" else 4, value,
                         kind == "autograd" or bool(case.get("adjoint")), bool(case.get("cov")))
        return {"bytes": b, "flops": f}
    hits, cells, links, rows = _sizes(case)
    hit_bytes = 8 if case.get("hits") == "f64" else 4
    b = hits * (3 * hit_bytes + 1 + 8) + cells * 9
    f = cells * 30.0
    if kind == "doublets":
        return {"bytes": b, "flops": f}
    b += cells * 9 + links * 8 + rows * (32 + 28 + 1 + 4)
    f += links * 40.0
    fb, ff = _fit_work(rows, hit_bytes, 8 if case.get("precision") == "f64" else 4,
                       bool(case.get("adjoint")) or case.get("stages") == "adjoint", case.get("stages") == "workflow")
    return {"bytes": b + fb, "flops": f + ff}


# ---------------------------------------------------------------------------
# the fit in 64 bits, in plain torch

def _solve(M, rhs):
    """Solves the symmetric positive systems M x = rhs, entries given as
    tensors over the tracks (elimination without pivoting)."""
    n = len(rhs)
    M = [list(r) for r in M]
    b = [list(v) for v in rhs]
    for i in range(n):
        for j in range(i + 1, n):
            f = M[j][i] / M[i][i]
            for k in range(i, n):
                M[j][k] = M[j][k] - f * M[i][k]
            b[j] = [u - f * v for u, v in zip(b[j], b[i])]
    x = [None] * n
    for i in reversed(range(n)):
        acc = b[i]
        for j in range(i + 1, n):
            acc = [u - M[i][j] * v for u, v in zip(acc, x[j])]
        x[i] = [u / M[i][i] for u in acc]
    return x


def _fit64(cfg, P, barrel):
    """Broken-line fit of tracks with N hits each in 64 bits: P [n, N, 3], barrel
    [n, N].  Returns (params [n, 5], chi2 [n], cov [n, 15])."""
    N = P.shape[1]
    r = P - P[:, :1]
    rx, ry, rz = (r[:, :, i] for i in range(3))
    ax, ay, bx, by = rx[:, N // 2], ry[:, N // 2], rx[:, -1], ry[:, -1]
    lb = torch.sqrt(bx * bx + by * by)
    kp = 2 * (ax * by - ay * bx) / (torch.sqrt(ax * ax + ay * ay) * lb * torch.sqrt((bx - ax) ** 2 + (by - ay) ** 2))
    sb = 0.5 * kp * lb
    cb = torch.sqrt(1 - sb * sb)
    tx, ty = (bx * cb + by * sb) / lb, (by * cb - bx * sb) / lb
    zero = torch.zeros_like(kp)
    s, u = [zero], [zero]
    for k in range(1, N):
        xt, xn = tx * rx[:, k] + ty * ry[:, k], tx * ry[:, k] - ty * rx[:, k]
        s.append(torch.atan2(kp * xt, 1 - kp * xn) / kp)
        a = 2 * xn - kp * (xt * xt + xn * xn)
        u.append(a / (1 + torch.sqrt(1 - kp * a)))
    d = [s[k + 1] - s[k] for k in range(N - 1)]
    t = rz[:, -1] / s[-1]
    sec2 = 1 + t * t
    sec = torch.sqrt(sec2)
    p = torch.clamp(0.299792458 * cfg["bfield"] / 100 / kp.abs() * sec, max=cfg["p_cap"])
    w_u = torch.full_like(kp, 1 / cfg["sigma_rphi"] ** 2)
    w_z = [torch.where(barrel[:, k], torch.full_like(kp, 1 / cfg["sigma_z"] ** 2), 1 / (cfg["sigma_r"] * t) ** 2)
           for k in range(N)]
    m = [rz[:, k] - t * s[k] for k in range(N)]
    A_ = [[zero] * (N + 1) for _ in range(N + 1)]
    B_ = [[zero] * N for _ in range(N)]
    for k in range(N):
        A_[k][k] = A_[k][k] + w_u
        B_[k][k] = B_[k][k] + w_z[k]
    kinks = []
    for j in range(1, N - 1):
        path = torch.where(barrel[:, j], sec, sec / t.abs())
        X = cfg["x_over_x0"] * path
        th2 = (cfg["highland_a"] / p) ** 2 * X * (1 + cfg["highland_b"] * torch.log(X)) ** 2
        wt, wz = 1 / (th2 * sec2), 1 / (th2 * sec2 * sec2)
        c = {j - 1: 1 / d[j - 1], j: -(1 / d[j - 1] + 1 / d[j]), j + 1: 1 / d[j]}
        cc = dict(c)
        cc[N] = -0.5 * (d[j - 1] + d[j])
        for q in cc:
            for v in cc:
                A_[q][v] = A_[q][v] + wt * cc[q] * cc[v]
        for q in c:
            for v in c:
                B_[q][v] = B_[q][v] + wz * c[q] * c[v]
        kinks.append((wt, wz, cc, c))
    one = torch.ones_like(kp)
    # the solution, then the columns of the inverses that the covariance needs
    xs = _solve(A_, [[w_u * u[k], *(one if k == q else zero for q in (0, 1))] + [zero] for k in range(N)] +
                [[zero, zero, zero, one]])
    ws = _solve(B_, [[w_z[k] * m[k], *(one if k == q else zero for q in (0, 1))] for k in range(N)])
    xc, wl = [v[0] for v in xs], [v[0] for v in ws]
    chi2 = sum(w_u * (u[k] - xc[k]) ** 2 + w_z[k] * (m[k] - wl[k]) ** 2 for k in range(N))
    for wt, wz, cc, c in kinks:
        chi2 = chi2 + wt * sum(v * xc[q] for q, v in cc.items()) ** 2 + wz * sum(v * wl[q] for q, v in c.items()) ** 2

    def perigee(u0, u1, dk, w0, w1):
        kappa = kp + dk
        qx, qy = P[:, 0, 0] - u0 * ty, P[:, 0, 1] + u0 * tx
        slope = (u1 - u0) / d[0] - 0.5 * dk * d[0]
        ca = 1 / torch.sqrt(1 + slope * slope)
        cps, sps = tx * ca - ty * slope * ca, ty * ca + tx * slope * ca
        v = kappa * (qx * qx + qy * qy) + 2 * (qy * cps - qx * sps)
        d0 = v / (1 + torch.sqrt(1 + kappa * v))
        hx, hy = cps + kappa * qy, sps - kappa * qx
        phi0 = torch.atan2(hy, hx)
        along, across = qx * torch.cos(phi0) + qy * torch.sin(phi0), qy * torch.cos(phi0) - qx * torch.sin(phi0)
        ds = torch.atan2(kappa * along, 1 + kappa * (d0 - across)) / kappa
        cot = t + (w1 - w0) / d[0]
        return torch.stack([kappa, phi0, cot, d0, P[:, 0, 2] + w0 - cot * ds], 1)

    inner = [xc[0], xc[1], xc[N], wl[0], wl[1]]
    params = perigee(*inner)
    return params, chi2, (perigee, inner, xs, ws)


def _cov64(fitted, N):
    perigee, inner, xs, ws = fitted
    with torch.enable_grad():
        at = [v.detach().requires_grad_() for v in inner]
        out = perigee(*at)
        J = [torch.autograd.grad(out[:, q].sum(), at, retain_graph=True) for q in range(5)]
    S = {}
    for i, a in enumerate((0, 1, N)):
        for j in range(3):
            S[i, j] = xs[a][1 + j]
    for i in range(2):
        for j in range(2):
            S[3 + i, 3 + j] = ws[i][1 + j]
    return torch.stack([sum(J[q][i] * v * J[k][j] for (i, j), v in S.items()) for q in range(5) for k in range(q, 5)], 1)


def exact(case, seed):
    """The fits in 64 bits; the other outputs are indices, counts and bytes, or
    follow from whole reconstructions that have no short plain form."""
    if case["kind"] not in ("fit", "autograd", "noalloc"):
        return None
    cfg = C.default_config()
    x, y, z, layer, module, rows, nhits = _tracks(case, seed)
    offsets = _fit_offsets(case, seed)
    adjoint = case["kind"] == "autograd" or bool(case.get("adjoint"))
    xyz = torch.stack([x, y, z], 1).double().requires_grad_(adjoint)
    off = None if offsets is None else offsets.double().requires_grad_(adjoint)
    n = case["tracks"]
    params = torch.zeros(n, 5, dtype=torch.float64, device=DEVICE)
    chi2 = torch.zeros(n, dtype=torch.float64, device=DEVICE)
    cov = torch.zeros(n, 15, dtype=torch.float64, device=DEVICE) if case.get("cov") else None
    g_hits = torch.zeros_like(xyz)
    g_off = torch.zeros(C.N_MODULES, 3, dtype=torch.float64, device=DEVICE)
    barrel = torch.tensor([bool(v) for v in cfg["layer_barrel"]], device=DEVICE)
    if adjoint:
        gp, gc = (t.double() for t in _cotangents(case, seed))
    for N in range(3, A.PT_MAX_HITS + 1):
        of_n = torch.nonzero(nhits == N)[:, 0]
        for at in of_n.split(250_000):
            h = rows[at, :N].long()
            P = xyz[h] if off is None else xyz[h] + off[module[h].long()]
            with torch.set_grad_enabled(adjoint):
                q, c, fitted = _fit64(cfg, P, barrel[layer[h].long()])
                if adjoint:
                    got = torch.autograd.grad((q, c), (xyz, off), (gp[at], gc[at]))
                    g_hits, g_off = g_hits + got[0], g_off + got[1]
            params[at], chi2[at] = q.detach(), c.detach()
            if cov is not None:
                cov[at] = _cov64(fitted, N).detach()
    if case["kind"] == "autograd":
        return {"params": params, "chi2": chi2, "status": None, "grads": [*g_hits.unbind(1), g_off]}
    out = {"params": params, "chi2": chi2, "track_status": None, "status": None}
    if cov is not None:
        out["cov"] = cov
    if adjoint:
        out.update(grad_hits=g_hits, grad_offsets=g_off)
    return out
