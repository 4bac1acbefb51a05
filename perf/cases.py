"""Performance cases: the calls a program makes of this library, over the range it makes them in.

``listed()`` names the cases, ``draw(rng)`` gives further ones of the same
ranges, ``prepare`` makes what a program holds before the call (the events on
the device, the context, the output buffers), ``run`` is one pass through the
public entry points, ``work`` the bytes and operations a pass cannot do
without, ``exact`` the float outputs in 64 bits where they have such a value.

A case is a dict of plain values:

``what``     "reconstruct" (tracks of a batch), "consolidate" (track
             coordinates and states of given tracks), "sequence" (event cut,
             reconstruction, consolidation) or "serve" (single events handed
             to the server and collected)
``recipe``   a recipe of ``paper_2207_03936_amd.synth``, or "mu1-5": the
             mu1-25 recipe at low pileup (1 to 5 vertices, events of up to
             about 2,500 hits)
``events``   events per call
``form``     "batched" (a context), "static" (the allocation-free entry) or
             "plain" (one launch per stage)
``f16``      hits as binary16 array-of-structures records
``own``      the call goes to a stream of the program's own (the batched form
             then replays a captured graph) instead of torch's current one
``reverse``, ``K``   method parameters: traversal direction, partners per
             middle hit
"""

import dataclasses

import numpy as np
import torch

from paper_2207_03936_amd import sbt, synth

# distinct events drawn for one batch; a longer batch repeats them, each time
# turned about the beam axis by an angle of its own (the detector and the
# recipes are symmetric under it), so that no two events of a batch are alike
POOL = {"mu30": 32}
POOL_DEFAULT = 240

HITS_PER_VERTEX = 410.0
VERTICES = {"tiny": 1.0, "mu7.6": 7.6, "mu1-25": 13.0, "mu30": 32.0, "pairs7.6": 7.6, "bw7.6": 7.6, "mu1-5": 3.0}
CUT_FRACTION = 0.1   # the sequence's event cut: the densest tenth of the events


def _case(name, what, recipe, events, form="batched", f16=False, own=False, reverse=1, K=4):
    return dict(name=name, what=what, recipe=recipe, events=events, form=form, f16=f16, own=own, reverse=reverse, K=K)


def listed():
    return [
        # one small event: the latency of a single call, launches and the step chain
        _case("tiny-1", "reconstruct", "tiny", 1),
        # one ordinary event from a program that may not allocate
        _case("mu7.6-1-static", "reconstruct", "mu7.6", 1, form="static"),
        # an online farm's small ragged batch, hits stored as binary16, replayed as a graph
        _case("mu1-25-37-f16", "reconstruct", "mu1-25", 37, f16=True, own=True),
        # many low-pileup events in one call
        _case("mu1-5-2048", "reconstruct", "mu1-5", 2048),
        # module pairs (two z per module) through the plain form, forward traversal
        _case("pairs7.6-201-plain", "reconstruct", "pairs7.6", 201, form="plain", reverse=0),
        # the benchmark's own batch: upgrade conditions, graph replay on a stream of its own
        _case("mu7.6-1000", "reconstruct", "mu7.6", 1000, own=True),
        # dense events with kinks and noise
        _case("mu30-400", "reconstruct", "mu30", 400),
        # the benchmark's long uneven batch
        _case("mu1-25-10000", "reconstruct", "mu1-25", 10000),
        # track states of a reconstructed batch
        _case("consolidate-mu7.6-1000", "consolidate", "mu7.6", 1000),
        # the paper's sequence: event cut, reconstruction, consolidation
        _case("sequence-mu7.6-500", "sequence", "mu7.6", 500),
        # single events through the server, host to host
        _case("serve-mu1-25-48", "serve", "mu1-25", 48),
    ]


def draw(rng):
    what = rng.choice(["reconstruct"] * 6 + ["consolidate", "sequence"])
    recipe = rng.choice(["tiny", "mu7.6", "mu7.6", "mu1-25", "mu1-25", "mu30", "pairs7.6", "bw7.6", "mu1-5"])
    if what == "consolidate" and recipe in ("pairs7.6", "bw7.6"):
        recipe = "mu7.6"
    most = {"tiny": 8000, "mu1-5": 8000, "mu7.6": 4000, "mu1-25": 4000, "mu30": 1200, "pairs7.6": 240, "bw7.6": 4000}[recipe]
    events = int(round(2.0 ** rng.uniform(0.0, np.log2(most))))
    form = rng.choice(["batched"] * 5 + ["plain", "static"]) if what == "reconstruct" else "batched"
    if form == "static":
        # the static form's 64 MiB hold about 600,000 hits
        events = max(1, min(events, int(5.0e5 / (HITS_PER_VERTEX * VERTICES[recipe] * 1.3))))
    f16 = what == "reconstruct" and form == "batched" and rng.random() < 0.25
    K = rng.choice([4, 4, 4, 4, 2, 8]) if what == "reconstruct" else 4
    c = _case("", what, recipe, events, form=form, f16=f16, own=rng.random() < 0.4,
              reverse=rng.choice([1, 1, 1, 0]), K=K)
    del c["name"]
    return c


# ---------------------------------------------------------------- inputs

def _recipe(name, seed):
    if name == "mu1-5":
        r = dataclasses.replace(synth.CONFIGS["mu1-25"], name="mu1-5", pv_max=5)
    else:
        r = synth.CONFIGS[name]
    return dataclasses.replace(r, seed=(r.seed << 32) + (int(seed) & 0xFFFFFFFF))


def _batch(case, seed):
    """The case's events as a host batch."""
    r = _recipe(case["recipe"], seed)
    n = case["events"]
    pool = POOL.get(case["recipe"], POOL_DEFAULT)
    k = min(n, pool)
    base = synth.concat([synth.make_event(r, i) for i in range(k)], synth.PLANE_Z)
    if k == n:
        return base
    rng = np.random.default_rng([int(seed) & 0xFFFFFFFF, 77])
    pick = np.concatenate([rng.permutation(k) for _ in range(-(-n // k))])[:n]
    phi = rng.uniform(0.0, 2.0 * np.pi, n)
    M = base.n_modules
    sizes = np.diff(base.event_offsets).astype(np.int64)
    counts = np.diff(base.module_offsets).astype(np.int64).reshape(k, M)
    eo = np.zeros(n + 1, np.int64)
    np.cumsum(sizes[pick], out=eo[1:])
    mo = np.zeros(n * M + 1, np.int64)
    np.cumsum(counts[pick].reshape(-1), out=mo[1:])
    x, y, z = (np.empty(int(eo[-1]), np.float32) for _ in range(3))
    truth = np.empty(int(eo[-1]) if case["what"] == "consolidate" else 0, np.int32)
    for i in range(n):
        s = slice(int(base.event_offsets[pick[i]]), int(base.event_offsets[pick[i] + 1]))
        d = slice(int(eo[i]), int(eo[i + 1]))
        c, t = np.float32(np.cos(phi[i])), np.float32(np.sin(phi[i]))
        x[d] = base.x[s] * c - base.y[s] * t
        y[d] = base.x[s] * t + base.y[s] * c
        z[d] = base.z[s]
        if truth.size:
            truth[d] = base.truth[s]
    return synth.Batch(x=x, y=y, z=z, event_offsets=eo.astype(np.int32), module_offsets=mo.astype(np.int32),
                       module_z=base.module_z, truth=truth)


def _truth_tracks(b):
    """The particles with three hits or more as tracks in the library's form:
    hits from the last plane to the first (one per plane), tracks of an event
    in the order of their second hit's id.  (event_track_offsets,
    track_hit_offsets, track_hits), host arrays."""
    E = b.n_events
    eto, tho, th = [0], [0], []
    nt = nh = 0
    for e in range(E):
        lo, hi = int(b.event_offsets[e]), int(b.event_offsets[e + 1])
        t = b.truth[lo:hi]
        ids = np.nonzero(t >= 0)[0]
        ids = ids[np.lexsort((-ids, t[ids]))]          # by particle, last plane first
        start = np.nonzero(np.diff(t[ids], prepend=-1))[0]
        length = np.diff(np.append(start, ids.size))
        ok = length >= 3
        start, length = start[ok], length[ok]
        if start.size:
            order = np.argsort(ids[start + 1], kind="stable")
            start, length = start[order], length[order]
            first = np.cumsum(length) - length
            th.append(ids[np.repeat(start - first, length) + np.arange(int(length.sum()))])
            tho.extend((nh + np.cumsum(length)).tolist())
            nt += int(length.size)
            nh += int(length.sum())
        eto.append(nt)
    hits = np.concatenate(th) if th else np.zeros(0, np.int64)
    return np.array(eto, np.int32), np.array(tho, np.int32), hits.astype(np.int32)


def _capacity(case):
    """Hits the buffers of the program are sized for: it keeps them from batch
    to batch, so they hold more than the present one."""
    n, mean = case["events"], HITS_PER_VERTEX * VERTICES[case["recipe"]]
    return int(mean * (1.4 * n + 8.0 * n ** 0.5))


_streams = {}


def _stream(case):
    """The stream of the call: torch's current one, or the program's own."""
    if not case["own"]:
        return torch.cuda.current_stream()
    d = torch.cuda.current_device()
    if d not in _streams:
        _streams[d] = torch.cuda.Stream()
    return _streams[d]


def prepare(case, seed):
    b = _batch(case, seed)
    cap = _capacity(case)
    assert b.n_hits <= cap
    s = dict(case=case, stream=_stream(case), cap=cap)
    params = sbt.make_params(b.module_z, reverse=case["reverse"], max_doublet_candidates=case["K"])
    if case["what"] == "serve":
        # events as they arrive, each in host memory of its own, and a running server
        s["events"] = []
        for i in range(b.n_events):
            ev = b.event(i)
            s["events"].append((ev.module_offsets, ev.x, ev.y, ev.z))
        s["server"] = sbt.Server(params, device_budget_bytes=1 << 30, n_slots=2, slot_events=64, slot_hits=1 << 19,
                                 max_wait_us=100)
        return s
    if case["what"] == "sequence":
        params.max_event_hits = sbt.sbt_gec_threshold(b.event_offsets, CUT_FRACTION)
    s["params"] = params
    s["batch"] = sbt.DeviceBatchF16(b) if case["f16"] else sbt.DeviceBatch(b)
    s["out"] = sbt.DeviceTracks(b.n_events, cap)
    if case["what"] in ("consolidate", "sequence"):
        s["states"] = sbt.TrackStates(cap)
    if case["what"] == "consolidate":
        out = s["out"]
        for dst, src in zip((out.eto, out.tho, out.th), _truth_tracks(b)):
            dst[:src.size] = torch.from_numpy(src).to(dst.device)
    elif case["form"] == "batched":
        s["ctx"] = sbt.Context(params, b.n_events, cap)
    elif case["form"] == "plain":
        s["ws"] = sbt.Workspace(b.n_events, cap)
    return s


# ---------------------------------------------------------------- one pass

def _serve(s):
    """Every event submitted, polled until all results are in, and their
    tracks kept in the order of the requests."""
    srv = s["server"]
    for i, (mo, x, y, z) in enumerate(s["events"]):
        if srv.submit(i, mo, x, y, z) != sbt.SBT_OK:
            raise RuntimeError("submit refused")
    got = {}
    while len(got) < len(s["events"]):
        for rid, status, tho, th, _, _ in srv.poll(wait_us=2000):
            got[rid] = (status, tho, th)
    status = np.zeros(len(got), np.int32)
    tho, th = np.zeros(s["cap"] // 3 + len(got), np.int32), np.zeros(s["cap"], np.int32)
    t = h = 0
    for i in range(len(got)):
        status[i] = got[i][0]
        tho[t:t + got[i][1].size] = got[i][1]
        th[h:h + got[i][2].size] = got[i][2]
        t, h = t + got[i][1].size, h + got[i][2].size
    return dict(status=status, tho=tho, th=th)


def run(state):
    s, case = state, state["case"]
    if case["what"] == "serve":
        return _serve(s)
    out, stream = s["out"], s["stream"]
    if case["what"] != "consolidate":
        if case["form"] == "static":
            sbt.sbt_reconstruct_batched_static(s["params"], s["batch"], out, stream)
        elif case["form"] == "plain":
            sbt.sbt_reconstruct(s["params"], s["batch"], out, s["ws"], stream)
        elif case["f16"]:
            s["ctx"].reconstruct_f16(s["batch"], out, stream)
        else:
            s["ctx"].reconstruct(s["batch"], out, stream)
    got = {}
    if case["what"] != "consolidate":
        got = dict(eto=out.eto, tho=out.tho, th=out.th, status=out.status)
    if case["what"] != "reconstruct":
        st = sbt.sbt_consolidate(s["batch"], out, s["states"], stream)
        got.update(hit_x=st.hit_x, hit_y=st.hit_y, hit_z=st.hit_z, state=st.state)
    return got


# ---------------------------------------------------------------- bounds and values

def work(case):
    E = case["events"]
    H = E * HITS_PER_VERTEX * VERTICES[case["recipe"]]
    M = synth.N_PLANES
    T, A = 0.08 * H, 0.9 * H          # tracks, and hits on them
    tracks_out = 4.0 * (A + T + 2 * E)
    hits_in = (8.0 if case["f16"] else 12.0) * H + 4.0 * (M + 1) * E
    # reconstruction: the angle of each hit (about 20 operations), and per hit on
    # a track one extrapolation, one angle and a scatter (about 40)
    rec = dict(bytes=hits_in + tracks_out, flops=20.0 * H + 40.0 * A)
    # consolidation: tracks and coordinates of their hits in, packed
    # coordinates and six numbers per track out; about 30 operations per hit
    con = dict(bytes=tracks_out + 12.0 * A + 12.0 * A + 24.0 * T, flops=30.0 * A)
    if case["what"] == "consolidate":
        return con
    if case["what"] == "sequence":
        return dict(bytes=rec["bytes"] + con["bytes"], flops=rec["flops"] + con["flops"])
    return rec


def exact(case, seed):
    """Tracks are whole numbers: no value here.  Consolidation: the copied
    coordinates and the least-squares states in 64 bits."""
    if case["what"] != "consolidate" or case["events"] > 2500:
        return None
    b = _batch(case, seed)
    _, tho, th = _truth_tracks(b)
    T, A = tho.size - 1, th.size
    n = np.diff(tho).astype(np.int64)
    eto = _truth_tracks(b)[0]
    ev = np.repeat(np.arange(b.n_events), np.diff(eto))
    g = np.repeat(b.event_offsets[ev].astype(np.int64), n) + th
    x, y, z = (a[g].astype(np.float64) for a in (b.x, b.y, b.z))
    t = np.repeat(np.arange(T), n)

    def total(v):
        return np.bincount(t, weights=v, minlength=T)
    xm, ym, zm = total(x) / n, total(y) / n, total(z) / n
    dz = z - zm[t]
    szz = total(dz * dz)
    tx, ty = total(dz * (x - xm[t])) / szz, total(dz * (y - ym[t])) / szz
    rx, ry = x - (xm[t] + tx[t] * dz), y - (ym[t] + ty[t] * dz)
    c2 = total(rx * rx + ry * ry) / (2 * n - 4)
    size = _capacity(case)

    def padded(v, m):
        o = np.zeros(m, np.float64)
        o[:v.size] = v
        return o
    state = np.stack([xm, ym, zm, tx, ty, c2], 1).reshape(-1)
    return dict(hit_x=padded(x, size), hit_y=padded(y, size), hit_z=padded(z, size),
                state=padded(state, 6 * (size // 3)))
