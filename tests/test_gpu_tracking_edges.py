"""The LDS form of the tracking stages at the sizes where it can go wrong,
against the oracle, byte for byte (tracks are whole numbers: no tolerance)."""

import numpy as np
import pytest

import oracle
from paper_2207_03936_amd import sbt, synth

pytestmark = pytest.mark.gpu


def _event(rng, counts, tracks, z0=-400.0, dup=0.0):
    """An event with counts[k] hits on plane k: straight tracks through all
    planes, the rest noise; a fraction of the hits is an exact copy of
    another one of its plane (equal scores in every comparison)."""
    M = len(counts)
    mz = (-100.0 + 30.0 * np.arange(M)).astype(np.float32)
    phi = rng.uniform(-np.pi, np.pi, tracks)
    slope = rng.uniform(0.02, 0.06, tracks)
    xs, ys, zs = [], [], []
    for k, n in enumerate(counts):
        t = min(tracks, n)
        r = slope[:t] * (mz[k] - z0)
        x = r * np.cos(phi[:t]) + rng.normal(0, 0.01, t)
        y = r * np.sin(phi[:t]) + rng.normal(0, 0.01, t)
        nr, nphi = rng.uniform(5, 40, n - t), rng.uniform(-np.pi, np.pi, n - t)
        x, y = np.append(x, nr * np.cos(nphi)), np.append(y, nr * np.sin(nphi))
        if dup and n > 1:
            d = np.nonzero(rng.random(n) < dup)[0]
            src = rng.integers(0, n, d.size)
            x[d], y[d] = x[src], y[src]
        o = rng.permutation(n)
        xs.append(x[o]); ys.append(y[o]); zs.append(np.full(n, mz[k]))
    cat = lambda a: np.concatenate(a).astype(np.float32)
    return dict(x=cat(xs), y=cat(ys), z=cat(zs), module_counts=np.array(counts, np.int64),
                truth=np.full(int(sum(counts)), -1, np.int32)), mz


def _check(events, mz, tuning=None, form="batched", **over):
    b = synth.concat(events, mz)
    print(f"[gpu] {b.n_events} events, modules up to {int(np.diff(b.module_offsets).max())}, {form}, {tuning}, {over}",
          flush=True)
    want = oracle.reconstruct(b, **over)
    p = sbt.make_params(b.module_z, **over)
    dev = sbt.DeviceBatch(b)
    if form == "plain":
        got = sbt.sbt_reconstruct(p, dev).to_host()
    else:
        ctx = sbt.Context(p, b.n_events, b.n_hits, sbt.make_tuning(*tuning) if tuning else None)
        got = ctx.reconstruct(dev).to_host()
        ctx.close()
    for g, w in zip(got[:3], want):
        assert np.array_equal(g, w)
    assert not got[3].any()


@pytest.mark.parametrize("n", [1, 2, 3, 31, 32, 63, 64, 65, 96, 97, 127, 128, 129, 192, 193, 255, 256])
def test_module_sizes_at_word_and_index_edges(n):
    """Modules around the edges of flag words (32, 64 bits), of the coarse
    index's widths and of the slots, in the widths that run them."""
    rng = np.random.default_rng(n)
    ev, mz = zip(*[_event(rng, [n] * 8, t) for t in (max(1, n // 4), n)])
    for tuning in (None, (64, 4, 256), (256, 5, 256), (512, 3, 448)):
        _check(ev, mz[0], tuning)
    _check(ev, mz[0], form="plain")


@pytest.mark.parametrize("B,slots", [(64, 256), (128, 448), (256, 672), (512, 768), (512, 1024), (1024, 1536)])
def test_slot_capacity_and_track_lanes(B, slots):
    """Modules at, below and above the slots' capacity, and more tracks at a
    step than the workgroup has lanes for (run again from memory)."""
    rng = np.random.default_rng(B + slots)
    ev, mz = zip(*[_event(rng, [n] * 6, t) for n, t in ((slots - 1, 10), (slots, slots), (slots, slots // 2),
                                                       (slots + 1, 20))])
    _check(ev, mz[0], (B, 1, slots, 65536 if B == 1024 else 16384))


@pytest.mark.parametrize("misses", [0, 1, 2, 3])
@pytest.mark.parametrize("K", [4, 2, 3, 16])
def test_equal_scores_and_misses(K, misses):
    """Exact copies of hits, so that claims of a stage tie and are settled over
    64-bit words, for each number of misses a bare seed may live through."""
    rng = np.random.default_rng(10 * K + misses)
    ev, mz = zip(*[_event(rng, [int(c) for c in rng.integers(0, 2 * t, 10)], t, dup=d)
                   for t, d in ((8, 0.5), (40, 0.3), (90, 0.2))])
    for form in ("batched", "plain"):
        _check(ev, mz[0], form=form, max_doublet_candidates=K, max_consecutive_misses=misses)


@pytest.mark.parametrize("window", [0, 300, 8000, 32767])
@pytest.mark.parametrize("tuning", [(64, 4, 256), (512, 3, 448), (512, 2, 672), (1024, 1, 1536)])
def test_windows_that_close_the_circle_of_small_modules(tuning, window):
    """Walks over modules of fewer hits than a walk takes at a time, with
    windows from nothing to the full circle."""
    rng = np.random.default_rng(window)
    ev, mz = zip(*[_event(rng, rng.permutation([n, 1, 2, 3, 4, 5, 7, n, 9, n]), 4) for n in (2, 3, 4, 6, 8, 13)])
    for K in (4, 3):
        _check(ev, mz[0], tuning, phi_window_seeding=window, phi_window_forwarding=window, max_doublet_candidates=K)


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1025, 4096, 4097])
def test_batch_sizes_at_the_launch_rules(n):
    """A workgroup per event at most one per CU (no order, no counter) and
    above, and the joint scan and write up to 4,096 events and above."""
    b = synth.make_batch("tiny", n)
    print(f"[gpu] tiny x {n}", flush=True)
    want = oracle.reconstruct(b)
    dev, p = sbt.DeviceBatch(b), sbt.make_params(b.module_z)
    for tuning in (None, (64, 4, 256, 4096, 4), (64, 1, 256, 4096, 3), (256, 2, 256), (1024, 1, 1536)):
        ctx = sbt.Context(p, b.n_events, b.n_hits, sbt.make_tuning(*tuning) if tuning else None)
        got = ctx.reconstruct(dev).to_host()
        for g, w in zip(got[:3], want):
            assert np.array_equal(g, w)
        assert got[3].size == n and not got[3].any()
        ctx.close()


@pytest.mark.parametrize("n,hits,want", [(1, 2500, (512, 2, 448)), (1, 2501, (512, 1, 1024)), (1, 4500, (512, 1, 1024)),
                                         (1, 4501, (1024, 1, 1536)), (2, 5002, (1024, 1, 1536)), (-1, 3000, (512, 2, 672)),
                                         (0, 3000, (512, 3, 448))])
def test_configuration_at_the_lines_of_the_rule(n, hits, want):
    """One event by its hits; n <= 0: 8.5 events per CU, and n fewer."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rng = np.random.default_rng(hits)
    mod = [250 if hits > 2000 else 100] * 10
    mod[5] += (hits if n in (1,) else 3000) - sum(mod)
    ev, mz = _event(rng, mod, 90)
    p = sbt.make_params(mz)
    E = n if n > 0 else (17 * cus + 1) // 2 + n
    ctx = sbt.Context(p, E, hits if n > 0 else hits * E)
    t = ctx.get_tuning()
    assert (t.threads_per_event, t.blocks_per_cu, t.lds_window_hits, t.deferred_window_hits) == want + (0,)
    ctx.close()
    if n == 1:
        _check([ev], mz)


@pytest.mark.parametrize("flags", [4096, 16384, 25000, 40000])
@pytest.mark.parametrize("deferred", [0, 768])
def test_slots_of_the_six_waves_instance(deferred, flags):
    """Modules around its 448 and 480 hits, with flags that leave LDS for the
    larger slots and that do not, in one pass and in two."""
    rng = np.random.default_rng(deferred + flags)
    ev, mz = zip(*[_event(rng, [n] * 6, 150) for n in (447, 448, 449, 479, 480, 481, 600)])
    _check(ev, mz[0], (512, 3, 448, flags, 1, deferred))


@pytest.mark.parametrize("seeding", [0.0, -1.0, 1e-40, 0.04, float("inf"), float("nan")])
@pytest.mark.parametrize("forwarding", [0.0, 1e-40, 0.04, float("inf"), float("nan")])
def test_scatter_bounds_at_the_edges_of_their_type(seeding, forwarding):
    """Bounds that nothing, almost nothing and everything lies under."""
    rng = np.random.default_rng(3)
    ev, mz = zip(*[_event(rng, [t + 5] * 8, t) for t in (3, 40, 120)])
    for form in ("batched", "plain"):
        _check(ev, mz[0], form=form, max_scatter_seeding=seeding, max_scatter_forwarding=forwarding)


@pytest.mark.parametrize("n", [640, 700, 1500])
def test_events_beyond_16384_hits(n):
    """Events of more than 16,384 hits with their flags in LDS (one 1,024-lane
    workgroup per CU)."""
    rng = np.random.default_rng(n)
    ev, mz = zip(*[_event(rng, [n] * 26, n // 3) for _ in range(2)])
    _check(ev, mz[0], (1024, 1, 1536, 16384))


def _fit32(x, y, z, tho):
    """The consolidation fit in binary32, every operation in the order the
    library defines (hits of a track one after another)."""
    f = np.float32
    lo, n = tho[:-1].astype(np.int64), np.diff(tho).astype(np.int64)
    fn = n.astype(f)

    def over(step):
        for j in range(int(n.max())):
            k = np.nonzero(n > j)[0]
            step(k, x[lo[k] + j], y[lo[k] + j], z[lo[k] + j])
    acc = lambda: np.zeros(n.size, f)
    sx, sy, sz, szz, sxz, syz, c2 = (acc() for _ in range(7))

    def means(k, a, b, c):
        sx[k] += a; sy[k] += b; sz[k] += c
    over(means)
    xm, ym, zm = sx / fn, sy / fn, sz / fn

    def centred(k, a, b, c):
        dz = c - zm[k]
        szz[k] += dz * dz; sxz[k] += dz * (a - xm[k]); syz[k] += dz * (b - ym[k])
    over(centred)
    tx, ty = sxz / szz, syz / szz

    def residuals(k, a, b, c):
        dz = c - zm[k]
        rx, ry = a - (xm[k] + tx[k] * dz), b - (ym[k] + ty[k] * dz)
        c2[k] += rx * rx + ry * ry
    over(residuals)
    return np.stack([xm, ym, zm, tx, ty, c2 / (2 * n - 4).astype(f)], 1)


@pytest.mark.parametrize("sizes", [(0, 90, 400), (2899, 2900, 2901), (2899, 2901, 0, 0, 0, 0), (11599, 11600, 11601, 0),
                                   (9200, 20000)])
def test_consolidation_at_the_lds_capacities(sizes):
    """Events around the sizes that consolidation holds in LDS, in each of its
    forms (chosen by the mean event): coordinates and states equal, bit for
    bit, the same binary32 operations done in numpy (no tolerance)."""
    import torch
    rng = np.random.default_rng(sum(sizes))
    M = 26
    evs = []
    for n in sizes:
        ev, mz = _event(rng, [n // M + (1 if k < n % M else 0) for k in range(M)], max(1, n // (2 * M)))
        evs.append(ev)
    b = synth.concat(evs, mz)
    print(f"[gpu] consolidation of events of {sizes} hits", flush=True)
    eto, tho, th = oracle.reconstruct(b)
    g = np.concatenate([b.event_offsets[e] + th[tho[eto[e]]:tho[eto[e + 1]]].astype(np.int64)
                        for e in range(b.n_events)])
    want = (b.x[g], b.y[g], b.z[g], _fit32(b.x[g], b.y[g], b.z[g], tho))
    dev = sbt.DeviceBatch(b)
    out = sbt.DeviceTracks(b.n_events, b.n_hits)
    for dst, src in zip((out.eto, out.tho, out.th), (eto, tho, th)):
        dst[:len(src)] = torch.from_numpy(src).to(dst.device)
    got = sbt.sbt_consolidate(dev, out).to_host(len(tho) - 1, len(th))
    assert len(tho) > 1
    for a, w in zip(got, want):
        assert a.dtype == w.dtype and np.array_equal(a.view(np.uint32), np.ascontiguousarray(w).view(np.uint32))


@pytest.mark.parametrize("tuning", [(64, 2, 256, 4096, 3), (128, 3, 256), (256, 2, 256), (512, 2, 672)])
def test_own_events_then_the_queue(tuning):
    """Batches around the number of event groups (each group's first event is
    its own, the rest come from the counter), alone and while a batch of
    another context holds the compute units, so that groups become resident
    late and others take their events."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    groups = cus * tuning[1] * (tuning[4] if len(tuning) > 4 else 1)
    pool = synth.make_batch("tiny", 64)
    evs = [pool.event(i % 64) for i in range(2 * groups + 5)]
    evs = [dict(x=e.x, y=e.y, z=e.z, module_counts=np.diff(e.module_offsets), truth=np.full(e.x.size, -1, np.int32))
           for e in evs]
    want = [oracle.reconstruct(pool.event(i)) for i in range(64)]
    side = synth.make_batch("mu7.6", 600)
    sdev, sp = sbt.DeviceBatch(side), sbt.make_params(side.module_z)
    sctx, sout = sbt.Context(sp, side.n_events, side.n_hits), sbt.DeviceTracks(side.n_events, side.n_hits)
    streams = [torch.cuda.Stream() for _ in range(2)]
    for n in (cus + 1, groups - 1, groups, groups + 1, 2 * groups + 5):
        b = synth.concat(evs[:n], pool.module_z)
        print(f"[gpu] {n} events on {groups} groups, {tuning}", flush=True)
        dev, p = sbt.DeviceBatch(b), sbt.make_params(b.module_z)
        ctx = sbt.Context(p, b.n_events, b.n_hits, sbt.make_tuning(*tuning))
        out = sbt.DeviceTracks(b.n_events, b.n_hits)
        for beside in (False, True, True):
            torch.cuda.synchronize()
            if beside:
                sctx.reconstruct(sdev, sout, streams[0])
            ctx.reconstruct(dev, out, streams[1])
            torch.cuda.synchronize()
            eto, tho, th, st = out.to_host()
            assert not st.any()
            assert np.array_equal(np.diff(eto), [want[i % 64][0][-1] for i in range(n)])
            assert np.array_equal(th, np.concatenate([want[i % 64][2] for i in range(n)]))
            assert np.array_equal(np.diff(tho), np.concatenate([np.diff(want[i % 64][1]) for i in range(n)]))
        ctx.close()
    sctx.close()


def _peak_bound(b, e, eto, tho, th, misses):
    """At least this many forming tracks meet at a step of event e where every
    unflagged middle hit makes a seed: a seed lives through misses + 1 steps,
    and a flagged hit is on a track of the result."""
    M = b.n_modules
    mo = b.module_offsets[e * M:e * M + M + 1] - b.event_offsets[e]
    hits = th[tho[eto[e]]:tho[eto[e + 1]]]
    taken = np.bincount(np.searchsorted(mo, hits, side="right") - 1, minlength=M)
    free = (np.diff(mo) - taken)[::-1]              # by traversal index
    seeds = [free[u] if u > 0 and u + 1 < M and free[u - 1] > 1 and free[u + 1] > 1 else 0 for u in range(M)]
    return max(sum(seeds[u:u + misses + 1]) for u in range(M))


@pytest.mark.parametrize("lanes,tuning,n", [
    (256, (64, 1, 256, 16384), 250), (448, (64, 1, 448, 4096, 3), 440), (704, (64, 1, 672, 16384), 600),
    (512, (128, 2, 448, 16384), 440), (768, (128, 1, 768, 16384), 700), (256, (256, 5, 256, 16384), 250),
    (768, (256, 2, 672, 16384), 650), (1024, (512, 2, 672, 16384), 660), (512, (512, 3, 448, 16384), 470),
    (512, (512, 3, 448, 16384, 1, 768), 470), (1024, (512, 2, 768, 16384), 760), (1024, (512, 1, 1024, 16384), 1000),
    (2048, (1024, 1, 1536, 16384), 1500), (1024, None, 660)])
def test_more_tracks_than_lanes(lanes, tuning, n):
    """Events that give up the LDS form half way, with flags, links and claims
    set, because more tracks meet at a step than the workgroup has lanes and
    sets for, and are run again from memory; ordinary events beside them.
    Noise modules under a window of the whole circle and no bound on the seeds'
    scatter: every unflagged middle hit makes a seed."""
    over = dict(phi_window_seeding=32767, max_scatter_seeding=float("inf"))
    rng = np.random.default_rng(n + lanes)
    ev, mz = zip(*[_event(rng, c, 30) for c in ([n] * 4 + [45] * 6, [40] * 10, [45] * 3 + [n] * 4 + [45] * 3)])
    b = synth.concat(ev, mz[0])
    want = oracle.reconstruct(b, **over)
    for e in (0, 2):
        assert np.diff(b.module_offsets[e * 10:e * 10 + 11]).max() <= (tuning[2] if tuning else 672) + 32
        assert _peak_bound(b, e, *want, misses=1) > lanes
    assert np.diff(want[0]).min() > 10      # tracks, and with them flags, before the noise
    _check(ev, mz[0], tuning, form="batched" if tuning else "plain", **over)


@pytest.mark.parametrize("tuning,n", [(None, 539), (None, 545), (None, 630), ((512, 2, 672), 576), ((512, 2, 672), 578),
                                      ((512, 3, 448), 420), ((512, 3, 448), 430), ((256, 5, 256), 240), ((256, 5, 256), 256),
                                      ((1024, 1, 1536), 1325), ((1024, 1, 1536), 1400)])
def test_compaction_with_the_ids_in_lds_and_in_memory(tuning, n):
    """Events of 26 modules around the hits that leave no room for the ids in
    the LDS of the compaction (None: the plain form)."""
    rng = np.random.default_rng(n)
    ev, mz = zip(*[_event(rng, [n] * 26, t) for t in (n, n // 3)])
    _check(ev, mz[0], tuning, form="batched" if tuning else "plain")


def _random_tracks(rng, n, longest):
    """Disjoint tracks over a random choice of n hits, as (lengths, hit ids)."""
    ids = rng.permutation(n)[:int(0.9 * n)]
    lengths = []
    while sum(lengths) + 3 <= ids.size:
        lengths.append(int(min(ids.size - sum(lengths), rng.choice([3, 4, 11, 16, 17, 26, longest]))))
    if lengths and lengths[-1] < 3:
        lengths.pop()
    return lengths, ids[:sum(lengths)]


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("fill,sizes", [
    (0, (3, 2899, 2900, 2901, 5801, 10150, 10151, 11600, 11601)),           # one event per CU: 1,024 lanes
    (0, (40600, 40601, 65535)),
    (400, (0, 2900, 2901, 10149, 10150, 10151, 20301, 31000)),              # 256 lanes, one to four columns
    (30, (2901, 10151)),                                                    # more events than workgroups
    (5200, (5799, 5800, 5801, 20300, 20301, 41000)),                        # 512 lanes
    (11000, (100, 11599, 11601, 40601))])                                   # 1,024 lanes by the mean
def test_consolidation_of_uneven_batches(fill, sizes, pinned):
    """Events around what each form holds whole, and in one column and several,
    among many of another size (fill), with tracks of up to 64 hits: packed
    coordinates and states equal, bit for bit, the same binary32 operations
    done in numpy (no tolerance); into device and into pinned host memory."""
    import torch
    cus = 256
    rng = np.random.default_rng(fill + len(sizes))
    n = list(sizes)
    if fill == 400:
        n += [int(v) for v in rng.integers(0, 800, cus + 40)]
    elif fill == 30:
        n += [int(v) for v in rng.integers(0, 60, 9000)]
    elif fill == 5200:
        n += [int(v) for v in rng.integers(3, 9000, 3 * cus + 10)]
    elif fill:
        n += [fill] * (cus + 7)
    n = [n[i] for i in rng.permutation(len(n))]
    eo = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    mean = int(eo[-1]) // len(n)
    assert {0: len(n) <= cus, 30: len(n) > 8192 and mean <= 2300, 400: len(n) > cus and mean <= 2300, 5200: len(n) > 3 * cus and 2300 < mean <= 5100,
            11000: len(n) > cus and mean > 5100}[fill]
    print(f"[gpu] {len(n)} events of {mean} hits, pinned {pinned}", flush=True)
    x, y, z = (rng.normal(0, s, eo[-1]).astype(np.float32) for s in (20, 20, 300))
    per = [_random_tracks(rng, v, 64) for v in n]
    th = np.concatenate([p[1] for p in per]).astype(np.int32)
    tho = np.concatenate([[0], np.cumsum(np.concatenate([p[0] for p in per]))]).astype(np.int32)
    eto = np.concatenate([[0], np.cumsum([len(p[0]) for p in per])]).astype(np.int32)
    g = np.concatenate([eo[e] + per[e][1] for e in range(len(n))])
    b = synth.Batch(x=x, y=y, z=z, event_offsets=eo, module_offsets=np.repeat(eo, 3)[:3 * len(n) + 1].astype(np.int32),
                    module_z=np.arange(3, dtype=np.float32), truth=np.zeros(0, np.int32))
    dev, out = sbt.DeviceBatch(b), sbt.DeviceTracks(b.n_events, b.n_hits)
    for dst, src in zip((out.eto, out.tho, out.th), (eto, tho, th)):
        dst[:len(src)] = torch.from_numpy(src).to(dst.device)
    want = (x[g], y[g], z[g], _fit32(x[g], y[g], z[g], tho))
    got = sbt.sbt_consolidate(dev, out, sbt.TrackStates(b.n_hits, pinned=pinned))
    torch.cuda.synchronize()
    for a, w in zip(got.to_host(len(tho) - 1, len(th)), want):
        assert np.array_equal(np.asarray(a).view(np.uint32), np.ascontiguousarray(w).view(np.uint32))
