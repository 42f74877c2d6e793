"""Parity of opattr_attribute's paths of at most 16384 operator rows: the
compact path (up to 2^20 launches), and the fused path (stream-major launches
with dense seq, or permuted into that order), where the matching stops at the
eligible launches, one pass resolves every launch's match with the dedup
broadcast, and one reduces the launches by operator row: runs in place (long
lists with few ranges; block partials sorted by row bucket, then added per
bucket), launches ordered by row in each block, or a table in LDS.

Random traces with ties, partitions, drops, extra profiled rows, range kinds
and non-default aggregation kinds, sized so that some blocks hold more runs
than they keep (the rest go through the row accumulators)."""
import numpy as np
import pytest

import cases
import parity
import paths
from oracle import oracle as O
from paper_2609_11938_amd import opattr, tracegen as tg

pytestmark = pytest.mark.gpu

HINTS = opattr.KERNELS_STREAM_MAJOR | opattr.SEQ_DENSE | opattr.RANGES_NESTED
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def _setup():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    opattr.library()
    O.build(force=False)


def _run(tr, flags=HINTS, path=None, **kw):
    import torch

    dt = opattr.to_device(tr, DEV) if isinstance(tr["seq"], np.ndarray) else tr
    if path:  # the path the test is meant for
        assert paths.attribute(dt, flags, **kw) == path
    out = opattr.opattr_attribute(dt, flags=flags, raise_strict=False, **kw)
    torch.cuda.synchronize()
    return out, opattr.read_diag(out["diag"])


@pytest.mark.parametrize("seed", range(16))
def test_fused_random(seed):
    """Compact, or fused in the seeds with range kinds."""
    T = 20_000 + 1777 * seed
    _random(seed, T, "fused" if seed % 5 == 3 else "compact")


@pytest.mark.parametrize("seed", [0, 2, 3, 7])
def test_run_reduction_random(seed):
    """The same from the launch count on from which runs are reduced in place:
    duplicate layers and extra rows, absent counters, range and aggregation
    kinds."""
    _random(seed, paths.LONG + 1777 * seed, "fused")


def _random(seed, T, path):
    tr = cases.random_trace(5000 + seed, T=T, S=1 + seed % 6, n_names=7 + 3 * seed,
                            R=T // (17 + 7 * (seed % 4)), n_ops=13 + 50 * seed,
                            t_max=T * (3 + seed % 5), max_depth=1 + seed % 7,
                            dedup=seed % 2 == 0, drop=0.1 if seed % 4 == 1 else 0.0,
                            extra_pf=0.05 if seed % 4 == 2 else 0.0)
    tr, _, _ = cases.stream_major(tr)
    if seed % 5 == 3:
        tr = cases.with_kinds(tr, seed)
    kw = {}
    if seed % 3 == 1:
        kw["agg_kind"] = np.array([(c * 7 + seed) % 3 for c in range(20)], np.uint8)
    if seed % 7 == 2:
        kw["absent_mask"] = (1 << 5) | (1 << 17)
    print(f"case fused seed={seed} T={T} R={tr['r_start'].size} G={tr['n_ops'] + 1}", flush=True)
    want = O.attribute(tr, **kw)
    out, diag = _run(tr, path=path, **kw)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("policy", [opattr.MISMATCH_PREFIX, opattr.MISMATCH_SKIP_NAME,
                                    opattr.MISMATCH_STRICT])
def test_fused_lstm_policies(policy):
    """The LSTM shape (5% of launches missing from the profiled list, 85% of
    kernel time outside every range) under the three count policies."""
    tr = tg.generate("lstm", emission="stream_major")
    want = O.attribute(tr, policy=policy)
    out, diag = _run(tr, policy=policy)
    parity.assert_attribute(out, want, diag)


def _regular_trace(T, run, n_ops, cycle, seed, with_ranges=True, NC=20):
    """One stream, launches 10 ns apart (5 ns long); each range covers `run`
    consecutive launches, the operators of consecutive ranges cycling over
    0 .. cycle-1; every launch has a profiled row in launch order."""
    rng = np.random.default_rng(seed)
    seq = np.arange(T, dtype=np.uint32)
    start = (np.arange(T, dtype=np.uint64) * 10).astype(np.uint64)
    dur = np.full(T, 5, dtype=np.uint32)
    name = (np.arange(T) % 7).astype(np.uint32)
    R = T // run if with_ranges else 0
    j = np.arange(R, dtype=np.uint64)
    r_start = (j * run * 10).astype(np.uint64)
    r_end = ((j * run + run - 1) * 10 + 5).astype(np.uint64)
    return dict(seq=seq, start_ns=start, dur_ns=dur, stream_id=np.zeros(T, np.uint16),
                name_id=name, part_id=None, pf_name=name.copy(),
                counters=rng.random((T, NC), dtype=np.float32), r_start=r_start, r_end=r_end,
                r_stream=np.zeros(R, np.uint16), r_op=(np.arange(R) % cycle).astype(np.uint32),
                part_rep=None, n_names=7, n_streams=1, n_ops=n_ops, n_parts=0)


@pytest.mark.parametrize("T,path", [(400_000, "compact"), (paths.LONG, "fused")])
def test_fused_combine_list_overflow(T, path):
    """More partial results for one bucket of operator rows in a combine
    wave's round than its LDS list holds: 64 operators of one bucket, each in
    every block, over more blocks than one round lists (the per-entry path)."""
    tr = _regular_trace(T=T, run=32, n_ops=16383, cycle=64, seed=91)
    print(f"case combine overflow T={tr['seq'].size} R={tr['r_start'].size}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, path=path)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("with_ranges", [False, True])
@pytest.mark.parametrize("T,path", [(300_000, "compact"), (paths.LONG, "fused")])
def test_fused_unattributed(with_ranges, T, path):
    """No ranges at all (every launch in the unattributed row, which has a
    partial in every block and combine waves of its own), and ranges whose
    operator rows all fall in the unattributed row's bucket."""
    tr = _regular_trace(T=T, run=40, n_ops=3, cycle=3, seed=92, with_ranges=with_ranges)
    print(f"case unattributed T={T} ranges={with_ranges}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, path=path)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("n_names", [9, paths.COMPACT_NAMES + 1])  # compact, or its own kernels
@pytest.mark.parametrize("T,per_range,n_ops,S", [
    (1, 1, 1, 1), (511, 2, 16383, 1), (512, 3, 2, 2), (513, 2, 700, 3),
    (2 ** 18 + 1, 2, 5000, 4), (2 ** 20 + 1, 3, 900, 5),  # four launches a lane
    (1023, 2, 703, 2), (1025, 2, 704, 2),                  # the largest table in LDS, one row more
    (2 ** 18 + 1, 40, 703, 3), (2 ** 19 + 1, 2, 50, 2), (2 ** 20 + 1, 5, 300, 4),
])
def test_row_order_edges(T, per_range, n_ops, S, n_names):
    """Launches ordered by operator row inside each block, or added to a
    table in LDS: block, wave and lane edges, one launch, the widest row
    table, the sizes at which the launches per lane change; rows inside a
    lane, across lanes and waves."""
    tr = cases.random_trace(6000 + T % 977, T=T, S=S, n_names=n_names, R=max(1, T // per_range),
                            n_ops=n_ops, t_max=4 * T + 8, max_depth=4)
    tr, _, _ = cases.stream_major(tr)
    print(f"case row order T={T} R={tr['r_start'].size} G={n_ops + 1} names={n_names}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, path="compact" if n_names == 9 and T <= paths.COMPACT_MAX else "fused")
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T,S,n_names,n_ops,order", [
    (1, 1, 1, 1, "any"), (1024, 3, 2048, 40, "any"), (1025, 3, 2048, 900, "gaps"),
    (1023, 2, 2049, 40, "stream"),            # more names than the compact tiles count
    (70_001, 5, 33, 703, "gaps"), (70_001, 5, 33, 704, "any"),
    (2 ** 18 + 3, 4, 700, 60, "any"),         # four launches a thread of a tile from here on
    (2 ** 20, 7, 300, 500, "stream"), (2 ** 20, 7, 300, 5000, "gaps"),
    (40_000, 1000, 20, 300, "any"),           # a range tile per stream
])
def test_compact_edges(T, S, n_names, n_ops, order):
    """At most a million launches in any order: tile and block edges, the
    most names, streams and rows of each form, dense seq in any order and
    seq with gaps, duplicate layers, drops, more rows than launches."""
    tr = cases.random_trace(6500 + T % 991 + S, T=T, S=S, n_names=n_names, R=T // 6, n_ops=n_ops,
                            t_max=8 * T + 8, max_depth=5, dedup=T > 100, drop=0.02,
                            extra_pf=0.5 if T < 2000 else 0.01, seq_gaps=order == "gaps")
    flags = {"any": opattr.SEQ_DENSE, "gaps": 0, "stream": HINTS}[order]
    if order == "stream":
        tr, _, _ = cases.stream_major(tr)  # and starts that do not decrease along a stream
        tr["start_ns"] = tr["start_ns"][np.lexsort((tr["start_ns"], tr["stream_id"]))]
    print(f"case compact T={T} S={S} names={n_names} ops={n_ops} {order}", flush=True)
    for extra in (0, opattr.VALIDATE):
        want = O.attribute(tr)
        out, diag = _run(tr, flags=flags | extra)
        parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T,kind", [
    (1, "even"), (1023, "even"), (50_001, "even"), (2 ** 20 + 9, "even"), (8192, "dense"),
    (70_000, "far"), (70_000, "ends"), (300_000, "captures"),
    (70_000, "pairs"), (20_000, "same"), (1025, "same"),
    (600_001, "far"), (600_001, "far_pair"), (300_000, "same"),
    (100_001, 4096), (100_001, 4097), (100_001, 8192), (100_001, 8193), (100_001, 33_000)])
def test_launch_ranks_by_buckets(T, kind):
    """Ranks of launches whose seq is not promised dense: the smallest and
    largest values, one far value beside a dense run (buckets of 2^18 values,
    most of them empty), two captures far apart, and equal values, whose
    ranks go by input index, in small buckets and in one larger than a
    bucket's own count of smaller launches takes (by the sort of all pairs, in
    stretches of one tile and of several). A number: clumps of that many
    consecutive values far apart, around the sizes from which a bucket is
    ranked in parts."""
    rng = np.random.default_rng(T)
    tr = cases.random_trace(6900 + T % 977, T=T, S=3, n_names=min(T, 70), R=T // 8, n_ops=50,
                            t_max=8 * T + 8, max_depth=5, dedup=False)
    if kind == "even":
        seq = np.sort(rng.choice(np.arange(0, 2 ** 32 - 1, 2 ** 32 // (2 * T)), T, replace=False))
    elif kind == "dense":
        seq = np.arange(T) + 77
    elif kind == "far":
        seq = np.append(np.arange(T - 1) + 5, 2 ** 32 - 1)
    elif kind == "far_pair":
        seq = np.append(np.arange(T - 1) + 5, 2 ** 32 - 1)
        seq[T // 3] = seq[T // 3 + 1]
    elif not isinstance(kind, str):
        seq = np.arange(T) // kind * (1 << 24) + np.arange(T) % kind
    elif kind == "ends":
        seq = np.append(np.arange(T // 2), 2 ** 32 - T + T // 2 + np.arange(T - T // 2))
    elif kind == "captures":
        seq = np.append(np.arange(T // 2), 3_000_000_000 + 7 * np.arange(T - T // 2))
    elif kind == "pairs":
        seq = np.arange(T) // 2 * 1000
    else:
        seq = np.full(T, 12345)
    tr["seq"] = rng.permutation(seq).astype(np.uint32)
    print(f"case launch ranks T={T} {kind}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, flags=0)
    parity.assert_attribute(out, want, diag)
    assert bool(diag["flags"] & opattr.F_ORDER) == (kind in ("pairs", "same", "far_pair"))


def test_launch_ranks_time_of_uneven_and_equal_values():
    """A far value beside a dense run, and equal values in a large bucket, cost
    a few times an even spread, not a serial pass over the list (500k launches:
    217 us the call for an even spread, 280 with a far value, 430 with a pair
    of equal ones too, 230 all equal)."""
    import torch

    T = 500_000
    rng = np.random.default_rng(1)
    tr = cases.random_trace(6990, T=T, S=3, n_names=70, R=T // 20, n_ops=50, t_max=8 * T + 8,
                            max_depth=5)
    far = np.append(np.arange(T - 1), 2 ** 32 - 1)
    pair = far.copy()
    pair[T // 3] = pair[T // 3 + 1]
    us = {}
    for kind, seq in (("even", 3 * np.arange(T)), ("far", far), ("pair", pair),
                      ("same", np.full(T, 7))):
        print(f"case launch ranks time {kind}", flush=True)
        tr["seq"] = rng.permutation(seq).astype(np.uint32)
        dt, ws = opattr.to_device(tr, DEV), opattr.Workspace(DEV)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(12)]
        for e in ev:
            opattr.opattr_attribute(dt, flags=0, ws=ws, raise_strict=False)
            e.record()
        torch.cuda.synchronize()
        us[kind] = np.median([a.elapsed_time(b) * 1e3 for a, b in zip(ev[1:], ev[2:])])
    print(us, flush=True)
    assert us["far"] < 2.5 * us["even"]
    assert us["pair"] < 6 * us["even"] and us["same"] < 6 * us["even"]


@pytest.mark.parametrize("R,t_max", [(1024, 4000), (1025, 50), (4097, 9000), (5000, 3),
                                     (2 ** 17, 300_000), (2 ** 17 + 1, 300_000)])
def test_unordered_ranges_merge_passes(R, t_max):
    """Ranges in any order around the tile of the sort, a group of runs and
    the size from which runs are merged in pairs, some with many ties."""
    rng = np.random.default_rng(R)
    tr = cases.random_trace(7200 + R % 97, T=20_000, S=3, n_names=20, R=64, n_ops=30, t_max=t_max)
    st = rng.integers(0, 3, R).astype(np.uint16)
    start = rng.integers(0, t_max + 1, R).astype(np.uint64)
    tr.update(r_stream=st, r_start=start, r_end=start + rng.integers(0, 4, R).astype(np.uint64),
              r_op=rng.integers(0, 30, R).astype(np.uint32))
    print(f"case merge passes R={R} t_max={t_max}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, flags=0)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T,S,kinds,dense", [
    (1, 1, False, False), (4095, 63, False, False), (4097, 63, True, True),
    (70_001, 5, True, False), (70_001, 63, False, True), (2 ** 20 + 1, 3, False, False)])
def test_permuted_launches(T, S, kinds, dense):
    """Launches in another order that the compact path leaves (more names,
    range kinds, more launches): permuted by their ranks, with gaps in seq or
    without, at tile edges, with the most streams and streams past the last."""
    tr = cases.random_trace(7100 + T % 983 + S, T=T, S=S, n_names=30 if kinds or T > 2 ** 20 else 2100,
                            R=max(1, T // 18), n_ops=90, t_max=6 * T + 8, max_depth=5,
                            dedup=T > 5000, drop=0.02, seq_gaps=not dense)
    if kinds:
        tr = cases.with_kinds(tr, 3)
    if S == 63:
        tr["stream_id"] = tr["stream_id"].copy()
        tr["stream_id"][::701] = 63 + np.arange(len(range(0, T, 701))) % 3
    print(f"case permuted T={T} S={S} kinds={kinds} dense={dense}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr, flags=opattr.SEQ_DENSE if dense else 0, path="permuted")
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("kinds", [False, True])
def test_row_order_more_partials_than_room(kinds):
    """Query points that jump back and forth change the innermost range far
    more often than the ranges' starts and ends: far more short stretches than
    ranges, kept as launch records."""
    rng = np.random.default_rng(5)
    T, R = 120_000, 400
    tr = _regular_trace(T=T, run=T // R, n_ops=900, cycle=R, seed=93)
    tr["start_ns"] = (rng.permutation(T).astype(np.uint64) * 10).astype(np.uint64)
    kw = dict(agg_kind=np.array([(c * 7 + 1) % 3 for c in range(20)], np.uint8)) if kinds else {}
    tr["counters"][::971, 5] = np.nan
    print(f"case row order overflow T={T} R={R} kinds={kinds}", flush=True)
    want = O.attribute(tr, **kw)
    out, diag = _run(tr, **kw)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T,n_ops,path", [
    (3 << 19, 900, "fused"), ((3 << 19) + 1, 900, "fused"),  # four, eight launches a lane
    (paths.ROW_MAX, 900, "fused"), (paths.ROW_MAX + 1, 900, "general"),
    (paths.ROW_MAX + 1, paths.TAB_ROWS - 1, "fused")])
def test_row_order_long_lists(T, n_ops, path):
    """Short runs of long stream-major lists: ordered by row up to a size, above
    it by the general path, and by row tables whatever the size. (The oracle
    would take minutes for so many flat ranges: launch i is in range i // run
    and takes row i.)"""
    run = 3
    tr = _regular_trace(T=T, run=run, n_ops=n_ops, cycle=n_ops, seed=95)
    print(f"case row order long T={T} n_ops={n_ops}", flush=True)
    out, diag = _run(tr, path=path, agg_kind=np.full(20, opattr.AGG_SUM, np.uint8))
    i = np.arange(T)
    rid = np.where(i // run < T // run, i // run, -1)
    op = np.where(rid < 0, n_ops, rid % n_ops)
    assert diag["status"] == 0
    assert np.array_equal(parity.host(out["match"]), i)
    assert np.array_equal(parity.host(out["range_id"]), rid)
    got, n = out.table_host(), np.bincount(op, minlength=n_ops + 1)
    for f, want in (("kernel_count", n), ("total_ns", 5 * n), ("matched_count", n),
                    ("matched_ns", 5 * n)):
        assert np.array_equal(got[f], want), f
    for c in range(20):
        want = np.bincount(op, weights=tr["counters"][:, c], minlength=n_ops + 1)
        want[n == 0] = np.nan
        parity.assert_values_close(got["value"][:, c], want, 1e-12)


@pytest.mark.parametrize("T,n_names,kinds,cols", [
    (700, 7, False, False), (40_000, 7, False, True), (40_000, 2100, True, False),
    (300_000, 7, True, False), (2 ** 20 + 700, 7, False, False)])
def test_row_order_short_and_long_stretches(T, n_names, kinds, cols):
    """Operators of one to a dozen launches in a wave, beside one that holds half
    of the launches and unattributed ones: stretches on both sides of the
    length from which a block adds them up itself, and more launch records of
    one bucket than a combine wave lists at once (64 operators of one bucket,
    each a few times in every block), with NaN counters."""
    rng = np.random.default_rng(T)
    tr = _regular_trace(T=T, run=1, n_ops=16383, cycle=1, seed=94)
    tr["name_id"] = (np.arange(T) % n_names).astype(np.uint32)
    tr["pf_name"], tr["n_names"] = tr["name_id"].copy(), n_names
    u = rng.random(T)
    op = np.select([u < 0.5, u < 0.7, u < 0.85], [np.full(T, 5000), rng.integers(0, 64, T),
                                                  rng.integers(200, 208, T)],
                   rng.integers(0, 16383, T))
    keep = rng.random(T) > 0.05
    for f in ("r_start", "r_end", "r_stream"):
        tr[f] = tr[f][keep]
    tr["r_op"] = op[keep].astype(np.uint32)
    tr["counters"][::971, 5] = np.nan
    tr["counters"][::973, 19] = np.nan
    kw = dict(agg_kind=np.array([(c * 7 + 1) % 3 for c in range(20)], np.uint8)) if kinds else {}
    print(f"case row order stretches T={T} names={n_names} kinds={kinds} cols={cols}", flush=True)
    want = O.attribute(tr, **kw)
    dt = opattr.to_device(tr, DEV)
    if cols:
        dt["counters"] = dt["counters"].t().contiguous().t()
    out, diag = _run(dt, **kw)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T,path", [(30_000, "compact"), (paths.LONG, "fused")])
def test_fused_dedup_errors(T, path):
    """Duplicates whose representative is shorter or has another name at a
    position, and a partition split in two: the same dedup errors, statuses
    and outputs as the oracle."""
    tr = cases.random_trace(4711, T=T, S=3, n_names=9, R=T // 25, n_ops=40, t_max=3 * T,
                            max_depth=4, dedup=True)
    tr, _, _ = cases.stream_major(tr)
    part = tr["part_id"].copy()
    names = tr["name_id"].copy()
    order = np.argsort(tr["seq"])
    ps = part[order]
    dup = np.flatnonzero(ps >= 0)
    # another name at some duplicate positions
    names[order[dup[5::97]]] = (names[order[dup[5::97]]] + 1) % tr["n_names"]
    t = dict(tr, name_id=names)
    want = O.attribute(t)
    out, diag = _run(t, path=path)
    assert want["diag"]["dedup_errors"] > 0
    parity.assert_attribute(out, want, diag)
    # a hole in one partition
    first = dup[0]
    ps2 = ps.copy()
    ps2[first + 1] = -1
    part2 = part.copy()
    part2[order] = ps2
    t2 = dict(tr, part_id=part2)
    want2 = O.attribute(t2)
    out2, diag2 = _run(t2, path=path)
    assert want2["diag"]["status"] == diag2["status"] != 0
    parity.assert_attribute(out2, want2, diag2)


@pytest.mark.parametrize("T,path", [(60_000, "compact"), (paths.LONG, "fused")])
def test_fused_graph_replay(T, path):
    """The compact path and the fused path (caller stream and both side
    streams) captured in a HIP graph replay to the oracle's outputs, replay
    after replay, with the outputs poisoned and eager work in between."""
    import torch

    tr = cases.random_trace(808, T=T, S=4, n_names=31, R=T // 25, n_ops=300, t_max=4 * T,
                            max_depth=5, dedup=True)
    tr, _, _ = cases.stream_major(tr)
    want = O.attribute(tr)
    dt = opattr.to_device(tr, DEV)
    assert paths.attribute(dt, HINTS) == path
    ws = opattr.Workspace(DEV)
    R = tr["r_start"].size
    o = opattr.Outputs(
        match=torch.empty(T, dtype=torch.int32, device=DEV),
        range_id=torch.empty(T, dtype=torch.int32, device=DEV),
        range_depth=torch.empty(R, dtype=torch.uint8, device=DEV),
        name_counts=torch.empty((tr["n_names"], 2), dtype=torch.int32, device=DEV),
        table=torch.empty((tr["n_ops"] + 1) * 192, dtype=torch.uint8, device=DEV),
        summary=torch.empty(40, dtype=torch.uint8, device=DEV))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        opattr.opattr_attribute(dt, flags=HINTS, ws=ws, outputs=o, raise_strict=False)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        opattr.opattr_attribute(dt, flags=HINTS, ws=ws, outputs=o, raise_strict=False)
    for rep in range(4):
        for k in ("match", "range_id", "table", "summary", "range_depth", "name_counts"):
            o[k].fill_(0x5A if o[k].dtype == torch.uint8 else -7)
        # eager work on the same workspace between replays
        opattr.opattr_attribute(dt, flags=HINTS, ws=ws, raise_strict=False)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        print(f"case fused graph replay {rep}", flush=True)
        parity.assert_attribute(o, want, opattr.read_diag(o["diag"]))


@pytest.mark.parametrize("n_names", [512, 513])
@pytest.mark.parametrize("dedup", [False, True])
def test_fused_ranking_waves(n_names, dedup):
    """On either side of the name count up to which a tile is ranked by
    sixteen waves, with full buckets and, by layer duplicates, mostly empty
    ones; bad names among the profiled rows and the launches."""
    T = (1 << 20) + 4_099
    tr = cases.random_trace(8100 + n_names, T=T, S=5, n_names=n_names, R=T // 40, n_ops=900,
                            t_max=20 * T, max_depth=3, dedup=dedup, drop=0.02)
    tr, _, _ = cases.stream_major(tr)
    tr["name_id"][::100_003] = n_names
    tr["pf_name"][::70_001] = n_names + 3
    print(f"case ranking waves names={n_names} dedup={dedup}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("T", [1 << 22, (1 << 22) + 1])
def test_fused_short_call_edge(T):
    """The launch count up to which a lane reduces four launches, not eight,
    and one launch scans the tiles' name counts, and one more."""
    tr = cases.random_trace(8300, T=T, S=3, n_names=70, R=T // 30, n_ops=900, t_max=20 * T,
                            max_depth=3)
    tr, _, _ = cases.stream_major(tr)
    print(f"case short call edge T={T}", flush=True)
    want = O.attribute(tr)
    out, diag = _run(tr)
    parity.assert_attribute(out, want, diag)


@pytest.mark.parametrize("n_ops", [705, 8_190, 8_192, 16_383])
def test_compact_row_sums_precision(n_ops):
    """One row in every block's partials, on either side of the rows a bucket's
    copies are halved at: the sums within 8 roundings (8.9e-16, relative) of
    sums in extended precision, where additions one after the other over 1500
    partials leave more."""
    T = 180_157
    tr = _regular_trace(T, 5, n_ops, min(n_ops, 900), seed=31)
    order = np.random.default_rng(5).permutation(T)
    tr["dur_ns"] = np.random.default_rng(6).integers(1, 5, size=T).astype(np.uint32)
    rs = tr["r_start"].size
    keep = np.arange(rs) % 7 == 0  # six launches in seven outside every range
    for f in ("r_start", "r_end", "r_stream", "r_op"):
        tr[f] = tr[f][keep]
    given = {f: (tr[f][order] if f in ("seq", "start_ns", "dur_ns", "stream_id", "name_id") else v)
             for f, v in tr.items()}
    print(f"case compact row sums n_ops={n_ops}", flush=True)
    want = O.attribute(given)
    out, diag = _run(given, flags=opattr.SEQ_DENSE)
    parity.assert_attribute(out, want, diag)
    row = out.table_host()[n_ops]
    un = parity.host(out["range_id"]) < 0
    c = tr["counters"].astype(np.longdouble)[given["seq"][un]]  # every launch has its own row
    d = given["dur_ns"][un].astype(np.longdouble)
    assert np.array_equal(parity.host(out["match"]), given["seq"])
    for k in range(20):
        if k in (17, 19):
            continue
        ref = c[:, k].sum() if k in (0, 1, 2, 10, 14, 18) else (c[:, k] * d).sum() / d.sum()
        assert abs(row["value"][k] - ref) <= 8.9e-16 * ref, (k, row["value"][k], ref)


@pytest.mark.parametrize("T,run,n_ops,cover", [
    (1_000_000, 4, 500, 1.0),            # tables in LDS
    (2 ** 20 + 50_000, 5, 600, 1.0),     # more launches than the compact path takes
    (2 ** 20 + 50_000, 40, 5000, 0.1)])  # unattributed launches: 32 shares of their row
def test_table_rounding(T, run, n_ops, cover):
    """The relative errors of duration-weighted means against extended precision,
    root mean square: a rounding of a value leaves 0.42 * 2^-53 = 4.7e-17; the
    division leaves one, a sum in pairs one in its last step, half the
    variance in the one before, and so on, together sqrt 3 times that, sqrt 4.5
    = 1.0e-16 with the steps inside the blocks. One after the other, the last
    ten partial results leave 1.1e-16 and 32 of them 1.6e-16."""
    tr = _regular_trace(T, run, n_ops, n_ops, seed=32)
    rng = np.random.default_rng(7)
    tr["r_op"] = rng.integers(0, n_ops, tr["r_op"].size).astype(np.uint32)
    keep = rng.random(tr["r_start"].size) < cover
    for f in ("r_start", "r_end", "r_stream", "r_op"):
        tr[f] = tr[f][keep]
    # products of 48 bits, so that their sums are not exact
    tr["dur_ns"] = rng.integers(2 ** 20, 2 ** 24, size=T).astype(np.uint32)
    tr["counters"] = np.exp(rng.standard_normal((T, 20), dtype=np.float32))
    print(f"case table rounding T={T} n_ops={n_ops} cover={cover}", flush=True)
    out, diag = _run(tr, agg_kind=np.full(20, opattr.AGG_DWMEAN, np.uint8))
    assert diag["status"] == 0 and np.array_equal(parity.host(out["match"]), tr["seq"])
    rid = parity.host(out["range_id"])
    op = np.where(rid < 0, n_ops, tr["r_op"][np.maximum(rid, 0)]).astype(np.int64)
    order = np.argsort(op, kind="stable")
    if cover < 1:  # the unattributed row
        order = order[op[order] == n_ops]
    first = np.flatnonzero(np.diff(op[order], prepend=-1))
    got = out.table_host()["value"][op[order][first]].astype(np.longdouble)
    d = tr["dur_ns"][order].astype(np.longdouble)[:, None]
    want = (np.add.reduceat(tr["counters"][order] * d, first) / np.add.reduceat(d, first))
    rms = float(np.sqrt((((got - want) / want) ** 2).mean()))
    print(f"error {rms:.2e}", flush=True)
    assert rms <= 1.0e-16
