"""The operator table has the same bits on every run of a call: a row's
fp64 sums are added up in an order that does not depend on scheduling.
(Except by the run reduction of the fused path, which adds a block's partials of
one row, and those past a wave's capacity, by atomics: more than 2^20 launches
with dense seq promised and at most one range per 16 launches, and noalloc calls
of such ranges that fit no other plan.)"""
import numpy as np
import pytest

import cases
import parity
from oracle import oracle as O
from paper_2609_11938_amd import opattr

pytestmark = pytest.mark.gpu

HINTS = opattr.KERNELS_STREAM_MAJOR | opattr.SEQ_DENSE | opattr.RANGES_NESTED
DEV = "cuda:0"
MIXED = np.array([(c * 7 + 2) % 3 for c in range(20)], np.uint8)


def _trace(seed, T, R, n_ops, order, n_names=30):
    tr = cases.random_trace(seed, T=T, S=4, n_names=n_names, R=R, n_ops=n_ops, t_max=4 * T,
                            max_depth=6, drop=0.01, seq_gaps=order == "gaps")
    if order == "stream":
        tr, _, _ = cases.stream_major(tr)
    # values and durations of many magnitudes, so that sums are not exact and
    # another order of the additions shows in the bits
    rng = np.random.default_rng(seed)
    tr["counters"] = np.exp(3 * rng.standard_normal(tr["counters"].shape)).astype(np.float32)
    tr["dur_ns"] = np.exp(8.5 + 1.2 * rng.standard_normal(T)).astype(np.uint32) + np.uint32(1)
    return tr, {"stream": HINTS, "dense": opattr.SEQ_DENSE, "gaps": 0}[order]


def _assert_repeats(tr, flags, runs=16, **kw):
    """Runs back to back, each beside a stream of copies that holds parts of
    the chip at other times."""
    import torch

    want = O.attribute(tr, **kw)
    dt, ws = opattr.to_device(tr, DEV), opattr.Workspace(DEV)
    side = torch.cuda.Stream()
    buf = torch.empty(2, 24 << 20, dtype=torch.uint8, device=DEV)
    outs = [opattr.opattr_attribute(dt, flags=flags, ws=ws, raise_strict=False, **kw)]
    torch.cuda.synchronize()
    parity.assert_attribute(outs[0], want, opattr.read_diag(outs[0]["diag"]))
    with torch.cuda.stream(side):
        for k in range(4 * runs):
            buf[k & 1].copy_(buf[(k + 1) & 1])
    for rep in range(runs):
        outs.append(opattr.opattr_attribute(dt, flags=flags, ws=ws, raise_strict=False, **kw))
    torch.cuda.synchronize()
    first = outs[0]["table"].view(torch.int64)
    differ = [int((o["table"].view(torch.int64) != first).sum()) for o in outs[1:]]
    assert not any(differ), differ


@pytest.mark.parametrize("T,R,n_ops,order,kind", [
    (10_000, 2_000, 200, "stream", None),         # one launch a thread
    (200_000, 50_000, 600, "gaps", None),
    (300_000, 40_000, 703, "stream", MIXED),      # two
    (1_000_000, 200_000, 400, "dense", None),     # four
    (1_100_000, 200_000, 400, "stream", None),    # more than the compact path takes
])
def test_table_in_lds_repeats(T, R, n_ops, order, kind):
    """Rows whose table fits in LDS: the waves of a block add to it in turns."""
    print(f"case repeat table T={T} R={R} ops={n_ops} {order}", flush=True)
    tr, flags = _trace(9700 + T % 97, T, R, n_ops, order)
    _assert_repeats(tr, flags, **({} if kind is None else {"agg_kind": kind}))


@pytest.mark.parametrize("T,R,n_ops,order,kind", [
    (10_000, 6_000, 5_000, "stream", None),       # two launches a lane
    (200_000, 120_000, 5_000, "gaps", None),
    (400_000, 100_000, 2_000, "dense", MIXED),    # four
    (300_000, 2_000, 1_500, "dense", None),       # few ranges: the rows change with the streams
    (1_100_000, 300_000, 3_000, "stream", None),  # more than the compact path takes
    (1_600_000, 300_000, 3_000, "stream", None),  # eight
    (1_100_000, 60_000, 1_000, "gaps", None),     # long runs, permuted by the launches' ranks
])
def test_rows_ordered_in_blocks_repeat(T, R, n_ops, order, kind):
    """Launches ordered by operator row in each block: the waves rank theirs in
    turns, and what a block keeps does not depend on the others."""
    print(f"case repeat rows T={T} R={R} ops={n_ops} {order}", flush=True)
    tr, flags = _trace(9800 + T % 97, T, R, n_ops, order)
    _assert_repeats(tr, flags, **({} if kind is None else {"agg_kind": kind}))
