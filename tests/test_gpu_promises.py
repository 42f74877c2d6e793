"""False layout promises without VALIDATE: the outputs are unspecified, but
every call stays inside its buffers and leaves ids in their ranges. Each call
runs on a workspace of exactly the size it asks for, with a guard behind it,
and on outputs that were filled with other values before."""
import numpy as np
import pytest

import cases
import parity
from paper_2609_11938_amd import opattr

pytestmark = pytest.mark.gpu

HINTS = opattr.KERNELS_STREAM_MAJOR | opattr.SEQ_DENSE | opattr.RANGES_NESTED
DEV = "cuda:0"
GUARD = 1 << 20


class _GuardedWorkspace(opattr.Workspace):
    """Exactly the bytes asked for, with a guard area behind them."""

    def get(self, nbytes):
        import torch

        self.whole = torch.full((nbytes + GUARD,), 0xA5, dtype=torch.uint8, device=self.device)
        return self.whole[:nbytes]

    def intact(self):
        return bool((self.whole[-GUARD:] == 0xA5).all())


def _poisoned(tr):
    import torch

    T, R = tr["seq"].size, tr["r_start"].size
    return opattr.Outputs(
        match=torch.full((T,), 0x5A5A5A5A, dtype=torch.int32, device=DEV),
        range_id=torch.full((T,), 0x5A5A5A5A, dtype=torch.int32, device=DEV),
        range_depth=torch.empty(R, dtype=torch.uint8, device=DEV),
        name_counts=torch.empty((tr["n_names"], 2), dtype=torch.int32, device=DEV),
        table=torch.empty((tr["n_ops"] + 1) * 192, dtype=torch.uint8, device=DEV),
        summary=torch.empty(40, dtype=torch.uint8, device=DEV))


def _run(tr, flags):
    import torch

    ws = _GuardedWorkspace(DEV)
    out = opattr.opattr_attribute(opattr.to_device(tr, DEV), flags=flags, raise_strict=False,
                                  ws=ws, outputs=_poisoned(tr))
    torch.cuda.synchronize()
    assert ws.intact()
    m, r = parity.host(out["match"]), parity.host(out["range_id"])
    assert m.min() >= -1 and m.max() < tr["pf_name"].size
    assert r.min() >= -1 and r.max() < tr["r_start"].size
    return m, r, opattr.read_diag(out["diag"])


def _stream_blocks(st, S):
    """The ranges' stream blocks as the library finds them (a 64-ary search
    for the first stream id that is not below s), whatever the order."""
    blk = []
    for s in range(S + 1):
        lo, hi = 0, st.size
        while hi - lo > 64:
            step = (hi - lo + 63) // 64
            p = np.minimum(lo + (np.arange(64) + 1) * step - 1, hi - 1)
            hit = np.flatnonzero(st[p] >= s)
            if hit.size == 0:
                lo = hi
                break
            f = int(hit[0])
            lo, hi = lo + f * step, int(p[f])
        rest = np.flatnonzero(st[lo:hi] >= s)
        blk.append(lo + int(rest[0]) if rest.size else hi)
    return blk


@pytest.mark.parametrize("n_names", [40, 2100])
@pytest.mark.parametrize("S", [3, 1100])
def test_false_nesting_promise_foreign_streams(n_names, S):
    """Ranges promised in nesting order with ranges of other streams inside a
    stream's block: of an id past the last one (first of a tile, so that no
    parent is found there), and of other valid streams with an end beyond all
    others. Their tiles are looked up by a stream whose block does not hold
    them. Compact path and range kernels of their own (names), tile bases
    found in the tiles and by a kernel (streams)."""
    tr = cases.random_trace(4100 + n_names + S, T=40_000, S=S, n_names=n_names, R=16, n_ops=60,
                            t_max=400_000)
    tr, _, _ = cases.stream_major(tr)
    # stream 1's block of several tiles, the others' small
    R = 8_003
    st = np.sort(np.where(np.arange(R) < 6_000, 1, np.arange(R) % S)).astype(np.uint16)
    first = int(np.searchsorted(st, 1))
    start = np.sort(np.random.default_rng(S).integers(0, 400_000, R)).astype(np.uint64)
    end = start + np.arange(R, dtype=np.uint64) % 50
    planted = [first + 1024 * k for k in (1, 2, 3)]
    st[planted] = [65535, S + 1, 60_000]
    others = [first + 1024 * k + 7 for k in (1, 2, 3)]
    st[others] = [S - 1, 0, S - 1]
    end[others] = (1 << 40) + np.arange(3)
    tr.update(r_start=start, r_end=end, r_stream=st, r_op=(np.arange(R) % 60).astype(np.uint32))
    blk = _stream_blocks(st, S)
    held = [any(blk[s] <= x < blk[s + 1] for s in range(S)) for x in planted + others]
    print(f"case false nesting names={n_names} S={S} R={R} held={held}", flush=True)
    assert any(held[:3]) and any(held[3:])
    _run(tr, HINTS)
    _, _, diag = _run(tr, HINTS | opattr.VALIDATE)
    assert diag["status"] in (-8, -9) and diag["flags"] & opattr.F_ORDER


@pytest.mark.parametrize("T", [30_000, (1 << 20) + 77])
@pytest.mark.parametrize("kind", ["shared", "past_end"])
def test_false_density_promise_any_order(T, kind):
    """Dense seq promised for launches in any order, with values shared by
    launches or past the end: launches that no rank holds have ids all the
    same (compact path, and the permutation of longer lists)."""
    tr = cases.random_trace(4200 + T % 97, T=T, S=3, n_names=20, R=T // 20, n_ops=30,
                            t_max=10 * T, max_depth=4)
    seq = tr["seq"].copy()
    seq[::3] = T // 2 if kind == "shared" else T + 5 + np.arange(seq[::3].size)
    tr["seq"] = seq
    print(f"case false density T={T} {kind}", flush=True)
    m, r, _ = _run(tr, opattr.SEQ_DENSE)
    if kind == "past_end":
        assert (m[::3] == -1).all() and (r[::3] == -1).all()
