"""Which path of opattr_attribute a call takes, and the sizes at which it
changes, so that a test runs the code it is meant for.

The limits are read from the library's own header. The path is told by the
probes that a call records: the compact path has no column scan, the general
path sorts items, and the fused path, which does neither, builds a launch-order
view when it permutes the launches first."""
import os
import re

from paper_2609_11938_amd import opattr

_IMPL = os.path.join(os.path.dirname(opattr.HERE), "paper_2609_11938_amd", "csrc", "impl.h")


def const(name):
    m = re.search(rf"constexpr \w+ {name} = ([\d<> ]+);", open(_IMPL).read())
    assert m, f"{name} is not in impl.h"
    return eval(m.group(1), {})  # digits and shifts only


COMPACT_MAX = const("kCompactMax")      # launches of the compact path
COMPACT_NAMES = const("kCompactNames")  # and its names
TAB_ROWS = const("kTabMaxRows")         # operator rows of a table in LDS
ROW_MAX = const("kRowOrderMax")         # stream-major launches that are ordered by row
# launches from which runs are reduced in place (dense seq, long runs)
LONG = max(COMPACT_MAX, const("kFusedShort")) + 1


def taken(call):
    """The path of one call: compact, fused, permuted (then fused) or general."""
    import torch

    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * len(opattr.PROBES))]
    for e in ev:
        e.record()
    torch.cuda.synchronize()
    mark = torch.cuda.Event(enable_timing=True)
    mark.record()
    opattr.set_probe_events(ev)
    try:
        call()
    finally:
        opattr.set_probe_events(None)
    torch.cuda.synchronize()
    ran = {p for k, p in enumerate(opattr.PROBES) if mark.elapsed_time(ev[2 * k]) > 0}
    if "item_sort" in ran:
        return "general"
    if "agg_runs" in ran:
        return "permuted" if "seq_view" in ran else "fused"
    assert "main_pass" in ran and "col_scan" not in ran, ran
    return "compact"


def attribute(dt, flags, **kw):
    return taken(lambda: opattr.opattr_attribute(dt, flags=flags, raise_strict=False, **kw))
