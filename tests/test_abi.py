"""Host-side checks of the C ABI (no GPU needed): the library loads, exports
every entry point declared in include/opattr.h, sizes its workspace, and
rejects bad arguments before enqueueing anything."""
import ctypes as C
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2609_11938_amd import opattr

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "opattr.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(opattr.LIB_PATH):
        from paper_2609_11938_amd import build

        build.build()
    return opattr.library()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(opattr_[a-z_]+)\s*\(", text)))


def test_header_declares_the_expected_calls():
    assert declared_functions() == sorted(opattr.EXPORTS)


def test_library_exports_every_declared_symbol(lib):
    out = subprocess.run(["nm", "-D", "--defined-only", opattr.LIB_PATH], check=True,
                         capture_output=True, text=True).stdout
    exported = set(re.findall(r"\sT\s(opattr_\w+)", out))
    for f in declared_functions():
        assert f in exported, f
        assert hasattr(lib, f)


def test_struct_layouts_match_header(tmp_path):
    """Sizes and field offsets of the binding's structs, against a C program
    compiled from the header."""
    structs = {"opattr_kernels": opattr.opattr_kernels, "opattr_profiled": opattr.opattr_profiled,
               "opattr_ranges": opattr.opattr_ranges, "opattr_dims": opattr.opattr_dims,
               "opattr_diag": opattr.opattr_diag}
    lines = ['#include <stdio.h>', '#include <stddef.h>', '#include "opattr.h"', "int main(void) {"]
    for name, cls in structs.items():
        lines.append(f'  printf("{name} %zu\\n", sizeof({name}));')
        for f, _ in cls._fields_:
            lines.append(f'  printf("{name}.{f} %zu\\n", offsetof({name}, {f}));')
    lines += ['  printf("opattr_op_row %zu\\n", sizeof(opattr_op_row));', "  return 0;", "}"]
    src = tmp_path / "layout.c"
    src.write_text("\n".join(lines) + "\n")
    exe = tmp_path / "layout"
    subprocess.run(["gcc", "-std=c11", "-I", os.path.dirname(HEADER), "-o", str(exe), str(src)],
                   check=True)
    got = dict(line.split() for line in subprocess.run([str(exe)], check=True, capture_output=True,
                                                       text=True).stdout.splitlines())
    for name, cls in structs.items():
        assert int(got[name]) == C.sizeof(cls), name
        for f, _ in cls._fields_:
            assert int(got[f"{name}.{f}"]) == getattr(cls, f).offset, f"{name}.{f}"
    assert int(got["opattr_op_row"]) == opattr.OP_ROW_DTYPE.itemsize == 192


def _structs(T=100, P=50, R=10, NN=8, NS=2, NOPS=4, flags=0):
    fake = C.c_void_p(0x1000)  # never dereferenced on the host
    k = opattr.opattr_kernels(T, fake, fake, fake, fake, fake, None, None)
    p = opattr.opattr_profiled(P, fake, fake, 20, 1, 0)
    r = opattr.opattr_ranges(R, fake, fake, fake, fake, None)
    d = opattr.opattr_dims(NN, NS, NOPS, 0, None, flags)
    return k, p, r, d


def test_workspace_size_is_pure_and_monotone(lib):
    sizes = []
    for T in (0, 1, 4096, 4097, 100_000):
        k, p, r, d = _structs(T=T)
        sizes.append(lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d)))
    assert all(s > 0 for s in sizes)
    assert sizes == sorted(sizes)
    # all hints drop the reordering buffers; dense seq in another order adds
    # the permuted launch arrays of opattr_attribute (about 34 B per launch)
    k, p, r, d = _structs(T=100_000, R=5_000)
    full = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d))
    d.flags = opattr.KERNELS_STREAM_MAJOR | opattr.SEQ_DENSE | opattr.RANGES_NESTED
    hinted = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d))
    assert hinted < full
    d.flags = opattr.SEQ_DENSE | opattr.RANGES_NESTED
    permuted = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d))
    assert permuted >= hinted + 100_000 * 34
    assert lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), None) == 0


def test_workspace_for_all_inputs_covers_every_entry_point(lib):
    """The header's contract: the size computed with every input covers each
    entry point, whose own plan leaves out the inputs it does not take."""
    for flags in (0, opattr.SEQ_DENSE, opattr.KERNELS_STREAM_MAJOR | opattr.SEQ_DENSE |
                  opattr.RANGES_NESTED):
        k, p, r, d = _structs(T=100_000, P=20_000, R=5_000, NN=300, NS=8, NOPS=64, flags=flags)
        d.n_parts, d.part_rep = 16, C.c_void_p(0x3000)
        k.part_id = C.c_void_p(0x4000)
        full = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d))
        for pp, rr in ((None, None), (None, r), (p, None), (p, r)):
            part = lib.opattr_workspace_bytes(C.byref(k), C.byref(pp) if pp else None,
                                              C.byref(rr) if rr else None, C.byref(d))
            assert part <= full, (flags, pp is None, rr is None)


@pytest.mark.parametrize("T,R,NN,NS,NOPS,flags,before", [
    (500_000, 25_000, 40, 4, 899, 7, 29.4), (500_000, 25_000, 40, 4, 899, 0, 34.8),
    (96_000, 62_800, 60, 4, 5014, 7, 7.2), (1_000_000, 600_000, 100, 8, 5000, 7, 69.5),
    (1_000_000, 600_000, 100, 8, 5000, 0, 112.4), (2_000_000, 400_000, 100, 8, 5000, 7, 118.1),
    (4_000_000, 2_000_000, 100, 8, 15_999, 7, 306.5),
    (10_000_000, 5_000_000, 100, 8, 15_999, 7, 763.2)])
def test_workspace_of_row_ordered_calls(lib, T, R, NN, NS, NOPS, flags, before):
    """Blocks that order their launches by operator row keep 200 / 6 + 16 bytes a
    launch (200 / 8 + 16 with at most a range for every sixteen), in the place of
    the general aggregation's arrays (about 40 bytes), and the combine sixteen
    shares of 200 bytes a row; MiB before: of the general aggregation alone."""
    k, p, r, d = _structs(T=T, P=min(T, 400_000), R=R, NN=NN, NS=NS, NOPS=NOPS, flags=flags)
    mib = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d)) / 2 ** 20
    more = 2 if R * 16 <= T else 10
    assert mib <= before + (more * T + 17 * 200 * NOPS) / 2 ** 20 + 6, mib


def test_workspace_of_few_launches_over_many_rows(lib):
    """The combine's shares go by the launches as well as by the rows: 20,000
    launches over 15,000 rows, with more names than the compact path takes, needed
    52 MiB when it always had sixteen (2.3 MiB by the general aggregation)."""
    k, p, r, d = _structs(T=20_000, P=20_000, R=15_000, NN=3000, NS=4, NOPS=14_999, flags=7)
    assert lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d)) < 14 << 20


@pytest.mark.parametrize("T,per_range,NN,NS,NOPS,flags", [
    (921087, 20, 40, 4, 899, 0), (952320, 20, 40, 4, 899, 4), (670528, 20, 40, 4, 899, 2),
    (1168736, 20, 40, 4, 899, 7), (1094592, 3, 40, 4, 899, 7), (1105919, 3, 40, 4, 299, 7),
    (716930, 3, 40, 4, 899, 0), (915456, 3, 40, 4, 899, 2), (888960, 20, 2100, 4, 899, 0),
    (652608, 20, 2100, 4, 899, 2), (491200, 20, 2100, 16, 8999, 7),
    (801600, 2, 2100, 16, 8999, 7), (847872, 20, 5000, 4, 899, 0),
    (669632, 5, 300, 200, 19999, 0), (956544, 5, 300, 200, 19999, 7), (1255424, 60, 12, 2, 99, 7),
    (729600, 60, 12, 2, 99, 6), (975680, 60, 12, 2, 99, 4), (780161, 2, 100, 8, 4999, 5)])
def test_noalloc_accepts_what_fits_the_general_path(lib, T, per_range, NN, NS, NOPS, flags):
    """The most launches of each shape whose arrays fit the scratch by the run
    reduction and the general path alone: not refused, whatever the other paths'
    plans take (without a device the scratch's address cannot be had; a launch
    more is not asserted, other plans may take it)."""
    import torch

    if torch.cuda.device_count() > 0:
        pytest.skip("the arrays are not there to be read")
    k, p, r, d = _structs(T=T, P=T // 4, R=T // per_range, NN=NN, NS=NS, NOPS=NOPS, flags=flags)
    fake = C.c_void_p(0x1000)
    assert lib.opattr_attribute_noalloc(C.byref(k), C.byref(p), C.byref(r), C.byref(d), 0, None,
                                        fake, fake, None, None, fake, fake, fake, None) == -3


def test_argument_errors_return_before_any_device_work(lib):
    k, p, r, d = _structs()
    fake = C.c_void_p(0x1000)
    ws = C.c_void_p(0x2000)
    INVALID, WORKSPACE = -1, -2
    # NULL diag / match
    assert lib.opattr_match(C.byref(k), C.byref(p), C.byref(d), 0, fake, None, None, ws,
                            C.c_size_t(1 << 40), None) == INVALID
    assert lib.opattr_match(C.byref(k), C.byref(p), C.byref(d), 0, None, None, fake, ws,
                            C.c_size_t(1 << 40), None) == INVALID
    # policy out of range
    assert lib.opattr_match(C.byref(k), C.byref(p), C.byref(d), 3, fake, None, fake, ws,
                            C.c_size_t(1 << 40), None) == INVALID
    # negative or too large sizes
    k.n = -1
    assert lib.opattr_enclose(C.byref(k), C.byref(r), C.byref(d), fake, None, fake, ws,
                              C.c_size_t(1 << 40), None) == INVALID
    k.n = 1 << 31
    assert lib.opattr_enclose(C.byref(k), C.byref(r), C.byref(d), fake, None, fake, ws,
                              C.c_size_t(1 << 40), None) == INVALID
    k.n = 100
    # too many names, unknown flag bits
    d.n_names = 1 << 20
    assert lib.opattr_match(C.byref(k), C.byref(p), C.byref(d), 0, fake, None, fake, ws,
                            C.c_size_t(1 << 40), None) == INVALID
    d.n_names = 8
    d.flags = 1 << 7
    assert lib.opattr_match(C.byref(k), C.byref(p), C.byref(d), 0, fake, None, fake, ws,
                            C.c_size_t(1 << 40), None) == INVALID
    d.flags = 0
    # missing range arrays
    r2 = opattr.opattr_ranges(10, fake, None, fake, fake)
    assert lib.opattr_enclose(C.byref(k), C.byref(r2), C.byref(d), fake, None, fake, ws,
                              C.c_size_t(1 << 40), None) == INVALID
    # aggregation kinds out of range
    bad_kind = (C.c_uint8 * 20)(*([3] + [0] * 19))
    assert lib.opattr_aggregate(C.byref(k), C.byref(p), fake, fake, C.byref(r), C.byref(d),
                                bad_kind, fake, fake, fake, ws, C.c_size_t(1 << 40),
                                None) == INVALID
    # undersized workspace
    need = lib.opattr_workspace_bytes(C.byref(k), C.byref(p), C.byref(r), C.byref(d))
    assert lib.opattr_attribute(C.byref(k), C.byref(p), C.byref(r), C.byref(d), 0, None, fake,
                                fake, None, None, fake, fake, fake, ws, C.c_size_t(need - 1),
                                None) == WORKSPACE
    # workspace off a 256-byte boundary
    assert lib.opattr_attribute(C.byref(k), C.byref(p), C.byref(r), C.byref(d), 0, None, fake,
                                fake, None, None, fake, fake, fake, C.c_void_p(0x2010),
                                C.c_size_t(need + 256), None) == WORKSPACE
    assert lib.opattr_diag_clear(None, None) == INVALID
    assert lib.opattr_read_diag(None, None, None) == INVALID


def test_strerror_names_every_status():
    for code in range(-10, 1):
        s = opattr.strerror(code)
        assert s and s != "unknown status"
    assert opattr.strerror(-99) == "unknown status"


def test_binding_fails_loudly_without_library(tmp_path):
    with pytest.raises(RuntimeError, match="not built"):
        opattr.library(str(tmp_path / "missing.so"))


def test_to_device_rejects_bad_counters():
    tr = dict(counters=np.zeros((2, 20), np.float64))
    with pytest.raises(TypeError):
        opattr.to_device(tr, "cpu")
