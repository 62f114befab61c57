"""Lists of plain ints are converted in C, everything else with numpy: the same calls are accepted, with the same
results and the same errors, whichever way a list goes."""
import numpy as np
import pytest

import paper_2006_15704_amd as d


def context(n=5, R=2):
    ctx = d.ddp_create(R, d.DDP_DEVICE_NONE)
    d.ddp_register_params(ctx, [10 + i for i in range(n)], [0] * n, None)
    d.ddp_build_buckets(ctx, 100)
    return ctx


FORMS = [list, tuple, lambda v: np.array(v), lambda v: np.array(v, dtype=np.int64), lambda v: [np.int32(x) for x in v],
         lambda v: [float(x) for x in v], lambda v: range(4, -1, -1)]


@pytest.mark.parametrize("form", FORMS)
def test_ids_in_any_form(form):
    ctx = context()
    d.ddp_mark_ready_many(ctx, form([4, 3, 2, 1, 0]))
    assert d.ddp_get_ready_order(ctx, 0) == [4, 3, 2, 1, 0]
    d.ddp_finalize_backward(ctx)
    d.ddp_mark_ready_many(ctx, form([4, 3, 2, 1, 0])[:0])
    d.ddp_mark_ready_many(ctx, [True, 0])
    assert d.ddp_get_ready_order(ctx, 0) == [1, 0]
    d.ddp_destroy(ctx)


@pytest.mark.parametrize("ids,error", [([7], d.DdpError), ([-1], d.DdpError), ([1, 1], d.DdpError), ([1 << 31], OverflowError),
                                       ([-(1 << 31) - 1], OverflowError), ([1 << 80], OverflowError), (["x"], ValueError)])
def test_refused_ids(ids, error):
    for form in (list, tuple):
        ctx = context()
        with pytest.raises(error):
            d.ddp_mark_ready_many(ctx, form(ids))
        d.ddp_destroy(ctx)


def test_null_contexts():
    for ctx in (None, d.binding.C.c_void_p()):
        with pytest.raises(d.DdpError):
            d.ddp_mark_ready_many(ctx, [0])
        with pytest.raises(d.DdpError):
            d.ddp_no_sync_accumulate(ctx, [0])


def test_pointers():
    ctx = context()
    for ptrs in ([None] * 10, [0] * 10, tuple([256, None] * 5), np.zeros(10, dtype=np.uint64), [(1 << 64) - 4] * 10):
        with pytest.raises(d.DdpError) as e:       # nothing is computed without a device
            d.ddp_no_sync_accumulate(ctx, ptrs)
        assert e.value.code == d.DDP_ERR_NO_DEVICE
    for ptrs in ([-1] * 10, [1 << 64] * 10):
        with pytest.raises(OverflowError):
            d.ddp_no_sync_accumulate(ctx, ptrs)
    d.ddp_destroy(ctx)


@pytest.mark.parametrize("form", [list, tuple, lambda v: np.array(v, dtype=np.uint64), lambda v: [np.uint64(x) for x in v], iter])
def test_pointer_lists_of_other_lengths(form):
    """A list with an entry too few is refused before the library reads past its end; further entries are not read."""
    ctx = context(n=5, R=2)
    for length in (0, 1, 5, 9):
        with pytest.raises(ValueError):
            d.ddp_no_sync_accumulate(ctx, form([256] * length))
    for length in (10, 11):
        with pytest.raises(d.DdpError) as e:
            d.ddp_no_sync_accumulate(ctx, form([256] * length))
        assert e.value.code == d.DDP_ERR_NO_DEVICE
    d.ddp_destroy(ctx)


def test_context_free_call():
    """What is refused before a device is touched."""
    big = 1 << 30
    for form in (list, tuple, lambda v: np.array(v, dtype=np.int64)):
        with pytest.raises(d.DdpError) as e:
            d.ddp_sync_static(2, 0, 0, form([big]), [0], form([256, 256]), 100)
        assert e.value.code == d.DDP_ERR_UNSUPPORTED
        with pytest.raises(d.DdpError) as e:
            d.ddp_sync_static(2, 0, 0, form([8]), [7], form([256, 256]), 100)
        assert e.value.code == d.DDP_ERR_ARG
        with pytest.raises(d.DdpError) as e:
            d.ddp_sync_static(2, 0, 0, form([8]), [0], form([256, 2]), d.DDP_CAP_WHOLE_MODEL)
        assert e.value.code == d.DDP_ERR_ARG
        with pytest.raises(ValueError):
            d.ddp_sync_static(2, 0, 0, form([8]), [0], form([256]), 100)
    with pytest.raises(OverflowError):
        d.ddp_sync_static(2, 0, 0, [8], [0], [-1, 256], 100)


EDGES = [0, 1, (1 << 15) - 1, 1 << 15, (1 << 30) - 1, 1 << 30, (1 << 31) - 1, 1 << 31, (1 << 32) + 5, (1 << 45) - 3, (1 << 60) - 1, 1 << 60,
         (1 << 62) + 1, (1 << 63) - 1, 1 << 63, (1 << 64) - 1]


@pytest.mark.parametrize("form", [list, tuple])
def test_values_arrive_as_they_are(form):
    """Ints of every number of the interpreter's digits, as pointers, sizes and ids."""
    from ctypes import CFUNCTYPE, POINTER, c_int32, c_int64, c_uint64, c_void_p, cast
    B = d.binding
    got = []

    @CFUNCTYPE(c_int32, c_void_p, POINTER(c_uint64))
    def accumulate(ctx, p):
        got.append(p[:len(EDGES) + 1])
        return 0

    @CFUNCTYPE(c_int32, c_void_p, POINTER(c_int32), c_int32)
    def many(ctx, p, n):
        got.append(p[:n])
        return 0

    @CFUNCTYPE(c_int32, c_int32, c_int32, c_void_p, c_int32, POINTER(c_int64), POINTER(c_int32), POINTER(c_uint64), c_uint64)
    def static(R, device, stream, n, numel, dtype, p, cap):
        got.append((numel[:n], dtype[:n], p[:R * n]))
        return 0

    sizes = [v for v in EDGES if v < 1 << 63] + [-1, -(1 << 30), -(1 << 63)]
    ids = [v for v in EDGES if v < 1 << 31] + [-1, -(1 << 30), -(1 << 31)]
    address = lambda f: cast(f, c_void_p).value
    B._fast.bind(B._mark, B._finalize, B._mark_local, c_int32, address(many), address(accumulate), address(static))
    try:
        assert B._fast_accumulate(1, form(EDGES + [None]), len(EDGES) + 1) == 0
        assert B._fast_many(1, form(ids)) == 0
        assert B._fast_static(1, 0, 0, form(sizes), form(ids[:1] * len(sizes)), form((EDGES * 2)[:len(sizes)]), 0) == 0
        assert B._fast_many(1, form([1 << 31])) is None and B._fast_many(1, form([-(1 << 31) - 1])) is None
        assert B._fast_accumulate(1, form([1 << 64] * 17), 17) is None and B._fast_accumulate(1, form([True] * 17), 17) is None
    finally:
        B._fast.bind(B._mark, B._finalize, B._mark_local, c_int32, B._many, B._accumulate, B._static)
    assert got[0] == EDGES + [0]
    assert got[1] == ids
    assert got[2] == (sizes, [ids[0]] * len(sizes), (EDGES * 2)[:len(sizes)])


@pytest.mark.parametrize("version", ["0x030A00F0", "0x030B00F0", "0x030C00F0"])
def test_the_marshalling_module_compiles_for_newer_interpreters(version, tmp_path):
    """As interpreters before 3.11, of 3.11 and from 3.12 on have the headers: 3.11 gives the layout of ints with Python.h and has no
    longintrepr.h of its own, and from 3.12 on the layout is another one, which the module must not use."""
    import os
    import shutil
    import subprocess
    import sys
    import sysconfig
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None or sys.version_info >= (3, 11):
        pytest.skip("needs a C compiler and an interpreter older than the ones it stands in for")
    real = sysconfig.get_paths()["include"]
    layout = '#include_next <longintrepr.h>\n' if version == "0x030B00F0" else ""
    (tmp_path / "Python.h").write_text(f"#include_next <Python.h>\n#define TAKES_LAYOUT\n{layout}#undef TAKES_LAYOUT\n"
                                       f"#undef PY_VERSION_HEX\n#define PY_VERSION_HEX {version}\n")
    if version != "0x030A00F0":
        (tmp_path / "longintrepr.h").write_text("#ifdef TAKES_LAYOUT\n#include_next <longintrepr.h>\n#else\n"
                                                "#error longintrepr.h: No such file\n#endif\n")
    csrc = os.path.join(os.path.dirname(os.path.abspath(d.__file__)), "csrc", "fastcall.c")
    done = subprocess.run([cc, "-fsyntax-only", "-Wall", "-Wno-unused", f"-I{tmp_path}", f"-I{real}", csrc], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
