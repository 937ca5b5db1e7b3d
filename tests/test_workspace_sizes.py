"""Workspace sizes (host only): what the size entry points return holds what the
calls lay out in it."""
import ctypes

import pytest

import paper_2607_04489_amd as eg


@pytest.fixture(scope="module")
def lib():
    if not eg.available():
        import __graft_entry__
        __graft_entry__.build()
    return eg.lib()


def col(n, dtype):
    return eg.Column(None, n, dtype, 0)


def join_size(lib, variant, kdt, bdt, pdt, n_build, n_probe, span, bits=0, passes=0):
    plan = eg.PlanT()
    plan.variant, plan.radix_bits, plan.radix_passes, plan.key_dtype = variant, bits, passes, kdt
    plan.load_factor, plan.build_min, plan.build_max = 0.5, 0, span
    size = ctypes.c_size_t()
    assert lib.eiger_join_workspace_size(ctypes.byref(plan), col(n_build, kdt), col(n_build, bdt), col(n_probe, kdt),
                                         col(n_probe, pdt), ctypes.byref(size)) == 0
    return size.value


def sort_size(lib, key_bytes, n):
    size = ctypes.c_size_t()
    assert lib.eiger_sort_pairs_workspace_size(key_bytes, n, 8 * key_bytes, ctypes.byref(size)) == 0
    return size.value - 256


def up(n):
    return (n + 255) // 256 * 256


# rows from which the radix sort takes its large tiles, by key width
LARGE = {4: 512 * 10240, 8: 512 * 6144}


@pytest.mark.parametrize("code_bytes", [4, 8])
@pytest.mark.parametrize("bdt,pdt", [(eg.INT32, eg.INT32), (eg.INT32, eg.INT64), (eg.INT64, eg.INT32), (eg.INT64, eg.INT64)])
def test_sort_merge_workspace_holds_both_sorts(lib, code_bytes, bdt, pdt):
    """SORT_MERGE keeps two code arrays and a row-id array of each side and runs the two
    sides' sorts in what remains, whichever side needs more: the tiles change with the
    row count, and with them the count table."""
    at = LARGE[code_bytes]
    kdt = eg.INT32 if code_bytes == 4 else eg.INT64
    span = 1 << 20 if code_bytes == 4 else 1 << 40
    for a in (1, 5000, at - 40000, at - 1, at, at + 1, at + 9999, 2 * at):
        for b in (1, 70001, at - 40000, at - 1, at, at + 1, at + 9999):
            for n_build, n_probe in ((a, b), (b, a)):
                size = join_size(lib, eg.SORT_MERGE, kdt, bdt, pdt, n_build, n_probe, span)
                kept = 256 + sum(2 * up(code_bytes * n) + up(4 * n) for n in (n_build, n_probe))
                for n in (n_build, n_probe):
                    assert size - kept >= sort_size(lib, code_bytes, n), (n_build, n_probe, n)


@pytest.mark.parametrize("n,payload,fits", [(1_600_000, eg.INT32, True), (1_680_000, eg.INT32, False),
                                            (1_900_000, eg.INT32, False), (1_380_000, eg.INT64, True), (1_410_000, eg.INT64, False)])
def test_noalloc_takes_the_same_sort_merge_joins(lib, n, payload, fits):
    """The 64 MiB scratch array holds the code and row-id arrays, the payloads and one
    sort beside them (40.1 or 48.1 bytes a row of each side); what is larger is refused on
    the host."""
    size = join_size(lib, eg.SORT_MERGE, eg.INT32, payload, payload, n, n, 1 << 20)
    assert (size <= eg.NOALLOC_SCRATCH_BYTES) == fits
    if not fits:
        plan = eg.PlanT()
        plan.variant, plan.key_dtype, plan.build_max, plan.load_factor = eg.SORT_MERGE, eg.INT32, 1 << 20, 0.5
        k, p = eg.Column(4096, n, eg.INT32, 0), eg.Column(4096, n, payload, 0)
        cnt, cs = ctypes.c_int64(), ctypes.c_int64()
        assert lib.eiger_join_noalloc(k, p, k, p, ctypes.byref(plan), None, None, 0, ctypes.byref(cnt), ctypes.byref(cs),
                                      None) == eg.EIGER_ERR_TOO_LARGE


def rising(sizes):
    return all(a <= b for a, b in zip(sizes, sizes[1:]))


# row counts around every bound of the radix sort's paths, up to twice the last
ROWS = sorted({1, 1000, 16384, 16385, 70001, 1 << 20, (1 << 20) + 1} |
              {at * f // 8 + d for at in LARGE.values() for f in (7, 8, 9, 10, 12, 14, 16) for d in (-1, 0, 1)})


@pytest.mark.parametrize("key_bytes", [4, 8])
def test_sort_workspace_rises_with_the_rows(lib, key_bytes):
    """A workspace sized for the largest input of a program takes every smaller one."""
    assert rising([sort_size(lib, key_bytes, n) for n in ROWS])


@pytest.mark.parametrize("bits", [1, 8, 9, 10, 11, 16, 17, 18])
@pytest.mark.parametrize("kdt", [eg.INT32, eg.INT64])
@pytest.mark.parametrize("vals", [(), (eg.INT32,), (eg.INT32, eg.INT32), (eg.INT64, eg.INT64)])
def test_groupby_workspace_rises_with_the_rows(lib, bits, kdt, vals):
    plan = eg.GroupByPlanT()
    plan.variant, plan.radix_bits, plan.key_dtype, plan.slots = eg.GB_PARTITION, bits, kdt, 1024
    plan.sentinel = -(1 << 63)
    sizes = []
    for n in ROWS:
        size = ctypes.c_size_t()
        cols = (eg.Column * 2)(*[col(n, v) for v in vals])
        assert lib.eiger_groupby_workspace_size(ctypes.byref(plan), col(n, kdt), cols, len(vals), ctypes.byref(size)) == 0
        sizes.append(size.value)
    assert rising(sizes)


@pytest.mark.parametrize("sort", [0, 1])
def test_fusion_workspace_rises_with_the_rows(lib, sort):
    plan = eg.SkfPlanT()
    plan.n_keys = 2
    for k, code in zip(plan.key, (eg.SKF_FOR, eg.SKF_DICT)):
        k.code, k.dtype, k.bits, k.slots, k.range_bits = code, eg.INT32, 8, 1024, 32
    sizes = []
    for n in ROWS:
        size = ctypes.c_size_t()
        assert lib.eiger_skf_workspace_size(ctypes.byref(plan), n, 0, sort, ctypes.byref(size)) == 0
        sizes.append(size.value)
    assert rising(sizes)


@pytest.mark.parametrize("variant,bits,passes", [(eg.GLOBAL_HASH, 0, 0), (eg.RADIX, 8, 1), (eg.RADIX, 9, 2), (eg.RADIX, 16, 2),
                                                 (eg.RADIX, 18, 2), (eg.SORT_MERGE, 0, 0)])
@pytest.mark.parametrize("kdt,pdt", [(eg.INT32, eg.INT32), (eg.INT64, eg.INT32), (eg.INT64, eg.INT64)])
def test_join_workspace_rises_with_the_rows(lib, variant, bits, passes, kdt, pdt):
    def size(a, b):
        return join_size(lib, variant, kdt, pdt, pdt, a, b, 1 << 20 if kdt == eg.INT32 else 1 << 40, bits, passes)

    for other in (1000, LARGE[4] - 1, LARGE[4], LARGE[8] - 1, LARGE[8]):
        assert rising([size(n, other) for n in ROWS])
        assert rising([size(other, n) for n in ROWS])


@pytest.mark.parametrize("bits", [8, 9, 10, 16, 18])
@pytest.mark.parametrize("kdt", [eg.INT32, eg.INT64])
def test_wide_join_workspace_rises_with_the_rows(lib, bits, kdt):
    plan = eg.PlanT()
    plan.variant, plan.radix_bits, plan.radix_passes, plan.key_dtype, plan.load_factor = eg.RADIX, bits, 2, kdt, 0.5

    def size(a, b):
        out = ctypes.c_size_t()
        bc, pc = (eg.Column * 1)(col(a, eg.INT32)), (eg.Column * 2)(col(b, eg.INT32), col(b, eg.INT64))
        assert lib.eiger_join_wide_workspace_size(ctypes.byref(plan), eg.MAT_GFTR, col(a, kdt), bc, 1, col(b, kdt), pc, 2,
                                                  ctypes.byref(out)) == 0
        return out.value

    for other in (1000, LARGE[4] - 1, LARGE[8] - 1):
        assert rising([size(n, other) for n in ROWS])
        assert rising([size(other, n) for n in ROWS])
