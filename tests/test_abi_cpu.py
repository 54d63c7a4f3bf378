"""Host-side checks that need no GPU: the library loads, exports every symbol the header
declares, and rejects bad arguments with a status before anything is launched."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    from paper_2401_14021_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2401_14021_amd import build
        build.build()
    return binding.lib()


def test_every_declared_symbol_is_exported(L):
    text = open(os.path.join(ROOT, "include", "ralm.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = set(re.findall(r"\b(ralm_[a-z0-9_]+)\s*\(", text))
    assert {"ralm_retrieve_topk", "ralm_retrieve_topk_ex", "ralm_retrieve_topk_seq", "ralm_cache_lookup",
            "ralm_verify", "ralm_cache_insert", "ralm_knnlm_probs", "ralm_os3_stride", "ralm_cache_lookup_topk",
            "ralm_cache_lookup_static",
            "ralm_release_buffers",
            "ralm_workspace_bytes", "ralm_build_scan_copy", "ralm_last_error"} <= names
    for n in names:
        assert hasattr(L, n), n


def _ds(binding, N=1000, d=768, exact=0x1000, exact_dtype=0, scan=0x2000, scan_dtype=1):
    ds = binding.ralm_datastore_t()
    ds.exact, ds.exact_dtype, ds.scan, ds.scan_dtype = exact, exact_dtype, scan, scan_dtype
    ds.N, ds.d, ds.exact_stride, ds.scan_stride = N, d, 0, 0
    return ds


def test_argument_errors_return_status_without_a_device(L):
    from paper_2401_14021_amd import binding as b
    P = 0x10000   # fake, aligned, never dereferenced: every call below fails validation first
    ds = _ds(b)
    ref = ctypes.byref
    ws = L.ralm_workspace_bytes(8, ref(ds), 5, 0)
    assert ws > 0
    call = L.ralm_retrieve_topk_ex
    assert call(None, 8, ref(ds), 5, 0, P, P, None, P, ws, None) == 1            # NULL queries
    assert b"NULL" in L.ralm_last_error()
    assert call(P, 0, ref(ds), 5, 0, P, P, None, P, ws, None) == 2               # Q < 1
    assert call(P, 8, ref(ds), 0, 0, P, P, None, P, ws, None) == 3               # k < 1
    assert call(P, 8, ref(ds), 2000, 0, P, P, None, P, ws, None) == 3            # k > N and > max
    assert call(P, 8, ref(ds), 5, 4, P, P, None, P, ws, None) == 3               # k' < k
    assert call(P, 8, ref(ds), 5, 8192, P, P, None, P, ws, None) == 3            # k' > max
    assert call(P, 8, ref(_ds(b, exact_dtype=1)), 5, 0, P, P, None, P, ws, None) == 4   # bf16 exact copy
    assert call(P, 8, ref(_ds(b, scan_dtype=7)), 5, 0, P, P, None, P, ws, None) == 4
    assert call(P, 8, ref(_ds(b, d=770)), 5, 0, P, P, None, P, ws, None) == 2    # d not a multiple of 8
    assert call(P, 8, ref(_ds(b, exact=0x1004)), 5, 0, P, P, None, P, ws, None) == 5
    assert call(P + 4, 8, ref(ds), 5, 0, P, P, None, P, ws, None) == 5
    assert call(P, 8, ref(ds), 5, 0, P, P, None, None, ws, None) == 6            # no workspace
    assert call(P, 8, ref(ds), 5, 0, P, P, None, P + 16, ws, None) == 6          # misaligned workspace
    assert call(P, 8, ref(ds), 5, 0, P, P, None, P, ws - 1, None) == 6           # too small
    wide = _ds(b)
    wide.scan_stride = 1 << 23                                                   # 16 MiB row pitch
    assert call(P, 8, ref(wide), 5, 0, P, P, None, P, 1 << 30, None) == 2
    assert b"pitch" in L.ralm_last_error()
    huge = _ds(b, N=2_000_000_000)
    assert call(P, 1 << 20, ref(huge), 5, 0, P, P, None, P, 1 << 62, None) == 2  # too many tile pairs
    assert b"split the batch" in L.ralm_last_error()
    l2 = _ds(b)
    l2.metric = 1
    l2.scan_stride = 770
    assert call(P, 8, ref(l2), 5, 0, P, P, None, P, 1 << 30, None) == 2          # scan pitch below d + 8
    l2.scan_stride = 776
    assert L.ralm_workspace_bytes(8, ref(l2), 5, 0) > 0                          # accepted with d + 8 columns
    l2.scan = None
    assert call(P, 8, ref(l2), 5, 0, P, P, None, P, 1 << 30, None) == 1          # squared distance needs a scan copy
    l2 = _ds(b, scan_dtype=0)
    l2.metric = 1
    assert call(P, 8, ref(l2), 5, 0, P, P, None, P, 1 << 30, None) == 4          # ... in bf16 or fp16
    bad = _ds(b)
    bad.metric = 5
    assert call(P, 8, ref(bad), 5, 0, P, P, None, P, 1 << 30, None) == 4
    bl2 = L.ralm_build_scan_copy_l2
    assert bl2(P, 0, 0, None, 1, 0, 10, 768, None) == 1
    assert bl2(P, 1, 0, P, 1, 0, 10, 768, None) == 4                             # bf16 is not an exact copy
    assert bl2(P, 0, 0, P, 0, 0, 10, 768, None) == 4                             # fp32 is not a scan copy
    assert bl2(P, 0, 0, P, 1, 770, 10, 768, None) == 2                           # dst pitch below d + 8
    assert bl2(P, 2, 776, P, 1, 776, 10, 768, None) == 2                         # in place needs equal dtypes
    assert L.ralm_workspace_bytes(8, ref(ds), 0, 0) == 0
    assert L.ralm_workspace_bytes(0, ref(ds), 5, 0) == 0
    # workspace grows with Q and with k'
    assert L.ralm_workspace_bytes(1024, ref(ds), 5, 0) > ws
    assert L.ralm_workspace_bytes(8, ref(ds), 1000, 0) > ws
    # simple form
    assert L.ralm_retrieve_topk(None, 8, P, 1000, 768, 5, P, P) == 1
    assert L.ralm_retrieve_topk(P, 8, P, 1000, 768, 1001, P, P) == 3
    # cache lookup / verify / scan copy
    assert L.ralm_cache_lookup(None, P, 4, 2, P, 6, P, ref(ds), P, P, None, 0, None) == 1
    assert L.ralm_cache_lookup(P, P, 0, 2, P, 6, P, ref(ds), P, P, None, 0, None) == 2
    assert L.ralm_cache_lookup(P, P, 4, 2, P, -1, P, ref(ds), P, P, None, 0, None) == 7
    assert L.ralm_cache_lookup(P, P, 4, 2, P, 6, P, ref(ds), P, P, P, 40, None) == 6     # 8 bytes per query needed
    assert L.ralm_cache_lookup(P, P, 4, 2, P, 6, P, ref(ds), P, P, P + 4, 64, None) == 6 # misaligned scratch
    st = L.ralm_cache_lookup_static
    assert st(P, None, 4, 2, P, 6, P, ref(ds), P, P, None) == 1                   # argument errors come first,
    assert st(P, P, 0, 2, P, 6, P, ref(ds), P, P, None) == 2                      # before any device call
    assert st(P, P, 4, 2, P, 65537, P, ref(ds), P, P, None) == 7                  # beyond the built-in scratch
    assert L.ralm_cache_lookup_workspace_bytes(6) >= 48 and L.ralm_cache_lookup_workspace_bytes(-1) == 0
    ins = L.ralm_cache_insert
    assert ins(P, P, None, 4, 2, P, 5, 6, P, None, 1, 0, 1000, None) == 1         # no head array
    assert ins(P, P, P, 0, 2, P, 5, 6, P, None, 1, 0, 1000, None) == 2            # C < 1
    assert ins(P, P, P, 20000, 2, P, 5, 6, P, None, 1, 0, 1000, None) == 2        # C above the LDS limit
    assert ins(P, P, P, 4, 2, P, 5, 6, P, None, 6, 0, 1000, None) == 3            # p > true_stride
    assert ins(P, P, P, 4, 2, P, 5, 6, P, None, 0, 0, 1000, None) == 3            # p < 1
    assert ins(P, P, P, 4, 2, P, 5, -1, P, None, 1, 0, 1000, None) == 7           # Qt < 0
    assert ins(P, P, P, 4, 2, P, 5, 6, P, None, 1, -1, 1000, None) == 7           # n_next < 0
    assert ins(P, P, P, 4, 2, P, 5, 6, P, None, 1, 0, 0, None) == 2               # N < 1
    kp = L.ralm_knnlm_probs
    assert kp(P, P, 4, 8, None, 100, 1.0, P, P, P, P, None) == 1                  # no values array
    assert kp(P, P, 4, 0, P, 100, 1.0, P, P, P, P, None) == 3                     # k < 1
    assert kp(P, P, 4, 2000, P, 100, 1.0, P, P, P, P, None) == 3                  # k > max
    assert kp(P, P, 4, 8, P, 100, 0.0, P, P, P, P, None) == 7                     # temperature not positive
    assert kp(P, P, 4, 8, P, 0, 1.0, P, P, P, P, None) == 2                       # N < 1
    tk = L.ralm_cache_lookup_topk
    wsk = L.ralm_cache_lookup_topk_workspace_bytes(6, 64)
    assert wsk >= 6 * 64 * 8 + 6 * 4 and L.ralm_cache_lookup_topk_workspace_bytes(6, 0) == 0
    assert tk(P, P, 64, 2, P, 6, P, ref(ds), 8, None, P, P, wsk, None) == 1        # no output
    assert tk(P, P, 5000, 2, P, 6, P, ref(ds), 8, P, P, P, 1 << 30, None) == 2     # C above the limit
    assert tk(P, P, 64, 2, P, 6, P, ref(ds), 65, P, P, P, wsk, None) == 3          # k > C
    assert tk(P, P, 64, 2, P, 6, P, ref(ds), 8, P, P, None, wsk, None) == 6        # no workspace
    assert tk(P, P, 64, 2, P, 6, P, ref(ds), 8, P, P, P, wsk - 1, None) == 6       # too small
    assert L.ralm_verify(P, None, 1, 6, P, 2, P, None) == 1
    assert L.ralm_verify(P, P, 0, 6, P, 2, P, None) == 7
    assert L.ralm_verify(P, P, 1, 6, P, -1, P, None) == 2
    assert L.ralm_build_scan_copy(P, 0, P, 0, 0, 10, 768, None) == 4             # fp32 is not a scan copy
    assert L.ralm_build_scan_copy(P, 0, P, 1, 0, 10, 12, None) == 2
    assert L.ralm_build_scan_copy(P, 0, None, 1, 0, 10, 768, None) == 1
    n, arr = ctypes.c_int32(0), (ctypes.c_int64 * b.RALM_MAX_LADDER_STAGES)()
    assert L.ralm_workspace_stage_entries(None, None, ref(n), arr) == 1             # accessors check their pointers
    assert L.ralm_workspace_stage_entries(P, None, None, arr) == 1
    assert L.ralm_workspace_counters(None, None, ref(b.ralm_counters_t())) == 1
    routes = (ctypes.c_int32 * b.RALM_MAX_LADDER_STAGES)()
    assert L.ralm_scan_routes(8, ref(ds), 5, 0, None, routes) == 1 and L.ralm_scan_routes(8, ref(ds), 5, 0, ref(n), None) == 1
    assert L.ralm_scan_routes(0, ref(ds), 5, 0, ref(n), routes) == 2
    assert L.ralm_scan_routes(8, ref(ds), 0, 0, ref(n), routes) == 3


def _routes(L, Q, k, N, d, scan_dtype=1, pitch=0, k_prime=0, metric=0):
    from paper_2401_14021_amd import binding as b
    ds = _ds(b, N=N, d=d, scan_dtype=scan_dtype)
    ds.scan_stride, ds.metric = pitch, metric
    n, arr = ctypes.c_int32(0), (ctypes.c_int32 * b.RALM_MAX_LADDER_STAGES)()
    assert L.ralm_scan_routes(Q, ctypes.byref(ds), k, k_prime, ctypes.byref(n), arr) == 0
    assert not any(arr[n.value:])
    return [b.SCAN_ROUTES[v] for v in arr[:n.value]]


# The rules' sides, one reason each (a device with 256 compute units; k = 10 keeps 64 candidates)
@pytest.mark.parametrize("Q,N,d,more,want", [
    (81, 1_000_000, 768, {}, ["all_quarters", "parked", "held"]),        # the second stage admits 10 scores per 32 rows
    (64, 4_000_000, 768, {}, ["all_quarters", "parked", "parked"]),      # few queries over whole lines stay in tiles
    (32, 4_000_000, 768, {}, ["all", "parked", "parked"]),               # ... and have no quarter tiles
    (200, 6_000_000, 768, {}, None),
    (90, 777_001, 392, dict(scan_dtype=2), ["all_quarters", "held", "held"]),
    (1, 1_000_000, 392, {}, None),                                       # no whole lines: any number of queries
    (1, 1_000_000, 392, dict(pitch=448), "parked"),                      # the same in whole lines
    (100, 4_000_000, 256, {}, "parked"),                                 # rows too short
    (100, 4_000_000, 1152, {}, "parked"),                                # ... and too long for the registers
    (100, 4_000_000, 1088, {}, None),
    (200, 4_000_000, 1024, {}, "parked"),                                # 128 queries a tile, whole lines
    (200, 4_000_000, 1000, {}, None),
    (1024, 10_000_000, 768, {}, None),
    (512, 10_000_000, 512, {}, "parked"),                                # several query tiles over short rows in whole lines
    (512, 10_000_000, 504, {}, None),
    (2341, 4_000_000, 768, {}, "parked"),                                # ten query tiles on 32 compute units of an XCD
    (100, 4_000_000, 768, dict(scan_dtype=0), "parked"),                 # fp32 rows
    (100, 4_000_000, 1024, dict(metric=1, pitch=1088, scan_dtype=2), None),
    (256, 10_000_000, 1024, dict(k=1024, scan_dtype=2), "parked"),
])
def test_scan_routes(L, Q, N, d, more, want):
    """The kernel of every stage, or of the last one (None: the queries are held in registers)."""
    more = dict(more)
    got = _routes(L, Q, more.pop("k", 10), N, d, **more)
    if isinstance(want, list):
        assert got == want
    else:
        assert got[-1] == (want or "held"), got


@pytest.mark.parametrize("Q,N,d,want", [
    (700, 4_000_000, 768, "held"), (600, 4_000_000, 768, "held"), (550, 4_000_000, 768, "parked"),   # idle columns: up to a quarter
    (300, 4_000_000, 768, "parked"), (300, 4_000_000, 712, "held"),      # two tiles over rows that are no whole lines: any size
    (2048, 4_000_000, 768, "held"), (2100, 4_000_000, 768, "parked"), (2200, 4_000_000, 768, "held"),   # nine tiles: a twentieth
    (400, 4_000_000, 904, "held"), (700, 4_000_000, 904, "parked"),      # tiles of 128 queries: up to four
    (768, 300_000, 768, "parked"),                                       # few rows for a workgroup
])
def test_scan_routes_of_several_query_tiles(L, Q, N, d, want):
    assert _routes(L, Q, 10, N, d)[-1] == want


@pytest.mark.parametrize("Q,N,d,want", [
    (600, 1_000_000, 328, ["parked", "parked"]), (1100, 600_000, 392, ["parked", "parked"]), (1100, 1_000_000, 392, ["parked", "held"]),
    (2304, 2_000_000, 328, ["parked", "held"]), (1500, 600_000, 456, ["parked", "parked"]), (1500, 4_000_000, 456, ["held", "held"]),
    (450, 1_000_000, 392, ["held", "held"]), (600, 1_000_000, 520, ["held", "held"]),      # two tiles, longer rows: as ever
])
def test_scan_routes_of_short_rows_that_are_no_whole_lines(L, Q, N, d, want):
    """Several query tiles: the two last stages."""
    assert _routes(L, Q, 10, N, d)[-2:] == want
    if want[-1] == "held":
        assert _routes(L, Q, 10, N, d, k_prime=4096)[-1] != "held"       # many candidates, many admitted scores


def test_scan_routes_with_compute_units_reserved(L):
    from paper_2401_14021_amd import binding as b
    try:
        b.ralm_scan_reserve_cus(8)
        assert _routes(L, 20, 10, 1_000_000, 392)[-1] == "parked"        # half of each unit's LDS stays free
        assert _routes(L, 40, 10, 1_000_000, 392)[-1] == "held"
        b.ralm_scan_reserve_cus(300)                                     # one unit per XCD is left: two tiles do not fit
        assert _routes(L, 129, 10, 4_000_000, 904)[-1] == "parked"
    finally:
        b.ralm_scan_reserve_cus(0)


# (k = 10 and 32 keep 64 candidates, 33 keeps 128)
@pytest.mark.parametrize("Q,k,N,k_prime,want", [
    (81, 10, 1_000_000, 0, True), (1, 32, 100_000, 0, True), (2341, 20, 4_000_000, 0, True), (600, 10, 16_385, 0, True),
    (81, 33, 1_000_000, 0, False), (81, 10, 1_000_000, 65, False), (81, 10, 1_000_000, 64, True), (8, 10, 16_384, 0, False),
])
def test_first_stage_scores(L, Q, k, N, k_prime, want):
    """Up to 64 candidates and more than one stage."""
    from paper_2401_14021_amd import binding as b
    ds = _ds(b, N=N, scan_dtype=1)
    out = ctypes.c_int32(-1)
    assert L.ralm_first_stage_scores(Q, ctypes.byref(ds), k, k_prime, ctypes.byref(out)) == 0
    assert out.value == int(want)
    assert L.ralm_first_stage_scores(Q, ctypes.byref(ds), k, k_prime, None) == 1
    assert L.ralm_first_stage_scores(0, ctypes.byref(ds), k, k_prime, ctypes.byref(out)) == 2


def _lookup(L, R, C, d, dtype=0, metric=0, Qt=None, k=0):
    from paper_2401_14021_amd import binding as b
    ds = _ds(b, d=d, exact_dtype=dtype, scan=None)
    ds.metric = metric
    out = [ctypes.c_int32(-1) for _ in range(3)]
    assert L.ralm_lookup_route(R, R if Qt is None else Qt, C, ctypes.byref(ds), k, *map(ctypes.byref, out)) == 0
    return tuple(v.value for v in out)


def test_lookup_routes(L):
    """(workgroups per request, pieces in flight, a launch that clears)"""
    from paper_2401_14021_amd import binding as b
    assert _lookup(L, 64, 1024, 768) == (4, 4, 1)
    assert _lookup(L, 64, 64, 768) == (1, 8, 0)
    assert _lookup(L, 600, 1024, 768) == (1, 8, 0)           # many requests are not split
    assert _lookup(L, 5000, 64, 768)[2] == 1                 # ... and for more than 4096 a launch answers unowned queries
    assert _lookup(L, 64, 1024, 776)[1] == 0                 # not a whole number of steps: vector units
    assert _lookup(L, 64, 1024, 768, metric=1)[1] == 0
    assert _lookup(L, 16, 1024, 768, k=10)[0] > 1
    assert _lookup(L, 256, 2048, 1000, dtype=2, metric=1, k=10) == (0, 0, 0)   # the re-score ranks these
    # up to 256 requests: one round of workgroups at least, also where rows are short or their sums are what takes the time
    assert _lookup(L, 1, 256, 392, dtype=2)[0] == 4 and _lookup(L, 96, 500, 392, dtype=2)[0] == 2
    assert _lookup(L, 8, 129, 1000, dtype=2, metric=1)[0] == 3 and _lookup(L, 33, 1024, 64)[0] == 7
    assert _lookup(L, 127, 4096, 64)[0] == 2 and _lookup(L, 64, 300, 512, dtype=2)[0] == 4
    assert _lookup(L, 33, 1024, 768)[0] == 7 and _lookup(L, 300, 1024, 768)[0] == 3 and _lookup(L, 200, 300, 768)[0] == 1
    assert [_lookup(L, 33, C, 64)[0] for C in (129, 300, 625, 626)] == [1, 1, 1, 7]   # few cached rows
    assert [_lookup(L, 8, C, d)[0] for C, d in ((128, 640), (128, 704), (129, 448), (129, 512), (256, 256))] == [1, 2, 1, 3, 1]
    assert [_lookup(L, 8, C, d, dtype=2)[0] for C, d in ((128, 1024), (160, 512), (200, 512), (300, 128), (300, 256))] == [1, 1, 4, 1, 5]
    assert [_lookup(L, 8, C, 392, Qt=Qt)[0] for C, Qt in ((128, 32), (128, 33), (160, 8), (160, 9), (161, 8))] == [1, 2, 1, 3, 3]
    assert [_lookup(L, 8, C, d)[0] for C, d in ((128, 632), (128, 648), (160, 440), (160, 456))] == [1, 2, 1, 3]
    assert _lookup(L, 8, 128, 392, dtype=2)[0] == 2 and _lookup(L, 8, 128, 392, metric=1)[0] == 2 and _lookup(L, 8, 128, 776)[0] == 2
    # the k best: pieces as long as they can be unless a workgroup has one step of rows
    assert [_lookup(L, R, 2048, 1024, dtype=2, k=64)[:2] for R in (16, 32, 33, 128, 600)] == [(32, 4), (16, 4), (15, 8), (4, 8), (1, 8)]
    assert _lookup(L, 33, 1024, 768, k=64)[:2] == (15, 4) and _lookup(L, 256, 64, 192, k=5)[:2] == (1, 6)
    assert [_lookup(L, R, 64, 768, k=5)[:2] for R in (256, 257, 512, 513)] == [(1, 8), (1, 4), (1, 4), (1, 8)]
    # ... and as many workgroups as run at once, or one more where they would leave too many of the places empty
    assert [_lookup(L, R, 2048, 1024, dtype=2, k=64)[0] for R in (150, 171, 200, 205, 257, 300, 410, 511, 512, 600)] == [3, 3, 3, 2, 2, 2, 1, 1, 1, 1]
    assert [_lookup(L, R, 2048, 392, k=64)[0] for R in (128, 171, 257, 383, 384, 500)] == [4, 3, 2, 2, 1, 1]
    assert [_lookup(L, R, 1024, 1544, k=64)[0] for R in (20, 100, 150)] == [12, 2, 1]
    # unowned queries: by the lookup's first workgroup up to 4096 requests and queries
    assert [_lookup(L, 100, 64, 64, Qt=Qt)[2] for Qt in (107, 4096, 4097, 1 << 20)] == [0, 0, 1, 1]
    assert [_lookup(L, R, 40, 64, Qt=4096)[2] for R in (4096, 4097)] == [0, 1]
    # the best one: four pieces where two workgroups to a unit pay, but not with many rows each
    assert [_lookup(L, 400, C, 1024, dtype=2)[:2] for C in (300, 512, 700, 4096)] == [(1, 4), (1, 4), (1, 8), (1, 8)]
    assert [_lookup(L, 64, C, 1024, dtype=2)[:2] for C in (1024, 2048, 4096)] == [(4, 4), (4, 4), (4, 8)]
    assert [_lookup(L, 450, C, 768)[:2] for C in (700, 1024, 2048)] == [(1, 4), (1, 4), (1, 8)] and _lookup(L, 400, 4096, 256)[:2] == (1, 4) and _lookup(L, 200, 300, 768)[1] == 8
    ds, n = _ds(b), [ctypes.c_int32(0) for _ in range(3)]
    ref = list(map(ctypes.byref, n))
    assert L.ralm_lookup_route(0, 1, 64, ctypes.byref(ds), 0, *ref) == 2
    assert L.ralm_lookup_route(1, -1, 64, ctypes.byref(ds), 0, *ref) == 7
    assert L.ralm_lookup_route(1, 1, 64, ctypes.byref(ds), 65, *ref) == 3
    assert L.ralm_lookup_route(1, 1, 64, None, 0, *ref) == 1
    assert L.ralm_lookup_route(1, 1, 64, ctypes.byref(ds), 0, ref[0], ref[1], None) == 1
    assert L.ralm_lookup_route(1, 1, 64, ctypes.byref(_ds(b, d=4096)), 0, *ref) == 2


def test_binding_refuses_to_run_without_the_library(monkeypatch):
    from paper_2401_14021_amd import binding
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "LIB_PATH", "/nonexistent/libralm.so")
    with pytest.raises(FileNotFoundError):
        binding.lib()


# ---- stride scheduler: host-only functions of the library against the oracle (no GPU involved) ----
def test_os3_matches_oracle(L, oracle):
    from paper_2401_14021_amd import binding as b
    import numpy as np
    from test_oracle_pins import _read_os3_cases
    objective, gamma = _read_os3_cases()
    for g, a, bb, s, asy, val in objective:
        assert b.ralm_os3_objective(g, a, bb, s, asy) == pytest.approx(val, rel=1e-14)
    for st, m, gmax, est in gamma:
        assert b.ralm_os3_gamma(st, m, gmax) == est
    rng = np.random.default_rng(12)
    for _ in range(400):
        g = float(rng.choice([0.0, 1.0, rng.random()]))
        a, bb = float(rng.random() * 5 + 1e-3), float(rng.random() * 50)
        asy = bool(rng.integers(0, 2))
        for s in (1, 2, 3, 7, 32):
            assert b.ralm_os3_objective(g, a, bb, s, asy) == pytest.approx(oracle.os3_objective(g, a, bb, s, asy), rel=1e-12)
        s_lib = b.ralm_os3_stride(g, a, bb, 32, asy)
        s_or = oracle.os3_stride(g, a, bb, 32, asy)
        # equal, or tied within rounding (the two sum the expectation in different orders)
        assert s_lib == s_or or oracle.os3_objective(g, a, bb, s_lib, asy) == pytest.approx(
            oracle.os3_objective(g, a, bb, s_or, asy), rel=1e-12)
        w = int(rng.integers(0, 8))
        st = rng.integers(1, 9, size=w)
        m = np.minimum(rng.integers(0, 10, size=w), st)
        assert b.ralm_os3_gamma(st, m, 0.6) == oracle.os3_gamma(st, m, 0.6) if w else b.ralm_os3_gamma(st, m) == 0.0
    assert b.ralm_os3_stride(0.5, 1, 4, 16) == 2 and b.ralm_os3_stride(0.0, 1, 4, 16) == 1
    # the combined call = the oracle's pieces put together; 1 while there is no history
    assert b.ralm_os3_next_stride([], [], [1.0], [4.0], 16) == 1
    assert b.ralm_os3_next_stride([3], [3], [], [4.0], 16) == 1
    for _ in range(200):
        w = int(rng.integers(1, 6))
        st = rng.integers(1, 9, size=w)
        m = np.minimum(rng.integers(0, 10, size=w), st)
        a_s, b_s = rng.random(int(rng.integers(1, 6))) + 0.05, rng.random(int(rng.integers(1, 6))) * 20
        asy = bool(rng.integers(0, 2))
        want = oracle.os3_stride(oracle.os3_gamma(st, m, 0.6), oracle.os3_latency(a_s), oracle.os3_latency(b_s), 16, asy)
        got = b.ralm_os3_next_stride(st, m, a_s, b_s, 16, 0.6, asy)
        g, a, bb = oracle.os3_gamma(st, m, 0.6), oracle.os3_latency(a_s), oracle.os3_latency(b_s)
        assert got == want or oracle.os3_objective(g, a, bb, got, asy) == pytest.approx(
            oracle.os3_objective(g, a, bb, want, asy), rel=1e-12)
    assert b.ralm_os3_objective(0.5, 1, 4, 0) != b.ralm_os3_objective(0.5, 1, 4, 0)      # NaN for s < 1
    assert b.ralm_os3_objective(1.5, 1, 4, 2) != b.ralm_os3_objective(1.5, 1, 4, 2)      # NaN for gamma > 1
