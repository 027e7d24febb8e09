"""Host-side checks that need no GPU: the library loads and exports every symbol that
include/csd.h declares, and host-side argument validation returns the documented codes."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def L():
    import paper_2312_11462_amd as P
    if not os.path.exists(P.library_path()):
        from paper_2312_11462_amd import build
        build.build()
    return P.lib()


def _declared():
    src = open(os.path.join(ROOT, "include", "csd.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(csd_[a-z0-9_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported(L):
    import paper_2312_11462_amd as P
    names = _declared()
    assert len(names) >= 14
    for n in names:
        assert hasattr(L, n), n
    assert sorted(P.EXPORTS) == names
    assert b"gfx950" in L.csd_version()


def test_null_and_domain_errors_without_a_device(L):
    from paper_2312_11462_amd.binding import Cfg
    out = C.c_void_p()
    cfg = Cfg(0, 1, 2, 64, 4, 16, 256, 512, 1, 64, 8, 0, 1e-5, 10000.0)
    assert L.csd_model_create(None, None, 0, None, C.byref(out)) == -3
    ptrs = (C.c_void_p * 21)(*([1] * 21))
    assert L.csd_model_create(C.byref(cfg), ptrs, 20, None, C.byref(out)) == -1          # wrong weight count
    bad = Cfg(2, 1, 2, 64, 4, 16, 256, 512, 1, 64, 8, 0, 1e-5, 10000.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -5          # arch
    bad = Cfg(1, 1, 2, 64, 4, 16, 256, 512, 1, 64, 8, 0, 1e-6, 0.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -1          # arch 1 needs enc_len
    bad = Cfg(1, 1, 2, 64, 4, 16, 256, 512, 1, 64, 8, 16, 1e-6, 0.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -1          # arch 1: 4 + 14 L tensors
    bad = Cfg(0, 1, 2, 64, 4, 16, 256, 512, 1, 64, 8, 16, 1e-5, 10000.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -1          # arch 0 has no encoder
    assert L.csd_cross_kv_init(None, None, None, 1, None) == -3
    bad = Cfg(0, 1, 2, 64, 4, 15, 256, 512, 1, 64, 8, 0, 1e-5, 10000.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -1          # odd head_dim
    bad = Cfg(0, 1, 2, 64, 4, 16, 256, 512, 1, 4, 8, 0, 1e-5, 10000.0)
    assert L.csd_model_create(C.byref(bad), ptrs, 21, None, C.byref(out)) == -2          # block > seq
    assert L.csd_accept(None, None, None, None, None, None, 1, 1, 8, C.c_float(1.0), 0, None, None, None) == -3
    one = C.c_void_p(1)
    assert L.csd_accept(one, None, None, one, one, one, 1, 1, 8, C.c_float(0.5), 0, one, one, None) == -1
    assert L.csd_accept(one, None, None, one, one, one, 1, 1, 8, C.c_float(1.0), 7, one, one, None) == -1
    assert L.csd_bigram_fit(one, 9000, 10, one, None) == -2
    assert L.csd_bigram_draft(None, one, 1, 8, one, 10, 2, 0, one, None, None) == -3
    assert L.csd_bigram_draft(one, one, 1, 0, one, 10, 2, 0, one, None, None) == -1
    assert L.csd_kv_bytes(None) == 0
    assert L.csd_verify_block(None, one, one, one, 1, 1, C.c_float(1.0), one, None, None) == -3


def test_gemm_plan_of_tall_blocks_fills_the_compute_units(L):
    """Host logic only: for blocks of 33 to 144 rows the row-split GEMM picks column tiles per workgroup and K
    splits per matrix, by one function for the launch and for this call.  Properties that hold for every shape, and the plans of
    the 7B-shaped matrices (the launches the batch-8 profiles name), which are the same at every row count."""
    def plan(N, K, rows, max_splits=16):
        ct, S = C.c_int32(), C.c_int32()
        assert L.csd_debug_gemm_plan(N, K, rows, max_splits, C.byref(ct), C.byref(S)) == 0
        return ct.value, S.value
    d, F, V = 4096, 11008, 32000
    for rows in (33, 40, 64, 65, 128, 129, 136, 144):
        assert plan(3 * d, d, rows) == (12, 4)  # QKV: 64 groups x 4 = 256 workgroups
        assert plan(d, d, rows) == (8, 8)       # O: 32 x 8 = 256
        assert plan(d, F, rows) == (8, 8)       # down
        assert plan(2 * F, d, rows) == (11, 2)  # gate|up: 126 x 2 = 252
        assert plan(V, d, rows) == (16, 2)      # LM head: 125 x 2 = 250, the wider workgroup wins the tie with (8, 1)
    for N, K in [(3 * d, d), (d, d), (d, F), (2 * F, d), (V, d), (768 * 3, 768), (768, 3072), (1040, 256), (16, 32)]:
        for rows in (33, 64, 100, 128, 129, 144):
            for ms in (1, 2, 16):
                ct, S = plan(N, K, rows, ms)
                assert ct in (16, 12, 11, 8, 6)
                assert 1 <= S <= min(8, ms)
                assert S == 1 or (K // 32) // S >= 8                     # a K slice holds at least two chunks of four k-steps
                groups = -(-(N // 16) // ct)
                assert S == 1 or groups * S <= 256                       # K is split only while the chip has room
    bad = C.c_int32()
    assert L.csd_debug_gemm_plan(100, 64, 128, 4, C.byref(bad), C.byref(bad)) == -1
    assert L.csd_debug_gemm_plan(64, 64, 145, 4, C.byref(bad), C.byref(bad)) == -1
    assert L.csd_debug_gemm_plan(64, 64, 64, 4, None, C.byref(bad)) == -3


def test_tall_gemm_plan_stays_in_bounds(L):
    """Host logic only: forms that exist, K splits that the partial-sum buffer holds and that leave six k-steps each, and the
    forms of the 7B- and 160M-shaped matrices at the block sizes that the profiles name."""
    def plan(N, K, rows, ms=1):
        v = [C.c_int32() for _ in range(4)]
        assert L.csd_debug_tall_plan(N, K, rows, ms, *[C.byref(x) for x in v]) == 0
        return tuple(x.value for x in v)
    for N, K in [(12288, 4096), (4096, 11008), (22016, 4096), (32000, 4096), (2304, 768), (768, 3072), (1040, 256), (16, 32), (32, 64)]:
        for rows in (1, 16, 65, 145, 192, 193, 289, 512, 1000, 4096):
            for ms in (1, 2, 8):
                ctw, rtw, stages, S = plan(N, K, rows, ms)
                assert (ctw, stages) in ((4, 4), (6, 2), (6, 3)) and rtw in (2, 3, 4)
                assert 1 <= S <= ms and (S == 1 or K // 32 // S >= 6)
                wgs = -(-N // (32 * ctw)) * -(-rows // (32 * rtw)) * S
                assert stages == (4 if ctw == 4 else 2 if wgs > 256 else 3)
    assert plan(12288, 4096, 512) == (6, 4, 3, 1) and plan(12288, 4096, 384) == (6, 3, 3, 1)
    assert plan(22016, 4096, 512) == (6, 4, 2, 1) and plan(32000, 4096, 512) == (6, 3, 2, 1)
    assert plan(4096, 4096, 512, 8)[:3] == (4, 4, 4) and plan(2304, 768, 512) == (4, 2, 4, 1)
    v = C.c_int32()
    p = C.byref(v)
    assert L.csd_debug_tall_plan(24, 64, 200, 1, p, p, p, p) == -1 and L.csd_debug_tall_plan(32, 48, 200, 1, p, p, p, p) == -1
    assert L.csd_debug_tall_plan(32, 64, 0, 1, p, p, p, p) == -1 and L.csd_debug_tall_plan(32, 64, 200, 0, p, p, p, p) == -1
    assert L.csd_debug_tall_plan(32, 64, 200, 1, None, p, p, p) == -3
