"""Which kernels serve a call: the rules by sizes and types that the launchers ask, read through the library's internal C++ symbols
(no GPU needed).  The lines lie where both sides were measured; the figures stand beside the rules."""
import ctypes as C

import numpy as np
import pytest

from paper_2512_09963_amd import binding as gsb


def _rule(symbol, restype, *argtypes):
    f = getattr(gsb.lib(), symbol)
    f.restype, f.argtypes = restype, list(argtypes)
    return f


def _wide_serves(M, N, K):
    return _rule("_ZN2gs11wide_servesEiii", C.c_bool, C.c_int, C.c_int, C.c_int)(M, N, K)


@pytest.mark.parametrize("M", [17, 33, 64])
@pytest.mark.parametrize("N,K,wide", [
    (1024, 1024, False), (1024, 4096, False), (512, 8192, False), (2048, 2048, False),       # a few workgroups, short launches
    (4096, 2048, False), (1024, 8192, False), (8192, 1024, False),                           # exactly one workgroup per compute unit
    (4224, 2048, True), (1536, 6144, True), (3072, 3072, True), (2048, 8192, True),          # more
    (4096, 4096, True), (6144, 4096, True), (4096, 14336, True), (8192, 28672, True),
    (1024, 512, True), (28672, 4096, True), (128256, 4096, True),                            # no K split
    (512, 20480, False), (896, 20480, False), (1024, 20480, True),                           # fewer than eight column blocks
    (1088, 4096, False),                                                                     # no multiple of 128 columns
])
def test_bf16_projections_of_up_to_64_rows(M, N, K, wide):
    assert _wide_serves(M, N, K) == wide


@pytest.mark.parametrize("N,K", [(1024, 1024), (1024, 4096), (2048, 2048), (4096, 14336)])
def test_bf16_projections_of_more_rows_are_wide(N, K):
    assert _wide_serves(65, N, K) and _wide_serves(2047, N, K) and not _wide_serves(65, N + 64, K)


def attention_key_groups(n_kv, group, gamma, ctx):
    """(key groups per workgroup, steps per split) of the attention launch."""
    g, c = np.ascontiguousarray(gamma, np.int32), np.ascontiguousarray(ctx, np.int32)
    sps, splits, groups = C.c_int(), C.c_int(), C.c_int()
    ip = C.POINTER(C.c_int)
    plan = _rule("_ZN2gs14attention_planEiiliPKiS1_PiS2_S2_", None, C.c_int, C.c_int, C.c_long, C.c_int, C.c_void_p, C.c_void_p, ip, ip, ip)
    plan(n_kv, group, int(g.max()) + 1, g.size, g.ctypes.data, c.ctypes.data, C.byref(sps), C.byref(splits), C.byref(groups))
    return groups.value, sps.value


@pytest.mark.parametrize("n", [1, 2, 8, 16, 24])
def test_attention_of_short_contexts_has_one_key_group(n):
    """A split of two steps of 32 keys is over before the start of four rings and their merge pay."""
    for keys in range(1, 65):
        assert attention_key_groups(8, 4, [0] * n, [keys - 1] * n)[0] == 1
    for keys in range(65, 193):
        assert attention_key_groups(8, 4, [0] * n, [keys - 1] * n) == (4, (keys + 31) // 32)


@pytest.mark.parametrize("gamma,ctx,groups", [
    ([0], [700], 4), ([7], [2040], 4), ([3] * 4, [500] * 4, 4),
    ([3] * 8, [2048] * 8, 1),      # more than 192 workgroups
    ([8], [700], 1),               # 36 query rows: two tiles
    ([40], [700], 1),
])
def test_attention_key_groups(gamma, ctx, groups):
    assert attention_key_groups(8, 4, gamma, ctx)[0] == groups


@pytest.mark.parametrize("dtype,M,d,hq,qkv,F,fused", [
    (1, 16, 4096, 4096, 6144, 14336, True), (1, 17, 4096, 4096, 6144, 14336, False),
    (1, 8, 8192, 8192, 10240, 28672, True), (1, 9, 8192, 8192, 10240, 28672, False),
    (1, 8, 256, 8192, 10240, 2048, True), (1, 8, 256, 8256, 10240, 2048, False),              # heads and features: 10240 up to 8 rows,
    (1, 9, 256, 8192, 10240, 1024, True), (1, 9, 256, 8192, 10240, 1088, False),              # 9216 beyond
    (1, 8, 1024, 6144, 7680, 4096, True), (1, 9, 1024, 6144, 7680, 4096, False), (1, 8, 1024, 8192, 10240, 4096, False),
    (1, 16, 1024, 4096, 5120, 4096, True), (1, 16, 1024, 1024, 2048, 8192, True),
    (1, 8, 2048, 12288, 15360, 8192, True), (1, 16, 2048, 8192, 10240, 8192, True), (1, 16, 2048, 2048, 3072, 16384, False),
    (1, 1, 2048, 16384, 20480, 4096, False), (1, 1, 512, 16384, 20480, 2048, False),
    (1, 1, 2048, 6144, 16384, 8192, True), (1, 1, 2048, 6144, 18432, 8192, False),            # columns of QKV
    (1, 8, 3072, 6144, 18432, 8192, False), (1, 8, 4096, 8192, 24576, 16384, True), (1, 9, 4096, 8192, 24576, 16384, False),
    (1, 1, 512, 512, 1024, 4096, True), (1, 1, 512, 512, 1024, 4160, False),
    (1, 1, 8256, 8192, 10240, 28672, False), (1, 1, 4128, 4096, 6144, 14336, False),
    (0, 64, 256, 256, 768, 1024, True), (0, 65, 256, 256, 768, 1024, False), (0, 64, 256, 32768, 98304, 1024, True),
    (0, 1, 192, 128, 384, 72, False), (2, 1, 4096, 4096, 6144, 14336, False),
])
def test_layers_of_a_few_rows_in_five_launches(dtype, M, d, hq, qkv, F, fused):
    rule = _rule("_ZN2gs10rows_fusedEiiiiii", C.c_bool, *[C.c_int] * 6)
    assert rule(dtype, M, d, hq, qkv, F) == fused and not rule(dtype, 0, d, hq, qkv, F)


def gemm_splits(dtype, M, N, K):
    return _rule("_ZN2gs11gemm_splitsEiiii", C.c_int, *[C.c_int] * 4)({"f32": 0, "bf16": 1, "w4": 2}[dtype], M, N, K)


@pytest.mark.parametrize("N,K,splits", [
    (4096, 14336, 4), (4096, 4096, 4), (3072, 12288, 5), (5120, 5120, 3), (7168, 5120, 2),       # 64 columns, four K groups
    (1024, 2048, 2), (1024, 16384, 16), (6144, 2048, 2), (512, 640, 1),                          # as many splits as K allows
    (6144, 4096, 4), (6144, 6144, 5), (6144, 12288, 5),      # 192 workgroups of 64 columns: 128 columns and two K groups
    (8192, 8192, 4),
])
def test_w4_splits_at_33_to_64_rows(N, K, splits):
    assert [gemm_splits("w4", M, N, K) for M in (33, 53, 64)] == [splits] * 3


@pytest.mark.parametrize("dtype,most", [(1, 16), (0, 64)])
def test_layers_of_five_launches_refuse_more_rows(dtype, most):
    """The launchers hold one row tile (bf16) or one row chunk (fp32): more rows are refused before anything is launched."""
    args = [C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p]
    residual = _rule("_ZN2gs20launch_rows_residualEiPKvS1_RKNS_11ResidualOutEiiiP12ihipStream_t", C.c_int, *args)
    out = (C.c_char * 64)()
    assert residual(dtype, None, None, C.addressof(out), most + 1, 256, 256, None) == -5      # GS_EUNSUPPORTED
    assert b"at most %d" % most in gsb.lib().gs_last_error()
    gate_up = _rule("_ZN2gs19launch_rows_gate_upEiPKvS1_RKNS_7RowNormEPviiiP12ihipStream_t", C.c_int,
                    C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_int, C.c_void_p)
    assert gate_up(dtype, None, None, C.addressof(out), None, most + 1, 256, 256, None) == -5
    qkv = _rule("_ZN2gs15launch_rows_qkvEiPKvS1_RKNS_7RowNormERKNS_6QkvOutEiiP12ihipStream_t", C.c_int,
                C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_int, C.c_void_p)
    assert qkv(dtype, None, None, C.addressof(out), C.addressof(out), most + 1, 256, None) == -5


@pytest.mark.parametrize("gamma,ctx,groups", [
    ([2046], [0], 2), ([127] * 8, [0] * 8, 1), ([300] * 4, [500] * 4, 2),      # the longest split of a prompt has 64, 4 and 26 steps
    ([223] * 5, [0] * 5, 1), ([255] * 5, [0] * 5, 2),                          # 7 and 8
    ([120], [700], 1),                                                         # groups that leave compute units idle are split instead
])
def test_attention_key_groups_of_prompts(gamma, ctx, groups):
    assert attention_key_groups(8, 4, gamma, ctx)[0] == groups


class _QkvOut(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("row_slot", "rope", "q", "k_pages", "v_pages")] + [(n, C.c_int) for n in ("page_size", "n_heads", "n_kv", "hd")]


@pytest.mark.parametrize("M,fused", [(17, False), (64, False), (128, False), (324, False), (512, False), (640, False), (800, True), (1024, True),
                                     (1280, True), (1500, False), (1800, True), (2047, True)])
def test_qkv_projections_of_many_rows_store_heads(M, fused):
    """Where whole sums are modelled no slower, and operands and places are aligned; bf16 alone."""
    rule = _rule("_ZN2gs9qkv_fusedEiPKvS1_RKNS_6QkvOutEii", C.c_bool, C.c_int, C.c_void_p, C.c_void_p, C.POINTER(_QkvOut), C.c_int, C.c_int)

    def ask(dtype=1, x=4096, w=4096, q=4096, k=4096, v=4096):
        return rule(dtype, x, w, C.byref(_QkvOut(4096, 4096, q, k, v, 16, 32, 8, 128)), M, 4096)

    assert ask() == fused and ask(k=4100, v=4104) == fused
    assert not ask(dtype=0) and not ask(dtype=2)
    assert not ask(x=4104) and not ask(w=4104) and not ask(k=4098) and not ask(v=4100)
