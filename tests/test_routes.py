"""Which kernels serve a call: the rules by sizes and types that the launchers ask, read through the library's internal C++ symbols
(no GPU needed).  The lines lie where both sides were measured; the figures stand beside the rules."""
import ctypes as C

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
    (1088, 4096, False),                                                                     # no multiple of 128 columns
])
def test_bf16_projections_of_up_to_64_rows(M, N, K, wide):
    assert _wide_serves(M, N, K) == wide


@pytest.mark.parametrize("N,K", [(1024, 1024), (1024, 4096), (2048, 2048), (4096, 14336)])
def test_bf16_projections_of_more_rows_are_wide(N, K):
    assert _wide_serves(65, N, K) and _wide_serves(2047, N, K) and not _wide_serves(65, N + 64, K)
