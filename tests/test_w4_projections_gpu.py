"""4-bit projections launched through the library's internal C++ symbols, on both sides of the line between one and two column tiles of a wave
beyond 96 rows, at row counts around the chunks of 128 and with K splits of unequal length, and the shapes with one step of activations ahead.

Codes, zero points, scales that are powers of two and small whole activations: products and fp32 sums are exact, so the result has to be
the float64 product.  The same with one scale group so large that its weights are repaired, as the only one that meets non-zero
activations."""
import ctypes as C

import pytest
import torch

from paper_2512_09963_amd import binding as gsb

pytestmark = pytest.mark.gpu


def run(x, packed, M, N, K):
    lib, V, I = gsb.lib(), C.c_void_p, C.c_int
    splits = lib._ZN2gs14gemm_w4_splitsEiii
    splits.restype, splits.argtypes = I, [I, I, I]
    launch = lib._ZN2gs14launch_gemm_w4EPKvS1_PfiiiP12ihipStream_t
    launch.restype, launch.argtypes = I, [V, V, V, I, I, I, V]
    out = torch.full((splits(M, N, K), M, N), 7.0, device="cuda")
    assert launch(x.data_ptr(), packed.data_ptr(), out.data_ptr(), M, N, K, torch.cuda.current_stream().cuda_stream) == 0
    return out.double().sum(0)


@pytest.mark.parametrize("rows,N,K", [
    ([97, 128], 8192, 6144), ([129], 4096, 6144), ([300], 4096, 4096),      # two tiles: exactly 192 workgroups' worth
    ([640], 5120, 2304), ([97, 129], 8192, 5120),                           # two tiles, K splits that do not divide; one tile
    ([128, 250], 4096, 4096), ([512], 2560, 1024), ([257], 384, 1152),      # one tile; no multiple of 256 columns
    ([1, 16, 33, 64, 96], 1024, 1152), ([17, 53], 448, 640),                # up to 96 rows
])
def test_sums_are_exact(rows, N, K):
    g = torch.Generator(device="cuda")
    g.manual_seed(N + K)
    codes = torch.randint(0, 16, (N, K), generator=g, device="cuda", dtype=torch.uint8)
    zeros = torch.randint(0, 16, (N, K // 128), generator=g, device="cuda", dtype=torch.uint8)
    scales = torch.ldexp(torch.ones((), device="cuda"), torch.randint(-3, 1, (N, K // 128), generator=g, device="cuda")).to(torch.bfloat16)
    for large in (None, 0, K // 256, K // 128 - 1):      # scale group of 2^118
        s = scales.clone()
        if large is not None:
            s[::3, large] = 2.0 ** 118
        packed = gsb.gs_pack_weight_w4(codes, s, zeros)
        w = ((codes.view(N, K // 128, 128).double() - zeros.double()[:, :, None]) * s.double()[:, :, None]).view(N, K)
        for M in rows:
            x = torch.randint(-4, 5, (M, K), generator=g, device="cuda").to(torch.bfloat16)
            if large is not None:
                x[:, :128 * large] = 0
                x[:, 128 * (large + 1):] = 0
                x[:, 128 * large + 1:128 * (large + 1)] = 0      # (one term: the sum of many would overflow)
            assert torch.equal(run(x, packed, M, N, K), x.double() @ w.t().contiguous()), (M, large)
