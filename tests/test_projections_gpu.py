"""bf16 projections of many rows, launched through the library's internal C++ symbols: every shape of the kernel that takes weights and
activations through LDS, and the plans of the launcher, at the edges of their tiles.

Inputs are small multiples of powers of two, so that every product and every fp32 sum is exact, whatever the order: the sums have to be
equal to a float64 product.  SwiGLU: one rounding to bfloat16 (2^-9 of the value) and expf (1e-6).  Statistics: fp32 exponentials and at
most a few hundred terms a block (1e-5)."""
import ctypes as C

import pytest
import torch

from paper_2512_09963_amd import binding as gsb

pytestmark = pytest.mark.gpu

PLAIN, GATE_UP, STATS = 0, 1, 2
SHAPES = [(4, 2, 1, 4, 8), (4, 2, 1, 4, 7), (2, 2, 1, 4, 6), (2, 2, 1, 4, 4), (1, 4, 2, 8, 4), (1, 4, 2, 10, 4), (1, 4, 2, 11, 4)]


class Plan(C.Structure):
    _fields_ = [(n, C.c_int) for n in "wm wn kg mt nt m_chunks n_blocks splits k_per".split()] + [("block", C.c_bool), ("us", C.c_float)]


def _symbol(name, *argtypes):
    f = getattr(gsb.lib(), name)
    f.restype, f.argtypes = C.c_int, list(argtypes)
    return f


V, I = C.c_void_p, C.c_int


def operands(M, N, K, offset=0):
    """x, w row-major (exactly summable) and w packed, both `offset` elements off their allocation."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M * 7 + N * 3 + K)
    x = torch.randint(-4, 5, (M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-4, 5, (N, K), generator=g, device="cuda").to(torch.bfloat16) / 64
    xs = torch.empty(M * K + offset, dtype=torch.bfloat16, device="cuda")[offset:].view(M, K).copy_(x)
    packed = gsb.gs_pack_weight(w).view(-1)
    ws = torch.empty(packed.numel() + offset, dtype=packed.dtype, device="cuda")[offset:].copy_(packed)
    return x, w, xs, ws


def check(mode, got, x, w, stats=None):
    ref = x.double() @ w.double().t().contiguous()
    if mode == GATE_UP:
        F = w.shape[0] // 2
        ref = torch.nn.functional.silu(ref[:, :F]) * ref[:, F:]
        assert ((got.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-30).all()
        return
    assert torch.equal(got.double(), ref)
    if mode == STATS:
        m, s = stats[..., 0].double(), stats[..., 1].double()
        lse = torch.logsumexp(m + torch.log(s), 1)
        assert torch.allclose(lse, torch.logsumexp(ref, 1), rtol=1e-5, atol=1e-5)
        assert torch.equal(m.amax(1), ref.amax(1))


def stream():
    return torch.cuda.current_stream().cuda_stream


def columns(shape):
    return 16 * shape[1] * shape[4]


@pytest.mark.parametrize("mode", [PLAIN, GATE_UP, STATS])
@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("rows,blocks,K,splits", [
    (0, 1, 64, 1), (1, 3, 128, 1), (-1, 2, 192, 1),      # a whole row chunk, a row more, a row less; 1 to 3 steps
    (None, 9, 320, 1), (17, 5, 1024, 1),                 # one row; column blocks that the XCDs do not share evenly
    (5, 2, 704, 4), (0, 3, 1024, 16),                    # K splits of 3, 3, 3 and 2 steps, of one step
])
def test_shapes_at_their_edges(mode, shape, rows, blocks, K, splits):
    if (splits > 1 and mode != PLAIN) or (mode == STATS and columns(shape) % 128):
        pytest.skip("whole sums; statistics of 128 or 256 columns")
    wm, wn, kg, mt, nt = shape
    chunk = 16 * wm * mt
    M, N = 1 if rows is None else chunk + rows, blocks * columns(shape)
    if N % 64 or (mode == GATE_UP and N % 128):
        N *= 2
    x, w, xs, ws = operands(M, N, K)
    k_per = -(-(-(-K // splits)) // 64) * 64
    assert -(-K // k_per) == splits
    plan = Plan(wm, wn, kg, mt, nt, -(-M // chunk), N // columns(shape), splits, k_per, True, 0.0)
    out = torch.full((splits, M, N // 2 if mode == GATE_UP else N), 7.0, dtype=torch.bfloat16 if mode == GATE_UP else torch.float32, device="cuda")
    stats = torch.empty(M, plan.n_blocks, 2, device="cuda")
    launch = _symbol("_ZN2gs12launch_blockEiRKNS_8WidePlanEPKtS4_PfiiiP15HIP_vector_typeIfLj2EEP12ihipStream_t", I, C.POINTER(Plan), V, V, V, I, I, I, V, V)
    assert launch(mode, C.byref(plan), xs.data_ptr(), ws.data_ptr(), out.data_ptr(), M, N, K, stats.data_ptr(), stream()) == 0
    check(mode, out[0] if splits == 1 else out.sum(0), x, w, stats)


@pytest.mark.parametrize("offset", [0, 2])      # (operands off a multiple of 16 bytes: no direct loads into LDS)
@pytest.mark.parametrize("M,N,K", [(65, 1152, 1024), (129, 3072, 2048), (200, 2304, 512), (300, 1280, 5120), (324, 1792, 256), (511, 4480, 128), (1025, 768, 3072)])
def test_planned_launches(M, N, K, offset):
    x, w, xs, ws = operands(M, N, K, offset)
    splits = _symbol("_ZN2gs11gemm_splitsEiiii", I, I, I, I)(1, M, N, K)
    out = torch.full((splits, M, N), 7.0, device="cuda")
    launch = _symbol("_ZN2gs11launch_gemmEiPKvS1_PfiiiP12ihipStream_t", I, V, V, V, I, I, I, V)
    assert launch(1, xs.data_ptr(), ws.data_ptr(), out.data_ptr(), M, N, K, stream()) == 0
    check(PLAIN, out.sum(0), x, w)
    act = torch.full((M, N // 2), 7.0, dtype=torch.bfloat16, device="cuda")
    launch = _symbol("_ZN2gs19launch_gemm_gate_upEiPKvS1_PviiiP12ihipStream_t", I, V, V, V, I, I, I, V)
    assert launch(1, xs.data_ptr(), ws.data_ptr(), act.data_ptr(), M, N // 2, K, stream()) == 0
    check(GATE_UP, act, x, w)
    blocks = _symbol("_ZN2gs16gemm_stat_blocksEiiii", I, I, I, I)(1, M, N, K)
    if blocks:
        logits, stats = torch.full((M, N), 7.0, device="cuda"), torch.empty(M, blocks, 2, device="cuda")
        launch = _symbol("_ZN2gs17launch_gemm_statsEPKvS1_PfPviiiP12ihipStream_t", V, V, V, V, I, I, I, V)
        assert launch(xs.data_ptr(), ws.data_ptr(), logits.data_ptr(), stats.data_ptr(), M, N, K, stream()) == 0
        check(STATS, logits, x, w, stats)
