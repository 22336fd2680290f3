"""The QKV projection of many rows with the rotation and the KV append in its epilogue, launched through the library's internal C++ symbols: every
shape of its kernel and both head sizes, rows at the edges of its tiles, pages of 16 and 48 slots, blocks that start anywhere in a page.

Inputs are small multiples of powers of two, so the sums are exact: V has to be the bfloat16 rounding of a float64 product.  Q and K: a rotation
in fp32 (2^-22 of the larger of its two terms) and one rounding to bfloat16 (2^-9 of the value, a unit more where the first one moves it over a tie)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2512_09963_amd import binding as gsb
from tests.test_projections_gpu import Plan, operands

pytestmark = pytest.mark.gpu


class QkvOut(C.Structure):
    _fields_ = [(n, C.c_void_p) for n in ("row_slot", "rope", "q", "k_pages", "v_pages")] + [(n, C.c_int) for n in ("page_size", "n_heads", "n_kv", "hd")]


def launch(plan, x, w, out, M, N, K):
    f = gsb.lib()._ZN2gs16launch_block_qkvERKNS_8WidePlanEPKtS4_RKNS_6QkvOutEiiiP12ihipStream_t
    f.restype, f.argtypes = C.c_int, [C.c_void_p] * 4 + [C.c_int] * 3 + [C.c_void_p]
    return f(C.addressof(plan), x.data_ptr(), w.data_ptr(), C.addressof(out), M, N, K, torch.cuda.current_stream().cuda_stream)


SHAPES = [(4, 2, 1, 4, 8), (2, 2, 1, 4, 6), (2, 2, 1, 4, 4), (1, 4, 2, 8, 4)]


@pytest.mark.parametrize("page", [16, 48])
@pytest.mark.parametrize("hd,H,Hk", [(128, 2, 2), (128, 4, 1), (64, 8, 2), (64, 4, 4)])      # (768 columns)
@pytest.mark.parametrize("shape", SHAPES)
def test_heads(shape, hd, H, Hk, page):
    wm, wn, kg, mt, nt = shape
    rows, cols, N = wm * mt * 16, wn * nt * 16, (H + 2 * Hk) * hd
    for M, K in ((rows - 1, 64), (rows + 1, 192), (2 * rows + 17, 128)):
        x, w, xs, ws = operands(M, N, K)
        r = np.random.RandomState(M + page)
        page_of, slot_of, used = np.zeros(M, np.int64), np.zeros(M, np.int64), 0
        a = 0
        while a < M:      # blocks of 1 to 70 rows, each in pages of its own from some slot on
            n, first = min(M - a, r.randint(1, 71)), r.randint(0, page)
            pos = first + np.arange(n)
            page_of[a:a + n], slot_of[a:a + n] = used + pos // page, pos % page
            used += int(pos[-1] // page) + 1
            a += n
        slots = torch.from_numpy(np.stack([page_of, slot_of, np.zeros(M), np.zeros(M)], 1).astype(np.int32)).cuda()
        ang = torch.rand(M, hd // 2, device="cuda") * 6.28
        rope = torch.stack([torch.cos(ang), torch.sin(ang)], 2).contiguous()
        q = torch.full((M, H, hd), 7.0, dtype=torch.bfloat16, device="cuda")
        k = torch.full((used, Hk, page, hd), 7.0, dtype=torch.bfloat16, device="cuda")
        v = torch.full((used, Hk, hd, page), 7.0, dtype=torch.bfloat16, device="cuda")
        plan = Plan(wm, wn, kg, mt, nt, -(-M // rows), N // cols, 1, K, True, 0.0)
        out = QkvOut(slots.data_ptr(), rope.data_ptr(), q.data_ptr(), k.data_ptr(), v.data_ptr(), page, H, Hk, hd)
        assert launch(plan, xs, ws, out, M, N, K) == 0
        ref = (x.double() @ w.double().t().contiguous()).view(M, H + 2 * Hk, hd)
        a_, b_ = ref[:, :H + Hk, :hd // 2], ref[:, :H + Hk, hd // 2:]
        cos, sin = rope[:, None, :, 0].double(), rope[:, None, :, 1].double()
        want = torch.cat([a_ * cos - b_ * sin, b_ * cos + a_ * sin], 2)
        size = torch.maximum(a_.abs(), b_.abs()).repeat(1, 1, 2)
        pg, sl = torch.from_numpy(page_of).cuda(), torch.from_numpy(slot_of).cuda()
        got = torch.cat([q, k[pg, :, sl]], 1).double()
        assert ((got - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -21 * size).all()
        assert torch.equal(v[pg, :, :, sl], ref[:, H + Hk:].to(torch.bfloat16))
        rest = torch.ones(used, page, dtype=torch.bool, device="cuda")      # slots of no row stay as they were
        rest[pg, sl] = False
        assert (k.transpose(1, 2)[rest] == 7.0).all() and (v.permute(0, 3, 1, 2)[rest] == 7.0).all()
