"""Edges of the kernels that serve blocks of a few rows: the fp32 attention (chunks of 128 keys, page sizes) and the layers of
five launches (norms, rotation and residual inside the projections)."""
import numpy as np
import pytest

from paper_2512_09963_amd import synth
from tests.test_routes import attention_key_groups
from tests.test_verify_gpu import _run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,page,gamma,ctx", [
    (64, 16, [0, 1, 2, 0], [0, 126, 127, 128]),        # 1 key; the last row at, the first past a chunk of 128
    (64, 7, [3, 0, 5], [13, 255, 300]),                # pages that are no multiple of 4: scalar loads
    (128, 1, [2, 1], [3, 130]),
    (128, 12, [4, 6], [253, 40]),                      # a multiple of 4 but not of 16
    (128, 64, [1, 15], [512, 1]),
    (64, 16, [1, 0], [30, 12]),                        # 32 keys: no look-up ahead
    (64, 16, [1, 0], [31, 12]),                        # 33
    (64, 16, [127], [300]),                            # 128 rows of 4 heads: the last launch that looks its pages up ahead
    (64, 16, [128], [300]),
    (128, 4, [100, 27, 2], [130, 0, 513]),             # past it
])
def test_f32_attention_chunks_and_page_sizes(hd, page, gamma, ctx):
    """Against the float64 oracle within 1e-4 of the row scale (float32 sums of at most a few hundred terms: about 1e-6)."""
    ms = synth.ModelShape(2, 4 * hd, 4, 2, hd, 384, 320, 10000.0, dtype="f32")
    _run_case(ms, 41 + page, np.array(gamma, np.int32), np.array(ctx, np.int32), page, 0.05)


@pytest.mark.parametrize("d,heads,n_kv,hd,ffn,rows", [
    (64, 1, 1, 64, 16, 2),             # the narrowest: 4 column tiles, one pair of gate and up
    (64, 2, 1, 128, 48, 16),           # head size 128: 4 pairs of tiles a head; 16 rows: the last of one row tile
    (128, 4, 2, 64, 400, 17),
    (320, 4, 4, 64, 1040, 33),         # K of 20 steps in slices of unequal length
    (192, 2, 2, 64, 72, 48),           # features that are no multiple of 16: the separate kernels
    (100, 2, 1, 64, 64, 9),            # a width that is no multiple of 64: the separate kernels
    (256, 4, 4, 64, 1024, 64),
    (256, 4, 4, 64, 1024, 65),         # past the last fused row
    (4160, 1, 1, 64, 32, 3),           # sums of squares of 260 tiles: five loads per lane
])
def test_f32_layer_of_five_launches(d, heads, n_kv, hd, ffn, rows):
    ms = synth.ModelShape(2, d, heads, n_kv, hd, ffn, 272, 10000.0, dtype="f32")
    gamma = np.array([rows - 1 - rows // 3, rows // 3 - 1] if rows >= 3 else [rows - 1], np.int32)
    _run_case(ms, 300 + rows, gamma, np.array([37, 5][:gamma.size], np.int32), 16, 0.06)


@pytest.mark.parametrize("d,heads,n_kv,hd,ffn,rows", [
    (64, 1, 1, 64, 64, 2),             # one k step: three waves of four have none
    (128, 2, 1, 128, 192, 16),
    (192, 4, 2, 64, 576, 11),          # 3 and 9 steps over 8 and 4 waves; head size 64: 2 tiles a half
    (320, 8, 1, 64, 2496, 15),         # 39 steps: past the ring of 8 x 4 steps
    (192, 4, 2, 64, 576, 17),          # past the last row: K splits and separate norms
    (320, 8, 1, 64, 2496, 31),
    (256, 8, 8, 128, 1024, 32),
    (256, 8, 8, 128, 1024, 33),
    (128, 4, 4, 64, 1088, 9),          # F > 8 d: the kernels with K splits
    (256, 64, 8, 128, 512, 12),        # 10240 columns: two pairs of tiles per workgroup
    (256, 63, 63, 64, 512, 13),        # 12096 columns: 189 workgroups of two pairs
    (256, 63, 63, 64, 512, 20),
    (4160, 2, 2, 64, 128, 7),          # 260 column tiles: two per workgroup; sums of squares of 260 tiles
    (4160, 2, 2, 64, 128, 27),
])
def test_bf16_layer_of_five_launches(d, heads, n_kv, hd, ffn, rows):
    """Against the oracle within 2e-2 of the row scale, K and V rows as well (one bf16 rounding of h, before instead of after the
    division by the root mean square, is as large as the one it replaces)."""
    ms = synth.ModelShape(2, d, heads, n_kv, hd, ffn, 384, 10000.0, dtype="bf16")
    gamma = np.array([rows - 1 - rows // 3, rows // 3 - 1] if rows >= 3 else [rows - 1], np.int32)
    # scores have a standard deviation of d std^2 sqrt(hd), and a rounding of q or k is amplified by that factor: at most
    # 1.44 sqrt(hd) = 16 (0.05 at d = 4160 would be 83, where softmax is nearly an argmax)
    _run_case(ms, 500 + rows, gamma, np.array([250, 5][:gamma.size], np.int32), 16, min(0.05, 1.2 / d ** 0.5))


@pytest.mark.parametrize("rows", [17, 32, 33, 49, 64, 65])
def test_bf16_projections_with_four_k_groups(rows):
    """5120 x 3584 in 3 K splits of 19, 19 and 18 steps (groups of 5, 5, 5 and 4 or 3 steps) and 3584 x 4096 in 4 of 16; two and four row
    tiles, of which a K group owns none, one or two; 65 rows: past them.  The down projection (K = 192) has no split."""
    ms = synth.ModelShape(1, 3584, 32, 4, 128, 192, 512, 10000.0, dtype="bf16")
    gamma = np.array([rows - 20, 11, 6] if rows > 20 else [rows - 3, 0, 1], np.int32)
    # (std: see above)
    _run_case(ms, 700 + rows, gamma, np.array([40, 0, 19], np.int32), 16, 0.02)


@pytest.mark.parametrize("rows", [17, 33, 64, 65])
def test_bf16_projections_of_small_matrices(rows):
    """2048 x 1024, 1024 x 1024 and 1024 x 2048 in two, two and four K splits of the skinny kernel, two and four row tiles; 65 rows: past
    them."""
    ms = synth.ModelShape(1, 1024, 8, 4, 128, 2048, 512, 10000.0, dtype="bf16")
    gamma = np.array([rows - 12, 0, 9], np.int32)
    _run_case(ms, 600 + rows, gamma, np.array([40, 0, 19], np.int32), 16, 0.035)


@pytest.mark.parametrize("heads,n_kv,hd,gamma,ctx,page,key_groups", [
    (4, 1, 128, [7, 0], [0, 60], 16, 1),                   # short contexts: one wave and one ring
    (4, 1, 128, [7, 0], [80, 60], 16, 4),                  # three and two steps: a key group has none
    (4, 1, 128, [7, 0], [0, 300], 16, 4),                  # one step (three key groups have none) beside splits of five
    (4, 2, 128, [3, 0], [40, 190], 16, 4),                 # two and six steps
    (8, 2, 64, [4, 2], [700, 129], 32, 4),                 # splits of six and five steps
    (8, 1, 128, [3], [8190], 16, 4),                       # 29 splits of nine and eight, the longest context here; a block across a step's end
    (2, 2, 64, [31, 5, 0], [333, 64, 1], 48, 4),           # a full tile of rows; page size that is no power of two
])
def test_bf16_attention_with_key_groups(heads, n_kv, hd, gamma, ctx, page, key_groups):
    """Few workgroups of one tile of query rows: four waves share the steps of a split."""
    assert attention_key_groups(n_kv, heads // n_kv, gamma, ctx)[0] == key_groups
    ms = synth.ModelShape(1, 128, heads, n_kv, hd, 192, 320, 10000.0, dtype="bf16")
    _run_case(ms, 900 + page + heads, np.array(gamma, np.int32), np.array(ctx, np.int32), page, 0.08)


@pytest.mark.parametrize("rows,page", [(1, 16), (12, 16), (40, 32)])
def test_bf16_attention_quotient_is_correctly_rounded(rows, page):
    """Attention of equal scores is the mean of V.  Here every mean is an integer plus one half, halfway between two bf16 values from
    128 on, and the float32 sums are exact, so a quotient that is off by one bit in float32 is off by one bf16 step in the result.
    Among the key counts are those (14, 30, 56, 60, 126, ...) whose rounded reciprocal times the sum is not the quotient."""
    import torch
    from paper_2512_09963_amd import binding as gsb
    d, hd, vocab = 256, 128, 64
    dev = torch.device("cuda:0")
    counts = [14, 30, 56, 60, 122, 126, 120, 112, 28, 52, 104, 26, 110, 94, 4, 6, 100, 128, 64][:rows]
    counts += [10 + 2 * i for i in range(rows - len(counts))]
    bf = dict(dtype=torch.bfloat16, device=dev)
    zeros = lambda n, k: gsb.gs_pack_weight(torch.zeros(n, k, **bf))
    layer = dict(wqkv=zeros(2 * d + d, d), wo=gsb.gs_pack_weight(torch.eye(d, **bf)), wgu=zeros(2 * 64, d), wd=zeros(d, 64),
                 norm1=torch.ones(d, device=dev), norm2=torch.ones(d, device=dev))
    top = dict(embed=torch.zeros(vocab, d, **bf), lm_head=zeros(vocab, d), final_norm=torch.ones(d, device=dev))
    desc = dict(n_layers=1, d_model=d, n_heads=2, n_kv_heads=2, head_dim=hd, d_ffn=64, vocab=vocab, rope_theta=10000.0, rms_eps=1e-5,
                dtype="bf16")
    ver = gsb.Verifier(desc, top, [layer])
    gamma, ctx = np.zeros(rows, np.int32), np.array([n - 1 for n in counts], np.int32)
    batch = synth.make_batch(3, gamma, ctx, page, permute_pages=True)
    k = torch.zeros(1, batch.n_pages, 2, page, hd, **bf)
    v = torch.zeros(1, batch.n_pages, 2, hd, page, **bf)
    a = torch.arange(128, 256, device=dev, dtype=torch.float32).repeat(2).view(2, hd)
    for i, n in enumerate(counts):      # the block's own value is 0: n / 2 values a + 1, n / 2 - 2 values a and one 2 a
        vals = [a + 1] * (n // 2) + [a] * (n // 2 - 2) + [2 * a]
        assert len(vals) == n - 1
        for p, val in enumerate(vals):
            v[0, int(batch.block_table[i, p // page]), :, :, p % page] = val.to(torch.bfloat16)
    trace = torch.empty(2, rows, d, device=dev)
    ver.gs_trace_residual(trace)
    logits = torch.empty(rows, vocab, device=dev)
    ws = torch.empty(ver.gs_workspace_bytes(rows, rows, int(max(counts))), dtype=torch.uint8, device=dev)
    ver.gs_verify_batch(k, v, page, batch.n_pages, gamma, ctx, torch.from_numpy(batch.cu_rows).to(dev), torch.from_numpy(ctx).to(dev),
                        torch.zeros(rows, dtype=torch.int32, device=dev), torch.from_numpy(batch.block_table).to(dev), None, None, None,
                        None, logits, ws)
    torch.cuda.synchronize()
    want = (a + 0.5).view(1, d).to(torch.bfloat16).float().expand(rows, d)
    assert torch.equal(trace[1], want)


@pytest.mark.parametrize("rows", [1, 20, 64, 70])
def test_f32_row_factor_is_that_of_a_quotient(rows):
    """Rows of ones have a mean square of exactly 1 and a factor of exactly 1, whatever the width.  2624 is 41 * 64: its rounded reciprocal times
    2624 is one bit below 1, and the factor would be one bit above it."""
    import torch
    from paper_2512_09963_amd import binding as gsb
    d, hd, vocab = 2624, 64, 96
    dev = torch.device("cuda:0")
    f32 = dict(dtype=torch.float32, device=dev)
    pick = torch.zeros(vocab, d, **f32)
    pick[torch.arange(vocab), torch.arange(vocab) * 27] = 1.0      # logit j is element 27 j of the normed row
    layer = dict(wqkv=torch.zeros(3 * hd, d, **f32), wo=torch.zeros(d, hd, **f32), wgu=torch.zeros(2 * 16, d, **f32),
                 wd=torch.zeros(d, 16, **f32), norm1=torch.ones(d, **f32), norm2=torch.ones(d, **f32))
    top = dict(embed=torch.ones(vocab, d, **f32), lm_head=pick, final_norm=torch.ones(d, **f32))
    desc = dict(n_layers=1, d_model=d, n_heads=1, n_kv_heads=1, head_dim=hd, d_ffn=16, vocab=vocab, rope_theta=10000.0, rms_eps=0.0,
                dtype="f32")
    ver = gsb.Verifier(desc, top, [layer])
    gamma, ctx = np.array([rows - 1], np.int32), np.zeros(1, np.int32)
    batch = synth.make_batch(5, gamma, ctx, 16)
    k, v = torch.zeros(1, batch.n_pages, 1, 16, hd, **f32), torch.zeros(1, batch.n_pages, 1, hd, 16, **f32)
    logits = torch.empty(rows, vocab, **f32)
    ws = torch.empty(ver.gs_workspace_bytes(rows, 1, rows), dtype=torch.uint8, device=dev)
    ver.gs_verify_batch(k, v, 16, batch.n_pages, gamma, ctx, torch.from_numpy(batch.cu_rows).to(dev), torch.from_numpy(ctx).to(dev),
                        torch.zeros(rows, dtype=torch.int32, device=dev), torch.from_numpy(batch.block_table).to(dev), None, None, None,
                        None, logits, ws)
    torch.cuda.synchronize()
    assert torch.equal(logits, torch.ones_like(logits))


def _small_model(dtype):
    return synth.ModelShape(2, 256, 4, 2, 64, 512, 1024, 10000.0, dtype=dtype)


def _prepare(ms, seed, gamma, ctx, std=0.08):
    """(verifier, KV cache, device batch, workspace) and what the oracle starts from."""
    import torch
    from paper_2512_09963_amd import workload as wl
    top = synth.top_weights(ms, seed, std=std)
    layers = [synth.layer_weights(ms, seed, l, std=std) for l in range(ms.n_layers)]
    batch = synth.make_batch(seed, np.array(gamma, np.int32), np.array(ctx, np.int32), 16, permute_pages=True)
    tokens, q, ua, ur = synth.verify_side_inputs(seed, ms.vocab, batch.gamma, sigma=0.5)
    ver = wl.upload_model(ms, top, lambda l: layers[l])
    kv = wl.KVCache(ms, batch.n_pages, 16)
    cache = [(synth.kv_layer_cache(ms, seed, l, "k", batch.n_pages, 16), synth.kv_layer_cache(ms, seed, l, "v", batch.n_pages, 16))
             for l in range(ms.n_layers)]
    for l in range(ms.n_layers):
        kv.set_layer(l, *cache[l])
    db = wl.DeviceBatch(batch, tokens, q, ua, ur)
    ws = torch.empty(ver.gs_workspace_bytes(db.n_rows, db.n_servers, db.max_ctx), dtype=torch.uint8, device="cuda:0")
    return ver, kv, db, ws, (top, layers, batch, tokens, cache)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layers_of_five_launches_under_capture(dtype):
    """Replays, with eager work and synchronisations between them, give the eager result bit for bit."""
    import torch
    from paper_2512_09963_amd import binding as gsb, workload as wl
    ms = _small_model(dtype)
    ver, kv, db, ws, _ = _prepare(ms, 61, [4, 0, 2, 5], [37, 5, 260, 0])
    ref_out, ref_logits, _ = wl.verify(ver, kv, db, workspace=ws)
    torch.cuda.synchronize()
    ref_out, ref_logits = {k: v.clone() for k, v in ref_out.items()}, ref_logits.clone()
    out, logits = gsb.make_accept_out(db.n_servers, db.n_draft, torch.device("cuda:0")), torch.empty_like(ref_logits)
    args = (kv.k, kv.v, kv.page_size, kv.n_pages, db.gamma, db.ctx_len_host, db.cu_rows, db.ctx_len, db.tokens, db.block_table,
            db.q_probs, db.u_accept, db.u_resample, out, logits, ws)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        ver.gs_verify_batch(*args)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ver.gs_verify_batch(*args)
    for rep in range(3):
        logits.zero_()
        ws.fill_(0xff)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(logits, ref_logits), f"replay {rep}"
        for k, v in ref_out.items():
            assert torch.equal(out[k], v), f"replay {rep}: {k}"
        wl.verify(ver, kv, db, workspace=ws)
        torch.cuda.synchronize()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_residual_trace_of_layers_of_five_launches(dtype):
    """Entry l is the residual stream that enters layer l.  The last entry, normed and multiplied by the LM head on the host, gives the
    logits: to 1e-5 of the row scale in fp32, to the rounding of the normed row in bf16 (2^-9 an element, 1e-2 with 256 of them)."""
    import torch
    from paper_2512_09963_amd import workload as wl
    ms = _small_model(dtype)
    ver, kv, db, ws, (top, layers, batch, tokens, _) = _prepare(ms, 62, [4, 0, 2, 5], [37, 5, 260, 0])
    trace = torch.full((ms.n_layers + 1, db.n_rows, ms.d_model), float("nan"), device="cuda:0")
    ver.gs_trace_residual(trace)
    _, logits, _ = wl.verify(ver, kv, db, workspace=ws)
    torch.cuda.synchronize()
    ver.gs_trace_residual(None)
    tr = trace.cpu().numpy().astype(np.float64)
    np.testing.assert_array_equal(tr[0], np.asarray(top["embed"], np.float64)[tokens])
    assert np.isfinite(tr).all() and (np.abs(tr[1:] - tr[:-1]).max(axis=(1, 2)) > 0).all()
    x = tr[-1]
    h = x * np.asarray(top["final_norm"], np.float64) / np.sqrt((x * x).mean(axis=1, keepdims=True) + ms.rms_eps)
    want = h @ np.asarray(top["lm_head"], np.float64).T
    err = np.abs(logits.cpu().numpy() - want) / np.abs(want).max(axis=1, keepdims=True)
    assert err.max() <= (1e-5 if dtype == "f32" else 1e-2)


def test_f32_weights_that_are_not_16_byte_aligned():
    """Matrices four bytes past an aligned address take scalar loads; the sums are formed in the same order."""
    import torch
    from paper_2512_09963_amd import binding as gsb, workload as wl
    ms = _small_model("f32")
    ver, kv, db, ws, _ = _prepare(ms, 63, [4, 0, 2, 5], [37, 5, 260, 0])
    _, want, _ = wl.verify(ver, kv, db, workspace=ws)
    want = want.clone()

    def moved(t):
        m = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:]
        m.view(t.shape).copy_(t)
        assert m.data_ptr() % 16 == 4
        return m
    top, layers = ver._keep
    mats = ("wqkv", "wo", "wgu", "wd")
    other = gsb.Verifier(ver.desc, dict(top, lm_head=moved(top["lm_head"])),
                         [dict(l, **{k: moved(l[k]) for k in mats}) for l in layers])
    _, got, _ = wl.verify(other, kv, db, workspace=ws)
    torch.cuda.synchronize()
    assert float((got - want).abs().max()) <= 1e-6 * float(want.abs().max())
