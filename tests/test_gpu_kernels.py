"""GPU parity of single kernels at the sizes where their tilings end: against the same operation in 64 bits.

Tolerances: a fp32 dot product of n terms summed in pieces of at most s carries a relative error of about
sqrt(s) * 2^-24 against the norm of its terms; with activations, queries or probabilities as a bf16 hi + lo pair every
factor adds at most 2^-17.  The bounds below are a few times that."""
import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc():
    import paper_2311_08263_amd as m
    return m


def rel(a, b):
    import torch
    a, b = a.double(), b.double()
    return float(torch.linalg.norm(a - b) / torch.linalg.norm(b))


def attn64(q, k, v, n):
    import torch
    W, H, Dh = q.shape
    G = H // k.shape[1]
    kk, vv = k.double().repeat_interleave(G, 1).permute(1, 0, 2), v.double().repeat_interleave(G, 1).permute(1, 0, 2)
    s = torch.bmm(q.double().permute(1, 0, 2).contiguous(), kk.transpose(1, 2).contiguous()) / Dh ** 0.5
    seen = torch.arange(n + W, device="cuda")[None, :] <= n + torch.arange(W, device="cuda")[:, None]
    p = torch.softmax(s.masked_fill(~seen[None], float("-inf")), -1)
    return torch.bmm(p, vv.contiguous()).permute(1, 0, 2).reshape(W, H * Dh)


def attn_inputs(n, W, H, Hkv, Dh, dtype, seed=3):
    import torch
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    q = torch.randn(W, H, Dh, generator=g, device="cuda")
    k = torch.randn(n + W, Hkv, Dh, generator=g, device="cuda").to(dtype)
    v = torch.randn(n + W, Hkv, Dh, generator=g, device="cuda").to(dtype)
    return q, k, v


@pytest.mark.parametrize("n,W,H,Hkv,Dh,f32", [(0, 1, 2, 2, 32, 1), (31, 1, 4, 4, 64, 1), (32, 9, 4, 2, 64, 1), (777, 3, 3, 1, 96, 1),
                                              (130, 40, 4, 2, 256, 1), (500, 2, 4, 2, 64, 0), (15900, 2, 2, 1, 128, 1)])
def test_plain_attention(fc, n, W, H, Hkv, Dh, f32):
    """fp32 caches, and bf16 ones the matrix-core kernel does not cover: half blocks of 16 keys, the last partial
    octet, head sizes of 1 to 8 groups, a cache whose scores need more than 64 KB of LDS.  Dot products are summed
    in at most Dh + (n + W) / 32 terms at a time."""
    import torch
    say(f"plain attention n={n} W={W} H={H}/{Hkv} Dh={Dh} f32={f32}")
    q, k, v = attn_inputs(n, W, H, Hkv, Dh, torch.float32 if f32 else torch.bfloat16)
    S = (n + W + 31) // 32 * 32
    kc, vc = fc.kv_scatter(k, v, S)
    out = fc.attn_window(q, kc, vc, n)
    assert rel(out, attn64(q, k, v, n)) < 2e-6


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("S,n,W,H,Hkv,Dh", [(32, 0, 1, 3, 1, 32), (128, 125, 3, 4, 2, 64), (128, 96, 8, 64, 64, 32), (128, 3, 16, 33, 33, 64), (160, 3, 8, 4, 4, 64),
                                            (160, 150, 10, 4, 2, 32), (640, 127, 1, 512, 8, 64), (640, 600, 2, 257, 257, 32)])
def test_plain_attention_with_its_first_blocks_requested_early(fc, f32, S, n, W, H, Hkv, Dh):
    """Heads of 32 and 64 on both sides of the lines: caches of up to 128 positions and larger ones, up to two workgroups per CU and
    more; what lies behind the last position is infinite or NaN.  Bound as above."""
    import torch
    say(f"plain attention, early blocks S={S} n={n} W={W} H={H}/{Hkv} Dh={Dh} f32={f32}")
    q, k, v = attn_inputs(n, W, H, Hkv, Dh, torch.float32 if f32 else torch.bfloat16)
    kp, vp = (torch.full((S, Hkv, Dh), float("nan"), dtype=k.dtype, device="cuda") for _ in range(2))
    vp[n + W::2] = float("inf")
    kp[:n + W], vp[:n + W] = k, v
    assert rel(fc.attn_window(q, *fc.kv_scatter(kp, vp, S), n), attn64(q, k, v, n)) < 2e-6


@pytest.mark.parametrize("n,W,H,Hkv", [(0, 33, 2, 2), (1024, 64, 40, 40), (37, 48, 8, 2), (4000, 49, 4, 1), (5, 300, 3, 3), (777, 96, 64, 8)])
def test_wide_window_attention(fc, n, W, H, Hkv):
    """More than 32 rows: units of 16 rows with three-part queries and probabilities, with and without key splits,
    the last unit of 1 row, grouped heads.  The three parts hold 24 bits, so the bound is that of fp32 sums."""
    say(f"wide window attention n={n} W={W} H={H}/{Hkv}")
    import torch
    q, k, v = attn_inputs(n, W, H, Hkv, 128, torch.bfloat16)
    kc, vc = fc.kv_scatter(k, v, (n + W + 31) // 32 * 32)
    assert rel(fc.attn_window(q, kc, vc, n), attn64(q, k, v, n)) < 1e-6


@pytest.mark.parametrize("n,W,H,Hkv", [(250, 5, 4, 2), (5, 16, 2, 2), (40, 17, 4, 4), (2000, 32, 8, 2), (0, 33, 2, 1), (777, 33, 8, 8), (3001, 64, 4, 4)])
def test_attention_takes_nothing_from_hidden_positions(fc, n, W, H, Hkv):
    """Positions past the window hold NaN and infinities (nobody has to fill them), and so do two head elements of V in
    the last window row, which only that row sees: every other row is what it is without them, and the last row is
    infinite and NaN in those two elements alone.  Bounds as in the tests above."""
    import torch
    say(f"hidden positions n={n} W={W} H={H}/{Hkv}")
    q, k, v = attn_inputs(n, W, H, Hkv, 128, torch.bfloat16)
    S = (n + W + 31) // 32 * 32
    assert S > n + W
    want = attn64(q, k, v, n).view(W, H, 128)
    kp, vp = (torch.full((S, Hkv, 128), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    kp[n + W::2], vp[n + W::2] = float("inf"), float("-inf")
    kp[:n + W], vp[:n + W] = k, v
    vp[n + W - 1, :, 37], vp[n + W - 1, :, 90] = float("inf"), float("nan")
    out = fc.attn_window(q, *fc.kv_scatter(kp, vp, S), n).view(W, H, 128)
    assert torch.isinf(out[-1, :, 37]).all() and torch.isnan(out[-1, :, 90]).all()
    out[-1, :, 37], out[-1, :, 90] = want[-1, :, 37].float(), want[-1, :, 90].float()
    assert rel(out, want) < (1e-6 if W > 32 else 1.5e-5)


@pytest.mark.parametrize("W", [9, 20, 33])
def test_attention_over_the_range_of_fp32(fc, W):
    """Queries that round to a bf16 infinity, and rows all of whose scores lie below -1e33."""
    import torch
    say(f"attention at the ends of the range W={W}")
    n, H = 300, 2
    q, k, v = attn_inputs(n, W, H, H, 128, torch.bfloat16)
    big = q.clone(); big[1::3] = torch.sign(big[1::3]) * 3.4e38
    small = (k.float() * 1e-30).bfloat16()
    for qq, kk in ((big, small), (q.abs() * 1e18, -(k.abs().float() * 1e15).bfloat16())):
        out = fc.attn_window(qq.contiguous(), *fc.kv_scatter(kk, v, (n + W + 31) // 32 * 32), n)
        assert rel(out, attn64(qq, kk, v, n)) < (1e-6 if W > 32 else 1.5e-5)


@pytest.mark.parametrize("W", [9, 20, 33])
def test_attention_of_very_large_scores(fc, W):
    """Scores of about 1e11, which rounding alone moves by thousands: the largest score's weight is still one.  (Two keys
    that lie within the 2^-17 of a query would change places; none do here: the result is that of 64 bits.)"""
    import torch
    say(f"attention of very large scores W={W}")
    n, H = 300, 4
    q, k, v = attn_inputs(n, W, H, 2, 128, torch.bfloat16)
    q, k = q * 1e5, (k.float() * 1e5).bfloat16()
    out = fc.attn_window(q, *fc.kv_scatter(k, v, (n + W + 31) // 32 * 32), n)
    assert rel(out, attn64(q, k, v, n)) < 1.5e-5


@pytest.mark.parametrize("W,planes", [(16, 2), (16, 3), (24, 2), (24, 1), (48, 2)])
def test_steps_of_very_large_scores(fc, W, planes):
    """The same in a model (query and key weights times 2^20, scores of about 1e13): a prompt through the many-row
    attention kernel and one step, against the plain kernels.  A row in which two keys do change places differs
    altogether, so the bound is on the median row."""
    import torch
    import synthgen
    say(f"step of very large scores W={W} planes={planes}")
    shape, B, P = synthgen.ModelShape(2, 512, 4, 2, 128, 768, 1040, init_std=0.05), 1, 140
    cfg = fc.Config.from_shape(shape, B, 256, W)

    def weights():
        for sp in synthgen.weight_tensors(shape):
            a = synthgen.weight_array(shape, sp, as_bf16_bits=True)
            if sp.name in ("wq", "wk"):
                a = np.where(a & 0x7F80, a + (20 << 7), a).astype(np.uint16)
            yield sp.name, sp.layer, a
    packed = fc.pack_weights(cfg, weights())
    prompts, buf = synthgen.prompts(B, P, shape.vocab, seed=7), synthgen.buffer_init(B, 2 * W + 8, shape.vocab, seed=8)
    out = []
    for plain in (0, 1):
        ctx = fc.Context(cfg, packed)
        ctx.set_option(fc.binding.OPT_KV_PLANES, planes)
        ctx.set_option(fc.binding.OPT_PLAIN_KERNELS if plain else fc.binding.PLAN_ATTN_MANY_ROWS, 1 if plain else 2)
        ctx.prefill(prompts, [P], buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg[:W].double())
        ctx.close()
    assert torch.isfinite(out[0]).all()
    err = torch.linalg.norm(out[0] - out[1], dim=1) / torch.linalg.norm(out[1], dim=1)
    assert float(err.median()) < (2e-2 if planes == 1 else 1e-4)


@pytest.mark.parametrize("n,W,H,Hkv", [(4050, 32, 64, 8), (4080, 32, 64, 8), (4100, 17, 64, 16), (9000, 24, 40, 8), (3000, 20, 128, 8), (200, 17, 512, 8)])
def test_two_tile_attention_splits(fc, n, W, H, Hkv):
    """17 to 32 rows over grouped heads: on both sides of the line beyond which two workgroups share a CU, with as many and
    with fewer key splits than asked for, and more heads than CUs."""
    say(f"two-tile attention n={n} W={W} H={H}/{Hkv}")
    import torch
    q, k, v = attn_inputs(n, W, H, Hkv, 128, torch.bfloat16)
    kc, vc = fc.kv_scatter(k, v, (n + W + 31) // 32 * 32)
    assert rel(fc.attn_window(q, kc, vc, n), attn64(q, k, v, n)) < 1.5e-5


@pytest.mark.parametrize("n,W,H,Hkv,splits", [(511, 1, 257, 257, 8), (3000, 16, 341, 31, 3), (3000, 16, 342, 9, 1), (440, 40, 100, 4, 1), (441, 40, 100, 4, 5),
                                              (2000, 113, 40, 40, 4), (600, 64, 66, 66, 8), (1740, 20, 300, 4, 1), (1741, 20, 300, 4, 5), (2100, 20, 300, 4, 5),
                                              (464, 16, 257, 257, 1), (465, 16, 257, 257, 8)])
def test_attention_cut_last_round(fc, n, W, H, Hkv, splits):
    """More units than CUs (256): those past the last full round in three to eight key splits, one unit and as many as are cut at
    most, one more than that (not cut), one and two query tiles, the longest context that is not cut and the shortest that is."""
    import ctypes
    import torch
    say(f"attention, cut last round n={n} W={W} H={H}/{Hkv}")
    got = ctypes.c_int32(0)
    units = H * ((W + 15) // 16 if W > 32 else 1)
    rest = fc.lib()["_Z14fc_attn16_restiiiiiiPi"](W, 16 if W > 32 else 0, units, 1, 1, n + W, ctypes.byref(got))
    assert (got.value, rest) == (splits, units % 256 if splits > 1 else 0)
    q, k, v = attn_inputs(n, W, H, Hkv, 128, torch.bfloat16)
    kc, vc = fc.kv_scatter(k, v, (n + W + 31) // 32 * 32)
    out = fc.attn_window(q, kc, vc, n)
    assert rel(out, attn64(q, k, v, n)) < (1e-6 if W > 32 else 1.5e-5)
    assert torch.equal(out, fc.attn_window(q, kc, vc, n))


def test_one_scratch_for_calls_of_different_shapes(fc):
    """A scratch zeroed once serves any order of shapes it is large enough for."""
    import torch
    say("attention: one scratch, several shapes")
    shapes = [(2048, 16, 32, 32), (700, 64, 64, 8), (300, 5, 4, 4), (2000, 40, 8, 8), (900, 32, 64, 64), (3000, 33, 4, 4)]
    scratch = torch.zeros(max(fc.lib().fastcot_attn_scratch_bytes(W, H, 128) for _, W, H, _ in shapes), dtype=torch.uint8, device="cuda")
    for n, W, H, Hkv in shapes + shapes[::-1]:
        q, k, v = attn_inputs(n, W, H, Hkv, 128, torch.bfloat16)
        kc, vc = fc.kv_scatter(k, v, (n + W + 31) // 32 * 32)
        assert rel(fc.attn_window(q, kc, vc, n, scratch), attn64(q, k, v, n)) < 1.5e-5


@pytest.mark.parametrize("M,d,V", [(1, 32, 16), (9, 96, 1040), (17, 160, 16 * 2001), (40, 608, 16 * 1027)])
def test_plain_lmhead(fc, M, d, V):
    """Widths that are no multiple of 256 go through the plain product: k-tiles that leave waves idle, rows past the
    last block of eight, one and four column tiles per workgroup with a remainder of one and three."""
    import torch
    say(f"plain lm head M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(5)
    w = (0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16()
    act = torch.randn(M, d, generator=g, device="cuda")
    ids, top, logits, top2 = fc.lmhead_argmax(act, fc.lmhead_pack(w), V, want_logits=True, want_top2=True)
    want = act.double() @ w.double()
    assert rel(logits, want) < 1e-6
    assert torch.equal(ids.long(), logits.argmax(1)) and torch.equal(top, logits.max(1).values)
    two = torch.topk(logits, 2, dim=1).values
    assert torch.equal(top2, two[:, 1])


@pytest.mark.parametrize("d", [272, 256, 16])
def test_plain_product_past_the_last_octet(fc, d):
    """A fp32 head of a width that ends in the middle of a k-tile: an infinite weight among the first eight rows (which
    octets past the end read instead of nothing) makes its logit infinite and no other one."""
    import torch
    import synthgen
    say(f"plain product d={d}, infinite weight")
    shape = synthgen.ModelShape(0, d, 2, 2, 32, 48, 64, dtype="f32")
    cfg = fc.Config.from_shape(shape, 1, 32, 4)
    tensors = {sp.name: synthgen.weight_array(shape, sp) for sp in synthgen.weight_tensors(shape)}
    tensors["wlm"][3, 17] = np.inf
    ctx = fc.Context(cfg, fc.pack_weights(cfg, [(n, -1, t) for n, t in tensors.items()]))
    prompt, buf = np.array([[5]], dtype=np.int32), np.arange(16, dtype=np.int32).reshape(1, 16)
    ctx.prefill(prompt, [1], buf)
    dbg = ctx.debug_logits(True)
    torch.cuda.synchronize()
    ctx.step()
    torch.cuda.synchronize()
    x = tensors["emb"][[5, 0, 1, 2]].astype(np.float64)
    x /= np.sqrt((x * x).mean(1, keepdims=True) + shape.rms_eps)
    want = torch.from_numpy(x @ tensors["wlm"].astype(np.float64)).cuda()
    got = dbg[:4].clone()
    assert torch.equal(got[:, 17].double(), want[:, 17]) and torch.isinf(want[:, 17]).all()
    got[:, 17], want[:, 17] = 0, 0
    assert rel(got, want) < 1e-6
    ctx.close()


@pytest.mark.parametrize("M,d,V", [(33, 256, 16), (40, 256, 16 * 65), (256, 1024, 16 * 501), (77, 512, 32000), (300, 2048, 16 * 999), (1030, 256, 4096)])
def test_many_row_lmhead(fc, M, d, V):
    """More than 32 rows through the many-row kernel on three-part activations: every tile width, last column blocks
    of one tile, last row blocks of one row, the narrowest K; ids, top and runner-up are read off the same logits."""
    import torch
    say(f"many-row lm head M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(6)
    w = (0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16()
    act = torch.randn(M, d, generator=g, device="cuda")
    packed = fc.lmhead_pack(w)
    ids, top, logits, top2 = fc.lmhead_argmax(act, packed, V, want_logits=True, want_top2=True)
    assert rel(logits, act.double() @ w.double()) < 1e-6
    assert torch.equal(ids.long(), logits.argmax(1)) and torch.equal(top, logits.max(1).values)
    if V > 16:
        assert torch.equal(top2, torch.topk(logits, 2, dim=1).values[:, 1])
    ids2, top_2, none, two = fc.lmhead_argmax(act, packed, V, want_top2=True)      # logits in the scratch
    assert none is None and torch.equal(ids, ids2) and torch.equal(top, top_2) and torch.equal(top2, two)


@pytest.mark.parametrize("M,d,V", [(33, 256, 1040), (70, 512, 16 * 65), (40, 96, 1040)])
def test_lmhead_of_infinite_activations(fc, M, d, V):
    """Rows with an infinity, a NaN, and values that round up to a bf16 infinity, among ordinary ones; the last shape goes
    through the plain product.  An infinite activation makes the logits infinite by the sign of its weights, and the
    lowest id of the positive ones wins."""
    import torch
    say(f"lm head, infinite activations M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(8)
    w = (0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16()
    w[w == 0] = 0.01
    act = torch.randn(M, d, generator=g, device="cuda")
    act[2, 5], act[9, 40], act[17, 63] = float("inf"), float("-inf"), float("nan")
    act[20, 8], act[20, 9], act[M - 1, d - 1] = 3.4e38, -3.395e38, -3.402823466e38
    ids, top, logits, top2 = fc.lmhead_argmax(act, fc.lmhead_pack(w), V, want_logits=True, want_top2=True)
    want = act.double() @ w.double()
    for m, f, s in ((2, 5, 1), (9, 40, -1)):
        assert torch.equal(logits[m].double(), want[m]) and torch.isinf(want[m]).all()
        assert int(ids[m]) == int((s * w[f] > 0).nonzero()[0]) and float(top[m]) == float(top2[m]) == float("inf")
    assert torch.isnan(logits[17]).all()
    rows = torch.tensor([m for m in range(M) if m not in (2, 9, 17)], device="cuda")
    for m in rows.tolist():
        assert rel(logits[m], want[m]) < 1e-6
    assert torch.equal(ids[rows].long(), logits[rows].argmax(1)) and torch.equal(top[rows], logits[rows].max(1).values)


@pytest.mark.parametrize("M,d", [(5, 256), (20, 512), (33, 256), (40, 96)])
def test_lmhead_ids_stay_in_the_vocabulary(fc, M, d):
    """A row of NaN has no largest logit and a row of -infinity only ties: id 0 for both, as the oracle's scan from the
    first id has it, in all three kernels."""
    import torch
    say(f"lm head, rows without a winner M={M} d={d}")
    V = 1040
    g = torch.Generator(device="cuda"); g.manual_seed(9)
    w = (0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16()
    w[3] = -w[3].abs() - 0.01
    act = torch.randn(M, d, generator=g, device="cuda")
    act[1, 7], act[3, 3] = float("nan"), float("inf")
    ids, top, logits, top2 = fc.lmhead_argmax(act, fc.lmhead_pack(w), V, want_logits=True, want_top2=True)
    assert int(ids[1]) == int(ids[3]) == 0
    if M > 32:
        assert torch.equal(logits[3], torch.full_like(logits[3], float("-inf"))) and float(top[3]) == float(top2[3]) == float("-inf")
    rows = torch.tensor([m for m in range(M) if m not in (1, 3)], device="cuda")
    assert torch.equal(ids[rows].long(), logits[rows].argmax(1)) and torch.equal(top[rows], logits[rows].max(1).values)


@pytest.mark.parametrize("B,W,P", [(1, 33, 20), (3, 16, 40), (1, 77, 30), (1, 80, 81), (2, 65, 97), (9, 16, 130), (1, 250, 300), (1, 33, 1027)])
def test_many_row_steps(fc, B, W, P):
    """Passes of more than 32 rows, row counts that end blocks of three and of four row tiles early, prompts in one and in
    two chunks: the logits of the same step through the plain kernels.  Activations are hi + lo pairs in one and fp32 in
    the other path (2^-17 per product, a few layers of them)."""
    import torch
    import synthgen
    say(f"many-row step B={B} W={W} P={P}")
    shape = synthgen.ModelShape(2, 512, 4, 2, 128, 768, 1040, init_std=0.05)
    cfg = fc.Config.from_shape(shape, B, (P + 3 * W + 63) // 32 * 32, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(B, P, shape.vocab, seed=7), synthgen.buffer_init(B, 2 * W + 8, shape.vocab, seed=8)
    lens = [P - b for b in range(B)]
    out = []
    for plain in (0, 1):
        ctx = fc.Context(cfg, packed)
        if plain:
            ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, 1)
        ctx.prefill(prompts, lens, buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg[:B * W].clone())
        ctx.close()
    assert rel(out[0], out[1]) < 1e-4


WIDE_HEADS = dict(n_layers=1, d_model=512, n_heads=32, n_kv_heads=32, head_dim=128, d_ffn=768, vocab=1040, init_std=0.05)


def test_attention_form_follows_the_context(fc):
    """Steps of 17 to 32 rows choose between one and two query tiles by the length of the context: a short one in a large
    cache runs what it runs in a small one, bit for bit."""
    import torch
    import synthgen
    shape, W, P = synthgen.ModelShape(**WIDE_HEADS), 32, 300
    prompts, buf = synthgen.prompts(1, P, shape.vocab, seed=7), synthgen.buffer_init(1, 2 * W + 8, shape.vocab, seed=8)
    out = []
    for S in (512, 8192):
        say(f"attention form, capacity {S}")
        cfg = fc.Config.from_shape(shape, 1, S, W)
        ctx = fc.Context(cfg, fc.load_synth_weights(cfg, shape))
        ctx.prefill(prompts, [P], buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg.clone())
        ctx.close()
    assert torch.equal(out[0], out[1])


def test_attention_form_changes_during_a_run(fc):
    """Four sequences grow past the line between the two forms (1024 positions for 128 units of two tiles): with and
    without a captured graph the same bits at every step, and the plain kernels' logits on both sides of it."""
    import torch
    import synthgen
    shape, B, W, P, steps = synthgen.ModelShape(**WIDE_HEADS), 4, 32, 990, 6
    cfg = fc.Config.from_shape(shape, B, 1152, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(B, P, shape.vocab, seed=7), synthgen.buffer_init(B, 2 * W + 24, shape.vocab, seed=8)
    runs = []
    for opt in ((), (fc.binding.OPT_GRAPH, 0), (fc.binding.OPT_PLAIN_KERNELS, 1)):
        say(f"attention form, run {opt}")
        ctx = fc.Context(cfg, packed)
        if opt:
            ctx.set_option(*opt)
        ctx.prefill(prompts, [P - b for b in range(B)], buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        got = []
        for _ in range(steps):
            ctx.step()
            torch.cuda.synchronize()
            got.append(dbg.clone())
        runs.append(got)
        ctx.close()
    for a, b, c in zip(*runs):
        assert torch.equal(a, b)
        assert rel(a, c) < 1e-4


@pytest.mark.parametrize("W,P,longest_first", [(16, 205, 0), (16, 205, 1), (9, 700, 1), (32, 830, 0)])
def test_attention_cut_last_round_in_steps(fc, W, P, longest_first):
    """Nine sequences of 32 heads, the last of which runs in key splits once the longest one and its window pass 224 positions (864 with
    two query tiles): the step before and after that, the cut one the longest or short enough to stay whole, with and
    without a captured graph and through the plain kernels."""
    import torch
    import synthgen
    shape, B, steps = synthgen.ModelShape(**WIDE_HEADS), 9, 6
    cfg = fc.Config.from_shape(shape, B, (P + W + 95) // 32 * 32, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(B, P, shape.vocab, seed=7), synthgen.buffer_init(B, 2 * W + 24, shape.vocab, seed=8)
    lens = [P - b * (P // 10) if longest_first else P - (B - 1 - b) for b in range(B)]
    runs = []
    for opt in ((), (fc.binding.OPT_GRAPH, 0), (fc.binding.OPT_PLAIN_KERNELS, 1)):
        say(f"attention, cut last round in steps W={W} P={P} longest first {longest_first}, run {opt}")
        ctx = fc.Context(cfg, packed)
        if opt:
            ctx.set_option(*opt)
        ctx.prefill(prompts, lens, buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        got = []
        for _ in range(steps):
            ctx.step()
            torch.cuda.synchronize()
            got.append(dbg[:B * W].clone())
        runs.append(got)
        ctx.close()
    for a, b, c in zip(*runs):
        assert torch.equal(a, b)
        assert rel(a, c) < 1e-4


@pytest.mark.parametrize("W,wins,planes", [(16, [16, 3, 9, 16, 1, 12, 5, 16, 2], 1), (16, [16, 3, 9, 16, 1, 12, 5, 16, 2], 3), (16, [1, 3, 9, 2, 1, 12, 5, 4, 16], 2),
                                           (20, [3, 20, 16, 17, 1, 20, 8, 20, 5], 1), (20, [3, 20, 16, 17, 1, 20, 8, 5, 20], 2), (20, [3, 20, 16, 17, 1, 20, 8, 20, 5], 3),
                                           (40, [40, 3, 33, 40, 5], 2), (40, [5, 3, 32, 20, 40], 1), (40, [40, 16, 3, 17, 33], 3)])
def test_attention_cut_last_round_of_packed_rows(fc, W, wins, planes):
    """Cut units of sequences with windows of their own (units with few rows, and second units without any), one to three cache planes:
    against whole units.  One layer, so both runs cache the same bits and differ by the order in which fp32 partial results of the
    attention are added."""
    import ctypes
    import torch
    import synthgen
    shape, B = synthgen.ModelShape(**WIDE_HEADS), len(wins)
    P = (600 if W == 16 else 1800) if planes == 1 else (300 if W == 16 else 900)
    cfg = fc.Config.from_shape(shape, B, P + 160, W)
    packed = fc.load_synth_weights(cfg, shape)
    units, got = 32 * B * (2 if W > 32 else 1), ctypes.c_int32(0)
    assert fc.lib()["_Z14fc_attn16_restiiiiiiPi"](W, 0, units, 1, planes, P, ctypes.byref(got)) == units - 256 and got.value > 2
    prompts, buf = synthgen.prompts(B, P, shape.vocab, seed=7), synthgen.buffer_init(B, 2 * W + 24, shape.vocab, seed=8)
    out = []
    for opt in ((), (fc.binding.OPT_GRAPH, 0), (fc.binding.PLAN_ATTN_SPLITS, 1)):
        say(f"cut last round, packed rows W={W} windows {wins} planes {planes} {opt}")
        ctx = fc.Context(cfg, packed)
        ctx.set_option(fc.binding.OPT_KV_PLANES, planes)
        if opt:
            ctx.set_option(*opt)
        ctx.prefill(prompts, [P - b for b in range(B)], buf)
        ctx.set_windows(wins)
        rows = int(ctx.step_rows()[-1])
        assert rows == sum(wins)
        dbg = ctx.debug_logits(True)
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg[:rows].clone())
        ctx.close()
    assert torch.equal(out[0], out[1])
    assert 0 < rel(out[0], out[2]) < 1e-5


def test_splits_option_counts_for_every_unit(fc):
    """Nine equal sequences, one in key splits by default: with the number of splits set, 1 included, all nine are computed alike, to
    the last bit."""
    import torch
    import synthgen
    shape, B, W, P = synthgen.ModelShape(**WIDE_HEADS), 9, 16, 300
    cfg = fc.Config.from_shape(shape, B, 448, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(1, P, shape.vocab, seed=7).repeat(B, 0), synthgen.buffer_init(1, 2 * W + 24, shape.vocab, seed=8).repeat(B, 0)
    alike = []
    for splits in (0, 1, 2):
        say(f"splits of the attention launch: {splits}")
        ctx = fc.Context(cfg, packed)
        if splits:
            ctx.set_option(fc.binding.PLAN_ATTN_SPLITS, splits)
        ctx.prefill(prompts, [P] * B, buf)
        dbg = ctx.debug_logits(True)
        ctx.step()
        torch.cuda.synchronize()
        lg = dbg.view(B, W, -1)
        alike.append([bool(torch.equal(lg[b], lg[0])) for b in range(B)])
        ctx.close()
    assert alike[0] == [True] * 8 + [False] and all(alike[1]) and all(alike[2])


def test_workgroups_of_the_o_projection(fc):
    """Grids that go with four K slices of 4096 inputs, or with two where four do not fit; odd ones and those that leave an owner too many
    tiles stay refused, and so does what does not fit slices that were asked for.  Logits against the plain kernels."""
    import torch
    import synthgen
    shape, W, P = synthgen.ModelShape(1, 512, 32, 32, 128, 512, 1040, init_std=0.05), 8, 20
    cfg = fc.Config.from_shape(shape, 1, 96, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(1, P, shape.vocab, seed=7), synthgen.buffer_init(1, 2 * W + 8, shape.vocab, seed=8)
    O = fc.binding.PLAN_NW + 1

    def logits(*opts):
        say(f"workgroups of the O projection {opts}")
        ctx = fc.Context(cfg, packed)
        for o in opts:
            ctx.set_option(*o)
        ctx.prefill(prompts, [P], buf)
        dbg = ctx.debug_logits(True)
        ctx.step()
        torch.cuda.synchronize()
        out = dbg[:W].clone()
        ctx.close()
        return out
    plain, default = logits((fc.binding.OPT_PLAIN_KERNELS, 1)), logits()
    for nw in (6, 8, 12, 30, 32):
        assert rel(logits((O, nw)), plain) < 1e-4
    assert torch.equal(logits((O, 30), (O, 32)), default)
    for refused in (((O, 31),), ((O, 4),), ((fc.binding.PLAN_KS + 1, 4), (O, 30))):
        with pytest.raises(fc.FastcotError):
            logits(*refused)


@pytest.mark.parametrize("W,F", [(33, 768), (40, 1024), (41, 1280), (47, 1536), (48, 1792), (49, 2048), (63, 512), (65, 2048)])
def test_reduction_of_k_slices(fc, W, F):
    """Many-row residual products in two to eight K slices (F / 256 of them), rows that fill the eight-row workgroups of their
    reduction and that do not: logits of a prompt and a step through the matrix-core and the plain kernels (activations as
    hi + lo pairs in one and fp32 in the other, 2^-17 per product)."""
    import torch
    import synthgen
    shape = synthgen.ModelShape(2, 512, 4, 4, 128, F, 1040, init_std=0.05)
    cfg = fc.Config.from_shape(shape, 1, 256, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts, buf = synthgen.prompts(1, W + 2, shape.vocab, seed=7), synthgen.buffer_init(1, 2 * W + 8, shape.vocab, seed=8)
    out = []
    for plain in (0, 1):
        say(f"reduction of K slices W={W} F={F} plain={plain}")
        ctx = fc.Context(cfg, packed)
        if plain:
            ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, 1)
        ctx.prefill(prompts, [W + 2], buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg[:W].clone())
        ctx.close()
    assert rel(out[0], out[1]) < 1e-4


@pytest.fixture(scope="module")
def wide_model(fc):
    """One layer whose QKV, gate/up and LM head have more column tiles than 8 * (CUs / 8 / row blocks) * 16."""
    import synthgen
    shape = synthgen.ModelShape(1, 512, 64, 64, 128, 28672, 32000, init_std=0.05)
    return shape, fc.load_synth_weights(fc.Config.from_shape(shape, 1, 512, 16), shape)


@pytest.mark.parametrize("W", [65, 77, 96, 129, 130, 144])
def test_many_row_steps_over_wide_matrices(fc, wide_model, W):
    """Row counts that run as blocks of three row tiles with the eight waves side by side: gate/up of 65 to 96 rows, QKV,
    gate/up and LM head of 129 to 144, the ends of both ranges; the logits and the argmax of the same step through the
    plain kernels (activations as hi + lo pairs in one and fp32 in the other path, 2^-17 per product)."""
    import torch
    import synthgen
    say(f"many-row step over wide matrices W={W}")
    shape, packed = wide_model
    P = 9
    cfg = fc.Config.from_shape(shape, 1, 512, W)
    prompts, buf = synthgen.prompts(1, P, shape.vocab, seed=7), synthgen.buffer_init(1, 2 * W + 8, shape.vocab, seed=8)
    out = []
    for plain in (0, 1):
        ctx = fc.Context(cfg, packed)
        ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, plain)
        ctx.prefill(prompts, [P], buf)
        dbg = ctx.debug_logits(True)
        torch.cuda.synchronize()
        ctx.step()
        torch.cuda.synchronize()
        out.append(dbg[:W].clone())
        assert (ctx.state()["o"][0] == dbg[:W].argmax(1).cpu().numpy()).all()
        ctx.close()
    assert rel(out[0], out[1]) < 1e-4
