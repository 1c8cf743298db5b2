"""GPU parity of the matrix-core (bf16) path against the oracle on small Llama-shaped models and
on the kernel-isolation shapes (window-causal attention with 32 heads x 128, cache 2048, 16 window
queries; LM-head argmax of a 16x4096 activation against 4096x32000 weights).

Bars: |dlogit| <= 2e-2 (the bf16 bar; measured values are printed and are far smaller), argmax
equal wherever the oracle's top-1/top-2 margin exceeds 0.05, and the integer path (verified count,
accepted ids, committed length, next window) bit-exact given the GPU's own argmax."""
import numpy as np
import pytest

import oracle
import synthgen
from gpu_util import follow_steps, margins, say

pytestmark = pytest.mark.gpu
TOL = 2e-2

# head_dim 128 models small enough for the oracle to follow in seconds; init std raised so that
# logits are O(1) and attention is far from uniform
SMALL = synthgen.ModelShape(3, 512, 4, 2, 128, 768, 2048, init_std=0.05)
SMALL_MHA = synthgen.ModelShape(2, 256, 2, 2, 128, 512, 1024, init_std=0.06)


@pytest.fixture(scope="module")
def fc():
    import paper_2311_08263_amd as m
    return m


def setup(fc, shape, B, S, W):
    cfg = fc.Config.from_shape(shape, B, S, W)
    packed = fc.load_synth_weights(cfg, shape)
    return fc.Context(cfg, packed), oracle.model_from_synth(shape)


@pytest.mark.parametrize("shape,B,W,P", [(SMALL, 1, 16, 45), (SMALL, 2, 16, 33), (SMALL_MHA, 1, 8, 20),
                                         (SMALL, 1, 32, 70), (SMALL_MHA, 3, 5, 12), (SMALL, 4, 32, 40),
                                         (SMALL_MHA, 3, 16, 30), (SMALL, 1, 64, 75), (SMALL_MHA, 2, 40, 300),
                                         # the largest window of the window sweep, and a prompt of 4k tokens
                                         (SMALL, 1, 128, 140), (SMALL_MHA, 2, 128, 200), (SMALL_MHA, 1, 16, 4099)])
def test_follow_mode_small_models(fc, shape, B, W, P):
    say(f"bf16 follow shape d={shape.d_model} B={B} W={W} P={P}")
    N = 48
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    lens = [P - 3 * b for b in range(B)]
    prompts = synthgen.prompts(B, P, shape.vocab, seed=21)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=22)
    ctx.prefill(prompts, lens, buf)
    r = follow_steps(ctx, om, prompts, lens, 6, TOL)
    print(f"max |dlogit| {r['max_err']:.3e} over {r['rows']} rows ({r['low_margin_rows']} low-margin)")
    assert r["max_err"] < 2e-3          # far inside the bf16 bar thanks to hi/lo activations


@pytest.mark.parametrize("shape,B,W,P,planes", [(SMALL, 1, 128, 140, 2), (SMALL_MHA, 2, 128, 200, 2), (SMALL_MHA, 1, 16, 4099, 2),
                                                (SMALL, 3, 40, 300, 2), (SMALL, 2, 64, 1100, 2), (SMALL, 2, 48, 333, 1)])
def test_many_row_attention(fc, shape, B, W, P, planes):
    """The attention kernel for passes of many rows per sequence (128-row workgroups that walk the keys once),
    forced on for every pass of more than 32 rows: prompt chunks of up to 1024 rows with ragged lengths, steps with
    windows of 40 to 128 rows (waves without rows, rows past the window), grouped K/V heads.  With the pair cache
    the oracle follows; with the one-plane cache (plain bf16, outside the oracle's bar) the step kernel is the
    reference, on identical cache contents."""
    say(f"many-row attention d={shape.d_model} B={B} W={W} P={P} planes={planes}")
    N = 48
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    lens = [P - 37 * b for b in range(B)]
    prompts = synthgen.prompts(B, P, shape.vocab, seed=25)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=26)
    if planes == 2:
        ctx.set_option(fc.binding.PLAN_ATTN_MANY_ROWS, 2)
        ctx.prefill(prompts, lens, buf)
        r = follow_steps(ctx, om, prompts, lens, 3, TOL)
        print(f"many-row attention: max |dlogit| {r['max_err']:.3e} over {r['rows']} rows")
        assert r["max_err"] < 2e-3
    else:
        logits = []
        for many in (0, 2):
            ctx.set_option(fc.binding.OPT_KV_PLANES, 1)
            ctx.set_option(fc.binding.PLAN_ATTN_MANY_ROWS, many)
            ctx.prefill(prompts, lens, buf)
            dbg = ctx.debug_logits(True)
            ctx.step()
            logits.append(dbg.cpu().numpy().copy())
        err = float(np.abs(logits[0] - logits[1]).max())
        print(f"many-row attention, one plane: max |dlogit| against the step kernel {err:.3e}")
        assert err < 2e-3
    ctx.close()


@pytest.mark.parametrize("shape,B,W,P,plain", [(SMALL, 1, 16, 45, 0), (SMALL, 4, 32, 40, 0), (SMALL_MHA, 2, 40, 300, 0),
                                               (SMALL, 2, 24, 70, 0), (SMALL, 2, 8, 33, 1)])
def test_three_byte_kv_cache(fc, shape, B, W, P, plain):
    """FASTCOT_OPT_KV_PLANES = 3: cached K/V as bf16 hi + an 8-bit residual (the upper 24 bits of the fp32 value),
    through the column-owner and the many-row QKV epilogues, the attention kernel's expansion of the residual bytes,
    and the plain kernels; same bar as the pair cache."""
    say(f"3-byte kv cache d={shape.d_model} B={B} W={W} P={P} plain={plain}")
    N = 48
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    ctx.set_option(fc.binding.OPT_KV_PLANES, 3)
    if plain:
        ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, 1)
    lens = [P - 3 * b for b in range(B)]
    prompts = synthgen.prompts(B, P, shape.vocab, seed=23)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=24)
    ctx.prefill(prompts, lens, buf)
    r = follow_steps(ctx, om, prompts, lens, 5, TOL)
    print(f"3-byte kv cache: max |dlogit| {r['max_err']:.3e} over {r['rows']} rows")
    assert r["max_err"] < 2e-3
    # finished sequences trading slots carry their residual planes with them
    if B > 1 and not plain:
        ctx.prefill(prompts, lens, buf)
        a = ctx.generate(N, eos_id=int(om.greedy_ar(prompts[0, :lens[0]], 6)[-1]))
        ctx.set_option(fc.binding.OPT_COMPACT, 0)
        ctx.prefill(prompts, lens, buf)
        b = ctx.generate(N, eos_id=int(om.greedy_ar(prompts[0, :lens[0]], 6)[-1]))
        assert (a["ids"] == b["ids"]).all() and (a["len"] == b["len"]).all()


@pytest.mark.parametrize("W", [16, 24])
def test_without_autotune(fc, W):
    """The option that used to switch timing runs at prefill off is still accepted and has no effect: same bar as everywhere, bits of the default."""
    shape, B, P, N = SMALL, 2, 37, 48
    say(f"bf16 follow without autotune W={W}")
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    ctx.set_option(fc.binding.OPT_AUTOTUNE, 0)
    lens = [P, P - 4]
    prompts = synthgen.prompts(B, P, shape.vocab, seed=61)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=62)
    ctx.prefill(prompts, lens, buf)
    r = follow_steps(ctx, om, prompts, lens, 4, TOL)
    assert r["max_err"] < 2e-3
    logits = []
    for off in (0, 1):
        ctx = fc.Context(ctx.cfg, ctx.packed)
        if off:
            ctx.set_option(fc.binding.OPT_AUTOTUNE, 0)
        ctx.prefill(prompts, lens, buf)
        dbg = ctx.debug_logits(True)
        ctx.step()
        logits.append(dbg.clone())
    assert bool((logits[0] == logits[1]).all())


def test_fast_path_matches_plain_path_and_oracle_stream(fc):
    """Same model through the MFMA kernels and through the plain kernels: same tokens; and the
    accepted stream is the oracle's greedy continuation up to the first low-margin row."""
    shape, W, P, N = SMALL, 16, 40, 64
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, 1, S, W)
    prompts = synthgen.prompts(1, P, shape.vocab, seed=31)
    buf = synthgen.buffer_init(1, N + 2 * W, shape.vocab, seed=32)
    outs = {}
    for plain in (0, 1):
        say(f"bf16 generate plain={plain}")
        ctx.set_option(1, plain)
        ctx.prefill(prompts, [P], buf)
        outs[plain] = ctx.generate(N)
    ref = om.jacobi_generate(prompts[0], buf[0], W, N)
    # the oracle's own margins along its trajectory decide how far equality is required
    ss = om.session(S)
    ss.forward(prompts[0, :-1], 0, want_logits=False)
    lg, _, _ = ss.forward(np.concatenate([prompts[0, -1:], ref["ids"][:-1]]), P - 1)
    low = np.where(margins(lg) <= 0.05)[0]
    upto = int(low[0]) if len(low) else N
    for plain in (0, 1):
        assert (outs[plain]["ids"][0, :upto] == ref["ids"][:upto]).all(), plain
    if upto == N:
        assert outs[0]["steps"][0] == ref["steps"] and (outs[0]["ids"][0] == outs[1]["ids"][0]).all()


def test_answer_phase_bf16(fc):
    """Answer phase (Sec. 4.4 "Trigger Answer") on a bf16 model, batch of two stopping differently (one by
    the iteration cap with a glimpse, both with a trigger): the MFMA kernels and the plain kernels give the
    same answer tokens, and they are the oracle's greedy continuation of the combined context up to the
    first low-margin row."""
    shape, W, P, N, NA = SMALL, 16, 40, 48, 10
    S = ((P + N + 3 * W + NA + 31) // 32) * 32
    ctx, om = setup(fc, shape, 2, S, W)
    prompts = synthgen.prompts(2, P, shape.vocab, seed=51)
    lens = [P, P - 5]
    buf = synthgen.buffer_init(2, N + 2 * W, shape.vocab, seed=52)
    trigger = np.array([11, 222, 333, 44], dtype=np.int32)
    res = {}
    for plain in (0, 1):
        say(f"bf16 answer phase plain={plain}")
        ctx.set_option(1, plain)
        ctx.prefill(prompts, lens, buf)
        out = ctx.generate(N, max_steps=4)
        st = ctx.state()
        ans = ctx.answer(trigger, NA)
        res[plain] = (out, st, ans)
    (out, st, ans), (out1, st1, ans1) = res[0], res[1]
    assert (out["ids"] == out1["ids"]).all() and (st["window"] == st1["window"]).all()
    for b in range(2):
        g = int(st["g"][b])
        exact = out["ids"][b][:g]
        assert int(out["len"][b]) == g and exact[-1] == st["window"][b][0]
        combined = np.concatenate([prompts[b, :lens[b]], exact, st["window"][b][1:], trigger]).astype(np.int32)
        want = om.greedy_ar(combined, NA)
        ss = om.session(S)
        ss.forward(combined[:-1], 0, want_logits=False)
        lg, _, _ = ss.forward(np.concatenate([combined[-1:], want[:-1]]), len(combined) - 1)
        low = np.where(margins(lg) <= 0.05)[0]
        upto = int(low[0]) if len(low) else NA
        assert ans["ids"][b][:upto].tolist() == want[:upto].tolist(), (b, upto)
        assert ans1["ids"][b][:upto].tolist() == want[:upto].tolist(), (b, upto)
        print(f"answer phase seq {b}: {upto} of {NA} tokens above the margin, all equal")


def test_early_finishers_bf16(fc):
    """bf16 model, batch of three of which one has a perfect draft: after it has left the batch the other two run
    through the kernels for fewer rows; every sequence's accepted stream is still the oracle's greedy continuation
    up to its first low-margin row."""
    shape, W, P, N, B = SMALL, 16, 40, 64, 3
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    prompts = synthgen.prompts(B, P, shape.vocab, seed=81)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=82)
    lens = [P, P - 6, P - 1]
    greedy = [om.greedy_ar(prompts[b, :lens[b]], N + 2 * W) for b in range(B)]
    buf[1, :] = greedy[1]                              # slot j of a window drafts generated token g + j - 1
    say("bf16 batch with an early finisher")
    ctx.prefill(prompts, lens, buf)
    out = ctx.generate(N)
    assert out["steps"][1] <= N // W + 2 and out["steps"][0] > 2 * out["steps"][1]
    for b in range(B):
        ss = om.session(S)
        if lens[b] > 1: ss.forward(prompts[b, :lens[b] - 1], 0, want_logits=False)
        lg, _, _ = ss.forward(np.concatenate([prompts[b, lens[b] - 1:lens[b]], greedy[b][:N - 1]]), lens[b] - 1)
        low = np.where(margins(lg) <= 0.05)[0]
        upto = int(low[0]) if len(low) else N
        assert (out["ids"][b, :upto] == greedy[b][:upto]).all(), (b, upto)
        print(f"sequence {b}: {out['steps'][b]} steps, {upto} of {N} tokens above the margin, all equal")


def test_join_bf16(fc):
    """bf16 model on the matrix-core path, follow mode: two prompts join a running batch of three (one into slot
    2, with a prompt long enough for several prefill passes of a batch of one, one into slot 0); at every step
    the logits of every sequence -- newcomers and the ones that stayed, whose caches moved aside and back -- are
    the oracle's for that sequence's own context."""
    shape, W, B, N = SMALL, 8, 3, 48
    Pmax = 300
    S = ((Pmax + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    first = synthgen.prompts(B, 40, shape.vocab, seed=91)
    lens = [40, 23, 31]
    late = synthgen.prompts(2, Pmax, shape.vocab, seed=92)
    bufs = synthgen.buffer_init(B + 2, N + 2 * W, shape.vocab, seed=93)
    say("bf16 batch with joining sequences")
    ctx.prefill(first, lens, bufs[:B])
    r = follow_steps(ctx, om, first, lens, 10, TOL, joins={3: (2, late[0, :Pmax], bufs[3]), 6: (0, late[1, :17], bufs[4])})
    print(f"join follow: max |dlogit| {r['max_err']:.2e} over {r['rows']} rows, {r['low_margin_rows']} low-margin")


def test_per_sequence_windows_bf16(fc):
    """bf16 model, follow mode with per-sequence window sizes: the
    verified count, accepted tokens and committed length come from the first W_b rows of a sequence; one sequence
    has a perfect draft so that the cut at W_b, not a mismatch, is what ends its verification."""
    shape, W, B, P, N = SMALL, 8, 2, 30, 40
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    prompts = synthgen.prompts(B, P, shape.vocab, seed=111)
    lens = [P, P - 5]
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=112)
    buf[1, :] = om.greedy_ar(prompts[1, :lens[1]], N + 2 * W)
    say(f"bf16 per-sequence windows")
    ctx.prefill(prompts, lens, buf)
    ctx.set_windows([6, 3])
    r = follow_steps(ctx, om, prompts, lens, 6, TOL, wins=[6, 3])
    ks = r["K"][1::2]
    assert max(ks) == 2 and max(r["K"][0::2]) <= 5
    print(f"per-sequence windows: verified counts {r['K']}")


@pytest.mark.parametrize("B,W,wins", [(4, 16, [16, 4, 4, 4]), (3, 32, [32, 5, 20]), (2, 8, [8, 8]), (4, 64, [3, 64, 17, 40])])
def test_packed_rows(fc, B, W, wins):
    """Sequences with windows of their own: the step computes only their rows, packed one sequence after the
    other (28 rows instead of 64 through the column-owner kernels, 57 instead of 96 and 124 instead of 256 through
    the many-row kernels), and with the option off all B x W rows; the oracle follows both, and a generation to
    the end gives the same tokens and step counts either way."""
    shape, P, N = SMALL, 41, 40
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, om = setup(fc, shape, B, S, W)
    prompts = synthgen.prompts(B, P, shape.vocab, seed=131)
    lens = [P - 4 * b for b in range(B)]
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=132)
    say(f"packed rows B={B} W={W} wins={wins}")
    outs = []
    for packed in (1, 0):
        ctx.set_option(fc.binding.OPT_PACKED_ROWS, packed)
        ctx.prefill(prompts, lens, buf)
        ctx.set_windows(wins)
        rows = int(ctx.step_rows()[B])
        assert rows == (sum(wins) if packed and min(wins) < W else B * W)
        r = follow_steps(ctx, om, prompts, lens, 4, TOL, wins=wins)
        assert r["max_err"] < 2e-3
        ctx.prefill(prompts, lens, buf)
        ctx.set_windows(wins)
        outs.append(ctx.generate(N))
    assert (outs[0]["len"] == outs[1]["len"]).all()
    for b in range(B):
        assert (outs[0]["ids"][b, :outs[0]["len"][b]] == outs[1]["ids"][b, :outs[1]["len"][b]]).all()
    assert (outs[0]["steps"] == outs[1]["steps"]).all()
    ctx.close()


def test_deterministic_replay(fc):
    shape, W, P, N = SMALL, 16, 30, 40
    S = ((P + N + 2 * W + 31) // 32) * 32
    ctx, _ = setup(fc, shape, 2, S, W)
    prompts = synthgen.prompts(2, P, shape.vocab, seed=41)
    buf = synthgen.buffer_init(2, N + 2 * W, shape.vocab, seed=42)
    res = []
    for graph in (1, 1, 0):
        ctx.set_option(2, graph)
        ctx.prefill(prompts, [P, P - 7], buf)
        res.append(ctx.generate(N))
    for r in res[1:]:
        assert (r["ids"] == res[0]["ids"]).all() and (r["steps"] == res[0]["steps"]).all()


@pytest.mark.parametrize("shape,B,W", [(synthgen.small_variant(synthgen.SHAPES["7b"], n_layers=3), 1, 16),
                                       (synthgen.small_variant(synthgen.SHAPES["13b"], n_layers=2), 1, 32)])
def test_fresh_contexts_give_identical_bits(fc, shape, B, W):
    """Same inputs, same logits bits, same verified counts and lengths in any context: three contexts, the second and third with two and
    with one pair of k-tiles under way in every product of up to 32 rows (that only moves loads)."""
    import torch
    P, N = 70, 32
    S = ((P + N + 2 * W + 31) // 32) * 32
    cfg = fc.Config.from_shape(shape, B, S, W)
    packed = fc.load_synth_weights(cfg, shape)
    prompts = synthgen.prompts(B, P, shape.vocab, seed=71)
    buf = synthgen.buffer_init(B, N + 2 * W, shape.vocab, seed=72)
    runs = []
    for variant in range(3):
        say(f"fresh context {variant}: d={shape.d_model} W={W}")
        ctx = fc.Context(cfg, packed)
        if variant:
            ctx.set_option(fc.binding.PLAN_CO_SINGLE, variant - 1)
        ctx.prefill(prompts, [P] * B, buf)
        dbg = ctx.debug_logits(True)
        steps = []
        for s in range(3):
            nacc, acc, win = ctx.step()
            st = ctx.state()
            steps.append((dbg.clone(), nacc.copy(), st["o"].copy(), st["K"].copy(), st["n"].copy()))
        torch.cuda.synchronize()
        runs.append(steps)
        ctx.close()
    for variant in (1, 2):
        for a, b in zip(runs[0], runs[variant]):
            assert torch.equal(a[0], b[0]), "logits differ between two fresh contexts"
            for x, y in zip(a[1:], b[1:]):
                assert (x == y).all()


@pytest.mark.parametrize("n,W,H,Hkv", [(2048, 16, 32, 32), (0, 16, 4, 4), (37, 5, 8, 2), (1000, 32, 8, 1), (2031, 16, 4, 4)])
def test_attention_isolation(fc, n, W, H, Hkv):
    """Kernel-isolation shape: K/V ~ N(0,1) in bf16, queries ~ N(0,1), causal inside the window."""
    import torch
    Dh, S = 128, 2080
    say(f"attention isolation n={n} W={W} H={H} Hkv={Hkv}")
    q = synthgen.normal_f32((W, H, Dh), 5, 1, 1.0, False)
    kb = synthgen.normal_bf16((n + W, Hkv, Dh), 5, 2, 1.0)
    vb = synthgen.normal_bf16((n + W, Hkv, Dh), 5, 3, 1.0)
    ref = oracle.attention_window(q, synthgen.bf16_bits_to_f32(kb), synthgen.bf16_bits_to_f32(vb), n)
    kc, vc = fc.kv_scatter(torch.from_numpy(kb.view(np.int16)).cuda().view(torch.bfloat16),
                           torch.from_numpy(vb.view(np.int16)).cuda().view(torch.bfloat16), S)
    out = fc.attn_window(torch.from_numpy(q).cuda(), kc, vc, n)
    torch.cuda.synchronize()
    err = np.abs(out.cpu().numpy() - ref).max()
    print(f"attention max |d| {err:.3e}")
    assert err < 1e-4
    # garbage (finite) beyond the visible range must not matter: positions >= n+W are never read as visible
    kg = np.concatenate([kb, np.full((S - n - W, Hkv, Dh), 0x40E0, dtype=kb.dtype)])      # bf16 7.0
    vg = np.concatenate([vb, np.full((S - n - W, Hkv, Dh), 0xC110, dtype=vb.dtype)])      # bf16 -9.0
    kc2, vc2 = fc.kv_scatter(torch.from_numpy(kg.view(np.int16)).cuda().view(torch.bfloat16),
                             torch.from_numpy(vg.view(np.int16)).cuda().view(torch.bfloat16), S)
    assert not torch.equal(kc, kc2) and not torch.equal(vc, vc2)
    out2 = fc.attn_window(torch.from_numpy(q).cuda(), kc2, vc2, n)
    assert torch.equal(out, out2)


@pytest.mark.parametrize("M,d,V", [(16, 4096, 32000), (5, 512, 2048), (32, 1024, 4096)])
def test_lmhead_argmax_isolation(fc, M, d, V):
    import torch
    say(f"lm head isolation M={M} d={d} V={V}")
    act = synthgen.normal_f32((M, d), 6, 1, 1.0, False)
    wb = synthgen.normal_bf16((d, V), 6, 2, 0.02)
    ref_logits, ref_ids = oracle.lmhead_argmax(act, wb, wdtype=1)
    packed = fc.lmhead_pack(torch.from_numpy(wb.view(np.int16)).cuda().view(torch.bfloat16))
    ids, top, logits = fc.lmhead_argmax(torch.from_numpy(act).cuda(), packed, V, want_logits=True)
    torch.cuda.synchronize()
    lg = logits.cpu().numpy()
    err = np.abs(lg - ref_logits).max()
    print(f"lm head max |dlogit| {err:.3e}")
    assert err < 1e-3
    ids = ids.cpu().numpy()
    assert (ids == lg.argmax(-1)).all()                      # lowest index among equal maxima
    clear = margins(ref_logits) > 2e-3
    assert (ids[clear] == ref_ids[clear]).all()
    assert np.allclose(top.cpu().numpy(), lg.max(-1), rtol=0, atol=0)
    # without the debug logits the result is the same
    ids2, _, _ = fc.lmhead_argmax(torch.from_numpy(act).cuda(), packed, V, want_logits=False)
    assert (ids2.cpu().numpy() == ids).all()
    # the runner-up: the largest logit among the other ids (the oracle's, within the logit tolerance; the
    # kernel's own, exactly)
    ids3, top3, _, top2 = fc.lmhead_argmax(torch.from_numpy(act).cuda(), packed, V, want_top2=True)
    torch.cuda.synchronize()
    assert (ids3.cpu().numpy() == ids).all() and (top3.cpu().numpy() == lg.max(-1)).all()
    masked = lg.copy()
    masked[np.arange(M), ids] = -np.inf
    assert (top2.cpu().numpy() == masked.max(-1)).all()
    assert np.abs(top2.cpu().numpy() - np.partition(ref_logits, -2, axis=-1)[:, -2]).max() < 1e-3


def test_pack_weights_whole_model_equals_tensor_by_tensor(fc):
    """fastcot_pack_weights (one canonical buffer, offsets from fastcot_canonical_offset) gives the same packed
    bytes as fastcot_pack_tensor called per tensor, gains included."""
    import torch
    shape = SMALL
    cfg = fc.Config.from_shape(shape, 1, 64, 8)
    rng = np.random.default_rng(3)
    gains = {"gf": rng.uniform(0.5, 1.5, shape.d_model).astype(np.float32),
             "g1": [rng.uniform(0.5, 1.5, shape.d_model).astype(np.float32) for _ in range(shape.n_layers)],
             "g2": [None] * shape.n_layers}

    def gen():
        for spec in synthgen.weight_tensors(shape):
            yield spec.name, spec.layer, synthgen.weight_array(shape, spec, as_bf16_bits=True)
    say("pack_weights: whole model against tensor by tensor")
    a = fc.pack_weights(cfg, gen(), gains)
    b = fc.pack_weights_whole(cfg, gen(), gains)
    torch.cuda.synchronize()
    assert torch.equal(a, b)
