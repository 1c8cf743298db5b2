"""Coded copies of the weights: the kernels that read them compute with every weight as it was packed.

A row with a single 1 picks one row of W out of the product: every other term is an exact zero, so the logits are W's row itself."""
import ctypes

import numpy as np
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fc():
    import paper_2311_08263_amd as m
    return m


def edge_rows(d):
    """Rows of two pairs of wave 0, of three of wave 1 and, where it has them, of the first and the 65th pair of wave 3 (no K slices)."""
    PT = d // 64
    begin = [w * PT // 8 for w in range(9)]
    pairs = [(0, 0), (0, 1), (1, 0), (1, 1), (1, 2)] + ([(3, 0), (3, 64)] if begin[4] - begin[3] > 64 else [])
    return [64 * (begin[w] + i) + 9 * (w + 1) for w, i in pairs]


def special(w, kind, seed):
    """Weights outside their columns' windows: few (flagged pairs taken one by one), edge (two flagged pairs of a wave are taken one by one, three
    are not; where waves have more than 64 pairs, the first and the 65th share a bit), many (whole walks over the plain tiles), columns of
    zeros, tiny or huge ones, a column whose largest weight leaves all others outside; zeros, which have a code of their own."""
    import torch
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    d, V = w.shape
    if kind == "few":
        for i in range(6):
            w[(i * 7919 + 5) % d, (i * 104729 + 3) % V] = 2.0 ** -60
        w[d - 1, V - 1] = -0.0; w[0, 0] = 2.0 ** -100
    elif kind == "edge":
        for k in edge_rows(d):
            w[k, k // 64 % 8] = 2.0 ** -60
    elif kind == "many":
        w[torch.rand(d, V, generator=g, device="cuda") < 0.5] = 2.0 ** -60
    elif kind == "zeros":
        w[torch.rand(d, V, generator=g, device="cuda") < 0.5] = 0.0
        w[torch.rand(d, V, generator=g, device="cuda") < 0.01] = -0.0
    elif kind == "columns":
        w[:, 0] = 0.0; w[:, 15] = 0.0; w[3, 15] = 1.5
        w[:, 5] *= 2.0 ** -120; w[:, 6] *= 2.0 ** 120; w[:, 7] = -w[:, 7].abs(); w[0, 8] = 2.0 ** 126
        for c, e in ((9, -29), (10, -30), (11, -31), (12, -32)):  # the last exponents inside the window and the first ones outside
            w[:, c] = 2.0 ** e; w[1, c] = 1.9921875
    return w


@pytest.mark.parametrize("kind", ["none", "few", "many", "zeros", "columns"])
@pytest.mark.parametrize("M,d,V", [(16, 256, 16), (16, 512, 592), (5, 768, 4112), (32, 1024, 2000), (17, 256, 8208)])
def test_every_weight_comes_out_as_it_went_in(fc, kind, M, d, V):
    """One to three n-tiles per workgroup (256 CUs), waves of no, one and two pairs of k-tiles, one and two row tiles; every row."""
    import torch
    say(f"coded weights {kind} M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(7)
    w = special((0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16(), kind, 11)
    packed = fc.lmhead_pack(w)
    scratch = torch.zeros(fc.lib().fastcot_lmhead_scratch_bytes(M, d, V), dtype=torch.uint8, device="cuda")
    for k0 in range(0, d, M):
        act = torch.zeros(M, d, device="cuda")
        rows = torch.arange(k0, min(k0 + M, d), device="cuda")
        act[torch.arange(len(rows), device="cuda"), rows] = 1.0
        _, _, logits = fc.lmhead_argmax(act, packed, V, True, scratch)
        assert torch.equal(logits[:len(rows)], w[rows].float()), k0


@pytest.mark.parametrize("kind", ["few", "edge", "many", "columns"])
@pytest.mark.parametrize("M,d,V", [(16, 4096, 16 * 1000), (5, 4096, 16 * 1300), (16, 4096, 16 * 1800), (16, 4096, 16 * 2900), (16, 4096, 16 * 3400), (24, 4096, 16 * 1000),
                                   (32, 4096, 16 * 1300), (17, 4096, 16 * 1800), (16, 33280, 16 * 20), (32, 33280, 16 * 300)])
def test_weights_of_wide_workgroups(fc, kind, M, d, V):
    """Four, six, eight, twelve and fourteen n-tiles per workgroup (256 CUs) up to 16 rows, four, six and eight of more, waves of eight pairs; waves
    of 65 pairs.  The rows that hold weights outside the windows, the first and the last ones."""
    import torch
    say(f"wide workgroups {kind} M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(7)
    w = special((0.02 * torch.randn(d, V, generator=g, device="cuda")).bfloat16(), kind, 11)
    packed = fc.lmhead_pack(w)
    scratch = torch.zeros(fc.lib().fastcot_lmhead_scratch_bytes(M, d, V), dtype=torch.uint8, device="cuda")
    for k0 in sorted({k // M * M for k in [0, 1, 3, d - 1] + [(i * 7919 + 5) % d for i in range(6)] + edge_rows(d)}):
        act = torch.zeros(M, d, device="cuda")
        rows = torch.arange(k0, min(k0 + M, d), device="cuda")
        act[torch.arange(len(rows), device="cuda"), rows] = 1.0
        _, _, logits = fc.lmhead_argmax(act, packed, V, True, scratch)
        assert torch.equal(logits[:len(rows)], w[rows].float()), k0


def tensors(shape, kind, seed):
    import torch
    L, d, H, Hkv, F, V = shape
    g = torch.Generator(device="cuda"); g.manual_seed(seed)
    def t(r, c, s): return (s * torch.randn(r, c, generator=g, device="cuda")).bfloat16()
    emb = t(V, d, 1.0)
    yield "emb", 0, emb
    yield "wlm", 0, special(t(d, V, 0.02), kind, seed)
    for l in range(L):
        for n, r, c in (("wq", d, H * 128), ("wk", d, Hkv * 128), ("wv", d, Hkv * 128), ("wo", H * 128, d), ("wg", d, F), ("wu", d, F), ("wd", F, d)):
            yield n, l, special(t(r, c, 0.02 if n not in ("wo", "wd") else 0.01), kind, seed + l)


def pack(fc, cfg, items, packed=None):
    import torch
    L, st = fc.lib(), torch.cuda.current_stream().cuda_stream
    if packed is None:
        packed = torch.zeros(L.fastcot_weight_bytes(ctypes.byref(cfg)), dtype=torch.uint8, device="cuda")
    for n, l, t in items:
        assert L.fastcot_pack_tensor(ctypes.byref(cfg), fc.binding.T[n], l, t.data_ptr(), packed.data_ptr(), st) == 0
    for n, l in [("gf", 0)] + [(g, l) for g in ("g1", "g2") for l in range(cfg.n_layers)]:
        assert L.fastcot_pack_tensor(ctypes.byref(cfg), fc.binding.T[n], l, None, packed.data_ptr(), st) == 0
    torch.cuda.synchronize()
    return packed


def first_logits(ctx, prompts, buf, rows):
    logits = ctx.debug_logits(True)
    ctx.prefill(prompts, [prompts.shape[1]] * prompts.shape[0], buf)
    ctx.step()
    return logits[:rows].clone()


@pytest.mark.parametrize("kind", ["none", "few", "many", "zeros"])
@pytest.mark.parametrize("B,W", [(1, 1), (1, 16), (2, 12)])
def test_steps_on_coded_weights(fc, kind, B, W):
    """Every product of a step (K slices, flagged pairs, plain walks) against the plain kernels on the plain tiles: fp32 arithmetic there,
    activations of 17 bits here, so logits that differ by a few 2^-17 of their size per product (nine in a row; 1e-4 is ten times that)."""
    import torch
    say(f"step on coded weights {kind} B={B} W={W}")
    shape = (2, 4096, 32, 8, 8192, 1008) if W == 16 else (2, 512, 4, 2, 768, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, B, 128, W)
    packed = pack(fc, cfg, tensors(shape, kind, 3))
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (B, 21)).astype(np.int32), r.randint(0, V, (B, 3 * W)).astype(np.int32)
    out = []
    for plain in (0, 1):
        ctx = fc.Context(cfg, packed)
        if plain:
            ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, 1)
        out.append(first_logits(ctx, prompts, buf, B * W))
        ctx.close() if hasattr(ctx, "close") else None
    a, b = out[0].double(), out[1].double()
    assert float(torch.linalg.norm(a - b) / torch.linalg.norm(b)) < 1e-4


@pytest.mark.parametrize("kind", ["few", "many"])
@pytest.mark.parametrize("W", [16, 24])
@pytest.mark.parametrize("copies", [0, 1])
def test_orders_of_a_walk(fc, kind, W, copies):
    """Pairs of k-tiles under way (two, one) move loads and no bits; a walk in rotated order, or in order where it is rotated by default, moves
    additions alone (fp32 sums, 1e-5), with K slices, flagged pairs and plain walks, over the copies and without them."""
    import torch
    shape = (2, 4096, 32, 8, 8192, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, W)
    packed = pack(fc, cfg, tensors(shape, kind, 3))
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 3 * W)).astype(np.int32)

    def logits(*opts):
        say(f"order of a walk {kind} W={W} copies={copies} {opts}")
        ctx = fc.Context(cfg, packed, None if copies else sizes(fc, cfg)[0])
        for o in opts:
            ctx.set_option(*o)
        out = first_logits(ctx, prompts, buf, W)
        ctx.close()
        return out
    default = logits()
    for n in (0, 1):
        assert torch.equal(logits((fc.binding.PLAN_CO_SINGLE, n)), default)
        other = logits(*[(fc.binding.PLAN_ROT + g, n) for g in range(5)])
        assert float(torch.linalg.norm(other - default) / torch.linalg.norm(default)) < 1e-5
        assert torch.equal(other, default) == (n == 1 - copies)


def test_weights_packed_again_are_coded_again(fc):
    """A prefill after other weights were packed computes with those, as a context that never saw the first ones does."""
    import torch
    say("weights packed again")
    shape = (2, 512, 4, 2, 768, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, 8)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 24)).astype(np.int32)
    packed = pack(fc, cfg, tensors(shape, "none", 3))
    ctx = fc.Context(cfg, packed)
    first = first_logits(ctx, prompts, buf, 8)
    assert torch.equal(first, first_logits(ctx, prompts, buf, 8))
    pack(fc, cfg, tensors(shape, "few", 9), packed)
    again = first_logits(ctx, prompts, buf, 8)
    fresh = first_logits(fc.Context(cfg, pack(fc, cfg, tensors(shape, "few", 9))), prompts, buf, 8)
    assert not torch.equal(first, again) and torch.equal(again, fresh)


def _unsampled_change(items):
    """The same tensors with weights of wo and the LM head changed in all columns but the first."""
    for n, l, t in items:
        if n in ("wo", "wlm"):
            t = t.clone(); t[:, 1:] *= -1
        yield n, l, t


@pytest.mark.parametrize("how", ["packed over zeros", "copied over"])
def test_every_new_set_of_weights_is_noticed(fc, how):
    """Other weights in the same buffer, packed after clearing it or copied over as a whole packed image: the next prefill and its
    step are those of a context that never saw the first ones, whichever weights differ."""
    import torch
    say(f"other weights {how}")
    shape = (1, 4096, 32, 8, 512, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, 8)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 24)).astype(np.int32)
    packed, other = pack(fc, cfg, tensors(shape, "none", 3)), pack(fc, cfg, _unsampled_change(tensors(shape, "none", 3)))
    ctx = fc.Context(cfg, packed)
    first = first_logits(ctx, prompts, buf, 8)
    if how == "copied over":
        packed.copy_(other)
        torch.cuda.synchronize()
    else:
        packed.zero_()
        torch.cuda.synchronize()
        pack(fc, cfg, _unsampled_change(tensors(shape, "none", 3)), packed)
    again = first_logits(ctx, prompts, buf, 8)
    assert torch.equal(again, first_logits(fc.Context(cfg, other), prompts, buf, 8)) and not torch.equal(first, again)


@pytest.mark.parametrize("graph", [0, 1])
def test_steps_between_packing_and_prefill(fc, graph):
    """A step after other weights were packed computes with those, also as a replay captured before; against the plain kernels on the same
    cache (nine products in a row, 1e-4 as above)."""
    import torch
    say(f"weights packed between steps graph={graph}")
    shape = (2, 512, 4, 2, 768, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, 8)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 64)).astype(np.int32)
    packed = pack(fc, cfg, tensors(shape, "none", 3))
    ctx = fc.Context(cfg, packed)
    ctx.set_option(fc.binding.OPT_GRAPH, graph)
    logits = ctx.debug_logits(True)
    ctx.prefill(prompts, [21], buf)
    ctx.step()
    pack(fc, cfg, tensors(shape, "few", 9), packed)
    n, win = ctx.state()["n"][0], ctx.state()["window"]
    ctx.step()
    got = logits[:8].clone()
    plain = fc.Context(cfg, pack(fc, cfg, tensors(shape, "none", 3)))
    plain.set_option(fc.binding.OPT_PLAIN_KERNELS, 1)
    ref = plain.debug_logits(True)
    plain.prefill(prompts, [21], buf)
    plain.step()
    assert plain.state()["n"][0] == n and (plain.state()["window"] == win).all()
    pack(fc, cfg, tensors(shape, "few", 9), plain.packed)
    plain.step()
    a, b = got.double(), ref[:8].double()
    assert float(torch.linalg.norm(a - b) / torch.linalg.norm(b)) < 1e-4


def test_contexts_that_share_a_workspace_in_turn(fc):
    """Two contexts of one configuration over different weights, one workspace, used one after the other, each from its own prefill on."""
    import ctypes as ct
    import torch
    say("shared workspace")
    shape = (2, 512, 4, 2, 768, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, 8)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 24)).astype(np.int32)
    a, b = fc.Context(cfg, pack(fc, cfg, tensors(shape, "none", 3))), fc.Context(cfg, pack(fc, cfg, tensors(shape, "none", 4)))
    want = [first_logits(c, prompts, buf, 8) for c in (a, b)]
    lib, h = fc.lib(), ct.c_void_p()
    assert lib.fastcot_init(ct.byref(cfg), b.packed.data_ptr(), a.workspace.data_ptr(), a.workspace.numel(), b.stream.cuda_stream, ct.byref(h)) == 0
    lib.fastcot_free(b.h); b.h = h; b.workspace = a.workspace
    for _ in range(2):
        for c, w in zip((a, b), want):
            assert torch.equal(first_logits(c, prompts, buf, 8), w)


@pytest.mark.parametrize("M,d,V", [(16, 20736, 24592), (32, 20736, 24592), (16, 23552, 53264), (1, 35072, 48), (32, 35072, 48)])
def test_isolated_lm_head_of_many_inputs(fc, M, d, V):
    """An LM head without a norm in front keeps no gain in LDS, so the number of its inputs is not limited by that: seven, fourteen and one
    n-tile per workgroup, waves of up to 69 pairs."""
    import torch
    say(f"LM head of many inputs M={M} d={d} V={V}")
    g = torch.Generator(device="cuda"); g.manual_seed(7)
    w = special((0.02 * torch.randn(d, V, generator=g, device="cuda", dtype=torch.float32)).bfloat16(), "few", 11)
    packed = fc.lmhead_pack(w)
    scratch = torch.zeros(fc.lib().fastcot_lmhead_scratch_bytes(M, d, V), dtype=torch.uint8, device="cuda")
    for k0 in (0, 7 * 7919 % d, d - M):
        act = torch.zeros(M, d, device="cuda")
        rows = torch.arange(k0, min(k0 + M, d), device="cuda")
        act[torch.arange(len(rows), device="cuda"), rows] = 1.0
        _, _, logits = fc.lmhead_argmax(act, packed, V, True, scratch)
        assert torch.equal(logits[:len(rows)], w[rows].float()), k0


def test_model_of_the_most_inputs(fc):
    """21504 inputs, the most whose norm gain fits the LDS beside the partial tiles of seven or eight n-tiles (the LM head here); against the
    plain kernels as above."""
    import torch
    say("model of 21504 inputs")
    shape = (1, 21504, 2, 2, 256, 24592)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 64, 16)
    packed = pack(fc, cfg, tensors(shape, "none", 3))
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 9)).astype(np.int32), r.randint(0, V, (1, 48)).astype(np.int32)
    out = []
    for plain in (0, 1):
        ctx = fc.Context(cfg, packed)
        ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, plain)
        out.append(first_logits(ctx, prompts, buf, 16).double())
        ctx.close()
    assert float(torch.linalg.norm(out[0] - out[1]) / torch.linalg.norm(out[1])) < 1e-4


def test_plan_options_take_what_a_launch_takes(fc):
    """Gate/up of 13.5 n-tiles per CU: its own grid (one round of 14) and slice count are accepted, other grids up to 14 tiles too, 15 are not;
    one K slice computes the default's bits, other grids the same logits."""
    import torch
    shape = (1, 256, 2, 2, 27648, 1008)
    L, d, H, Hkv, F, V = shape
    cfg = fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, 1, 128, 16)
    packed = pack(fc, cfg, tensors(shape, "none", 3))
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, V, (1, 21)).astype(np.int32), r.randint(0, V, (1, 48)).astype(np.int32)
    NW, KS, NT = fc.binding.PLAN_NW + 2, fc.binding.PLAN_KS + 2, 2 * F // 16
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def logits(*opts):
        say(f"gate/up plan {opts}")
        ctx = fc.Context(cfg, packed)
        for o in opts:
            ctx.set_option(*o)
        out = first_logits(ctx, prompts, buf, 16).double()
        ctx.close()
        return out
    default, fewest = logits(), (NT + 13) // 14
    for same in (((KS, 1),), ((NW, cus),), ((NW, 2 * cus), (NW, cus), (KS, 1))):
        assert torch.equal(logits(*same), default)
    for other in (((NW, 2 * cus),), ((NW, fewest),)):
        assert float(torch.linalg.norm(logits(*other) - default) / torch.linalg.norm(default)) < 1e-5
    for refused in (((NW, fewest - 1),), ((NW, NT + 1),), ((KS, 2),), ((KS, 9),)):
        with pytest.raises(fc.FastcotError):
            logits(*refused)


SMALL = (2, 512, 4, 2, 768, 1008)


def small_cfg(fc, B, W):
    L, d, H, Hkv, F, V = SMALL
    return fc.Config(L, d, H, Hkv, 128, F, V, 1e-5, 1e4, 1, B, 128, W)


def sizes(fc, cfg):
    return fc.lib().fastcot_workspace_bytes_min(ctypes.byref(cfg)), fc.lib().fastcot_workspace_bytes(ctypes.byref(cfg))


def test_workspaces_without_room_for_every_copy(fc, monkeypatch):
    """From the least workspace on any size does, with the same logits but for the order of additions (fp32 sums of 17-bit activations times
    weights: 1e-5 as between grids); less is refused; without memory for the copies a context takes the least."""
    import torch
    cfg = small_cfg(fc, 1, 8)
    packed, (least, full) = pack(fc, cfg, tensors(SMALL, "none", 3)), sizes(fc, cfg)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, 1008, (1, 21)).astype(np.int32), r.randint(0, 1008, (1, 24)).astype(np.int32)
    want = first_logits(fc.Context(cfg, packed), prompts, buf, 8)
    for n in (least, least + 1, least + (full - least) // 3, (least + full) // 2, full - 1, full + 4096):
        say(f"workspace of {n} bytes, {least} to {full}")
        ctx = fc.Context(cfg, packed, n)
        got = first_logits(ctx, prompts, buf, 8)
        assert ctx.workspace.numel() == n and float(torch.linalg.norm(got - want) / torch.linalg.norm(want)) < 1e-5
    with pytest.raises(fc.FastcotError):
        fc.Context(cfg, packed, least - 1)
    empty = torch.empty

    def short(n, *a, **k):
        if n == full:
            raise torch.cuda.OutOfMemoryError("no room")
        return empty(n, *a, **k)
    monkeypatch.setattr(torch, "empty", short)
    ctx = fc.Context(cfg, packed)
    got = first_logits(ctx, prompts, buf, 8)
    assert ctx.workspace.numel() == least and torch.equal(got, first_logits(fc.Context(cfg, packed, least), prompts, buf, 8))


@pytest.mark.parametrize("B,W,plain", [(1, 8, 0), (1, 8, 1), (3, 12, 0)])
def test_copies_are_made_where_steps_read_them(fc, B, W, plain):
    """Steps of up to 32 rows by the matrix-core kernels: made by the prefill; the plain kernels and steps of more rows: never; made by the
    first step that has few rows because its sequences have windows of their own."""
    import torch
    say(f"copies made B={B} W={W} plain={plain}")
    cfg = small_cfg(fc, B, W)
    packed, (least, full) = pack(fc, cfg, tensors(SMALL, "none", 3)), sizes(fc, cfg)
    r = np.random.RandomState(5)
    prompts, buf = r.randint(0, 1008, (B, 21)).astype(np.int32), r.randint(0, 1008, (B, 5 * W)).astype(np.int32)
    ctx = fc.Context(cfg, packed)
    ctx.set_option(fc.binding.OPT_PLAIN_KERNELS, plain)
    ctx.workspace[least:] = 0x5A
    torch.cuda.synchronize()
    ctx.prefill(prompts, [21] * B, buf)
    if plain or B * W > 32:
        ctx.step()
        assert bool((ctx.workspace[least:] == 0x5A).all())
    else:
        assert float((ctx.workspace[least:] != 0x5A).float().mean()) > 0.9
    if B * W > 32:
        ctx.set_windows([4] * B)
        logits = ctx.debug_logits(True)
        ctx.step()
        assert float((ctx.workspace[least:] != 0x5A).float().mean()) > 0.9
        got = logits[:4 * B].clone()
        ref = fc.Context(cfg, packed, least)
        ref.prefill(prompts, [21] * B, buf)
        ref.step(); ref.set_windows([4] * B)
        logits = ref.debug_logits(True)
        ref.step()
        assert float(torch.linalg.norm(got - logits[:4 * B]) / torch.linalg.norm(got)) < 1e-5
