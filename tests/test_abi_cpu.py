"""Host-only checks of the C ABI: the library loads, exports every symbol the header declares,
sizes configurations, and rejects bad arguments before touching a GPU."""
import ctypes

import numpy as np
import os
import re

import synthgen
from paper_2311_08263_amd import binding


def test_library_exports_every_declared_symbol():
    hdr = open(os.path.join(os.path.dirname(__file__), "..", "include", "fastcot.h")).read()
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(fastcot_[a-z_0-9]+)\s*\(", hdr))
    assert declared, "no declarations found"
    L = ctypes.CDLL(binding._build.SO) if os.path.exists(binding._build.SO) else binding.lib()
    for name in declared:
        assert hasattr(L, name), f"{name} is declared in fastcot.h but not exported"
    assert declared == set(binding.SYMBOLS), declared ^ set(binding.SYMBOLS)


def test_sizes_and_invalid_configs():
    L = binding.lib()
    s7 = synthgen.SHAPES["7b"]
    cfg = binding.Config.from_shape(s7, 1, 640, 16)
    wb = L.fastcot_weight_bytes(ctypes.byref(cfg))
    streamed = s7.n_params_streamed() * 2
    assert streamed < wb < streamed + s7.vocab * s7.d_model * 2 + (1 << 22)
    assert L.fastcot_workspace_bytes(ctypes.byref(cfg)) > 2 * 32 * 640 * 4096 * 2
    for field, bad in (("head_dim", 100), ("n_kv_heads", 5), ("dtype", 7), ("window", 0), ("max_seq", 10), ("vocab", 1001)):
        c = binding.Config.from_shape(s7, 1, 640, 16)
        setattr(c, field, bad)
        assert L.fastcot_weight_bytes(ctypes.byref(c)) == 0, field
        assert L.fastcot_workspace_bytes(ctypes.byref(c)) == 0, field


def test_logits_are_sized_for_the_rows_of_a_step():
    """Prompt passes of the plain kernels have more rows per sequence than a step, but no logits: a larger vocabulary adds
    four bytes per id and step row, and the winners of the argmax (eight bytes per sixteen ids and row)."""
    L = binding.lib()
    B, W, d = 4, 8, 256
    size = [L.fastcot_workspace_bytes(ctypes.byref(binding.Config(2, d, 4, 4, 64, 688, V, 1e-5, 1e4, 0, B, 640, W))) for V in (16000, 32000)]
    assert 0 < size[1] - size[0] <= 16000 * (B * W * 4 + 32 * 8 // 16) + 4096


def test_null_arguments_are_rejected_without_a_gpu():
    L = binding.lib()
    assert L.fastcot_prefill(None, 1, None, 1, None, None, 1) == -1
    assert L.fastcot_jacobi_step(None, None, None, None) == -1
    assert L.fastcot_generate(None, 1, 0, -1, None, None, None, None) == -1
    assert L.fastcot_get_state(None, None, None, None, None, None, None) == -1
    one = np.ones(4, dtype=np.int32)
    assert L.fastcot_set_window(None, 4) == -1
    assert L.fastcot_set_windows(None, one.ctypes.data) == -1
    assert L.fastcot_step_rows(None, one.ctypes.data) == -1
    assert L.fastcot_join(None, 0, one.ctypes.data, 4, one.ctypes.data) == -1
    assert L.fastcot_answer(None, one.ctypes.data, 1, 4, -1, one.ctypes.data, one.ctypes.data) == -1
    assert b"NULL" in L.fastcot_last_error(None)
    cfg = binding.Config.from_shape(synthgen.SHAPES["tiny"], 1, 64, 4)
    out = ctypes.c_void_p()
    assert L.fastcot_init(ctypes.byref(cfg), None, None, 0, None, ctypes.byref(out)) == -1
    assert L.fastcot_pack_tensor(ctypes.byref(cfg), 99, 0, None, None, None) == -1
    assert L.fastcot_attn_window(None, None, None, 0, 1, 1, 1, 16, 16, 0, None, None, None) == -1
    assert L.fastcot_lmhead_argmax(None, None, 1, 32, 16, None, None, None, None, None, None) == -1
    assert L.fastcot_pack_weights(ctypes.byref(cfg), None, None, None) == -1
    assert L.fastcot_canonical_offset(ctypes.byref(cfg), 3, 99) == ctypes.c_size_t(-1).value
    assert L.fastcot_kernel_name(4) == b"attention"


class _Dims(ctypes.Structure):              # KernelDims and FastPlan of the library's headers
    _fields_ = [(n, ctypes.c_int32) for n in "L d H Hkv Dh F V B S W M Wcap Rcap qkvN".split()] + [("eps", ctypes.c_float)] + \
               [(n, ctypes.c_int32) for n in "esz kvp actq kvq".split()]


class _Plan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in "attn_splits attn_cut attn_bpw attn_many co_single".split()] + \
               [(n, ctypes.c_int32 * k) for n, k in (("co_sb", 10), ("co_rot", 10), ("ks", 5), ("nw2", 5), ("ks2", 5), ("nw", 5), ("ks_rule", 5))]


def _attention_form(B, H, W, kvp, many, ctx_len):
    """Form of a step's attention launch, by which a captured step is kept or captured once more (256 CUs without a GPU)."""
    L = ctypes.CDLL(binding._build.SO)
    plan, form = L["_Z12fc_fast_planRK10KernelDimsP8FastPlan"], L["_Z12fc_attn_formRK10KernelDimsiRK8FastPlani"]
    kd = _Dims(2, H * 128, H, H, 128, H * 256, 1024, B, 4096, W, B * W, W, W, 3 * H * 128, 1e-5, 2, kvp, 0, 0)
    p = _Plan()
    plan(ctypes.byref(kd), ctypes.byref(p))
    p.attn_many = many
    assert p.attn_bpw == 2 and p.co_single == 2           # (the fields above are where the library has them)
    return form(ctypes.byref(kd), B, ctypes.byref(p), ctx_len)


def test_attention_form_of_a_captured_step():
    """A step keeps its graph while its launches stay what they are: the many-row kernel has one form for every context, the other
    one changes where its last units are first cut."""
    binding.lib()
    lengths = range(100, 3000, 50)
    for B, H, W in ((7, 40, 64), (9, 32, 64), (9, 32, 128)):
        assert len({_attention_form(B, H, W, 2, 1, n) for n in lengths}) == 1
    assert len({_attention_form(7, 40, 64, 2, 0, n) for n in lengths}) == 2
    assert len({_attention_form(7, 40, 64, 3, 1, n) for n in lengths}) == 2
    assert len({_attention_form(9, 32, 16, 2, 1, n) for n in lengths}) == 2


def test_end_of_a_step_in_one_launch_where_that_is_faster():
    """Rows and logits, or rows and partial winners, on both sides of the lines: one workgroup loses where a wave has much to walk."""
    fits = ctypes.CDLL(binding._build.SO)["_Z12fc_tail_fitsiiiib"]
    fits.argtypes, fits.restype = [ctypes.c_int32] * 4 + [ctypes.c_bool], ctypes.c_bool
    for M, V in ((1, 2048), (8, 1024), (16, 2048), (17, 256), (32, 256)):
        assert fits(1, M, M, V, False)
    for M, V in ((1, 2064), (1, 8192), (8, 4096), (16, 4096), (17, 272), (32, 512), (33, 16), (64, 128), (512, 16)):
        assert not fits(1, M, M, V, False)
    for M, parts in ((1, 256), (16, 256), (17, 128), (32, 128)):
        assert fits(2, M, M, parts, True)
    for M, parts in ((1, 512), (16, 257), (17, 129), (32, 256), (33, 16)):
        assert not fits(2, M, M, parts, True)
    assert fits(4, 256, 10, 64, True) and not fits(4, 257, 10, 64, True)


def test_workspaces_with_and_without_copies_of_the_weights():
    """Copies in 13 bits a weight of every matrix; of the 70B shape, where weights and workspace may have 208 GiB, as many layers as
    fit; none for fp32 models."""
    L = binding.lib()

    def sizes(name, B=1, S=640, W=16):
        c = binding.Config.from_shape(synthgen.SHAPES[name], B, S, W)
        return L.fastcot_weight_bytes(ctypes.byref(c)), L.fastcot_workspace_bytes_min(ctypes.byref(c)), L.fastcot_workspace_bytes(ctypes.byref(c))
    for name in ("7b", "13b"):
        _, least, full = sizes(name)
        streamed = synthgen.SHAPES[name].n_params_streamed() * 13 / 8
        assert streamed < full - least < streamed * 1.01
    s = synthgen.SHAPES["70b"]
    for B, S in ((1, 640), (8, 4096)):
        weights, least, full = sizes("70b", B, S)
        assert least < full and 0 <= (208 << 30) - weights - full < s.d_ffn * s.d_model * 13 / 8 * 1.01
    assert sizes("70b", 32, 8192)[1] == sizes("70b", 32, 8192)[2]
    assert sizes("tiny")[1] == sizes("tiny")[2]
