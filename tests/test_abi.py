"""CPU-side checks of the C ABI: the library loads, exports every entry point
that include/dard.h declares, validates arguments on the host (error codes
without touching a GPU) and sizes its buffers as documented."""
import ctypes
import os
import re

import pytest

from paper_2608_26574_amd import dard, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "dard.h")


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dard_[a-z_]+)\s*\(", text)))


def test_header_declares_the_boundary():
    names = declared_functions()
    for required in ("dard_build_state_mask", "dard_masked_attention", "dard_confidence",
                     "dard_commit_remask", "dard_step"):
        assert required in names


def test_library_exports_every_declared_symbol():
    L = dard.lib()
    missing = [n for n in declared_functions() if not hasattr(L, n)]
    assert not missing
    assert sorted(dard.EXPORTS) == declared_functions()


def test_version():
    assert dard.lib().dard_version() == 1


def _params(**kw):
    p = dict(tau_c=0.4, tau_u=0.9, lam=0.5 ** 0.125, p0=0.1, mask_id=5, flags=0)
    p.update(kw)
    return dard.make_params(**p)


def test_host_validation_errors():
    L = dard.lib()
    fake = ctypes.c_void_p(0x1000)   # never dereferenced: validation fails first
    # NULL pointers
    assert L.dard_build_state_mask(None, fake, 1, 4, 0, fake, None) == -1
    # B outside [1, 256]
    assert L.dard_build_state_mask(fake, fake, 1, 0, 0, fake, None) == -2
    assert L.dard_build_state_mask(fake, fake, 1, 257, 0, fake, None) == -2
    # unknown flag bits; two candidate orderings at once
    assert L.dard_build_state_mask(fake, fake, 1, 4, 1 << 12, fake, None) == -1
    assert b"flag" in L.dard_last_error()
    assert L.dard_build_state_mask(fake, fake, 1, 4, dard.F_C_BIDIR | dard.F_ORDER_L2R, fake, None) == -1
    assert b"ordering" in L.dard_last_error()
    # attention: P + 2B > cap, bad dh, GQA ratio
    args = [1, fake, fake, fake]
    assert L.dard_masked_attention(*args, 10, 11, fake, fake, 1, 1, 4, 4, 128, 0.1, 0, fake, None, 0, None) == -2
    assert L.dard_masked_attention(*args, 0, 64, fake, fake, 1, 8, 4, 4, 96, 0.1, 0, fake, None, 0, None) == -2
    assert L.dard_masked_attention(*args, 0, 64, fake, fake, 1, 8, 6, 4, 128, 0.1, 0, fake, None, 0, None) == -2
    # confidence: mixing without w, ld not a multiple of 4
    assert L.dard_confidence(fake, fake, None, None, 2, 10, 12, fake, fake, None, None, None, fake, 1 << 20,
                             None) == -1
    assert L.dard_confidence(fake, None, None, None, 2, 10, 10, fake, fake, None, None, None, fake, 1 << 20,
                             None) == -2
    # confidence: workspace too small
    assert L.dard_confidence(fake, None, None, None, 2, 16, 16, fake, fake, None, None, None, fake, 4, None) == -5
    # commit/remask: thresholds out of order, lambda outside (0, 1), unknown phase
    def remask(phase, p, *outs):
        rest = list(outs) + [None] * (4 - len(outs))
        return L.dard_commit_remask(phase, ctypes.byref(p), 1, 4, fake, fake, None, None, None, None, None, None,
                                    fake, *rest, None)
    assert remask(0, _params(tau_c=0.95, tau_u=0.9)) == -1
    assert remask(0, _params(lam=1.0)) == -1
    assert remask(7, _params()) == -1
    # fixed mixing weight outside [0, 1]; two orderings at once
    assert remask(0, _params(flags=dard.F_FIXED_W, w_fixed=1.5)) == -1
    assert b"w_fixed" in L.dard_last_error()
    assert remask(0, _params(flags=dard.F_ORDER_ENTROPY | dard.F_ORDER_MARGIN)) == -1
    # FINAL under the entropy ordering needs the caller's keys
    p = _params(flags=dard.F_ORDER_ENTROPY)
    assert L.dard_commit_remask(1, ctypes.byref(p), 1, 4, fake, fake, None, fake, fake, fake, None, None,
                                None, fake, fake, fake, None, None) == -1
    assert b"key" in L.dard_last_error()


def test_dims_validation_and_sizes():
    L = dard.lib()
    d = dard.make_dims(synth.LLADA8B)
    # packed image: weights + rotary table, each region 256-byte aligned
    n = L.dard_packed_weight_bytes(ctypes.byref(d))
    D, F, V, Lr = 4096, 12288, 126464, 32
    weights = 2 * (2 * V * D + Lr * (4 * D * D + 3 * D * F + 2 * D) + D)
    assert weights <= n <= weights + 256 * (4 + 6 * Lr) + 4096 * 64 * 2 * 4 + 256
    # KV cache [L][2][b][Hkv][cap][dh] bf16
    assert L.dard_kv_bytes(ctypes.byref(d), 1, 768) == 32 * 2 * 32 * 768 * 128 * 2
    # workspace holds at least the step's logits
    assert L.dard_workspace_bytes(ctypes.byref(d), 1, 32, 768) >= 64 * V * 4
    # cap smaller than the augmented block
    assert L.dard_workspace_bytes(ctypes.byref(d), 1, 32, 63) == 0
    bad = dard.make_dims(synth.Dims(2, 256, 4, 4, 96, 1024, 2048, 64, "f32"))
    assert L.dard_packed_weight_bytes(ctypes.byref(bad)) == 0
    assert b"head_dim" in L.dard_last_error()
    bad = dard.make_dims(synth.Dims(2, 256, 4, 3, 64, 1024, 2048, 64, "f32"))
    assert L.dard_packed_weight_bytes(ctypes.byref(bad)) == 0
    bad = dard.make_dims(synth.Dims(2, 4096, 32, 32, 128, 12288, 126460, 64, "bf16"))
    assert L.dard_packed_weight_bytes(ctypes.byref(bad)) == 0
    # a bf16 weight matrix of 4 GiB or more (LM head 262144 x 8192) is refused:
    # the tiled GEMM addresses weights with 32-bit byte offsets
    bad = dard.make_dims(synth.Dims(2, 8192, 64, 8, 128, 28672, 262144, 64, "bf16"))
    assert L.dard_packed_weight_bytes(ctypes.byref(bad)) == 0
    assert b"4 GiB" in L.dard_last_error()
    ok = dard.make_dims(synth.Dims(2, 8192, 64, 8, 128, 28672, 131072, 64, "bf16"))
    assert L.dard_packed_weight_bytes(ctypes.byref(ok)) > 0


def test_attention_workspace_sizing():
    L = dard.lib()
    # batch 1, 32 heads, 64 rows: a short prefix (3 key tiles) is walked by one
    # workgroup per head (room for the state mask only); a longer one is split
    # across workgroups (about 3 tiles each) and needs room for the partials
    short = L.dard_attention_workspace_bytes(1, 1, 32, 32, 128, 96)
    assert short == 64 * 8  # 64 rows x one 8-byte mask word
    long = L.dard_attention_workspace_bytes(1, 1, 32, 32, 128, 512)
    assert long > short + 3 * 64 * 32 * 128 * 4
    # many sequences fill the chip without splitting: room for the state mask only
    # (64 sequences x 64 rows x one 8-byte word)
    assert L.dard_attention_workspace_bytes(1, 64, 32, 32, 128, 512) == 64 * 64 * 8
    # the fp32 path never splits
    assert L.dard_attention_workspace_bytes(0, 1, 32, 4, 64, 64) == 0


def test_gemm_plan_query():
    """The host-side plan query reports the kernel and tiling launch_gemm runs
    (no GPU needed)."""
    # decoding step rows: the weight-streaming kernel; O / down split K
    assert dard.dard_gemm_plan(64, 24576, 4096)[0] == dard.GEMM_STREAM
    assert dard.dard_gemm_plan(64, 4096, 12288, partial=True)[3] > 1
    # 64 < M < 256 and M >= 256: the tiled kernel under its two codes
    assert dard.dard_gemm_plan(144, 1024, 512)[0] == dard.GEMM_PIPE
    assert dard.dard_gemm_plan(1024, 37888, 3584)[0] == dard.GEMM_BIG
    # a 700-row prefill of a wide FFN fills whole rounds with 128 x 192 tiles
    assert dard.dard_gemm_plan(700, 16256, 320)[:3] == (dard.GEMM_BIG, 4, 6)
    # the residual projection of those sizes takes another one (below 4096 rows
    # split-K partials never run on 128 x 192; this one runs unsplit on 256 x 192)
    assert dard.dard_gemm_plan(700, 16256, 320, partial=True)[1:3] != (4, 6)
    # row-major activations (dard_linear) and fp32
    assert dard.dard_gemm_plan(300, 256, 128, frag_x=False)[0] == dard.GEMM_TILED
    assert dard.dard_gemm_plan(300, 256, 128, dtype=dard.DTYPE_F32)[0] == dard.GEMM_F32
    L = dard.lib()
    plan = (ctypes.c_int32 * 4)()
    assert L.dard_gemm_plan(1, 64, 100, 64, 0, 1, plan) == -2      # N % 16 != 0
    assert L.dard_gemm_plan(1, 64, 128, 64, 0, 1, None) == -1


def test_state_check_validation():
    L = dard.lib()
    fake = ctypes.c_void_p(0x1000)
    assert L.dard_check_states(None, 4, fake, None) == -1
    assert L.dard_check_states(fake, 0, fake, None) == -2
    # a step under DARD_F_CHECK_STATES reports through block_done, which must be given
    p = _params(flags=dard.F_CHECK_STATES)
    assert L.dard_commit_remask(1, ctypes.byref(p), 1, 4, fake, fake, None, fake, fake, fake, None, None,
                                None, fake, fake, fake, None, None) == -1
    assert b"block_done" in L.dard_last_error()


def test_model_call_validation():
    """Host-side argument checks of the whole-model calls (nothing enqueued):
    the prefix refreshes and the three steps."""
    L = dard.lib()
    fake = ctypes.c_void_p(0x1000)
    d = dard.make_dims(synth.Dims(2, 256, 4, 2, 64, 512, 2048, 256, "bf16"))
    b, B, cap = 2, 16, 128
    ws = L.dard_workspace_bytes(ctypes.byref(d), b, B, cap)
    assert ws > 0
    dp = ctypes.byref(d)
    # extend-only refresh: NULL ids, Pn < 1, P + Pn past cap or max_pos, P < 0, workspace too small
    assert L.dard_prefill_extend(dp, fake, fake, cap, 10, b, 8, None, fake, ws, None) == -1
    assert L.dard_prefill_extend(dp, fake, fake, cap, 10, b, 0, fake, fake, ws, None) == -2
    assert L.dard_prefill_extend(dp, fake, fake, cap, 120, b, 9, fake, fake, ws, None) == -2
    assert L.dard_prefill_extend(dp, fake, fake, cap, -1, b, 8, fake, fake, ws, None) == -2
    assert L.dard_prefill_extend(dp, fake, fake, cap, 10, b, 8, fake, fake, 16, None) == -5
    # prefill: P outside [1, min(cap, max_pos)]
    assert L.dard_prefill(dp, fake, fake, cap, b, 0, fake, None, fake, ws, None) == -2
    assert L.dard_prefill(dp, fake, fake, cap, b, cap + 1, fake, None, fake, ws, None) == -2
    p = _params(mask_id=2047)
    pp = ctypes.byref(p)
    # step: P + 2B past cap; NULL outputs
    assert L.dard_step(dp, fake, fake, cap, cap - 2 * B + 1, pp, b, B, fake, fake, fake, fake, fake, fake, fake,
                       None, fake, ws, None) == -2
    assert L.dard_step(dp, fake, fake, cap, 8, pp, b, B, fake, fake, fake, None, fake, fake, fake,
                       None, fake, ws, None) == -1
    # full-sequence step: the block must lie inside the sequence, N + B <= cap
    assert L.dard_step_full(dp, fake, fake, cap, 64, 60, pp, b, B, fake, fake, fake, fake, fake, fake, fake,
                            None, fake, ws, None) == -2
    assert L.dard_step_full(dp, fake, fake, cap, cap - B + 1, 0, pp, b, B, fake, fake, fake, fake, fake, fake, fake,
                            None, fake, ws, None) == -2
    # shared-prompt step: the shared prompt is whole 64-key tiles and no longer than P
    assert L.dard_step_shared(dp, fake, fake, cap, fake, 128, 60, 64, pp, b, B, fake, fake, fake, fake, fake, fake,
                              fake, None, fake, ws, None) == -2
    assert L.dard_step_shared(dp, fake, fake, cap, fake, 128, 128, 64, pp, b, B, fake, fake, fake, fake, fake, fake,
                              fake, None, fake, ws, None) == -2
    assert L.dard_step_shared(dp, fake, fake, cap, None, 128, 64, 64, pp, b, B, fake, fake, fake, fake, fake, fake,
                              fake, None, fake, ws, None) == -1
