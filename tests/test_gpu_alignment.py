"""Buffers that are only as aligned as their element: the fp32 output of
dard_linear, captured logits in every form of the LM head, and image embeddings
(by both embedding kernels).  Each case is compared bit for bit with the same
call on 16-byte aligned buffers, since alignment only changes how values are
moved."""
import sys

import numpy as np
import pytest
import torch

from oracle import dard_oracle as O
from paper_2608_26574_amd import dard, synth

from parity import P, cparams, dev, step_buffers

pytestmark = pytest.mark.gpu


def announce(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


def shifted(shape, dtype, fill, by=1):
    """A contiguous tensor `by` elements past a 16-byte boundary."""
    n = int(np.prod(shape))
    t = torch.full((n + 16,), fill, dtype=dtype, device="cuda")[by:by + n].view(*shape)
    assert t.data_ptr() % 16 == by * t.element_size() % 16
    return t


# streaming, row-major tiles and fp32 in each of its tilings
@pytest.mark.parametrize("dtype,M,N,K", [("bf16", 33, 80, 128), ("bf16", 200, 272, 64), ("f32", 33, 100, 68),
                                         ("f32", 130, 516, 260), ("f32", 520, 2060, 132)])
def test_linear_output(dtype, M, N, K):
    announce("linear, output off alignment", dtype, M, N, K)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(M + N)
    X = torch.randn(M, K, generator=g, device="cuda").to(td)
    W = torch.randn(N, K, generator=g, device="cuda").to(td)
    Wp = torch.empty_like(W)
    dard.dard_pack_matrix(W, Wp)
    ref = torch.full((M, N), float("nan"), device="cuda")
    dard.dard_linear(X, Wp, N, ref)
    for by in (1, 2, 3):
        out = shifted((M, N), torch.float32, float("nan"), by)
        dard.dard_linear(X, Wp, N, out)
        torch.cuda.synchronize()
        assert torch.equal(out, ref), by


# the head over all rows, over listed rows (stored), over listed rows with fused
# partials, its two hidden-mixing passes, and the fp32 head
@pytest.mark.parametrize("dtype,b,B,flags", [("bf16", 1, 16, 0), ("bf16", 3, 24, 0), ("bf16", 2, 80, 0),
                                             ("bf16", 5, 64, O.F_HIDDEN_MIX), ("f32", 2, 16, 0)])
def test_captured_logits(dtype, b, B, flags):
    announce("captured logits off alignment", dtype, b, B, flags)
    dims = synth.Dims(1, 512, 4, 2, 128, 512, 1040, 512, dtype)
    w = {k: v.cuda() for k, v in synth.make_weights(dims, seed=3).items()}
    eng = dard.Engine(dims, w, b, B, 40 + 2 * B)
    eng.dard_prefill(dev(synth.prompt_ids(b, 40, dims.vocab, seed=4)))
    tok, state, conf = synth.tiny_block(b, B, dims.vocab, seed=5)
    prm = cparams(dard, P(dims.mask_id, flags))
    res = []
    for by in (0, 1, 3):
        out, dbg = step_buffers(b, B, dims.vocab)
        if by:
            dbg["logits"] = shifted((b, 2 * B, dims.vocab), torch.float32, float("nan"), by)
        eng.dard_step(40, prm, dev(tok), dev(state), dev(conf), out["tok_out"], out["state_out"], out["conf_out"],
                      out["block_done"], debug={"logits": dbg["logits"]})
        torch.cuda.synchronize()
        res.append([dbg["logits"].cpu().numpy()] + [t.cpu().numpy() for t in out.values()])
    # the rows that the decisions read are there (rows the head does not run over stay NaN)
    need = np.ones((b, 2 * B), dtype=bool)
    need[:, :B] = (state == O.STATE_M) & (flags != O.F_HIDDEN_MIX)
    assert np.all(np.isfinite(res[0][0][need]))
    for r in res[1:]:
        for x, y in zip(res[0], r):
            assert np.array_equal(x, y, equal_nan=x.dtype == np.float32)


# a workgroup per row, and a wave per row (2048 rows or more; unaligned rows there
# take the former); ids < 0 take the embedding row, the others the table's
@pytest.mark.parametrize("dtype,b,P_", [("bf16", 1, 37), ("f32", 2, 29), ("bf16", 3, 683), ("bf16", 1, 2048)])
def test_image_embeddings(dtype, b, P_):
    announce("image embeddings", dtype, b, P_)
    dims = synth.Dims(1, 256, 2, 1, 128, 256, 1040, 4096, dtype)
    td = synth.torch_dtype(dims)
    w = {k: v.cuda() for k, v in synth.make_weights(dims, seed=3).items()}
    g = torch.Generator(device="cuda").manual_seed(7)
    emb = torch.randn(b, P_, dims.d_model, generator=g, device="cuda").to(td)
    ids = dev(synth.prompt_ids(b, P_, dims.vocab, seed=4))
    image = torch.rand(b, P_, generator=g, device="cuda") < 0.5
    ids[image] = -1
    eng = dard.Engine(dims, w, b, 8, P_ + 16)
    caches = []
    for by in (0, 1):
        e = emb
        if by:
            e = shifted(emb.shape, td, 0.0, by)
            e.copy_(emb)
        eng.kv.zero_()
        eng.dard_prefill(ids, embeds=e)
        torch.cuda.synchronize()
        caches.append([t.clone() for t in eng.kv_view(td)])
    # V of the only layer from the embedding rows, in float64: norm, projection, two
    # storage roundings (bf16: 2^-9 each, and the sum over 256 terms of order one)
    h = torch.where(image[..., None], emb.double(), w["embed"][ids.clamp(min=0).long()].double())
    x = h / torch.sqrt((h * h).mean(-1, keepdim=True) + dims.norm_eps) * w["layers.0.attn_norm"].double()
    ref = (x @ w["layers.0.wv"].double().T).view(b, P_, 1, 128).transpose(1, 2)
    got = caches[0][1][0][:, :, :P_].double()
    err = ((got - ref).norm(dim=-1) / ref.norm(dim=-1)).max().item()
    assert err < (1e-2 if dtype == "bf16" else 1e-5), err
    for x, y in zip(*caches):
        # the two kernels sum a row's squares in another order: a last bit of the norm
        d = (x.double() - y.double()).norm() / x.double().norm()
        assert d < (2e-3 if dtype == "bf16" and b * P_ >= 2048 else 1e-12), d
