"""Projection GEMMs of a prefill over the tilings that the row count selects,
with ragged last tiles in both directions, against the same two layers in
float64 (plain torch).  Every case prints its name and sizes before touching
the GPU and asserts the tiling that it is there to cover."""
import sys

import pytest
import torch

from paper_2608_26574_amd import dard, synth

pytestmark = pytest.mark.gpu


def reference_kv(w, dims, ids):
    """K (natural dim order) and V of every layer, [L][b][P][Hkv][dh], in float64."""
    b, P = ids.shape
    dh, half = dims.head_dim, dims.head_dim // 2
    pos = torch.arange(P, device="cuda").double()
    ang = pos[:, None] * dims.rope_theta ** (-torch.arange(half, device="cuda").double() / half)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def rope(x):
        a, z = x[..., :half], x[..., half:]
        return torch.cat([a * cos - z * sin, z * cos + a * sin], -1)

    def norm(h, gain):
        return h / torch.sqrt((h * h).mean(-1, keepdim=True) + dims.norm_eps) * gain.double()

    h = w["embed"][ids.long()].double()
    ks, vs = [], []
    for layer in range(dims.n_layers):
        W = lambda n: w[f"layers.{layer}.{n}"].double()   # noqa: B023,E731
        x = norm(h, W("attn_norm"))
        q = rope((x @ W("wq").T).view(b, P, -1, dh))
        k = rope((x @ W("wk").T).view(b, P, -1, dh))
        v = (x @ W("wv").T).view(b, P, -1, dh)
        ks.append(k)
        vs.append(v)
        group = dims.n_heads // dims.n_kv_heads
        out = torch.empty_like(q)
        for s in range(b):
            for head in range(dims.n_heads):
                sc = q[s, :, head] @ k[s, :, head // group].T.contiguous() * dh ** -0.5
                out[s, :, head] = torch.softmax(sc, -1) @ v[s, :, head // group]
        h = h + out.reshape(b, P, -1) @ W("wo").T
        x = norm(h, W("ffn_norm"))
        h = h + (torch.nn.functional.silu(x @ W("w_gate").T) * (x @ W("w_up").T)) @ W("w_down").T
    return torch.stack(ks), torch.stack(vs)


@pytest.mark.parametrize("b,P,d,F,gu,down", [
    (1, 65, 512, 1088, (1, 2, 2, 1), (1, 2, 2, 2)),   # 64 x 64; 64 x 64, 2 splits
    (1, 97, 2048, 8256, (1, 4, 4, 1), (1, 2, 2, 4)),   # 128 x 128; 64 x 64, 4 splits
    (3, 41, 1024, 12288, (1, 4, 4, 1), (1, 2, 2, 8)),   # 128 x 128; 64 x 64, 8 splits
    (1, 150, 4096, 4096, (1, 4, 2, 1), (1, 3, 4, 4)),   # 128 x 64; 96 x 128, 4 splits
    (1, 160, 4096, 12288, (1, 6, 4, 1), (1, 3, 4, 4)),   # 192 x 128; 96 x 128, 4 splits
    (3, 83, 1024, 9472, (1, 4, 6, 1), (1, 4, 2, 8)),   # 128 x 192; 128 x 64, 8 splits
    (1, 255, 3584, 18944, (1, 4, 6, 1), (1, 4, 4, 4)),   # 128 x 192; 128 x 128, 4 splits
    (1, 257, 512, 1088, (2, 2, 2, 1), (2, 2, 2, 2)),   # 64 x 64; 64 x 64, 2 splits
    (1, 385, 512, 4160, (2, 4, 6, 1), (2, 2, 2, 4)),   # 128 x 192; 64 x 64, 4 splits
    (3, 171, 512, 5120, (2, 6, 4, 1), (2, 2, 2, 3)),   # 192 x 128; 64 x 64, 3 splits
    (1, 641, 2048, 4160, (2, 3, 4, 1), (2, 3, 4, 2)),   # 96 x 128; 96 x 128, 2 splits
    (1, 1000, 3584, 18944, (2, 4, 6, 1), (2, 8, 6, 3)),   # 128 x 192; 256 x 192, 3 splits
    (2, 2050, 1024, 4160, (2, 4, 6, 1), (2, 6, 4, 1)),   # 128 x 192; 192 x 128, one split
    (3, 683, 1024, 4160, (2, 4, 6, 1), (2, 6, 4, 2)),   # 192 x 128, 2 splits, added at 2049 rows
    (3, 513, 4096, 2112, (2, 4, 4, 1), (2, 8, 4, 1)),   # 128 x 128; 256 x 128, one round and one split (O as well)
    (3, 683, 4096, 1088, (2, 6, 4, 1), (2, 8, 6, 1)),   # 192 x 128; 256 x 192, one split (O as well)
])
def test_prefill_tilings(b, P, d, F, gu, down):
    print("[case] prefill tilings", b, P, d, F, gu, down, file=sys.stderr, flush=True)
    assert tuple(dard.dard_gemm_plan(b * P, 2 * F, d)) == gu
    assert tuple(dard.dard_gemm_plan(b * P, d, F, partial=True)) == down
    dims = synth.Dims(2, d, d // 128, max(1, d // 256), 128, F, 1040, 4096, "bf16")
    w = synth.make_weights(dims, seed=5, device="cuda")
    ids = torch.from_numpy(synth.prompt_ids(b, P, dims.vocab, seed=6)).cuda()
    eng = dard.Engine(dims, w, b, 8, P + 16)
    eng.dard_prefill(ids)
    kc, vc = (t[:, :, :, :P].double().transpose(2, 3) for t in eng.kv_view(torch.bfloat16))
    kc = torch.cat([kc[..., 0::2], kc[..., 1::2]], -1)
    # a value of the second layer is behind about ten storage roundings of at
    # most 2^-9 (norms, Q / K / V, probabilities, attention, SwiGLU, twice): each
    # adds about 2^-9 / sqrt(3) to a row's relative 2-norm error, in all 4e-3; a row
    # that missed a k unit or came from another tile is off by 0.1 and more
    for got, ref in zip((kc, vc), reference_kv(w, dims, ids)):
        err = (got - ref).norm(dim=(-2, -1)) / ref.norm(dim=(-2, -1))   # [L][b][P]
        assert err.max().item() < 3e-2, err.max().item()
