"""The fp32 kernels at the edges of their tiles: the projection GEMM in every
tiling, with ragged rows, columns and K and pointers that are only 4-byte
aligned, and the attention over ragged rows and keys, with values that a row
does not see set to infinity.  Every case prints its sizes first."""
import sys

import numpy as np
import pytest
import torch

from oracle import dard_oracle as O
from paper_2608_26574_amd import dard, synth

pytestmark = pytest.mark.gpu


def announce(*a):
    print("[case]", *a, file=sys.stderr, flush=True)


# tiles of 16 (K split over 4 or 16 waves), 32 and 64 rows and columns
@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (33, 100, 68), (17, 52, 1028), (130, 516, 260), (520, 2060, 132)])
@pytest.mark.parametrize("shift", [0, 1])
def test_linear_f32_tiles(M, N, K, shift):
    announce("linear f32", M, N, K, shift)
    g = torch.Generator().manual_seed(M + N)
    X, W = torch.randn(M, K, generator=g), torch.randn(N, K, generator=g)
    xb = torch.empty(M * K + 4, device="cuda")
    xd = xb[shift:shift + M * K].view(M, K)
    xd.copy_(X)
    Wp = torch.empty_like(W).cuda()
    dard.dard_pack_matrix(W.cuda(), Wp)
    Y = torch.full((M, N), float("nan"), device="cuda")
    dard.dard_linear(xd, Wp, N, Y)
    torch.cuda.synchronize()
    x, w = X.double().numpy(), W.double().numpy()
    # fp32 products summed in fp32: at most K roundings of 2^-24 of the sum of magnitudes
    err = np.abs(Y.cpu().double().numpy() - x @ w.T) / (np.abs(x) @ np.abs(w).T)
    assert err.max() < min(K, 64) * 2.0 ** -24, err.max()


@pytest.mark.parametrize("b,B,P,Hq,Hkv,dh", [(1, 1, 0, 2, 2, 64), (2, 7, 3, 4, 2, 64), (1, 24, 101, 6, 2, 128),
                                             (3, 16, 33, 2, 1, 128), (1, 65, 191, 4, 4, 64)])
@pytest.mark.parametrize("unseen", [None, "inf", "nan"])
def test_attention_f32_edges(b, B, P, Hq, Hkv, dh, unseen):
    announce("attention f32", b, B, P, Hq, Hkv, dh, unseen)
    cap = P + 2 * B + 3
    g = torch.Generator().manual_seed(B * 5 + P)
    q = torch.randn(b, 2 * B, Hq, dh, generator=g)
    k = torch.randn(b, Hkv, cap, dh, generator=g)
    v = torch.randn(b, Hkv, dh, cap, generator=g)
    _, state, conf = synth.tiny_block(b, B, 2048, seed=3)
    flags = 0
    see = np.ones((b, 2 * B, P + 2 * B), dtype=bool)
    for s in range(b):
        for r in range(2 * B):
            i, shadow = r % B, r >= B
            for j in range(B):
                si, sj = state[s, i], state[s, j]
                if si == O.STATE_U:
                    t = sj == O.STATE_U and not (i == j and shadow)
                elif si == O.STATE_C:
                    t = (sj == O.STATE_U or (sj == O.STATE_C and conf[s, i] <= conf[s, j])) and not (i == j and shadow)
                else:
                    t = sj == O.STATE_U if shadow else True
                see[s, r, P + j], see[s, r, P + B + j] = t, not t
    if unseen:
        # one block key that some row does not see: its value must reach only the rows that do
        key = P + int(np.argmax((~see[:, :, P:]).any(axis=(0, 1))))
        v[:, :, :, key] = float(unseen)
    out = torch.zeros(b, 2 * B, Hq, dh, device="cuda")
    dard.dard_masked_attention(q.cuda(), k.cuda(), v.cuda(), P, torch.from_numpy(state).cuda(),
                               torch.from_numpy(conf).cuda(), dh ** -0.5, flags, out)
    torch.cuda.synchronize()
    got = out.cpu().double()
    for h in range(Hq):
        hk = h // (Hq // Hkv)
        sc = torch.einsum("brd,bkd->brk", q[:, :, h].double(), k[:, hk, :P + 2 * B].double()) * dh ** -0.5
        sc = sc.masked_fill(~torch.from_numpy(see), -float("inf"))
        p = torch.softmax(sc, -1)
        for s in range(b):
            for r in range(2 * B):
                keys = np.flatnonzero(see[s, r])
                ref = v[s, hk][:, keys].double() @ p[s, r, keys]
                if unseen and key in keys:
                    assert not torch.isfinite(got[s, r, h]).any()
                else:
                    # scores, probabilities and sums in fp32: a few 2^-24 of values of order one
                    assert (got[s, r, h] - ref).abs().max() < 1e-5, (s, r, h)


@pytest.mark.parametrize("B,P", [(1, 0), (7, 160), (24, 101)])
def test_attention_f32_infinite_scores(B, P):
    """Keys whose score is minus infinity take no weight, also where a whole key
    tile holds nothing else; a row that sees only such keys has no softmax (NaN)."""
    announce("attention f32, scores of minus infinity", B, P)
    b, Hq, dh, n = 2, 2, 64, P + 2 * B
    g = torch.Generator().manual_seed(B + P)
    q, k, v = torch.randn(b, 2 * B, Hq, dh, generator=g), torch.randn(b, Hq, n, dh, generator=g), \
        torch.randn(b, Hq, dh, n, generator=g)
    q[..., 0] = q[..., 0].abs() + 0.1
    if P:
        k[0, :, 32:P, 0] = -float("inf")       # whole tiles of the first sequence ...
    k[1, :, :, 0] = -float("inf")              # ... and every key of the second
    # all positions U: a row reads every x key (a shadow row its own shadow key instead)
    state = np.full((b, B), O.STATE_U, dtype=np.uint8)
    conf = np.full((b, B), 0.95, dtype=np.float32)
    see = torch.ones(2 * B, n, dtype=torch.bool)
    see[:, P + B:] = False
    for i in range(B):
        see[B + i, P + i], see[B + i, P + B + i] = False, True
    out = torch.zeros(b, 2 * B, Hq, dh, device="cuda")
    dard.dard_masked_attention(q.cuda(), k.cuda(), v.cuda(), P, torch.from_numpy(state).cuda(),
                               torch.from_numpy(conf).cuda(), dh ** -0.5, 0, out)
    torch.cuda.synchronize()
    sc = torch.matmul(q.double().transpose(1, 2), k.double().transpose(-1, -2).contiguous()) * dh ** -0.5
    p = torch.softmax(sc.masked_fill(~see, -float("inf")), -1)
    ref = torch.matmul(p, v.double().transpose(-1, -2).contiguous()).transpose(1, 2)
    assert torch.isnan(out[1]).all() and torch.isnan(ref[1]).all()
    # scores, probabilities and sums in fp32: a few 2^-24 of values of order one
    assert (out[0].cpu().double() - ref[0]).abs().max() < 1e-5


def test_attention_f32_very_many_sequences():
    """More rows of heads than one launch takes (2^23 workgroups): blocks of one
    position and no prefix, where a U token's x row reads its own x key and its
    shadow row its shadow key, so that every row is one of the V vectors."""
    b, Hq, dh = (1 << 19) + 3, 32, 64          # 2^32 threads in one launch; 8.6 GB of queries
    announce("attention f32, sequences", b)
    g = torch.Generator(device="cuda").manual_seed(1)
    q = torch.randn(b, 2, Hq, dh, generator=g, device="cuda")
    k = torch.randn(b, 1, 2, dh, generator=g, device="cuda")
    v = torch.randn(b, 1, dh, 2, generator=g, device="cuda")
    state = torch.full((b, 1), O.STATE_U, dtype=torch.uint8, device="cuda")
    conf = torch.full((b, 1), 0.95, device="cuda")
    out = torch.zeros_like(q)
    dard.dard_masked_attention(q, k, v, 0, state, conf, dh ** -0.5, 0, out)
    ref = v.transpose(2, 3)[:, 0, :, None].expand(b, 2, Hq, dh)
    assert torch.equal(out, ref)
