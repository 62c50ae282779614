"""Isolated attention where the launch shape or the copy path changes: key
splits of grouped-query heads (fewest and most tiles, ragged ends, the largest
split count) and FP8 caches whose tiles take the straight-line copies, or only
some of them.  Tolerances as for the other attention cases: probabilities and
outputs are bf16 values of order one."""
import pytest

from test_gpu_ops import _attn_case, _attn_case_fp8, announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,B,P,Hq,Hkv,dh", [
    (1, 32, 384, 28, 4, 128),     # 7 tiles: not split
    (1, 32, 400, 28, 4, 128),     # 8 tiles, ragged prefix end: not split
    (1, 32, 650, 28, 4, 128),     # 12 tiles, ragged prefix end: the shortest split
    (4, 32, 760, 28, 4, 128),     # 64 workgroups, 13 tiles: not split
    (3, 64, 1390, 28, 4, 128),    # 84 workgroups, 24 tiles: the shortest split there
    (2, 24, 1000, 28, 4, 128),    # ragged block tile in the last split
    (1, 16, 4100, 14, 2, 128),    # 66 tiles: the largest split count
    (4, 64, 700, 8, 2, 64),       # head_dim 64
    (1, 256, 900, 4, 1, 128),     # maximum block
])
def test_attention_gqa_split(b, B, P, Hq, Hkv, dh):
    announce("attention gqa split", b, B, P, Hq, Hkv, dh)
    assert _attn_case(b, B, P, Hq, Hkv, dh, "bf16", 0.25, seed=4) < 2e-2


@pytest.mark.parametrize("b,B,P,Hq,Hkv,dh,extra", [
    (2, 32, 512, 4, 4, 128, 0),    # every full tile aligned
    (16, 32, 320, 16, 16, 128, 8),
    (1, 32, 100, 8, 8, 128, 4),    # aligned prefix tiles, block tiles off by four keys
    (2, 20, 333, 4, 2, 64, 3),     # no row aligned
    (1, 32, 900, 28, 4, 128, 4),   # grouped heads, split
])
def test_attention_fp8_copies(b, B, P, Hq, Hkv, dh, extra):
    announce("attention fp8 copies", b, B, P, Hq, Hkv, dh, extra)
    assert _attn_case_fp8(b, B, P, Hq, Hkv, dh, 0.25, seed=8, cap_extra=extra) < 2e-2
