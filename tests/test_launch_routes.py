"""What the library launches, on the CPU: a small C library takes the place of
hipExtLaunchKernel (every kernel start of libdard goes through it) and writes
down each kernel's name and grid and, for the tiled GEMM, its sizes.  Nothing
runs and no pointer is followed, so the tile, the K split and the order of a
forward's launches can be compared with what dard_gemm_plan reports."""
import json
import os
import re
import subprocess
import sys

import pytest

from paper_2608_26574_amd import dard

STAND_IN = r"""
#include <stdio.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void* f; const char* name; } known[4096];
static int n_known;
void __hipRegisterFunction(void** m, const void* f, char* dev, const char* name, unsigned t, void* a, void* b,
                           void* c, void* d, int* w) {
    if (n_known < 4096) { known[n_known].f = f; known[n_known++].name = name; }
}
int hipExtLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t lds, void* s, void* e0, void* e1, int fl) {
    const char* name = "?";
    for (int i = 0; i < n_known; ++i) if (known[i].f == f) name = known[i].name;
    int M = 0, K = 0, N = 0, kind = 0;
    if (strstr(name, "gemm_big_bf16")) { M = *(int*)args[1]; K = *(int*)args[2]; N = *(int*)args[4]; kind = *(int*)args[5]; }
    if (strstr(name, "gemm_stream_bf16")) { M = *(int*)args[1]; K = *(int*)args[2]; N = *(int*)args[5]; kind = *(int*)args[6]; }
    printf("[\"%s\", %u, %u, %u, %d, %d, %d, %d]\n", name, g.x, g.y, b.x, kind, M, N, K);
    return 0;
}
int hipGetLastError(void) { return 0; }
"""

# one prefill of one layer per line of the input (rows, d, ffn), or one step of no
# layer (sequences, block, d, vocabulary)
PROGRAM = r"""
import ctypes, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
L.dard_workspace_bytes.restype = ctypes.c_size_t
fake = ctypes.c_void_p(1 << 20)
class Params(ctypes.Structure):
    _fields_ = [("tau_c", ctypes.c_float), ("tau_u", ctypes.c_float), ("lambda_", ctypes.c_double),
                ("p0", ctypes.c_double), ("mask_id", ctypes.c_int32), ("flags", ctypes.c_uint32),
                ("w_fixed", ctypes.c_float)]
for line in sys.stdin:
    v = list(map(int, line.split()))
    step = len(v) == 4
    d, F, V = (v[2], 64, v[3]) if step else (v[1], v[2], 1040)
    dims = (ctypes.c_int32 * 12)(0 if step else 1, d, d // 128, max(1, d // 256), 128, F, V, 1 << 20, 1)
    ctypes.cast(dims, ctypes.POINTER(ctypes.c_float))[10] = 1e4
    if step:
        b, B = v[:2]
        params = Params(0.4, 0.9, 0.5, 0.1, V - 1, 0, 0.0)
        ws = L.dard_workspace_bytes(dims, b, B, 2 * B)
        rc = L.dard_step(dims, fake, fake, 2 * B, 0, ctypes.byref(params), b, B, *[fake] * 7, None, fake,
                         ctypes.c_size_t(ws), None)
    else:
        M = v[0]
        ws = L.dard_workspace_bytes(dims, 1, 1, M + 2)
        rc = L.dard_prefill(dims, fake, fake, M + 2, 1, M, fake, None, fake, ctypes.c_size_t(ws), None)
    ctypes.CDLL(None).fflush(None)
    print("end", rc, flush=True)
"""

STORE, RESID, SWIGLU, QKV, PARTIAL, LMHEAD = range(6)


@pytest.fixture(scope="module")
def forwards(tmp_path_factory):
    """cases, prefills (M, d, F) or steps (b, B, d, V) -> per case the launches
    (kernel, grid x, y, threads, kind, M, N, K)."""
    folder = tmp_path_factory.mktemp("standin")
    src, so = folder / "standin.c", folder / "standin.so"
    src.write_text(STAND_IN)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", "-o", str(so), str(src)], check=True)

    def run(cases):
        r = subprocess.run([sys.executable, "-c", PROGRAM, str(so), os.path.abspath(dard.LIB_PATH)],
                           input="".join(" ".join(map(str, c)) + "\n" for c in cases), capture_output=True, text=True,
                           timeout=120)
        assert r.returncode == 0, r.stderr
        out, cur = [], []
        for line in r.stdout.splitlines():
            if line.startswith("end"):
                assert line == "end 0", line
                out.append(cur)
                cur = []
            else:
                cur.append(json.loads(line))
        assert len(out) == len(cases)
        return out

    return run


def tile(launch):
    """(rows / 32, columns / 32, K split) of a launch of the tiled GEMM: template
    arguments TI, TJ, WM give 16 TI WM rows and 64 TJ columns."""
    ti, tj, wm = map(int, re.search(r"gemm_big_bf16ILi(\d+)ELi(\d+)ELi(\d+)E", launch[0]).groups())
    return ti * wm // 2, 2 * tj, launch[2]


# the projections of 4096 and 3584 wide models over row counts on both sides of
# every change of tile, K too short for a split, and full sums on 256 x 192 tiles
# (2560 x 4096 x 12288, 8192 x 4096 x 4096, 700 x 320 x 8192), one round of 256 x 128
# (1537 to 2048 rows of 4096 columns, 1793 to 2304 of 3584)
CASES = [(M, d, F) for d, F in ((4096, 12288), (3584, 18944), (1024, 4160))
         for M in (65, 97, 160, 255, 256, 300, 651, 1000, 1536, 1537, 2048, 2049, 2100, 2304, 2305, 2560, 2816, 3000, 3500, 4096, 5000, 6000, 8192,
                   16000)] + [(700, 8192, 320), (700, 512, 128)]


def test_tiles_that_run_are_the_tiles_of_the_plan(forwards):
    full_256 = one_round = 0
    for (M, d, F), launches in zip(CASES, forwards(CASES)):
        gemms = [x for x in launches if "gemm_big_bf16" in x[0]]
        assert len(gemms) == 4, (M, d, F, launches)   # QKV, O, gate/up, down
        for x, (N, K, kinds) in zip(gemms, (((d // 128 + 2 * max(1, d // 256)) * 128, d, (QKV,)), (d, d, (RESID, PARTIAL)),
                                            (2 * F, d, (SWIGLU,)), (d, F, (RESID, PARTIAL)))):
            assert x[5:] == [M, N, K] and x[4] in kinds, (M, d, F, x)
            plan = dard.dard_gemm_plan(M, N, K, partial=x[4] in (RESID, PARTIAL))
            assert tile(x) == plan[1:], (M, N, K, x[0], plan)
            assert (x[4] == PARTIAL) == (x[4] in (RESID, PARTIAL) and plan[3] > 1), (M, N, K, x, plan)
            full_256 += x[4] == RESID and tile(x) == (8, 6, 1)
            if tile(x)[:2] == (8, 4):
                assert x[4] == RESID and x[1] <= 256, (M, d, F, x)
                one_round += 1
            # exactly a round of 256 x 128 tiles: two rounds of 128 x 128 took longer
            assert (M, N, x[4]) != (2048, 4096, RESID) or tile(x) == (8, 4, 1), (K, x)
    # the full sums on 256 x 192 and 256 x 128 tiles are among the cases
    assert full_256 >= 3 and one_round >= 6


def test_streaming_tiles_that_run_are_the_tiles_of_the_plan(forwards):
    cases = [(M, d, F) for M in (1, 17, 64) for d, F in ((512, 1088), (4096, 12288), (384, 512), (1024, 960))]
    for (M, d, F), launches in zip(cases, forwards(cases)):
        gemms = [x for x in launches if "gemm_stream_bf16" in x[0]]
        assert len(gemms) == 4
        for x in gemms:
            plan = dard.dard_gemm_plan(x[5], x[6], x[7], partial=x[4] in (RESID, PARTIAL))
            nw = int(re.search(r"gemm_stream_bf16ILi(\d+)E", x[0]).group(1))
            assert (nw, x[2]) == (plan[2], plan[3]), (M, d, F, x, plan)


def test_few_key_tiles_of_a_prefill_are_not_split(forwards):
    """Key splits of a prefix pass in bf16: rows (64-key tiles), heads and workgroups on
    both sides of the rule."""
    cases = {(449, 4096): 1, (512, 4096): 1, (640, 512): 1, (700, 512): 1, (705, 512): 3, (1024, 1024): 4,
             (769, 1024): 1, (833, 1024): 3, (1400, 1024): 1, (1473, 1024): 2, (1500, 1536): 1}
    for ((M, d), ns), launches in zip(cases.items(), forwards([(M, d, 512) for M, d in cases])):
        att = [x for x in launches if "attn_mfma_kernel" in x[0]]
        assert len(att) == 1 and att[0][2] == ns, (M, d, att)
        assert len([x for x in launches if "attn_combine_kernel" in x[0]]) == (ns > 1)


def test_partials_are_added_by_a_workgroup_per_row(forwards):
    """From 2048 rows a wave takes a row of the norms that add no partials; those
    that add them keep a workgroup per row at every row count."""
    cases = [(2047, 4096, 12288), (2048, 1024, 4160), (2100, 4096, 12288), (2304, 3584, 18944), (3584, 4096, 12288)]
    split = 0
    for (M, d, F), launches in zip(cases, forwards(cases)):
        for x, norm in zip(launches, launches[1:]):
            if "gemm_big_bf16" not in x[0] or x[4] not in (RESID, PARTIAL) or "norm" not in norm[0]:
                continue
            by_wave = x[4] == RESID and M >= 2048
            assert ("resid_norm_rows_kernel" in norm[0]) == by_wave, (M, d, F, x, norm)
            assert norm[1] == (-(-M // 8) if by_wave else M)
            split += x[4] == PARTIAL and M >= 2048
    assert split >= 2


# listed rows (b * 2B) on both sides of every tile height
HEADS = [(2, 18), (3, 16), (2, 25), (2, 32), (3, 22), (2, 36), (5, 16), (3, 32), (7, 16), (4, 32), (3, 64), (16, 32),
         (8, 64)]


@pytest.mark.parametrize("d,V", [(4096, 126464), (3584, 152064), (512, 2048)])
def test_lm_head_holds_every_count_in_one_row_tile_up_to_192_rows(forwards, d, V):
    """The number of rows that the head runs over is known on the device only; at
    the first step of a block it is all of them."""
    for (b, B), launches in zip(HEADS, forwards([(b, B, d, V) for b, B in HEADS])):
        heads = [x for x in launches if "gemm_big_bf16" in x[0]]
        assert len(heads) == 1 and heads[0][4:] == [LMHEAD, 2 * b * B, V, d], launches
        ti, tj, split = tile(heads[0])
        row_tiles, col_tiles = -(-2 * b * B // (32 * ti)), -(-V // (32 * tj))
        assert heads[0][1] == row_tiles * col_tiles and split == 1
        if 2 * b * B <= 192 and V > 100000:
            assert row_tiles == 1, (b, B, ti, tj)
        # partials come from the head's epilogue (tiles of 128 columns or more) from 256 rows
        merges = [x for x in launches if "lm_merge_kernel" in x[0]]
        assert len(merges) == (2 * b * B >= 256) and (not merges or tj >= 4)
