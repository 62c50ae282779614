// Projection GEMMs Y = X * W^T (X [M][K] activations, W [N][K] weights) with
// fused epilogues:
//   STORE_F32  plain fp32 store (LM head logits, dard_linear)
//   RESID      fp32 residual add into the residual stream (O and down proj.)
//   SWIGLU     silu(gate) * up on interleaved gate/up rows, stored as dtype
//   QKV        rotary embedding on adjacent (t, t + dh/2) pairs, Q to its
//              buffer, K and V straight into the KV cache at the rows' keys
//              (K [cap][dh], V dims-major [dh][cap] per KV head)
//   PARTIAL    fp32 split-K partial [split][M][N], reduced by the consumer
//
// bf16 weights are packed fragment-major: the 16 x 64 block (row block nb,
// k unit u) is stored contiguously at element ((nb * K/64 + u) * 1024), as two
// halves of 512 (k 8h..8h+7 of each 16-wide group) in which lane l of a wave
// finds its 8 values at 8*l.  One 16-byte load per lane then reads exactly the
// A operand of v_mfma_f32_16x16x32_bf16 and a wave load is 1 KB contiguous;
// a wave streaming a row block over K reads one contiguous region.
//
// W is the A operand (16 output columns), X the B operand (16 tokens), so each
// lane ends with 4 consecutive output columns of one token.
//   gemm_stream: M <= 64 tokens (a decoding step).  Each wave owns 16*NW
//     columns; the KSPLIT waves of a workgroup take interleaved k units and are
//     summed in LDS in a fixed order; DEPTH units per wave are in flight in a
//     register ring.  Weights are read with non-temporal loads (streamed once).
//     Optional split of K across SPLIT workgroups writes fp32 partials.
//   gemm_big: M > 64 with fragment-major X, tiles of 64 x 64 to 256 x 192, X
//     through LDS, the weights straight to registers.
//   gemm_tiled: row-major X (dard_linear), 128 x 128 tiles through LDS.
#include "common.h"
#include "launch.h"

namespace dard {

namespace {

template <typename T>
__device__ __forceinline__ void store4(T* p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
}
template <>
__device__ __forceinline__ void store4<bf16_t>(bf16_t* p, float a, float b, float c, float d) {
    const uint32_t w0 = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
    const uint32_t w1 = (uint32_t)f2bf(c) | ((uint32_t)f2bf(d) << 16);
    *reinterpret_cast<uint2*>(p) = make_uint2(w0, w1);
}

// Two adjacent values (p 2-element aligned): one 4- or 8-byte store.
template <typename T>
__device__ __forceinline__ void store2(T* p, float a, float b);
template <>
__device__ __forceinline__ void store2<float>(float* p, float a, float b) {
    *reinterpret_cast<float2*>(p) = make_float2(a, b);
}
template <>
__device__ __forceinline__ void store2<bf16_t>(bf16_t* p, float a, float b) {
    *reinterpret_cast<uint32_t*>(p) = (uint32_t)f2bf(a) | ((uint32_t)f2bf(b) << 16);
}

// x * sigmoid(x) with the hardware exp2 and reciprocal (about 1 ulp each):
// exp2 of a large argument is +inf and its reciprocal 0, so the limits hold.
__device__ __forceinline__ float silu(float x) {
    return x * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(x * -1.4426950408889634f));
}

// The epilogue kind is uniform over a launch; kernels branch on it once and
// run a loop specialised for it (Kind<k>), so a tile's epilogue carries no
// per-tile dispatch and no code of the other kinds.
template <int K>
struct Kind {
    static constexpr int value = K;
};

template <typename F>
__device__ __forceinline__ void with_kind(int kind, F&& f) {
    switch (kind) {
    case EPI_STORE_F32: f(Kind<EPI_STORE_F32>{}); break;
    case EPI_PARTIAL: f(Kind<EPI_PARTIAL>{}); break;
    case EPI_RESID: f(Kind<EPI_RESID>{}); break;
    case EPI_SWIGLU: f(Kind<EPI_SWIGLU>{}); break;
    case EPI_QKV: f(Kind<EPI_QKV>{}); break;
    case EPI_LMHEAD: f(Kind<EPI_LMHEAD>{}); break;
    default: break;
    }
}

// Row m of the QKV output: sequence s, rotary position and cache index.
struct QkvRow {
    int s, pos, cidx;
};
__device__ __forceinline__ QkvRow qkv_row(const EpiArgs& e, int m) {
    const int s = m / e.rows_per_seq, r = m - s * e.rows_per_seq;
    if (e.step == 2)   // full sequence: the other positions, then the block's x and s rows
        return QkvRow{s, r < e.P ? (r < e.blk ? r : r + e.B) : e.blk + (r - e.P) % e.B, r};
    if (e.step == 3)   // positions after a shared prompt of P
        return QkvRow{s, e.P + r, e.P + r};
    return QkvRow{s, e.step ? e.P + (r % e.B) : r, e.step ? e.P + r : r};
}

// Epilogue for output columns n..n+3 (n % 4 == 0) of token row m, in two
// halves: epi_fetch loads what the epilogue reads (the residual, or the two
// rotary (cos, sin) pairs), epi_store combines and writes.  A kernel that
// owns several tiles fetches for all of them before its first store, so the
// loads overlap instead of each waiting behind the stores before it.  head_dim
// is 64 or 128, so dims and heads come from shifts.
template <int EK>
__device__ __forceinline__ float4 epi_fetch(const EpiArgs& e, int m, int n) {
    if constexpr (EK == EPI_RESID) return *reinterpret_cast<const float4*>(e.y + (size_t)m * e.ldy + n);
    if constexpr (EK == EPI_QKV) {
        const int qd = e.Hq * e.dh, kd = e.Hkv * e.dh;
        if (n < qd + kd) {
            const int ein = (n < qd ? n : n - qd) & (e.dh - 1);
            const float* t = e.rope + ((size_t)qkv_row(e, m).pos * (e.dh / 2) + ein / 2) * 2;
            const float2 c0 = *reinterpret_cast<const float2*>(t);
            const float2 c1 = *reinterpret_cast<const float2*>(t + 2);
            return make_float4(c0.x, c0.y, c1.x, c1.y);
        }
    }
    return make_float4(0.f, 0.f, 0.f, 0.f);
}

template <typename T, int EK>
__device__ __forceinline__ void epi_store(const EpiArgs& e, int m, int n, floatx4 v, float4 f) {
    if constexpr (EK == EPI_STORE_F32) {
        st_f4(e.y + (size_t)m * e.ldy + n, v);     // (dard_linear takes any float pointer)
    } else if constexpr (EK == EPI_PARTIAL) {
        *reinterpret_cast<float4*>(e.y + (size_t)m * e.ldy + n) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (EK == EPI_RESID) {
        *reinterpret_cast<float4*>(e.y + (size_t)m * e.ldy + n) =
            make_float4(f.x + v[0], f.y + v[1], f.z + v[2], f.w + v[3]);
    } else if constexpr (EK == EPI_SWIGLU) {
        // interleaved rows: (gate, up) pairs at (n, n+1) and (n+2, n+3)
        T* a = reinterpret_cast<T*>(e.act) + (e.act_frag ? frag_off(m, n / 2, e.ld_act) : (size_t)m * e.ld_act + n / 2);
        store2<T>(a, silu(v[0]) * v[1], silu(v[2]) * v[3]);
    } else if constexpr (EK == EPI_LMHEAD) {
        // a listed row of the LM head: stored at its logit row when its code says so
        const int code = e.rowmap[m];
        const size_t o = (size_t)(code & kLmRowMask) * e.ldy + n;
        if ((code & kLmStore) || e.store_all)
            *reinterpret_cast<float4*>(e.y + o) = make_float4(v[0], v[1], v[2], v[3]);
        if (e.y2) st_f4(e.y2 + o, v);              // (a captured-logits buffer off 16-byte alignment)
    } else if constexpr (EK == EPI_QKV) {
        const QkvRow row = qkv_row(e, m);
        const int qd = e.Hq * e.dh, kd = e.Hkv * e.dh;
        const int sh = e.dh == 128 ? 7 : 6;
        if (n < qd + kd) {
            // rotary pairs (v0, v1) and (v2, v3): natural dims (t, t + dh/2)
            const float a0 = v[0] * f.x - v[1] * f.y, b0 = v[1] * f.x + v[0] * f.y;
            const float a1 = v[2] * f.z - v[3] * f.w, b1 = v[3] * f.z + v[2] * f.w;
            if (n < qd) {
                store4<T>(reinterpret_cast<T*>(e.q) + (size_t)m * e.ldq + n, a0, b0, a1, b1);
            } else {
                const int nk = n - qd, kvh = nk >> sh, ein = nk & (e.dh - 1);
                const size_t ko = (((size_t)row.s * e.Hkv + kvh) * e.cap + row.cidx) * e.dh + ein;
                if (e.kv_fp8)
                    *reinterpret_cast<uint32_t*>(reinterpret_cast<uint8_t*>(e.kc) + ko) =
                        f2e4m3(a0) | (f2e4m3(b0) << 8) | (f2e4m3(a1) << 16) | (f2e4m3(b1) << 24);
                else
                    store4<T>(reinterpret_cast<T*>(e.kc) + ko, a0, b0, a1, b1);
            }
        } else {
            // the V cache is dims-major ([dh][cap] per KV head): four strided stores
            const int nv = n - qd - kd, kvh = nv >> sh, ein = nv & (e.dh - 1);
            const size_t vo = (((size_t)row.s * e.Hkv + kvh) * e.dh + ein) * e.cap + row.cidx;
            if (e.kv_fp8) {
                uint8_t* vc = reinterpret_cast<uint8_t*>(e.vc) + vo;
#pragma unroll
                for (int i = 0; i < 4; ++i) vc[(size_t)i * e.cap] = (uint8_t)f2e4m3(v[i]);
            } else {
                T* vc = reinterpret_cast<T*>(e.vc) + vo;
#pragma unroll
                for (int i = 0; i < 4; ++i) St<T>::st(vc + (size_t)i * e.cap, v[i]);
            }
        }
    }
}

// Rows of the launch whose results are kept: all M, or the device count of
// an LM-head launch over listed rows.
__device__ __forceinline__ int valid_rows(const EpiArgs& e, int M) {
    return e.rows_dev ? min(M, __builtin_amdgcn_readfirstlane(*e.rows_dev)) : M;
}

__device__ __forceinline__ bf16x8 ld_nt(const bf16_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(p));
}

// ---------------------------------------------------------------- streaming
template <int NW, int KSPLIT, int DEPTH, bool XF>
__global__ __launch_bounds__(64 * KSPLIT) void gemm_stream_bf16(const bf16_t* __restrict__ X, int M, int K, int ldx,
                                                               const bf16_t* __restrict__ W, int N, EpiArgs e) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, g = lane >> 4;
    const int nb0 = blockIdx.x * NW;
    const int KU = K / 64;
    // this workgroup's k units: [u_begin, u_end) of split blockIdx.y
    const int split = blockIdx.y, nsplit = gridDim.y;
    const int u_begin = (int)((long)KU * split / nsplit), u_end = (int)((long)KU * (split + 1) / nsplit);

    floatx4 acc[NW][4];
#pragma unroll
    for (int j = 0; j < NW; ++j)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) acc[j][mb] = floatx4{0.f, 0.f, 0.f, 0.f};

    const bf16_t* wp[NW];
#pragma unroll
    for (int j = 0; j < NW; ++j) wp[j] = W + (size_t)min(nb0 + j, N / 16 - 1) * KU * 1024 + 8 * lane;
    // X row-major: lane (lr, g) reads token 16mb+lr at k 64u + 16g + 8h; X
    // fragment-major: 1 KB block (mb, u), half h at +512h, lane at +8*lane.
    // Token blocks past the last one re-read it (their results are not stored).
    const bf16_t* xp[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
        xp[mb] = XF ? X + (size_t)min(mb, (M - 1) >> 4) * KU * 1024 + 8 * lane
                    : X + (size_t)min(16 * mb + lr, M - 1) * ldx + 16 * g;
    constexpr int xu = XF ? 1024 : 64, xh = XF ? 512 : 8;   // element steps per k unit / half

    bf16x8 wb[DEPTH][NW][2], xb[DEPTH][4][2];
    auto load = [&](int s, int u) {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            wb[s][j][0] = ld_nt(wp[j] + (size_t)u * 1024);
            wb[s][j][1] = ld_nt(wp[j] + (size_t)u * 1024 + 512);
        }
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
            xb[s][mb][0] = ld_bf16x8(xp[mb] + (size_t)xu * u);
            xb[s][mb][1] = ld_bf16x8(xp[mb] + (size_t)xu * u + xh);
        }
    };
#pragma unroll
    for (int s = 0; s < DEPTH; ++s) {
        const int u = u_begin + wave + s * KSPLIT;
        if (u < u_end) load(s, u);
    }
    for (int base = u_begin + wave; base < u_end; base += DEPTH * KSPLIT) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
            const int u = base + s * KSPLIT;
            if (u < u_end) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int j = 0; j < NW; ++j)
#pragma unroll
                        for (int mb = 0; mb < 4; ++mb) acc[j][mb] = mfma16x16x32(wb[s][j][h], xb[s][mb][h], acc[j][mb]);
                const int un = u + DEPTH * KSPLIT;
                if (un < u_end) load(s, un);
            }
        }
    }

    // Sum the KSPLIT partial tiles through LDS in wave order; wave w then
    // finishes token blocks [NQ w, NQ (w + 1)) so the epilogue runs on every wave.
    static_assert(4 % KSPLIT == 0, "KSPLIT divides the 4 token blocks");
    constexpr int NQ = 4 / KSPLIT;
    const int mb0 = wave * NQ;
    floatx4 res[NW][NQ];
    if constexpr (KSPLIT > 1) {
        __shared__ floatx4 red[KSPLIT][NW * 4][64];
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int mb = 0; mb < 4; ++mb) red[wave][j * 4 + mb][lane] = acc[j][mb];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                floatx4 t = red[0][j * 4 + mb0 + q][lane];
#pragma unroll
                for (int w = 1; w < KSPLIT; ++w) t += red[w][j * 4 + mb0 + q][lane];
                res[j][q] = t;
            }
    } else {
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int q = 0; q < NQ; ++q) res[j][q] = acc[j][q];
    }
    EpiArgs ee = e;
    if (e.kind == EPI_PARTIAL) ee.y = e.y + (size_t)split * M * e.ldy;
    const int Mv = valid_rows(e, M);
    with_kind(e.kind, [&](auto kind) {
        constexpr int EK = decltype(kind)::value;
        float4 pre[NW][NQ];
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int n = 16 * (nb0 + j) + 4 * g, m = 16 * (mb0 + q) + lr;
                pre[j][q] = (m < Mv && n < N) ? epi_fetch<EK>(ee, m, n) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
        for (int j = 0; j < NW; ++j)
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const int n = 16 * (nb0 + j) + 4 * g, m = 16 * (mb0 + q) + lr;
                if (m < Mv && n < N) epi_store<bf16_t, EK>(ee, m, n, res[j][q], pre[j][q]);
            }
    });
}

// ---------------------------------------------------------------- tiles
// M > 64 with fragment-major X.  A workgroup of
// 4 WM waves (WM x 4) owns a (16 TI WM)-token x (64 TJ)-column output tile; wave
// (wm, wn) computes 16 TI tokens x 16 TJ columns.
// What bounds such a tile is the traffic behind the MFMAs.  With both operands
// staged in LDS a 256 x 128 tile moved 72 KB through LDS (copies in and operand
// reads) per 512 MFMA cycles of the CU, 144 bytes per cycle where LDS serves 128.  Here only
// X, which the four column waves share, goes through LDS (copied straight from
// global memory, NST 64-wide k units deep); a wave's weight blocks are its own,
// and fragment-major weights already are MFMA operands, so they are loaded into
// registers WD (two to four) units ahead and never touch LDS.  A 128 x 192 tile then moves
// 80 KB through LDS per 768 MFMA cycles (16 in, and 16 read by each of four waves:
// 107 bytes per cycle, still near that limit), its barrier is one per 64-wide unit,
// and three workgroups share a CU, so one's prologue, epilogue and barrier
// waits lie under the others' MFMAs.
// Measured on MI355X (8192 x 37888 x 3584, SwiGLU): 2160 us (1030 TFLOP/s) with
// both operands in LDS, 1610 us (1380 TFLOP/s) now; 8192 x 4608 x 3584: 300 ->
// 208 us.
// The X fragments of a unit are read in four chunks (half of the row blocks of
// one 32-wide half), each a chunk ahead of its MFMAs.
__device__ __forceinline__ void copy16_lds(__amdgpu_buffer_rsrc_t r, char* dst, int voff, uint32_t soff) {
#if __HIP_DEVICE_COMPILE__   // (the host pass does not know the builtin)
    typedef __attribute__((address_space(3))) void* lds_ptr;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr)dst, 16, voff, soff, 0, 0);
#endif
}

// The counted wait in the middle of unit u (see the K loop of gemm_big_bf16): vector
// memory operations that may stay outstanding there.  Copies between the one waited
// for and the wait, and in the unrolled loop 2 TJ of the weight loads between them; a
// tail unit's weight loads are dead code and dropped, so its wait counts none.
constexpr int mid_wait(bool tail, int TJ, int NST, int CPW) { return (NST - 2) * CPW + (tail ? 0 : 2 * TJ); }

// Whether no wait of a launch of nu units can leave the copy of unit u + 1 in
// flight: at least mid_wait operations are certain to be issued after that copy.
// Certain are the copies, the weight loads of the loop's units, and of the prologue's
// weight loads those whose slots units 0..u have used (the compiler may sink the
// others).
constexpr bool waits_cover(int TJ, int NST, int WD, int CPW, int nu) {
    const int loop_end = nu / WD * WD;
    for (int u = 0; u + 1 < nu; ++u) {
        const int c = u + 1 - NST;                 // the unit that copied unit u + 1 (below 0: the prologue)
        int issued = (NST - 2) * CPW;
        if (c < 0) issued += 2 * TJ * (u + 1 < WD ? u + 1 : WD);
        for (int t = c < 0 ? 0 : c; t <= u; ++t)   // half of unit c's follow its copy, half of unit u's come before its wait
            if (t < loop_end) issued += t == c || t == u ? TJ : 2 * TJ;
        if (issued < mid_wait(u >= loop_end, TJ, NST, CPW)) return false;
    }
    return true;
}
constexpr bool waits_cover_all(int TJ, int NST, int WD, int CPW) {
    for (int nu = 1; nu <= 4 * WD + NST; ++nu)     // the counts repeat from there on
        if (!waits_cover(TJ, NST, WD, CPW, nu)) return false;
    return true;
}

template <int TI, int TJ, int WM, int NST, int WD, int OCC>
__global__ __launch_bounds__(256 * WM) __attribute__((amdgpu_waves_per_eu(OCC, OCC)))
void gemm_big_bf16(const bf16_t* __restrict__ X, int M, int K, const bf16_t* __restrict__ W, int N, EpiArgs e,
                   int tiles_n) {
    constexpr int BM = 16 * TI * WM;
    constexpr int STAGE = TI * WM * 2048;          // LDS bytes of one 64-wide unit of the X tile
    constexpr int CPW = TI / 2;                    // 1 KB copies per wave per unit
    constexpr int CH = TI / 2;                     // X fragments per chunk
    static_assert(TI % 2 == 0 && NST >= 3, "whole chunks; the wait counts below need three stages");
    static_assert((NST - 1) * CPW + 2 * TJ <= 63, "vmcnt range");
    static_assert(waits_cover_all(TJ, NST, WD, CPW), "a wait could leave the copy of the next unit in flight");
    static_assert(NST * STAGE >= WM * 4 * TI * 16 * 12, "the epilogue's row partials fit the stages");
    __shared__ __attribute__((aligned(16))) char smem[NST * STAGE];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const int lr = lane & 15, g = lane >> 4;
    // Tile order.  Only the row tiles that hold kept rows are dealt out (an
    // LM-head launch covers the largest possible count; tiles skipped in the
    // middle of the order would leave whole shader engines idle, since the
    // dispatcher deals workgroups to them in turn).  Workgroups go round-robin to
    // the 8 XCDs: each XCD gets a contiguous run of an order that walks groups
    // of 8 row tiles column by column, so the tiles in flight on an XCD form a
    // block that shares both its X rows and its weight panels in that L2.
    const int Mv = valid_rows(e, M);
    const int tiles_m = (Mv + BM - 1) / BM;
    const int total = tiles_m * tiles_n;
    if ((int)blockIdx.x >= total) return;
    const int xcd = blockIdx.x & 7;
    const int t = xcd * (total >> 3) + min(xcd, total & 7) + (int)(blockIdx.x >> 3);
    constexpr int GM = 8;
    const int grp = t / (GM * tiles_n), in = t - grp * GM * tiles_n;
    const int gm = min(GM, tiles_m - grp * GM);
    const int tm = grp * GM + in % gm, tn = in / gm;
    const int KU = K / 64, NB = N / 16, MB = (M + 15) / 16;
    const int split = blockIdx.y, nsplit = gridDim.y;
    const int u_begin = (int)((long)KU * split / nsplit), u_end = (int)((long)KU * (split + 1) / nsplit);
    const int nu = u_end - u_begin, last = nu - 1;

    // Loads go through buffer descriptors based at the tile, with scalar block
    // and unit offsets and one lane offset: few address registers, and the
    // compiler counts them exactly (global loads to LDS make it wait for every
    // load in flight before the first use of any).  Blocks past the matrix
    // re-read its last block and units past the range its last unit; neither
    // reaches a stored result.
    const int mb_first = tm * TI * WM, nb_first = tn * 4 * TJ;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(X + ((size_t)mb_first * KU + u_begin) * 1024), (short)0, -1, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(W + ((size_t)nb_first * KU + u_begin) * 1024), (short)0, -1, 0x00020000);
    const int voff = 16 * lane;
    uint32_t xo[CPW], wo[TJ];
#pragma unroll
    for (int j = 0; j < CPW; ++j) {
        const int c = wave * CPW + j;              // copy c of the stage: row block c / 2, half c % 2
        xo[j] = (uint32_t)min(c >> 1, MB - 1 - mb_first) * KU * 2048 + (c & 1) * 1024;
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) wo[j] = (uint32_t)min(wn * TJ + j, NB - 1 - nb_first) * KU * 2048;
    auto copy_x = [&](int u, int stage) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)min(u, last) * 2048;
        char* dst = smem + stage * STAGE + wave * CPW * 1024;
#pragma unroll
        for (int j = 0; j < CPW; ++j) copy16_lds(rx, dst + j * 1024, voff, xo[j] + off);
    };
    bf16x8 wf[WD][2][TJ];                          // [unit % WD][half][column block]
    auto load_w = [&](int u, int slot, int h) __attribute__((always_inline)) {
        const uint32_t off = (uint32_t)min(u, last) * 2048 + h * 1024;
#pragma unroll
        for (int j = 0; j < TJ; ++j)
            wf[slot][h][j] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rw, voff, wo[j] + off, 0));
    };

    floatx4 acc[TJ][TI];
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int i = 0; i < TI; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 xa[CH], xb[CH];
    auto read_x = [&](bf16x8 (&xf)[CH], int stage, int h, int i0) __attribute__((always_inline)) {
        const char* st = smem + stage * STAGE + wm * TI * 2048 + h * 1024 + 16 * lane;
#pragma unroll
        for (int i = 0; i < CH; ++i) xf[i] = *reinterpret_cast<const bf16x8*>(st + (i0 + i) * 2048);
    };
    auto mm = [&](const bf16x8 (&wv)[TJ], const bf16x8 (&xf)[CH], auto i0c) __attribute__((always_inline)) {
        constexpr int i0 = decltype(i0c)::value;
#pragma unroll
        for (int i = 0; i < CH; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j) acc[j][i0 + i] = mfma16x16x32(wv[j], xf[i], acc[j][i0 + i]);
#pragma unroll
        for (int q = 0; q < CH; ++q) {             // one LDS read behind every TJ MFMAs
            __builtin_amdgcn_sched_group_barrier(0x008, TJ, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };

    // Unit t lives in LDS stage t % NST and register slot t % WD.  In the middle
    // of unit t, once every wave has read the last chunk of stage t into
    // registers, the barrier also publishes stage t + 1; unit t + NST is then
    // copied over stage t.  Copies complete in issue order, so stage t + 1 has
    // arrived when at most the (NST - 2) CPW copies issued after it are
    // outstanding, plus the weight loads issued after it: 2 (NST - 1) TJ of
    // them in the loop.  The waits count only 2 TJ, and none in the prologue, from
    // where the compiler may sink weight loads, and in the tail units, whose weight
    // loads nothing uses, so that it drops them (mid_wait, waits_cover).
#pragma unroll
    for (int p = 0; p < NST; ++p) copy_x(p, p);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int p = 0; p < WD; ++p) {
        load_w(p, p, 0);
        load_w(p, p, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((NST - 1) * CPW));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read_x(xa, 0, 0, 0);
    int st0 = 0;
    auto unit = [&](int u, auto slotc, auto tailc) __attribute__((always_inline)) {
        constexpr int s = decltype(slotc)::value;
        constexpr bool tail = decltype(tailc)::value != 0;
        const int st1 = st0 + 1 == NST ? 0 : st0 + 1;
        read_x(xb, st0, 0, CH);
        mm(wf[s][0], xa, Kind<0>{});
        __builtin_amdgcn_sched_barrier(0);
        read_x(xa, st0, 1, 0);
        mm(wf[s][0], xb, Kind<CH>{});
        __builtin_amdgcn_sched_barrier(0);
        load_w(u + WD, s, 0);
        __builtin_amdgcn_sched_barrier(0);
        read_x(xb, st0, 1, CH);
        mm(wf[s][1], xa, Kind<0>{});
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(waitcnt_vm(mid_wait(tail, TJ, NST, CPW)));   // (and every LDS read)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        copy_x(u + NST, st0);
        read_x(xa, st1, 0, 0);
        mm(wf[s][1], xb, Kind<CH>{});
        __builtin_amdgcn_sched_barrier(0);
        load_w(u + WD, s, 1);
        __builtin_amdgcn_sched_barrier(0);
        st0 = st1;
    };
    int u = 0;
    for (; u + WD <= nu; u += WD) {
        unit(u, Kind<0>{}, Kind<0>{});
        if constexpr (WD > 1) unit(u + 1, Kind<1>{}, Kind<0>{});
        if constexpr (WD > 2) unit(u + 2, Kind<2>{}, Kind<0>{});
        if constexpr (WD > 3) unit(u + 3, Kind<3>{}, Kind<0>{});
    }
    if (u < nu) unit(u, Kind<0>{}, Kind<1>{});
    if constexpr (WD > 2) if (u + 1 < nu) unit(u + 1, Kind<1>{}, Kind<1>{});
    if constexpr (WD > 3) if (u + 2 < nu) unit(u + 2, Kind<2>{}, Kind<1>{});
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));     // no copy lands after this point

    EpiArgs ee = e;
    if (e.kind == EPI_PARTIAL) ee.y = e.y + (size_t)split * M * e.ldy;
    const int nb0 = nb_first + wn * TJ, m0 = tm * BM + wm * 16 * TI;
    with_kind(e.kind, [&](auto kind) {
        constexpr int EK = decltype(kind)::value;
#pragma unroll
        for (int ih = 0; ih < TI; ih += 2) {
            float4 pre[2][TJ];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int n = 16 * (nb0 + j) + 4 * g, m = m0 + 16 * (ih + i) + lr;
                    pre[i][j] = (m < Mv && n < N) ? epi_fetch<EK>(ee, m, n) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int n = 16 * (nb0 + j) + 4 * g, m = m0 + 16 * (ih + i) + lr;
                    if (m < Mv && n < N) epi_store<bf16_t, EK>(ee, m, n, acc[j][ih + i], pre[i][j]);
                }
        }
        if constexpr (EK == EPI_LMHEAD) {
            // fused confidence partials: per row, (max, first argmax, sum of
            // exp(l - max)) over the tile's columns (Eq. 1).  A lane's columns
            // of a row first, then its row's four lanes, then the four waves.
            if (!e.lpart) return;
            __builtin_amdgcn_s_barrier();          // every wave has read its last X fragments (and dropped the rest)
            float* red = reinterpret_cast<float*>(smem) + wave * TI * 16 * 3;
            constexpr float kL2e = 1.4426950408889634f;
#pragma unroll
            for (int i = 0; i < TI; ++i) {
                SmPart p{-INFINITY, 0x7fffffff, 0.f};
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int n = 16 * (nb0 + j) + 4 * g;
                    if (n < N) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (acc[j][i][q] > p.m) { p.m = acc[j][i][q]; p.a = n + q; }
                    }
                }
                // sum of exp2(l log2e - mb), mb = max log2e rounded once; its
                // rounding error, common to every term, is corrected at the end
                const float mb = p.m * kL2e;
#pragma unroll
                for (int j = 0; j < TJ; ++j) {
                    const int n = 16 * (nb0 + j) + 4 * g;
                    if (n < N) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) p.s += __builtin_amdgcn_exp2f(fmaf(acc[j][i][q], kL2e, -mb));
                    }
                }
                if (p.m != -INFINITY) p.s *= exp2f(-fmaf(p.m, kL2e, -mb));
#pragma unroll
                for (int o = 16; o < 64; o <<= 1) {
                    const SmPart y{__shfl_xor(p.m, o, 64), __shfl_xor(p.a, o, 64), __shfl_xor(p.s, o, 64)};
                    p = smpart_merge(p, y);
                }
                if (g == 0) {
                    red[(i * 16 + lr) * 3 + 0] = p.m;
                    red[(i * 16 + lr) * 3 + 1] = __int_as_float(p.a);
                    red[(i * 16 + lr) * 3 + 2] = p.s;
                }
            }
            __syncthreads();
            for (int r = tid; r < BM; r += 256 * WM) {
                const int m = tm * BM + r;
                if (m >= Mv) continue;
                const int w0 = r / (16 * TI) * 4, ro = r % (16 * TI);
                SmPart p{-INFINITY, 0x7fffffff, 0.f};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float* o = reinterpret_cast<const float*>(smem) + ((w0 + w) * TI * 16 + ro) * 3;
                    p = smpart_merge(p, SmPart{o[0], __float_as_int(o[1]), o[2]});
                }
                float* o = e.lpart + ((size_t)m * e.ntile + tn) * 3;
                o[0] = p.m;
                o[1] = __int_as_float(p.a);
                o[2] = p.s;
            }
        }
    });
}

// ---------------------------------------------------------------- tiled
constexpr int TBM = 128, TBN = 128, TBK = 64, TPAD = TBK + 8;

__global__ __launch_bounds__(256) void gemm_tiled_bf16(const bf16_t* __restrict__ X, int M, int K, int ldx,
                                                       const bf16_t* __restrict__ W, int N, EpiArgs e,
                                                       int tiles_m, int tiles_n) {
    __shared__ __attribute__((aligned(16))) bf16_t Ws[8 * 1024];      // 8 fragment blocks of one k unit
    __shared__ __attribute__((aligned(16))) bf16_t Xs[TBM * TPAD];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, g = lane >> 4;
    // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs, so give
    // each XCD a contiguous run of tiles (m fastest: tiles sharing a weight
    // panel then share that XCD's L2).
    const int total = tiles_m * tiles_n;
    int bid = blockIdx.x;
    if ((total & 7) == 0) bid = (bid & 7) * (total >> 3) + (bid >> 3);
    const int tm = bid % tiles_m, tn = bid / tiles_m;
    const int nb_base = tn * (TBN / 16), m0 = tm * TBM;
    const int wn = wave & 1, wm = wave >> 1;
    const int KU = K / 64, NB = N / 16;

    floatx4 acc[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};

    bf16x8 wr[4], xr[4];
    auto gload = [&](int u) {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int c = threadIdx.x + 256 * it;      // 16-byte chunk of the 16 KB tile
            const int nbl = c >> 7, off = c & 127;
            wr[it] = ld_bf16x8(W + ((size_t)min(nb_base + nbl, NB - 1) * KU + u) * 1024 + off * 8);
            const int row = c >> 3, c8 = c & 7;
            xr[it] = ld_bf16x8(X + (size_t)min(m0 + row, M - 1) * ldx + u * 64 + c8 * 8);
        }
    };
    auto sstore = [&]() {
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int c = threadIdx.x + 256 * it;
            *reinterpret_cast<bf16x8*>(&Ws[c * 8]) = wr[it];
            const int row = c >> 3, c8 = c & 7;
            *reinterpret_cast<bf16x8*>(&Xs[row * TPAD + c8 * 8]) = xr[it];
        }
    };
    gload(0);
    for (int u = 0; u < KU; ++u) {
        __syncthreads();
        sstore();
        __syncthreads();
        if (u + 1 < KU) gload(u + 1);
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            bf16x8 af[4], bfr[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                af[j] = *reinterpret_cast<const bf16x8*>(&Ws[(wn * 4 + j) * 1024 + hh * 512 + lane * 8]);
#pragma unroll
            for (int i = 0; i < 4; ++i)
                bfr[i] = *reinterpret_cast<const bf16x8*>(&Xs[(wm * 64 + 16 * i + lr) * TPAD + 16 * g + 8 * hh]);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[j][i] = mfma16x16x32(af[j], bfr[i], acc[j][i]);
        }
    }
    with_kind(e.kind, [&](auto kind) {
        constexpr int EK = decltype(kind)::value;
        float4 pre[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (nb_base + wn * 4 + j) + 4 * g, m = m0 + wm * 64 + 16 * i + lr;
                pre[j][i] = (m < M && n < N) ? epi_fetch<EK>(e, m, n) : make_float4(0.f, 0.f, 0.f, 0.f);
            }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int n = 16 * (nb_base + wn * 4 + j) + 4 * g, m = m0 + wm * 64 + 16 * i + lr;
                if (m < M && n < N) epi_store<bf16_t, EK>(e, m, n, acc[j][i], pre[j][i]);
            }
    });
}

// ---------------------------------------------------------------- fp32
// Row-major W and X on v_mfma_f32_16x16x4_f32 (fp32 products and sums).  A
// workgroup owns 16 MI tokens x 16 NJ columns; its KS waves take interleaved
// 16-wide k steps and are summed in LDS in wave order.  A lane's float4 of a step
// is the operand of four MFMAs (element e of lanes g = 0..3 is k = 4g + e on both
// sides), so nothing is staged.  fp32 models are small and their launches bound
// by latency: many small tiles and a short chain per wave.  One thread per four
// outputs walking K through LDS took 24 us at 64 x 2048 x 256 and 90 us at 64 x
// 256 x 1024, this 5.0 and 6.8 us.
template <int MI, int NJ, int KS>
__global__ __launch_bounds__(64 * KS) void gemm_f32(const float* __restrict__ X, int M, int K, int ldx,
                                                   const float* __restrict__ W, int N, EpiArgs e) {
    constexpr int U = MI > 1 ? 2 : 4;              // steps loaded together
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int lr = lane & 15, g = lane >> 4;
    const int m0 = blockIdx.y * 16 * MI, n0 = blockIdx.x * 16 * NJ;
    const int Mv = valid_rows(e, M);
    if (m0 >= Mv) return;                          // the whole row tile is past the kept rows
    const float *xp[MI], *wp[NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i) xp[i] = X + (size_t)min(m0 + 16 * i + lr, M - 1) * ldx;
#pragma unroll
    for (int j = 0; j < NJ; ++j) wp[j] = W + (size_t)min(n0 + 16 * j + lr, N - 1) * K;
    floatx4 acc[NJ][MI];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[j][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int steps = (K + 15) / 16;
    for (int s0 = wave; s0 < steps; s0 += KS * U) {
        floatx4 xv[U][MI], wv[U][NJ];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = 16 * (s0 + u * KS) + 4 * g;
            const int kc = min(k, K - 4);          // (K % 4 == 0)
            const bool in = k < K;
#pragma unroll
            for (int i = 0; i < MI; ++i) xv[u][i] = ld_f4(xp[i] + kc);
#pragma unroll
            for (int j = 0; j < NJ; ++j) wv[u][j] = ld_f4(wp[j] + kc);
#pragma unroll
            for (int i = 0; i < MI; ++i) xv[u][i] = in ? xv[u][i] : floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) wv[u][j] = in ? wv[u][j] : floatx4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int i = 0; i < MI; ++i) acc[j][i] = mfma16x16x4f(wv[u][j][q], xv[u][i][q], acc[j][i]);
    }
    __shared__ floatx4 red[KS][NJ * MI][64];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < MI; ++i) red[wave][j * MI + i][lane] = acc[j][i];
    __syncthreads();
    with_kind(e.kind, [&](auto kind) {
        constexpr int EK = decltype(kind)::value;
        for (int t = wave; t < NJ * MI; t += KS) {
            const int n = n0 + 16 * (t / MI) + 4 * g, m = m0 + 16 * (t % MI) + lr;
            if (m >= Mv || n >= N) continue;
            const float4 pre = epi_fetch<EK>(e, m, n);
            floatx4 v = red[0][t][lane];
#pragma unroll
            for (int w = 1; w < KS; ++w) v += red[w][t][lane];
            epi_store<float, EK>(e, m, n, v, pre);
        }
    });
}

// Fragment-major packing of a bf16 weight matrix (see the file comment), with
// an optional row permutation: mode 1 puts rotary pairs (t, t + dh/2) of each
// head on adjacent rows, mode 2 interleaves the rows of src0 (gate) and src1
// (up).  One thread per 16-byte piece.
__global__ void pack_frag_kernel(const bf16_t* __restrict__ src0, const bf16_t* __restrict__ src1,
                                 bf16_t* __restrict__ dst, int N, int K, int mode, int dh) {
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)N * K / 8;
    if (t >= total) return;
    const int KU = K / 64;
    const int lane = t & 63;
    const int h = (t >> 6) & 1;
    const size_t blk = t >> 7;                // (nb, u)
    const int u = blk % KU, nb = blk / KU;
    const int row = 16 * nb + (lane & 15);
    const int k0 = 64 * u + 16 * (lane >> 4) + 8 * h;
    const bf16_t* src;
    if (mode == 1) {
        const int head = row / dh, e = row % dh, tt = e / 2;
        src = src0 + (size_t)(head * dh + ((e & 1) ? tt + dh / 2 : tt)) * K;
    } else if (mode == 2) {
        src = ((row & 1) ? src1 : src0) + (size_t)(row / 2) * K;
    } else {
        src = src0 + (size_t)row * K;
    }
    *reinterpret_cast<bf16x8*>(dst + t * 8) = *reinterpret_cast<const bf16x8*>(src + k0);
}

}  // namespace

hipError_t launch_pack_frag(const void* src0, const void* src1, void* dst, int N, int K, int mode, int dh,
                            hipStream_t s) {
    const size_t total = (size_t)N * K / 8;
    launch(pack_frag_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       (const bf16_t*)src0, (const bf16_t*)src1, (bf16_t*)dst, N, K, mode, dh);
    return hipGetLastError();
}

// Configuration of the streaming kernel for one projection shape:
//   nw     16-column blocks per wave (wave tile 16*nw columns)
//   ks     waves per workgroup splitting K
//   depth  k units in flight per wave
//   split  workgroups splitting K (fp32 partials, reduced by the consumer)
// Chosen from measurements on MI355X at 64 tokens.  Every wave reads all 64
// token rows of its k units (8 KB per unit), so a wider wave tile amortises
// that over more weight columns: the widest of 8, 6, 4, 3 column blocks whose
// grid still covers the 256 CUs; otherwise the tile that fills the CUs most
// evenly, with 4 waves per workgroup.  The O and down projections, whose
// 4096-wide output has too few column tiles, split K 4 ways instead, with 4
// waves per workgroup splitting K again (3 k units in flight for the long K
// of the down projection).
struct StreamCfg {
    int nw, ks, depth, split;
};

StreamCfg stream_cfg(int N, int K, bool partial) {
    const int KU = K / 64;
    if (partial) {
        int S = 4;
        while (S > 1 && KU / S < 8) S /= 2;
        if (N % 64 == 0) return K > 4096 ? StreamCfg{4, 4, 3, S} : StreamCfg{4, 4, 2, S};
        return StreamCfg{1, 4, 2, S};
    }
    for (int c : {8, 6}) {
        if (N % (16 * c) == 0 && N / (16 * c) >= 256) return c == 8 ? StreamCfg{8, 2, 3, 1} : StreamCfg{6, 4, 3, 1};
    }
    int nw = 0;
    double best = -1.0;
    for (int c : {4, 3}) {
        if (N % (16 * c)) continue;
        const int grid = N / (16 * c);
        const double eff = (double)grid / (((grid + 255) / 256) * 256);
        if (eff > best + 1e-9) { best = eff; nw = c; }
    }
    if (nw == 0) nw = N % 32 == 0 ? 2 : 1;
    const int grid = N / (16 * nw);
    const int ks = grid <= 256 ? 4 : 2;
    const int depth = (nw == 3 && ks == 4) ? 3 : 2;
    return StreamCfg{nw, ks, depth, 1};
}

// Tile of the M > 64 kernel, by the time model below: a CU's tiles run side by
// side, so a launch computes for about as long as the CU with the most tiles,
// ceil(tiles / 256) times a tile's time (its work over the tile's rate plus a
// fixed part for prologue and epilogue), and reads the weights from HBM for
// 2 N K bytes / 5 TB/s + 4 us; the shorter of the two hides but for a third.
// Rates and fixed parts are fitted to a sweep on MI355X of 72 to 2048 rows over
// the projections of the 8B and 7B shapes, weights cold in cache (136 shapes; the
// pick is within 2 % of the best tile on average, and 17 % off at worst, 2048 x 4608 x
// 3584, where epilogues but the residual's leave the best one out).  No tile is best
// everywhere:
// 192 x 24576 x 4096 takes 55 us with 192 x 128 (71 with 128 x 128), 128 x 12288 x
// 4096 35 us with 96 x 128 (44 with 128 x 128), 96 x 4608 x 3584 18 us with 64 x 64
// (32 with 128 x 128), 1024 x 37888 x 3584 231 us with 128 x 192 (260 with 128 x
// 128), 1024 x 3584 x 18944 in three splits 114 us with 256 x 192 (127 with 192 x
// 128).  (Below 256 rows one 128 x 128 tile through a register ring and an LDS double
// buffer, two k units ahead, took 79, 50, 42 us for the first three.)
// Residual projections (O and down) may split K up to 4 ways, up to 8 below 256
// rows, at least 8 k units each; a split adds its partial's pass through the
// residual-norm kernel, about 4.4 bytes per nanosecond.  One list of tiles serves
// the decision, the partials and the full sum, so that what is priced is what runs.
// From 4096 rows, where one split fills the chip, full sums leave 256-row tiles out
// (8192 x 3584 x 18944: 914 us with 128 x 192, 1034 with 256 x 192; a prefill of 8192
// rows was 1.6 % slower with it); below, partials leave 128 x 192 out and full sums gain
// from 256 x 192 (2560 x 4096 x 12288: 221 us, 244 with 192 x 128) and, where one round
// of them covers the matrix, from 256 x 128 (2048 x 4096 x 4096: 71 us, 80 with 128 x
// 128 two to a CU; 1920 x 4096 x 12288: 187 and 206; 2304 x 3584 x 18944: 284 and 289;
// in a second round they lose, 3840 x 4096 x 12288: 364 us, 352 with 192 x 128, and their
// fixed part is set so that a short K leaves them out, 3328 x 2048 x 1088: 28 us and 27;
// with K = 2048 both take 40, with 8192 116 and 127).  Other epilogues leave 256 rows out: inside a step 128 x 192 was faster there (1024 x 37888 x
// 3584: 235 against 275 us), most of all for LM-head launches, whose row count the host
// does not know (320 of at most 1024 rows: 414 against 554 us); with fused partials
// those take tiles of 128 columns or more, the merge's limit.
struct BigCfg {
    int ti, tj, split;   // tile in units of 32 rows / columns
};
// resid: a residual projection, K split at most max_split ways.
BigCfg big_cfg(int M, int N, int K, bool resid, int max_split, bool fused_head) {
    struct Tile {
        int ti, tj;
        double rate, fixed_us;   // multiply-adds per microsecond and CU in millions; per tile
    };
    const Tile cand[8] = {{4, 6, 2.8, 5.0}, {6, 4, 2.8, 6.0}, {4, 4, 2.4, 4.0}, {3, 4, 2.0, 4.5},
                          {4, 2, 1.6, 2.0}, {2, 2, 1.2, 1.0}, {8, 6, 2.85, 10.0}, {8, 4, 2.45, 8.5}};
    BigCfg best{0, 0, 1};
    double best_t = 0.0;
    for (const Tile& c : cand) {
        const bool t128x192 = c.ti == 4 && c.tj == 6;
        if (!resid && c.ti == 8) continue;
        if (fused_head && c.tj < 4) continue;
        // a tile's 32-bit byte offsets: rows (columns) x K x 2 stay under 4 GiB
        if ((c.ti > 4 || c.tj > 4) && K > (1 << 22)) continue;
        const int bm = 32 * c.ti, bn = 32 * c.tj;
        const long tiles = (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
        for (int S = 1; S <= max_split; ++S) {
            if (S > 1 && K / 64 / S < 8) break;
            if (S == 5 || S == 7) continue;
            if (S == 1 ? c.ti == 8 && M >= 4096 : t128x192 && M < 4096) continue;
            const long per_cu = (tiles * S + 255) / 256;
            if (c.ti == 8 && c.tj == 4 && (S > 1 || per_cu > 1)) continue;
            // three 128 x 192 tiles share a CU: they reach their rate when more follow
            const double rate = t128x192 && per_cu <= 3 ? 2.65 : c.rate;
            const double calc = per_cu * ((double)bm * bn * K / S / (1e6 * rate) + c.fixed_us);
            const double mem = 2.0 * N * K / 5e6 + 4.0;
            const double us = (calc > mem ? calc + 0.35 * mem : mem + 0.35 * calc) +
                              (S > 1 ? 4.0 * S * M * N / 4.4e6 : 0.0);
            if (best.ti == 0 || us < best_t) {
                best = BigCfg{c.ti, c.tj, S};
                best_t = us;
            }
        }
    }
    return best;
}

// Rows that an LM-head launch over at most M listed rows is tiled for.  The count
// is device data: with logit mixing M at the first step of a block (every position
// masked), toward M / 2 at its end.  Up to 192 rows one row tile can hold any count
// and M it is: tiled for three quarters, 128 rows of the 8B head took 293 us with all
// of them listed and 224 to 231 with up to three quarters, tiled for M 244 and 231 to
// 238.  Above, three quarters: 256 rows take 260 to 263 us in one tile of 192 rows up
// to there and 360 in two beyond, 324 to 339 us throughout when tiled for M; from 320
// rows the two rarely differ.
int head_rows(int M) { return M <= 192 ? M : (3 * M + 3) / 4; }

// The tile of one launch of the M > 64 kernel; the split of a residual projection
// (EPI_PARTIAL) is the one whose time is least, and where that is 1 the full sum
// (EPI_RESID) runs on the very tile that was priced.
BigCfg launch_cfg(int kind, int M, int N, int K, bool fused_head) {
    switch (kind) {
    case EPI_PARTIAL: return big_cfg(M, N, K, true, M < 256 ? 8 : 4, false);
    case EPI_RESID: return big_cfg(M, N, K, true, 1, false);
    case EPI_LMHEAD: return big_cfg(head_rows(M), N, K, false, 1, fused_head);
    default: return big_cfg(M, N, K, false, 1, false);
    }
}

void gemm_plan(int dtype, int M, int N, int K, bool partial, bool xfrag, int32_t* plan, bool fused_head) {
    plan[1] = plan[2] = 0;
    plan[3] = 1;
    if (dtype == DARD_DTYPE_F32) {
        plan[0] = DARD_GEMM_F32;
        return;
    }
    if (M <= 64) {
        StreamCfg c = stream_cfg(N, K, partial);
        if (c.split == 1) c = stream_cfg(N, K, false);   // one split runs the full-sum epilogue
        plan[0] = DARD_GEMM_STREAM;
        plan[1] = 4;
        plan[2] = c.nw;
        plan[3] = c.split;
        return;
    }
    if (!xfrag) {
        plan[0] = DARD_GEMM_TILED;
        plan[1] = TBM / 32;
        plan[2] = TBN / 32;
        return;
    }
    const BigCfg c = launch_cfg(fused_head ? EPI_LMHEAD : (partial ? EPI_PARTIAL : EPI_STORE_F32), M, N, K, fused_head);
    plan[0] = M < 256 ? DARD_GEMM_PIPE : DARD_GEMM_BIG;
    plan[1] = c.ti;
    plan[2] = c.tj;
    plan[3] = c.split;
}

int gemm_split(int dtype, int M, int N, int K) {
    if (dtype != DARD_DTYPE_BF16) return 1;
    if (M > 64) return launch_cfg(EPI_PARTIAL, M, N, K, false).split;
    return stream_cfg(N, K, true).split;
}

hipError_t launch_gemm(int dtype, const void* X, int M, int K, int ldx, const void* W, int N,
                       const EpiArgs& e, int kernel_class, hipStream_t s, bool xfrag) {
    TraceScope ts(kernel_class, s);
    if (e.kind == EPI_LMHEAD && (!e.rowmap || !e.rows_dev || !e.y)) return hipErrorInvalidValue;
    // fused LM-head partials: only the tiled kernel forms them
    if (e.kind == EPI_LMHEAD && e.lpart && (dtype != DARD_DTYPE_BF16 || M <= 64 || !xfrag))
        return hipErrorInvalidValue;
    if (dtype == DARD_DTYPE_F32) {
        // the largest tile that still gives every CU a workgroup; with the
        // smallest, more waves split a longer K
        const float *x = reinterpret_cast<const float*>(X), *w = reinterpret_cast<const float*>(W);
        auto grid = [&](int t) { return dim3((N + 16 * t - 1) / (16 * t), (M + 16 * t - 1) / (16 * t)); };
        auto wgs = [&](int t) { return (long)grid(t).x * grid(t).y; };
        if (wgs(4) >= 256) launch((gemm_f32<4, 4, 4>), grid(4), dim3(256), 0, s, x, M, K, ldx, w, N, e);
        else if (wgs(2) >= 256) launch((gemm_f32<2, 2, 4>), grid(2), dim3(256), 0, s, x, M, K, ldx, w, N, e);
        else if (K < 1024) launch((gemm_f32<1, 1, 4>), grid(1), dim3(256), 0, s, x, M, K, ldx, w, N, e);
        else launch((gemm_f32<1, 1, 16>), grid(1), dim3(1024), 0, s, x, M, K, ldx, w, N, e);
        return hipGetLastError();
    }
    const bf16_t* x = reinterpret_cast<const bf16_t*>(X);
    const bf16_t* w = reinterpret_cast<const bf16_t*>(W);
    if (xfrag && !frag_rows(dtype, M)) return hipErrorInvalidValue;
    if (M <= 64) {
        const StreamCfg c = stream_cfg(N, K, e.kind == EPI_PARTIAL);
        const dim3 grid(N / (16 * c.nw), c.split), block(64 * c.ks);
#define DARD_GS(NW, KS, D)                                                                               \
    do {                                                                                                 \
        if (xfrag) launch((gemm_stream_bf16<NW, KS, D, true>), grid, block, 0, s, x, M, K, ldx, w, N, e);  \
        else launch((gemm_stream_bf16<NW, KS, D, false>), grid, block, 0, s, x, M, K, ldx, w, N, e);       \
    } while (0)
        if (c.nw == 8) DARD_GS(8, 2, 3);
        else if (c.nw == 6) DARD_GS(6, 4, 3);
        else if (c.nw == 4 && c.ks == 4 && c.depth == 3) DARD_GS(4, 4, 3);
        else if (c.nw == 4 && c.ks == 4) DARD_GS(4, 4, 2);
        else if (c.nw == 4) DARD_GS(4, 2, 2);
        else if (c.nw == 3 && c.ks == 4) DARD_GS(3, 4, 3);
        else if (c.nw == 3) DARD_GS(3, 2, 2);
        else if (c.nw == 2) DARD_GS(2, 4, 2);
        else DARD_GS(1, 4, 2);
#undef DARD_GS
        return hipGetLastError();
    }
    if (xfrag) {
        const bool parts = e.kind == EPI_LMHEAD && e.lpart;
        const BigCfg c = launch_cfg(e.kind, M, N, K, parts);
        const int tiles_m = (M + 32 * c.ti - 1) / (32 * c.ti), tiles_n = (N + 32 * c.tj - 1) / (32 * c.tj);
        if (parts && e.ntile != tiles_n) return hipErrorInvalidValue;
        const dim3 grid(tiles_m * tiles_n, c.split);
#define DARD_GB(TI, TJ, WM, NST, WD, OCC)                                                                       \
    launch((gemm_big_bf16<TI, TJ, WM, NST, WD, OCC>), grid, dim3(256 * WM), 0, s, x, M, K, w, N, e, tiles_n)
        if (c.ti == 8 && c.tj == 4) DARD_GB(8, 2, 2, 4, 4, 2);
        else if (c.ti == 8) DARD_GB(8, 3, 2, 4, 3, 2);
        else if (c.ti == 6) DARD_GB(12, 2, 1, 3, 3, 2);
        else if (c.ti == 3) DARD_GB(6, 2, 1, 4, 4, 3);
        else if (c.ti == 2) DARD_GB(4, 1, 1, 4, 4, 4);
        else if (c.tj == 6) DARD_GB(8, 3, 1, 3, 2, 3);
        else if (c.tj == 4) DARD_GB(8, 2, 1, 3, 4, 3);
        else DARD_GB(8, 1, 1, 3, 4, 3);
#undef DARD_GB
        return hipGetLastError();
    }
    const int tiles_m = (M + TBM - 1) / TBM, tiles_n = (N + TBN - 1) / TBN;
    launch(gemm_tiled_bf16, dim3(tiles_m * tiles_n), dim3(256), 0, s, x, M, K, ldx, w, N, e,
                       tiles_m, tiles_n);
    return hipGetLastError();
}

}  // namespace dard
