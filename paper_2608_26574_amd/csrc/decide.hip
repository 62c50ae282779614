// Decision part of one DARD step (Algorithm 1): candidate verification, the
// promotion / demotion sets, the guidance weight of masked tokens (Eq. 5-6)
// and the three-state transition with token fill (Eq. 8).  One workgroup per
// sequence, one thread per block position.  Distance-weighted sums are formed
// in float64 in position order from a table of lambda^k.  In step mode the
// vocab-chunk partials of the confidence reduction are first copied to LDS
// in one coalesced pass; the 256 / B lanes that a position has share the merge
// of its partials (runs combined by a butterfly), and the sums of Eq. 5-6 walk
// only the promoted and demoted positions.  The kernel is one workgroup per
// sequence and nothing but latency: verification and transitions took 8 and 9 us
// at B = 32 with one lane per position and every position in the sums, 16 and 14
// at B = 128, and take 8 and 6, 14 and 11 (reading the partials where they are
// instead of through LDS: 8 and 7, 17 and 10).
//
// Sec. 5.1 variants: with a fixed weight every M position takes w_fixed
// instead of Eq. 5-6; with the entropy or margin ordering the key carried to
// the next step's mask (conf_out) is -entropy or the margin of the row that
// gave the confidence, from the statistics partials (chunk stride 5).
#include "common.h"
#include "launch.h"

namespace dard {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ int transition(float c, float tau_c, float tau_u) {
    if (c <= tau_c) return DARD_STATE_M;
    if (c <= tau_u) return DARD_STATE_C;
    return DARD_STATE_U;
}

struct Red {
    float m;
    int a;
    float s;
    float t, m2;   // statistics partials only: sum e (l - max), second-largest l
};

__device__ __forceinline__ Red merge_red(const Red& x, const Red& y, bool stats) {
    Red r;
    const bool take = (y.m > x.m) || (y.m == x.m && y.a < x.a);
    r.m = fmaxf(x.m, y.m);
    r.a = take ? y.a : x.a;
    const float e1 = x.m == -INFINITY ? 0.f : exp2f((x.m - r.m) * kLog2e);
    const float e2 = y.m == -INFINITY ? 0.f : exp2f((y.m - r.m) * kLog2e);
    r.s = x.s * e1 + y.s * e2;
    r.t = 0.f;
    r.m2 = -INFINITY;
    if (stats) {
        const float t1 = x.m == -INFINITY ? 0.f : e1 * (x.t + (x.m - r.m) * x.s);
        const float t2 = y.m == -INFINITY ? 0.f : e2 * (y.t + (y.m - r.m) * y.s);
        r.t = t1 + t2;
        r.m2 = fmaxf(fminf(x.m, y.m), fmaxf(x.m2, y.m2));
    }
    return r;
}

// Merge the chunk partials of one row (stride K floats each): lane `sub` of the
// row's `lanes` (a power of two, consecutive lanes of one wave, all of them here)
// takes chunks sub, sub + lanes, ...; every lane of the row gets the result of the
// same merges.
__device__ Red combine(const float* p, int nchunk, int K, int sub, int lanes) {
    const bool stats = K == kConfStatsStride;
    Red t{-INFINITY, 0x7fffffff, 0.f, 0.f, -INFINITY};
    for (int c = sub; c < nchunk; c += lanes) {
        const float* q = p + (size_t)c * K;
        const Red y{q[0], __float_as_int(q[1]), q[2], stats ? q[3] : 0.f, stats ? q[4] : -INFINITY};
        t = c == sub ? y : merge_red(t, y, stats);
    }
    for (int o = 1; o < lanes; o <<= 1) {
        Red y{__shfl_xor(t.m, o, 64), __shfl_xor(t.a, o, 64), __shfl_xor(t.s, o, 64), 0.f, -INFINITY};
        if (stats) { y.t = __shfl_xor(t.t, o, 64); y.m2 = __shfl_xor(t.m2, o, 64); }
        // (lower lane first on both sides, so that both hold the same bits)
        t = (sub & o) ? merge_red(y, t, stats) : merge_red(t, y, stats);
    }
    return t;
}

__device__ __forceinline__ float red_entropy(const Red& t) { return logf(t.s) - t.t / t.s; }
__device__ __forceinline__ float red_margin(const Red& t) { return (1.f - expf(t.m2 - t.m)) / t.s; }

constexpr int kThreads = kMaxBlock;   // one thread per block position
constexpr size_t kStageBytes = 64 * 1024;   // chunk partials larger than this are read in place

// Copy n floats from global to LDS with all of a thread's loads in flight.
__device__ void stage(float* dst, const float* src, int n) {
    constexpr int U = 8;
    for (int base = 0; base < n; base += U * kThreads) {
        float v[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = base + k * kThreads + threadIdx.x;
            v[k] = t < n ? src[t] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int t = base + k * kThreads + threadIdx.x;
            if (t < n) dst[t] = v[k];
        }
    }
}

struct PosConf {
    float maxprob, pcur;
    int argmax;
    float entropy, margin, key;   // key: the caller's ordering key (array mode)
};

// Shadow-row confidence of position i: from its merged partials (step mode) or
// from the per-position arrays.
__device__ PosConf shadow_conf(const DecideArgs& a, const Red* red, int s, int i, int tok) {
    PosConf r{0.f, 0.f, 0, 0.f, 0.f, 0.f};
    const int pos = s * a.B + i;
    if (red) {
        const Red t = *red;
        r.maxprob = 1.f / t.s;
        r.argmax = t.a;
        if ((a.flags & DARD_F_VERIFY_PCUR) || a.dbg_pcur_s) {
            tok = min(max(tok, 0), (int)a.ld - 1);   // stay inside the row whatever the id
            const float lc = a.logits[((size_t)s * 2 * a.B + a.B + i) * a.ld + tok];
            r.pcur = exp2f((lc - t.m) * kLog2e) / t.s;
        }
        if (a.stride == kConfStatsStride) { r.entropy = red_entropy(t); r.margin = red_margin(t); }
    } else {
        r.maxprob = a.maxprob_s[pos];
        r.argmax = a.argmax_s ? a.argmax_s[pos] : 0;
        r.pcur = a.pcur_s ? a.pcur_s[pos] : 0.f;
        r.key = a.key_s ? a.key_s[pos] : 0.f;
    }
    return r;
}

// The key the next step's mask orders candidates by (Eq. 3 or its Sec. 5.1
// variants): the confidence, -entropy or the margin.
__device__ __forceinline__ float order_key(uint32_t flags, bool from_partials, float c, float entropy,
                                           float margin, float given) {
    if (!(flags & (DARD_F_ORDER_ENTROPY | DARD_F_ORDER_MARGIN))) return c;
    if (!from_partials) return given;
    return (flags & DARD_F_ORDER_ENTROPY) ? -entropy : margin;
}

__global__ __launch_bounds__(kThreads) void decide_kernel(DecideArgs a, int in_lds) {
    extern __shared__ float staged[];            // [2][B][nchunk][stride] in step mode (in_lds)
    __shared__ uint64_t promoted[kBlockWords], demoted[kBlockWords];
    __shared__ Red rows[kThreads];               // merged partials by position (step mode)
    __shared__ double lam_pow[kThreads];
    __shared__ int all_u, entered_u, bad_code;
    __shared__ float c_all[kThreads];
    __shared__ int nxt_all[kThreads], xhat_all[kThreads];
    const int s = blockIdx.x, i = threadIdx.x;
    const bool live = i < a.B;
    const int pos = s * a.B + i;
    const int st = live ? a.state_in[pos] : DARD_STATE_U;
    const bool pcur_mode = (a.flags & DARD_F_VERIFY_PCUR) != 0;
    const int per_seq = a.B * a.nchunk * a.stride;
    // the sequence's chunk partials: copied to LDS in one coalesced pass, or
    // (large blocks) read where they are
    const float* sv = a.part_v ? a.part_v + (size_t)s * per_seq : nullptr;
    const float* sm = a.part_m ? a.part_m + (size_t)s * per_seq : nullptr;
    if (in_lds) {
        if (a.part_v) stage(staged, sv, per_seq);
        if (a.part_m && a.phase == DARD_PHASE_FINAL) stage(staged + per_seq, sm, per_seq);
        sv = a.part_v ? staged : nullptr;
        sm = a.part_m ? staged + per_seq : nullptr;
    }

    if (a.phase == DARD_PHASE_VERIFY && live) lam_pow[i] = pow(a.lambda, (double)i);
    __syncthreads();
    // merged partials of every position that has any: 256 / B lanes each
    if (sv || sm) {
        int lanes = 1;
        while (lanes < 64 && lanes * 2 * a.B <= kThreads) lanes *= 2;
        const int row = i / lanes, sub = i & (lanes - 1);
        if (row < a.B) {                           // (uniform over a row's lanes)
            const int rst = a.state_in[s * a.B + row];
            const float* part = rst == DARD_STATE_C ? sv : (a.phase != DARD_PHASE_VERIFY ? sm : nullptr);
            if (part) {
                const Red t = combine(part + (size_t)row * a.nchunk * a.stride, a.nchunk, a.stride, sub, lanes);
                if (sub == 0) rows[row] = t;
            }
        }
        __syncthreads();
    }

    if (a.phase == DARD_PHASE_VERIFY) {
        bool up = false, down = false;
        if (live && st == DARD_STATE_C) {
            const int tok = a.tok_in ? a.tok_in[pos] : 0;
            const PosConf pc = shadow_conf(a, a.part_v ? &rows[i] : nullptr, s, i, tok);
            const float c = pcur_mode ? pc.pcur : pc.maxprob;
            const int nxt = transition(c, a.tau_c, a.tau_u);
            up = nxt == DARD_STATE_U;
            down = nxt == DARD_STATE_M;
        }
        const uint64_t bu = __ballot(up), bd = __ballot(down);
        if ((i & 63) == 0) { promoted[i >> 6] = bu; demoted[i >> 6] = bd; }
        __syncthreads();
        if (!live) return;
        float w = 0.f;
        if (st == DARD_STATE_M && (a.flags & DARD_F_FIXED_W)) {
            w = a.w_fixed;
        } else if (st == DARD_STATE_M) {
            double P = 0.0, D = 0.0;
            for (int q = 0; q < kBlockWords; ++q) {
                for (uint64_t u = promoted[q]; u; u &= u - 1) P += lam_pow[abs(i - (64 * q + __builtin_ctzll(u)))];
                for (uint64_t u = demoted[q]; u; u &= u - 1) D += lam_pow[abs(i - (64 * q + __builtin_ctzll(u)))];
            }
            w = (float)((P + a.p0) / (P + D + a.p0));
        }
        a.w_out[pos] = w;
        return;
    }

    // ---- FINAL: confidences of every position, transition, fill
    if (i == 0) { all_u = 1; entered_u = 0; bad_code = 0; }
    __syncthreads();
    if (live && st > DARD_STATE_U) atomicOr(&bad_code, 1);
    if (live) {
        const int tok = a.tok_in ? a.tok_in[pos] : 0;
        float c, key;
        int xhat;
        float mp_s = 0.f, pc_s = 0.f, mp_mix = 0.f, ent = 0.f, mrg = 0.f;
        int am_s = -1, am_mix = -1;
        const bool from_part = a.part_m != nullptr;
        if (st == DARD_STATE_M) {
            float given = 0.f;
            if (from_part) {
                const Red t = rows[i];
                mp_mix = 1.f / t.s;
                am_mix = t.a;
                if (a.stride == kConfStatsStride) { ent = red_entropy(t); mrg = red_margin(t); }
            } else {
                mp_mix = a.maxprob_mix[pos];
                am_mix = a.argmax_mix[pos];
                given = a.key_mix ? a.key_mix[pos] : 0.f;
            }
            c = mp_mix;
            xhat = am_mix;
            key = order_key(a.flags, from_part, c, ent, mrg, given);
        } else {
            const PosConf pc = shadow_conf(a, from_part ? &rows[i] : nullptr, s, i, tok);
            mp_s = pc.maxprob; pc_s = pc.pcur; am_s = pc.argmax;
            ent = pc.entropy; mrg = pc.margin;
            c = pcur_mode ? pc.pcur : pc.maxprob;
            xhat = pc.argmax;
            key = order_key(a.flags, from_part, c, ent, mrg, pc.key);
        }
        const int nxt = transition(c, a.tau_c, a.tau_u);
        if (nxt != DARD_STATE_U) atomicAnd(&all_u, 0);
        if (nxt == DARD_STATE_U && st != DARD_STATE_U) atomicOr(&entered_u, 1);
        c_all[i] = c;
        nxt_all[i] = nxt;
        xhat_all[i] = xhat;
        a.state_out[pos] = (uint8_t)nxt;
        a.tok_out[pos] = nxt == DARD_STATE_M ? a.mask_id : xhat;
        a.conf_out[pos] = key;
        if (a.dbg_maxprob_s) a.dbg_maxprob_s[pos] = mp_s;
        if (a.dbg_argmax_s) a.dbg_argmax_s[pos] = am_s;
        if (a.dbg_pcur_s) a.dbg_pcur_s[pos] = pc_s;
        if (a.dbg_maxprob_mix) a.dbg_maxprob_mix[pos] = mp_mix;
        if (a.dbg_argmax_mix) a.dbg_argmax_mix[pos] = am_mix;
        if (a.dbg_entropy) a.dbg_entropy[pos] = ent;
        if (a.dbg_margin) a.dbg_margin[pos] = mrg;
    }
    __syncthreads();
    // progress rule (DARD_F_PROGRESS): no position entered U in an unfinished
    // block -> the most confident non-U position (lowest on ties) becomes U
    if (i == 0 && (a.flags & DARD_F_PROGRESS) && !entered_u && !all_u) {
        int best = -1;
        for (int j = 0; j < a.B; ++j)
            if (nxt_all[j] != DARD_STATE_U && (best < 0 || c_all[j] > c_all[best])) best = j;
        const int bp = s * a.B + best;
        a.state_out[bp] = (uint8_t)DARD_STATE_U;
        a.tok_out[bp] = xhat_all[best];
        int done = 1;
        for (int j = 0; j < a.B; ++j)
            if (j != best && nxt_all[j] != DARD_STATE_U) done = 0;
        all_u = done;
    }
    if (i == 0 && a.block_done)
        a.block_done[s] = ((a.flags & DARD_F_CHECK_STATES) && bad_code) ? DARD_BAD_STATE : all_u;
}

}  // namespace

hipError_t launch_decide(const DecideArgs& a, hipStream_t s) {
    TraceScope ts(DARD_K_DECIDE, s);
    if (a.B < 1 || a.B > kThreads) return hipErrorInvalidValue;
    size_t lds = (a.part_v || a.part_m) ? (size_t)2 * a.B * a.nchunk * a.stride * sizeof(float) : 0;
    const int in_lds = lds > 0 && lds <= kStageBytes;
    if (!in_lds) lds = 0;
    launch(decide_kernel, dim3(a.b), dim3(kThreads), lds, s, a, in_lds);
    return hipGetLastError();
}

}  // namespace dard
