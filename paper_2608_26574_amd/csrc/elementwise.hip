// Row-wise kernels: embedding gather of the augmented block / prefix with the
// first RMSNorm fused, the RMSNorm between sub-layers, and the row copies
// used to pack the weight image.
#include "common.h"
#include "launch.h"

namespace dard {

namespace {

// Offset of element (row, c) of a [rows][d] activation, row-major or fragment-major.
__device__ __forceinline__ size_t act_off(int row, int c, int d, bool frag) {
    return frag ? frag_off(row, c, d) : (size_t)row * d + c;
}

// N consecutive values (16 bytes of T, aligned) as floats, and back.
template <typename T, int N>
__device__ __forceinline__ void load_vec(const T* p, float (&v)[N]) {
    static_assert(N * sizeof(T) == 16 || N * sizeof(T) == 8, "one 8- or 16-byte access");
    typedef T Vec __attribute__((ext_vector_type(N)));
    const Vec x = *reinterpret_cast<const Vec*>(p);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const T e = x[i];
        v[i] = St<T>::ld(&e);
    }
}
template <typename T, int N>
__device__ __forceinline__ void store_vec(T* p, const float (&v)[N]) {
    typedef T Vec __attribute__((ext_vector_type(N)));
    Vec x;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        T e;
        St<T>::st(&e, v[i]);
        x[i] = e;
    }
    *reinterpret_cast<Vec*>(p) = x;
}

// Source row of embedding row `row`; in_table is cleared for a row of `embeds`.
template <typename T>
__device__ __forceinline__ const T* embed_src(const int32_t* ids, const T* embeds, const T* table, size_t row, int d,
                                              int vocab, int step_B, int mask_id, bool* in_table) {
    int id;
    if (step_B > 0) {
        const int s = row / (2 * step_B), r = row % (2 * step_B);
        id = r < step_B ? ids[(size_t)s * step_B + r] : mask_id;
    } else {
        id = ids[row];
    }
    // ids are device data: keep every read inside its table
    if (id >= vocab || (id < 0 && embeds == nullptr)) id = id < 0 ? 0 : vocab - 1;
    *in_table = id >= 0;
    return id >= 0 ? table + (size_t)id * d : embeds + row * d;
}

// The embedding row is held in registers between its load, the store to h and
// the normalised store, in 16-byte pieces (an 8-element group of the
// fragment-major layout is contiguous), so the row costs one read and two
// writes: 64 rows of 4096 in 5.2 us, 640 rows in 10.6 us (15 and 27 us when h
// was read back and values were stored one by one).
template <typename T>
__global__ __launch_bounds__(256) void embed_norm_kernel(const int32_t* __restrict__ ids, const T* __restrict__ embeds,
                                                         const T* __restrict__ table, const T* __restrict__ gain,
                                                         int d, int vocab, float eps, int step_B, int mask_id,
                                                         float* __restrict__ h, T* __restrict__ xn, int frag,
                                                         int embeds_aligned) {
    constexpr int N = 16 / sizeof(T), kIt = 8192 / (256 * N);   // d <= 8192, a multiple of N
    __shared__ float red[4];
    const size_t row = blockIdx.x;
    bool in_table;
    const T* src = embed_src(ids, embeds, table, row, d, vocab, step_B, mask_id, &in_table);
    float v[kIt][N];
    if (in_table || embeds_aligned) {
#pragma unroll
        for (int q = 0; q < kIt; ++q) {
            const int c = (threadIdx.x + 256 * q) * N;
            if (c < d) load_vec<T, N>(src + c, v[q]);
        }
    } else {
#pragma unroll
        for (int q = 0; q < kIt; ++q) {
            const int c = (threadIdx.x + 256 * q) * N;
#pragma unroll
            for (int i = 0; i < N; ++i)
                if (c < d) v[q][i] = St<T>::ld(src + c + i);
        }
    }
    float ss = 0.f;
    float* hr = h + row * d;
#pragma unroll
    for (int q = 0; q < kIt; ++q) {
        const int c = (threadIdx.x + 256 * q) * N;
        if (c < d) {
#pragma unroll
            for (int i = 0; i < N; i += 4) {
                *reinterpret_cast<float4*>(hr + c + i) = make_float4(v[q][i], v[q][i + 1], v[q][i + 2], v[q][i + 3]);
                ss += v[q][i] * v[q][i] + v[q][i + 1] * v[q][i + 1] + v[q][i + 2] * v[q][i + 2] +
                      v[q][i + 3] * v[q][i + 3];
            }
        }
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float inv = rsqrtf((red[0] + red[1] + red[2] + red[3]) / (float)d + eps);
#pragma unroll
    for (int q = 0; q < kIt; ++q) {
        const int c = (threadIdx.x + 256 * q) * N;
        if (c < d) {
            float gn[N];
            load_vec<T, N>(gain + c, gn);
#pragma unroll
            for (int i = 0; i < N; ++i) gn[i] *= v[q][i] * inv;
            store_vec<T, N>(xn + act_off((int)row, c, d, frag != 0), gn);
        }
    }
}

// The same for many rows: a wave per row, eight adjacent rows per workgroup.  A
// row of the fragment-major layout is 16-byte pieces 256 bytes apart, so a
// workgroup that stores one row touches every 128-byte line of 16 rows for an
// eighth of it; eight adjacent rows stored together fill their lines in L2.
constexpr int kRowWaves = 8;

template <typename T>
__global__ __launch_bounds__(64 * kRowWaves) void embed_norm_rows_kernel(
    const int32_t* __restrict__ ids, const T* __restrict__ embeds, const T* __restrict__ table,
    const T* __restrict__ gain, int rows, int d, int vocab, float eps, int step_B, int mask_id, float* __restrict__ h,
    T* __restrict__ xn, int frag) {
    constexpr int N = 16 / sizeof(T), kIt = 4096 / (64 * N);   // d <= 4096
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * kRowWaves + (threadIdx.x >> 6);
    if (row >= (size_t)rows) return;
    bool in_table;
    const T* src = embed_src(ids, embeds, table, row, d, vocab, step_B, mask_id, &in_table);
    float* hr = h + row * d;
    typedef T Vec __attribute__((ext_vector_type(N)));
    Vec raw[kIt];                                  // the row as stored: half the registers of its floats
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < kIt; ++q) {
        const int c = (lane + 64 * q) * N;
        if (c < d) raw[q] = *reinterpret_cast<const Vec*>(src + c);
    }
#pragma unroll
    for (int q = 0; q < kIt; ++q) {
        const int c = (lane + 64 * q) * N;
        if (c < d) {
#pragma unroll
            for (int i = 0; i < N; i += 4) {
                float f[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const T e = raw[q][i + k];
                    f[k] = St<T>::ld(&e);
                }
                *reinterpret_cast<float4*>(hr + c + i) = make_float4(f[0], f[1], f[2], f[3]);
                ss += f[0] * f[0] + f[1] * f[1] + f[2] * f[2] + f[3] * f[3];
            }
        }
    }
    const float inv = rsqrtf(wave_sum(ss) / (float)d + eps);
#pragma unroll
    for (int q = 0; q < kIt; ++q) {
        const int c = (lane + 64 * q) * N;
        if (c < d) {
            float gn[N];
            load_vec<T, N>(gain + c, gn);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const T e = raw[q][i];
                gn[i] *= St<T>::ld(&e) * inv;
            }
            store_vec<T, N>(xn + act_off((int)row, c, d, frag != 0), gn);
        }
    }
}

// h[row] += sum_s part[s][row] (split-K partials of the preceding projection,
// added in split order), then xn[row] = RMSNorm(h[row]) * gain.  One
// workgroup of 512 threads per row, each thread holding up to kVec float4 of the row.
constexpr int kVec = 4;   // d <= 512 * 4 * kVec

// NS is the split count (0 = no partials); all loads of a thread are issued
// before the first add so that the row costs one memory round trip.
template <typename T, int NS>
__global__ __launch_bounds__(512) void resid_norm_kernel(float* __restrict__ h, const float* __restrict__ part,
                                                         size_t split_stride, const T* __restrict__ gain,
                                                         int d, float eps, T* __restrict__ xn, int frag) {
    __shared__ float red[8];
    const size_t row = blockIdx.x;
    float4* hr = reinterpret_cast<float4*>(h + row * d);
    const int n4 = d / 4;
    float4 v[kVec];
    float4 p[NS > 0 ? NS : 1][kVec];
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        const int c4 = threadIdx.x + 512 * q;
        v[q] = c4 < n4 ? hr[c4] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int s = 0; s < NS; ++s)
            p[s][q] = c4 < n4 ? reinterpret_cast<const float4*>(part + s * split_stride + row * d)[c4]
                              : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        const int c4 = threadIdx.x + 512 * q;
        float4 x = v[q];
#pragma unroll
        for (int s = 0; s < NS; ++s) { x.x += p[s][q].x; x.y += p[s][q].y; x.z += p[s][q].z; x.w += p[s][q].w; }
        if (NS > 0 && c4 < n4) hr[c4] = x;
        v[q] = x;
        ss += x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
    }
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < 8; ++w) tot += red[w];
    const float inv = rsqrtf(tot / (float)d + eps);
#pragma unroll
    for (int q = 0; q < kVec; ++q) {
        const int c4 = threadIdx.x + 512 * q;
        if (c4 < n4) {
            const int c = 4 * c4;   // c..c+3 stay inside one 8-element group of the fragment layout
            float gn[4];
            load_vec<T, 4>(gain + c, gn);
            const float o[4] = {v[q].x * inv * gn[0], v[q].y * inv * gn[1], v[q].z * inv * gn[2], v[q].w * inv * gn[3]};
            store_vec<T, 4>(xn + act_off((int)row, c, d, frag != 0), o);
        }
    }
}

// The same for many rows without partials, a wave per row and eight adjacent rows
// per workgroup (see embed_norm_rows_kernel).  8192 rows of 3584: 61 -> 40 us;
// embedding them 98 -> 58 us.  Partials are left to a workgroup per row, whose
// waves have more loads in flight: two of them at 2100 rows of 4096 take 35 us
// there and 51 here, at 4000 rows 60 and 69.
template <typename T, int IT>
__global__ __launch_bounds__(64 * kRowWaves) void resid_norm_rows_kernel(const float* __restrict__ h,
                                                                         const T* __restrict__ gain, int rows, int d,
                                                                         float eps, T* __restrict__ xn, int frag) {
    const int lane = threadIdx.x & 63;
    const size_t row = (size_t)blockIdx.x * kRowWaves + (threadIdx.x >> 6);
    if (row >= (size_t)rows) return;
    const float* hr = h + row * d;
    float4 v[IT];                                  // d <= 256 IT
    float ss = 0.f;
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int c = 4 * (lane + 64 * q);
        v[q] = c < d ? *reinterpret_cast<const float4*>(hr + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < IT; ++q) ss += v[q].x * v[q].x + v[q].y * v[q].y + v[q].z * v[q].z + v[q].w * v[q].w;
    const float inv = rsqrtf(wave_sum(ss) / (float)d + eps);
#pragma unroll
    for (int q = 0; q < IT; ++q) {
        const int c = 4 * (lane + 64 * q);
        if (c < d) {
            float gn[4];
            load_vec<T, 4>(gain + c, gn);
            const float o[4] = {v[q].x * inv * gn[0], v[q].y * inv * gn[1], v[q].z * inv * gn[2], v[q].w * inv * gn[3]};
            store_vec<T, 4>(xn + act_off((int)row, c, d, frag != 0), o);
        }
    }
}

__global__ void copy_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// Packed weight rows.  mode 0: identity; mode 1: per head of `dh` rows, packed
// row 2t <- row t and 2t+1 <- row t + dh/2 (rotary pairs adjacent); mode 2:
// packed row 2t <- row t of src0 (gate), 2t+1 <- row t of src1 (up).
__global__ void pack_rows_kernel(const uint8_t* __restrict__ src0, const uint8_t* __restrict__ src1,
                                 uint8_t* __restrict__ dst, int nrows, int rowbytes, int mode, int dh) {
    const int rd = blockIdx.x;
    if (rd >= nrows) return;
    const uint8_t* src;
    if (mode == 1) {
        const int head = rd / dh, e = rd % dh, t = e / 2;
        src = src0 + (size_t)(head * dh + ((e & 1) ? t + dh / 2 : t)) * rowbytes;
    } else if (mode == 2) {
        src = ((rd & 1) ? src1 : src0) + (size_t)(rd / 2) * rowbytes;
    } else {
        src = src0 + (size_t)rd * rowbytes;
    }
    const uint4* s4 = reinterpret_cast<const uint4*>(src);
    uint4* d4 = reinterpret_cast<uint4*>(dst + (size_t)rd * rowbytes);
    for (int i = threadIdx.x; i < rowbytes / 16; i += blockDim.x) d4[i] = s4[i];
}

}  // namespace

hipError_t launch_pack_rows(const void* src0, const void* src1, void* dst, int nrows, int rowbytes, int mode,
                            int dh, hipStream_t s) {
    launch(pack_rows_kernel, dim3(nrows), dim3(128), 0, s, (const uint8_t*)src0,
                       (const uint8_t*)src1, (uint8_t*)dst, nrows, rowbytes, mode, dh);
    return hipGetLastError();
}

// Rows from which a wave per row fills the chip (without partials; rows of 3584 and 4096: at 1024
// rows 11.0 us against 9.1 with a workgroup per row, at 2048 16.2 against 18.5).
constexpr int kManyRows = 2048;

hipError_t launch_embed_norm(int dtype, const int32_t* ids, const void* embeds, const void* table,
                             const void* gain, int rows, int d, int vocab, float eps, int step_B,
                             int mask_id, float* h, void* xn, bool frag, hipStream_t s) {
    TraceScope ts(DARD_K_NORM, s);
    if (frag && !frag_rows(dtype, rows)) return hipErrorInvalidValue;
    if (d > 8192 || d % (dtype == DARD_DTYPE_BF16 ? 8 : 4)) return hipErrorInvalidValue;
    const int aligned = (reinterpret_cast<uintptr_t>(embeds) & 15) == 0;
    if (dtype == DARD_DTYPE_BF16 && rows >= kManyRows && d <= 4096 && aligned) {
        launch(embed_norm_rows_kernel<bf16_t>, dim3((rows + kRowWaves - 1) / kRowWaves), dim3(64 * kRowWaves), 0, s,
               ids, (const bf16_t*)embeds, (const bf16_t*)table, (const bf16_t*)gain, rows, d, vocab, eps, step_B,
               mask_id, h, (bf16_t*)xn, (int)frag);
        return hipGetLastError();
    }
    if (dtype == DARD_DTYPE_BF16)
        launch(embed_norm_kernel<bf16_t>, dim3(rows), dim3(256), 0, s, ids,
                           (const bf16_t*)embeds, (const bf16_t*)table, (const bf16_t*)gain, d, vocab, eps, step_B,
                           mask_id, h, (bf16_t*)xn, (int)frag, aligned);
    else
        launch(embed_norm_kernel<float>, dim3(rows), dim3(256), 0, s, ids, (const float*)embeds,
                           (const float*)table, (const float*)gain, d, vocab, eps, step_B, mask_id, h, (float*)xn, 0,
                           aligned);
    return hipGetLastError();
}

hipError_t launch_resid_norm(int dtype, float* h, const float* part, int nsplit, int rows, int d,
                             const void* gain, float eps, void* xn, bool frag, hipStream_t s) {
    TraceScope ts(DARD_K_NORM, s);
    if (frag && !frag_rows(dtype, rows)) return hipErrorInvalidValue;
    const size_t stride = (size_t)rows * d;
    if (nsplit < 0 || nsplit > 8 || d > 512 * 4 * kVec) return hipErrorInvalidValue;
    if (dtype == DARD_DTYPE_BF16 && rows >= kManyRows && nsplit == 0 && d <= 4096) {
        launch((resid_norm_rows_kernel<bf16_t, 16>), dim3((rows + kRowWaves - 1) / kRowWaves), dim3(64 * kRowWaves), 0,
               s, h, (const bf16_t*)gain, rows, d, eps, (bf16_t*)xn, (int)frag);
        return hipGetLastError();
    }
#define DARD_RN(T, NS)                                                                                 \
    launch((resid_norm_kernel<T, NS>), dim3(rows), dim3(512), 0, s, h, part, stride,      \
                       (const T*)gain, d, eps, (T*)xn, (int)frag)
#define DARD_RN_ALL(T)                                                                                 \
    switch (nsplit) {                                                                                  \
    case 0: DARD_RN(T, 0); break; case 1: DARD_RN(T, 1); break; case 2: DARD_RN(T, 2); break;          \
    case 3: DARD_RN(T, 3); break; case 4: DARD_RN(T, 4); break; case 5: DARD_RN(T, 5); break;          \
    case 6: DARD_RN(T, 6); break; case 7: DARD_RN(T, 7); break; default: DARD_RN(T, 8); break;         \
    }
    if (dtype == DARD_DTYPE_BF16) {
        DARD_RN_ALL(bf16_t)
    } else {
        DARD_RN_ALL(float)
    }
#undef DARD_RN_ALL
#undef DARD_RN
    return hipGetLastError();
}

hipError_t launch_copy_rows(const void* src, void* dst, size_t bytes, hipStream_t s) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const size_t blocks = (n16 + 255) / 256;
    launch(copy_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s,
                       (const uint4*)src, (uint4*)dst, n16);
    return hipGetLastError();
}

// ---------------------------------------------------------------- full-sequence rows
__global__ void full_rows_kernel(const int32_t* __restrict__ seq, int N, int blk, int B, int mask_id,
                                 int32_t* __restrict__ row_ids, int32_t* __restrict__ tok) {
    const int s = blockIdx.y, R = N + B, Nc = N - B;
    const int32_t* sq = seq + (size_t)s * N;
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < R; r += gridDim.x * blockDim.x) {
        int id;
        if (r < Nc) id = sq[r < blk ? r : r + B];
        else if (r < N) id = sq[blk + (r - Nc)];
        else id = mask_id;
        row_ids[(size_t)s * R + r] = id;
        if (r >= Nc && r < N) tok[(size_t)s * B + (r - Nc)] = id;
    }
}

hipError_t launch_full_rows(const int32_t* seq, int b, int N, int blk, int B, int mask_id, int32_t* row_ids,
                            int32_t* tok, hipStream_t s) {
    if (b < 1 || B < 1 || N < B || blk < 0 || blk + B > N) return hipErrorInvalidValue;
    launch(full_rows_kernel, dim3((N + B + 255) / 256, b), dim3(256), 0, s, seq, N, blk, B, mask_id, row_ids, tok);
    return hipGetLastError();
}

// One thread per 16 bytes of a destination row.  In the fragment-major layout
// the 8 bf16 values k..k+7 (k % 8 == 0) of a row are contiguous.
template <typename T>
__global__ void gather_rows_kernel(const T* __restrict__ src, int R, int first, int count, int d, int frag,
                                   T* __restrict__ dst, size_t n16) {
    constexpr int E = 16 / sizeof(T);
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n16) return;
    const int per_row = d / E;
    const int mo = (int)(t / per_row), k = (int)(t % per_row) * E;
    const int s = mo / count, mi = s * R + first + mo % count;
    const size_t so = frag ? frag_off(mi, k, d) : (size_t)mi * d + k;
    const size_t dO = frag ? frag_off(mo, k, d) : (size_t)mo * d + k;
    *reinterpret_cast<uint4*>(dst + dO) = *reinterpret_cast<const uint4*>(src + so);
}

hipError_t launch_gather_rows(int dtype, const void* src, int b, int R, int first, int count, int d, bool frag,
                              void* dst, hipStream_t s) {
    if (b < 1 || count < 1 || first < 0 || first + count > R || d % (dtype == DARD_DTYPE_BF16 ? 64 : 4))
        return hipErrorInvalidValue;
    if (frag && !frag_rows(dtype, b * R)) return hipErrorInvalidValue;
    const size_t es = dtype == DARD_DTYPE_BF16 ? 2 : 4;
    const size_t n16 = (size_t)b * count * d * es / 16;
    const unsigned blocks = (unsigned)((n16 + 255) / 256);
    if (dtype == DARD_DTYPE_BF16)
        launch(gather_rows_kernel<bf16_t>, dim3(blocks), dim3(256), 0, s, (const bf16_t*)src, R, first, count, d,
               (int)frag, (bf16_t*)dst, n16);
    else
        launch(gather_rows_kernel<float>, dim3(blocks), dim3(256), 0, s, (const float*)src, R, first, count, d, 0,
               (float*)dst, n16);
    return hipGetLastError();
}

}  // namespace dard
