// Mean directions, Householder reflection and observed statistic on the GPU
// (Sec. 3.1 "Householder mean-direction alignment", eq:householder_fast,
// eq:tobs; Algorithm 1, Steps 1-4).  All reductions are FP64 and run in a
// fixed order, so results do not depend on timing.
#include <string.h>

#include <type_traits>

#include "hbt_launch.h"

namespace hbt {

// ---------------------------------------------------------------------------
// small utilities: table upload through kernel arguments, zero fill
// ---------------------------------------------------------------------------
struct UploadChunk {
    unsigned char b[3072];
};

__global__ void k_upload(unsigned char* dst, UploadChunk c, int bytes, uint64_t* clear, int clear_words) {
    for (int i = threadIdx.x; i < bytes; i += blockDim.x) dst[i] = c.b[i];
    for (int i = threadIdx.x; i < clear_words; i += blockDim.x) clear[i] = 0;
}

hipError_t upload(void* dst, const void* src, size_t bytes, hipStream_t s, void* clear, size_t clear_bytes) {
    const unsigned char* p = (const unsigned char*)src;
    unsigned char* q = (unsigned char*)dst;
    int words = (int)(clear_bytes / 8);
    while (bytes) {
        const size_t k = bytes < sizeof(UploadChunk) ? bytes : sizeof(UploadChunk);
        UploadChunk c;
        memcpy(c.b, p, k);
        hipLaunchKernelGGL(k_upload, dim3(1), dim3(256), 0, s, q, c, (int)k, (uint64_t*)clear, words);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        words = 0;
        p += k;
        q += k;
        bytes -= k;
    }
    return hipSuccess;
}

__global__ void k_zero(uint64_t* dst, int64_t words) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = 0;
}

hipError_t zero(void* dst, size_t bytes, hipStream_t s) {
    const int64_t words = (int64_t)(bytes / 8);
    if (!words) return hipSuccess;
    int64_t g = (words + 255) / 256;
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(k_zero, dim3((unsigned)g), dim3(256), 0, s, (uint64_t*)dst, words);
    return hipGetLastError();
}

// Unit-row check of the inputs (Sec. 3.1, Eq. 2: every embedding is
// l2-normalised before the test): a row fails when | |x| - 1 | > 1e-4,
// i.e. |x|^2 outside [(1 - 1e-4)^2, (1 + 1e-4)^2]; NaN fails too.  The
// column-sum pass reads every row once, so it tests them there and writes one
// flag per chunk (1 = some row of the chunk failed); the finalize step turns
// a pair's flags into the status HBT_ERR_NOT_UNIT.
__device__ __forceinline__ bool not_unit(double ss) {
    return !(ss >= 0.99980001 && ss <= 1.00020001);
}

// Sum of x over the 64 lanes of a wave, returned to every lane: an inclusive
// scan by DPP row shifts and row broadcasts (lane 63 ends with the total),
// then a read of lane 63.
__device__ __forceinline__ float wave_total_f32(float x) {
    float v = x;
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x111, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x112, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x114, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x118, 0xF, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xA, 0xF, false));
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xC, 0xF, false));
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// This lane's J x 4 columns 256 j + 64 e + lane of one row of d values (all
// zero when the row is not valid).
template <int J, typename Tin>
__device__ __forceinline__ void load_cols(Tin (&x)[J][4], const Tin* row, int d, bool valid) {
    const int lane = threadIdx.x & 63;
    const __amdgpu_buffer_rsrc_t rs = row_rsrc(row, valid ? (int)sizeof(Tin) * d : 0);
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int at = (int)sizeof(Tin) * (256 * j + 64 * e + lane);
            if constexpr (sizeof(Tin) == 4)
                x[j][e] = __builtin_bit_cast(Tin, __builtin_amdgcn_raw_buffer_load_b32(rs, at, 0, 0));
            else
                x[j][e] = __builtin_bit_cast(Tin, __builtin_amdgcn_raw_buffer_load_b64(rs, at, 0, 0));
        }
}

// Sum of x over the 64 lanes, returned to every lane: each adds the values of
// lanes l ^ 32, l ^ 16, ..., l ^ 1 (as __shfl_xor would, through LDS), which
// reach it by a swap of two registers' halves or rows, or by DPP.  (Bound by its
// latency: three such sums in a chain in the finalize step of one pair of d = 1024
// took 12.7 us, five of them by __shfl_xor 16.5.)
__device__ __forceinline__ double wave_sum_f64(double x) {
    typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
    auto join = [](uint32_t lo, uint32_t hi) {
        return __longlong_as_double((long long)((uint64_t)hi << 32 | lo));
    };
    auto lo = [](double a) { return (uint32_t)(uint64_t)__double_as_longlong(a); };
    auto hi = [](double a) { return (uint32_t)((uint64_t)__double_as_longlong(a) >> 32); };
    {
        const u32x2 l = __builtin_amdgcn_permlane32_swap(lo(x), lo(x), false, false);
        const u32x2 h = __builtin_amdgcn_permlane32_swap(hi(x), hi(x), false, false);
        x = join(l.x, h.x) + join(l.y, h.y);
    }
    {
        const u32x2 l = __builtin_amdgcn_permlane16_swap(lo(x), lo(x), false, false);
        const u32x2 h = __builtin_amdgcn_permlane16_swap(hi(x), hi(x), false, false);
        x = join(l.x, h.x) + join(l.y, h.y);
    }
#define HBT_DPP(v, ctrl) (uint32_t) __builtin_amdgcn_mov_dpp((int)(v), ctrl, 0xF, 0xF, true)
    x += join(HBT_DPP(lo(x), 0x128), HBT_DPP(hi(x), 0x128));  // row_ror:8
    {  // l ^ 7 (row_half_mirror), then ^ 3 (quad_perm 3 2 1 0)
        const uint32_t l = HBT_DPP(lo(x), 0x141), h = HBT_DPP(hi(x), 0x141);
        x += join(HBT_DPP(l, 0x1B), HBT_DPP(h, 0x1B));
    }
    x += join(HBT_DPP(lo(x), 0x4E), HBT_DPP(hi(x), 0x4E));  // quad_perm 2 3 0 1
    x += join(HBT_DPP(lo(x), 0xB1), HBT_DPP(hi(x), 0xB1));  // quad_perm 1 0 3 2
#undef HBT_DPP
    return x;
}

// ---------------------------------------------------------------------------
// column sums, any rows of d > 1024: one work-group = 64 columns x one chunk of
// rows, 4 row phases
// ---------------------------------------------------------------------------
template <typename Tin>
__global__ __launch_bounds__(256) void k_colsum(const PairDesc* __restrict__ pairs,
                                                int npairs, int d,
                                                double* __restrict__ partial,
                                                int32_t* __restrict__ chunk_bad, const PairTables tab) {
    write_tables(tab);
    PairDesc pd;
    const SumChunk ch = chunk_of(tab, pairs, npairs, blockIdx.x, &pd);
    const Tin* base = (const Tin*)(ch.side ? pd.Y : pd.X);
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    if (blockIdx.y == 0) {  // the first column tile also tests whole rows (wave ty: rows ty, ty + 4, ...)
        bool bad = false;
        for (int r = ch.r0 + ty; r < ch.r1; r += 4) {
            double ss = 0.0;
            for (int cc = tx; cc < d; cc += 64) {
                const double a = (double)base[(int64_t)r * d + cc];
                ss += a * a;
            }
            ss = wave_sum_f64(ss);
            bad |= not_unit(ss);
        }
        bad = __syncthreads_or(bad);
        if (threadIdx.x == 0) chunk_bad[blockIdx.x] = bad ? 1 : 0;
    }
    const int c = blockIdx.y * 64 + tx;
    double s0 = 0.0, s1 = 0.0;
    if (c < d) {
        int r = ch.r0 + ty;
        for (; r + 4 < ch.r1; r += 8) {
            const double a = (double)base[(int64_t)r * d + c];
            const double b = (double)base[(int64_t)(r + 4) * d + c];
            s0 += a;
            s1 += b;
        }
        if (r < ch.r1) s0 += (double)base[(int64_t)r * d + c];
    }
    __shared__ double red[4][64];
    red[ty][tx] = s0 + s1;
    __syncthreads();
    if (ty == 0 && c < d)
        partial[(int64_t)blockIdx.x * d + c] = (red[0][tx] + red[1][tx]) + (red[2][tx] + red[3][tx]);
}

// The same sums for rows of d <= 1024 that the 16-byte path does not take: one
// work-group = one chunk x all columns, each row read once for the sums and its
// test.  A chunk's sum is eight chains of rows, r0 + w, r0 + w + 8, ... (the two
// accumulators of each phase above), one to a wave, four rows in flight, added
// in k_colsum's order; so both give the same bits.  Bound by the latency of a
// wave's loads: n = 777, m = 1333, d = 301, 46 us as 64-column work-groups whose
// first tested the chunk's rows one by one, 8.7 us so.
template <typename Tin, int J>
__global__ __launch_bounds__(512) void k_colsum_rows(const PairDesc* __restrict__ pairs, int npairs, int d,
                                                     double* __restrict__ partial,
                                                     int32_t* __restrict__ chunk_bad, const PairTables tab) {
    __shared__ double red[4][256 * J];
    write_tables(tab);
    PairDesc pd;
    const SumChunk ch = chunk_of(tab, pairs, npairs, blockIdx.x, &pd);
    const Tin* base = (const Tin*)(ch.side ? pd.Y : pd.X);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double acc[J][4];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.0;
    bool bad = false;
    for (int r = ch.r0 + wave; r < ch.r1; r += 32) {
        Tin x[4][J][4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rr = r + 8 * q;
            load_cols<J>(x[q], base + (int64_t)(rr < ch.r1 ? rr : r) * d, d, rr < ch.r1);
        }
        double ss[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            ss[q] = 0.0;
            if (r + 8 * q >= ch.r1) continue;  // wave-uniform: nothing added past the chunk
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double a = (double)x[q][j][e];
                    acc[j][e] += a;
                    ss[q] += a * a;
                }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) ss[q] = wave_sum_f64(ss[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) bad |= r + 8 * q < ch.r1 && not_unit(ss[q]);
    }
    auto col = [&](int j, int e) { return 256 * j + 64 * e + lane; };
    if (wave >= 4)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave - 4][col(j, e)] = acc[j][e];
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) chunk_bad[blockIdx.x] = bad ? 1 : 0;
    if (wave < 4)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave][col(j, e)] = acc[j][e] + red[wave][col(j, e)];
    __syncthreads();
    for (int c = threadIdx.x; c < d; c += 512)
        partial[(int64_t)blockIdx.x * d + c] = (red[0][c] + red[1][c]) + (red[2][c] + red[3][c]);
}

hipError_t launch_colsum(int input_dtype, const PairDesc* pairs, int npairs, int nchunks, int d, int d_pad,
                         double* partial, int32_t* chunk_bad, hipStream_t s, const PairTables& tab) {
    if (nchunks <= 0) return hipSuccess;
    const bool f64 = input_dtype == HBT_IN_F64;
    auto go = [&](auto kern, dim3 grid, int threads) {
        hipLaunchKernelGGL(kern, grid, dim3(threads), 0, s, pairs, npairs, d, partial, chunk_bad, tab);
    };
    const dim3 tiles(nchunks, (d + 63) / 64), chunks(nchunks);
    switch ((d_pad + 255) / 256) {
        case 1: f64 ? go(k_colsum_rows<double, 1>, chunks, 512) : go(k_colsum_rows<float, 1>, chunks, 512); break;
        case 2: f64 ? go(k_colsum_rows<double, 2>, chunks, 512) : go(k_colsum_rows<float, 2>, chunks, 512); break;
        case 3: f64 ? go(k_colsum_rows<double, 3>, chunks, 512) : go(k_colsum_rows<float, 3>, chunks, 512); break;
        case 4: f64 ? go(k_colsum_rows<double, 4>, chunks, 512) : go(k_colsum_rows<float, 4>, chunks, 512); break;
        default: f64 ? go(k_colsum<double>, tiles, 256) : go(k_colsum<float>, tiles, 256); break;
    }
    return hipGetLastError();
}

// FP32 rows with d a multiple of 4 and 16-byte aligned rows: one
// work-group = one chunk of rows x all columns; wave w sums rows w, w+4, ...
// of the chunk with 16-byte loads (lane l: columns 4(l + 64 j) .. +3), the
// four waves' sums are added in a fixed order through LDS.
// (red: at least 3 rows of 256 J doubles)
template <int J>
__device__ __forceinline__ void colsum4_chunk(const SumChunk& ch, const PairDesc& pd, int d,
                                              double* __restrict__ partial_row,
                                              double (*red)[256 * J], int32_t* bad_out) {
    const float *xb = (const float*)pd.X, *yb = (const float*)pd.Y;
    const float* base = ch.side ? yb : xb;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    double acc[J][4];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[j][e] = 0.0;
    bool bad = false;
    // rows r, r + 4, r + 8, r + 12 per step, all loads issued first (rows past
    // the chunk read zero, see load_cols); the additions keep the row order
    for (int r = ch.r0 + wave; r < ch.r1; r += 16) {
        float4 x[4][J];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int rr = r + 4 * q;
            const __amdgpu_buffer_rsrc_t rs =
                row_rsrc(base + (int64_t)(rr < ch.r1 ? rr : r) * d, rr < ch.r1 ? 4 * d : 0);
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const u32x4 u = __builtin_amdgcn_raw_buffer_load_b128(rs, 16 * (lane + 64 * j), 0, 0);
                x[q][j] = make_float4(__uint_as_float(u.x), __uint_as_float(u.y),
                                      __uint_as_float(u.z), __uint_as_float(u.w));
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (r + 4 * q >= ch.r1) continue;  // wave-uniform: nothing added past the chunk
            float ss = 0.0f;
#pragma unroll
            for (int j = 0; j < J; ++j) {
                acc[j][0] += (double)x[q][j].x;
                acc[j][1] += (double)x[q][j].y;
                acc[j][2] += (double)x[q][j].z;
                acc[j][3] += (double)x[q][j].w;
                ss += x[q][j].x * x[q][j].x + x[q][j].y * x[q][j].y + x[q][j].z * x[q][j].z +
                      x[q][j].w * x[q][j].w;
            }
            bad |= not_unit((double)wave_total_f32(ss));
        }
    }
    if (wave > 0)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave - 1][4 * (lane + 64 * j) + e] = acc[j][e];
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) *bad_out = bad ? 1 : 0;
    if (wave == 0)
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 4 * (lane + 64 * j) + e;
                if (c < d) partial_row[c] = (acc[j][e] + red[0][c]) + (red[1][c] + red[2][c]);
            }
}

// hbt_align's column sums of one pair on the 16-byte path.  A CU takes in some
// 37 GB/s by itself, so the 128 rows of an X chunk, 512 KB at d = 1024, are spread
// over four work-groups, one to a phase (rows r0 + f, r0 + f + 4, ... of the chunk
// of k_colsum_store4, in one chain per column); a wave takes 256 columns, and the
// rows' squares meet in LDS for their test, added as colsum4_chunk adds them.
// Their sums are added by k_finalize<kFinPhases>, in the order of the four waves of
// colsum4_chunk.  (n = 3000, m = 2000, d = 1024: 14.3 us with a work-group per
// chunk, 8.0 so; the finalize step 12.8 and 13.4.)
template <int J>
__global__ __launch_bounds__(256) void k_colsum4(const PairDesc* __restrict__ pairs,
                                                 int npairs, int d,
                                                 double* __restrict__ partial,
                                                 int32_t* __restrict__ chunk_bad, const PairTables tab) {
    constexpr int kRun = kSumChunk / 4;  // rows of a phase
    __shared__ union {
        double red[3][256 * J];
        float sq[kRun][J][64];
    } sh;
    write_tables(tab);
    const int b = blockIdx.x;
    PairDesc pd;
    SumChunk ch = chunk_of(tab, pairs, npairs, 0, &pd);  // one pair, whose chunks begin at 0
    double* prow = partial + (int64_t)b * d;
    if (b >= 4 * pd.cx1) {  // work-group-uniform
        ch = chunk_of(pd, 0, b - 3 * pd.cx1);
        colsum4_chunk<J>(ch, pd, d, prow, sh.red, chunk_bad + b);
        return;
    }
    ch = chunk_of(pd, 0, b >> 2);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r0 = ch.r0 + (b & 3), nr = (ch.r1 - r0 + 3) >> 2;  // this phase's rows (may be none)
    const float* base = (const float*)pd.X;
    if (wave < J) {
        const int c0 = 4 * (lane + 64 * wave);
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int i = 0; i < nr; i += 16) {  // 16 rows in flight
            u32x4 u[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const bool in = i + q < nr;
                const __amdgpu_buffer_rsrc_t rs = row_rsrc(base + (int64_t)(r0 + 4 * (in ? i + q : 0)) * d, in ? 4 * d : 0);
                u[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, 4 * c0, 0, 0);
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                if (i + q >= nr) continue;  // uniform: nothing added past the chunk
                const float4 x = make_float4(__uint_as_float(u[q].x), __uint_as_float(u[q].y),
                                             __uint_as_float(u[q].z), __uint_as_float(u[q].w));
                acc[0] += (double)x.x;
                acc[1] += (double)x.y;
                acc[2] += (double)x.z;
                acc[3] += (double)x.w;
                sh.sq[i + q][wave][lane] = x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w;
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (c0 + e < d) prow[c0 + e] = acc[e];
    }
    __syncthreads();
    bool bad = false;
    for (int i = wave; i < nr; i += 4) {
        float ss = 0.0f;
#pragma unroll
        for (int j = 0; j < J; ++j) ss += sh.sq[i][j][lane];
        bad |= not_unit((double)wave_total_f32(ss));
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) chunk_bad[b] = bad ? 1 : 0;
}

bool vector_rows_ok(int input_dtype, int d, int d_pad) {
    return input_dtype == HBT_IN_F32 && d % 4 == 0 && d_pad <= 1024;
}

hipError_t launch_colsum_phases(const PairDesc* pairs, int nx, int ny, int d, int d_pad, double* partial,
                                int32_t* chunk_bad, hipStream_t s, const PairTables& tab) {
    const int npairs = 1;
    const int J = (d_pad + 255) / 256;
    const dim3 g(4 * nx + ny), b(256);
    switch (J) {
        case 1: hipLaunchKernelGGL(k_colsum4<1>, g, b, 0, s, pairs, npairs, d, partial, chunk_bad, tab); break;
        case 2: hipLaunchKernelGGL(k_colsum4<2>, g, b, 0, s, pairs, npairs, d, partial, chunk_bad, tab); break;
        case 3: hipLaunchKernelGGL(k_colsum4<3>, g, b, 0, s, pairs, npairs, d, partial, chunk_bad, tab); break;
        case 4: hipLaunchKernelGGL(k_colsum4<4>, g, b, 0, s, pairs, npairs, d, partial, chunk_bad, tab); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Householder coefficients 2 (v . x_i) / (v . v) of every X row, for pairs
// whose rows are stored unreflected (eq:householder_fast folded into the
// statistic): FP64 dot products of the FP32 rows (d <= 256 J).  One wave takes
// kFoldRows consecutive rows, all in flight, against v in registers, which it
// loads again where its rows pass from one pair to the next.  Bound by the loads
// and, beside the split kernel, by its share of the CUs: 512 pairs of 20 to 5000
// rows of d = 768, 850 to 920 us with one row a wave and v read for each, 212 so.
// ---------------------------------------------------------------------------
constexpr int kFoldRows = 4;  // 8 take more registers than the split kernel's waves leave
template <int J>
__global__ __launch_bounds__(256) void k_fold_coef(const PairDesc* __restrict__ pairs, int npairs,
                                                   const PairState* __restrict__ st,
                                                   const double* __restrict__ v, int d, int d_pad,
                                                   int64_t total, double* __restrict__ coef) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    int64_t r = ((int64_t)blockIdx.x * 4 + wave) * kFoldRows;
    if (r >= total) return;
    const int64_t rend = r + kFoldRows < total ? r + kFoldRows : total;
    int p = upper_index(npairs, r, [&](int k) { return pairs[k].coef0; });
    for (; r < rend; ++p) {  // wave-uniform
        const int64_t r0 = pairs[p].coef0, next = r0 + pairs[p].n;
        const int k = (int)((next < rend ? next : rend) - r);  // rows of this pair
        double w[kFoldRows];
#pragma unroll
        for (int q = 0; q < kFoldRows; ++q) w[q] = 0.0;
        const int identity = st[p].identity;
        if (!identity) {
            const float* x0 = (const float*)pairs[p].X + (r - r0) * d;
            float x[kFoldRows][J][4];
            double vc[J][4];
#pragma unroll
            for (int q = 0; q < kFoldRows; ++q) load_cols<J>(x[q], x0 + (q < k ? q : 0) * (int64_t)d, d, q < k);
            load_cols<J>(vc, v + (int64_t)p * d_pad, d, true);
#pragma unroll
            for (int q = 0; q < kFoldRows; ++q)
#pragma unroll
                for (int j = 0; j < J; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[q] += vc[j][e] * (double)x[q][j][e];
#pragma unroll
            for (int q = 0; q < kFoldRows; ++q) w[q] = wave_sum_f64(w[q]);
        }
        if (lane < k) {
            double wl = w[0];
#pragma unroll
            for (int q = 1; q < kFoldRows; ++q) wl = lane == q ? w[q] : wl;
            coef[r + lane] = identity ? 0.0 : 2.0 * wl / st[p].vv;
        }
        r += k;
    }
}

hipError_t launch_fold_coef(const PairDesc* pairs, int npairs, const PairState* st, const double* v, int d,
                            int d_pad, int64_t total, double* coef, hipStream_t s) {
    if (total <= 0) return hipSuccess;
    const dim3 g((unsigned)((total + 4 * kFoldRows - 1) / (4 * kFoldRows))), b(256);
    switch ((d_pad + 255) / 256) {
        case 1: hipLaunchKernelGGL(k_fold_coef<1>, g, b, 0, s, pairs, npairs, st, v, d, d_pad, total, coef); break;
        case 2: hipLaunchKernelGGL(k_fold_coef<2>, g, b, 0, s, pairs, npairs, st, v, d, d_pad, total, coef); break;
        case 3: hipLaunchKernelGGL(k_fold_coef<3>, g, b, 0, s, pairs, npairs, st, v, d, d_pad, total, coef); break;
        case 4: hipLaunchKernelGGL(k_fold_coef<4>, g, b, 0, s, pairs, npairs, st, v, d, d_pad, total, coef); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// finalize: one work-group per pair
// ---------------------------------------------------------------------------
// Bound by the memory rate of the CUs that read the chunk partials (n = 3000, m =
// 2000, d = 1024: 91 chunks, 745 KB).  kFinPair, for batches, where the pairs fill the chip: one
// work-group per pair, a column of a thread after the other, few registers (the
// split kernel's waves share the CUs).  kFinSplit, for few pairs: work-group
// (x, p) adds 64 columns of pair p, wave w the w-th quarter of X's chunks and of
// Y's, and the last of the pair's work-groups to end does the rest (they count
// themselves on the pair's ticket, each after its sums are visible to the whole
// device; nobody waits for anybody).  That pair: 13 to 14 us alone, 14 to 16 beside
// its splits, against 32 with one work-group.  kFinPhases is kFinSplit on sums of launch_colsum_phases, X's
// chunks by their four phases.  512 pairs, d = 768: 70 us with kFinPair, 1180 with
// kFinSplit, whose fences write back caches full of other pairs' rows, 177 as two
// launches.
// Both sum in one order, so a pair's results do not depend on the call it is in:
// a column's partials as four quarters, each in chunk order; a sum over columns
// as if by fin_threads(d_pad) threads, thread t taking columns t, t + threads, ...,
// then a butterfly in each wave, then the waves in order.
enum FinalizeMode { kFinPair, kFinSplit, kFinPhases };
constexpr int kFinCols = 64;
__host__ __device__ constexpr int fin_threads(int d_pad) { return d_pad >= 1024 ? 1024 : (d_pad + 255) / 256 * 256; }

template <int MODE>
__global__ __launch_bounds__(256) void k_finalize(
    const PairDesc* __restrict__ pairs, const double* __restrict__ partial, const int32_t* __restrict__ chunk_bad,
    int d, int d_pad, int align, int gd, double* sxy, PairState* st, double* v, double* t64, float* t32,
    PairCount* cnt, hbt_result* res, int p0, float* __restrict__ v32, uint32_t* ticket) {
    __shared__ double red[2][16];
    __shared__ double part[2][4][kFinCols];
    __shared__ uint32_t before;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int p = (MODE == kFinPair ? blockIdx.x : blockIdx.y) + p0;
    const PairDesc pd = pairs[p];
    double* sx = sxy + (int64_t)p * 2 * d_pad;
    double* sy = sx + d_pad;
    double* vp = v + (int64_t)p * d_pad;
    double* tp = t64 + (int64_t)p * d_pad;
    float* tq = t32 + (int64_t)p * d_pad;
    const int extra = MODE == kFinPhases ? 3 * pd.cx1 : 0;  // rows of `partial` that X takes more than its chunks
    // Step 1: sums of X and Y
    auto quarter = [&](int k0, int k1, int q, int c) {
        const int per = (k1 - k0 + 3) / 4, a = k0 + q * per, b = a + per < k1 ? a + per : k1;
        double acc = 0.0;
        if (MODE == kFinPhases && k0 == pd.cx0) {  // four chunks of four phases in flight
            for (int k = a; k < b; k += 4) {
                double t[4][4];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int f = 0; f < 4; ++f) t[u][f] = partial[(int64_t)(4 * (k + u < b ? k + u : b - 1) + f) * d + c];
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (k + u < b) acc += (t[u][0] + t[u][1]) + (t[u][2] + t[u][3]);
            }
            return acc;
        }
        for (int k = a; k < b; k += 16) {
            double t[16];
#pragma unroll
            for (int u = 0; u < 16; ++u) t[u] = partial[(int64_t)(extra + (k + u < b ? k + u : b - 1)) * d + c];
#pragma unroll
            for (int u = 0; u < 16; ++u)
                if (k + u < b) acc += t[u];  // uniform
        }
        return acc;
    };
    if constexpr (MODE != kFinPair) {
        const int c = kFinCols * blockIdx.x + lane;
        part[0][wave][lane] = c < d ? quarter(pd.cx0, pd.cx1, wave, c) : 0.0;
        part[1][wave][lane] = c < d ? quarter(pd.cy0, pd.cy1, wave, c) : 0.0;
        __syncthreads();
        if (wave < 2)
            store_shared(&(wave ? sy : sx)[c], (part[wave][0][lane] + part[wave][1][lane]) +
                                                   (part[wave][2][lane] + part[wave][3][lane]));
        stores_done();  // every wave's sums are there before thread 0 counts the work-group
        __syncthreads();
        if (threadIdx.x == 0)
            before = __hip_atomic_fetch_add(&ticket[p], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (before != gridDim.x - 1) return;
    }
    // this thread stands for the threads threadIdx.x + 256 j < nt, j < kSlots;
    // the sums and v of their first columns stay in registers, those of others
    // (d_pad > 1024) pass through memory
    constexpr int kSlots = 4;
    const int nt = fin_threads(d_pad);
    int bad = 0;
    for (int k = pd.cx0 + threadIdx.x; k < pd.cx1 + extra; k += 256) bad |= chunk_bad[k];
    for (int k = pd.cy0 + extra + threadIdx.x; k < pd.cy1 + extra; k += 256) bad |= chunk_bad[k];
    double x4[kSlots], y4[kSlots], v4[kSlots];
    if constexpr (MODE == kFinPair) {
        auto column = [&](int k0, int k1, int c) {  // four chunks of each quarter in flight
            const int per = (k1 - k0 + 3) / 4;
            double q[4] = {0.0, 0.0, 0.0, 0.0};
            for (int i = 0; i < per; i += 4) {
                double t[4][4];
#pragma unroll
                for (int h = 0; h < 4; ++h)
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int k = k0 + h * per + (i + u < per ? i + u : per - 1);
                        t[h][u] = partial[(int64_t)(k < k1 ? k : k1 - 1) * d + c];
                    }
#pragma unroll
                for (int h = 0; h < 4; ++h)
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (i + u < per && k0 + h * per + i + u < k1) q[h] += t[h][u];  // uniform
            }
            return (q[0] + q[1]) + (q[2] + q[3]);
        };
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const int c = threadIdx.x + 256 * j;
            x4[j] = c < d ? column(pd.cx0, pd.cx1, c) : 0.0;
            y4[j] = c < d ? column(pd.cy0, pd.cy1, c) : 0.0;
        }
        for (int c = threadIdx.x + 1024; c < d_pad; c += 256) {
            sx[c] = c < d ? column(pd.cx0, pd.cx1, c) : 0.0;
            sy[c] = c < d ? column(pd.cy0, pd.cy1, c) : 0.0;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const int c = threadIdx.x + 256 * j;
            x4[j] = c < d_pad ? load_shared(sx + c) : 0.0;
            y4[j] = c < d_pad ? load_shared(sy + c) : 0.0;
        }
    }
    auto columns = [&](auto f) {  // f(slot, c, x, y, v) of each column; f may set v
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            const int c0 = threadIdx.x + 256 * j;
            if (256 * j >= nt) continue;
            if (c0 < d_pad) f(j, c0, x4[j], y4[j], v4[j]);
            for (int c = c0 + nt; c < d_pad; c += nt) {
                if (MODE == kFinPair) f(j, c, sx[c], sy[c], vp[c]);
                else f(j, c, load_shared(sx + c), load_shared(sy + c), vp[c]);
            }
        }
    };
    // sums of x (and of y) over the slots of all threads; every thread gets them
    auto total = [&](double (&x)[kSlots], double (&y)[kSlots], auto both, double& sx_, double& sy_) {
        constexpr bool two = decltype(both)::value;
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            if (256 * j >= nt) continue;  // uniform: nt is a multiple of 256
            x[j] = wave_sum_f64(x[j]);
            if (two) y[j] = wave_sum_f64(y[j]);
        }
        __syncthreads();  // the previous total's readers are done with red
        if (lane == 0)
#pragma unroll
            for (int j = 0; j < kSlots; ++j) {
                if (256 * j >= nt) continue;
                red[0][wave + 4 * j] = x[j];
                if (two) red[1][wave + 4 * j] = y[j];
            }
        __syncthreads();
        sx_ = sy_ = 0.0;
        for (int q = 0; q < nt / 64; ++q) {
            sx_ += red[0][q];
            if (two) sy_ += red[1][q];
        }
    };
    constexpr std::true_type two{};
    constexpr std::false_type one{};
    double a1[kSlots], a2[kSlots], ssx, ssy, vv, w, vt, none;
    auto clear = [&](double (&x)[kSlots]) {
#pragma unroll
        for (int j = 0; j < kSlots; ++j) x[j] = 0.0;
    };
    clear(a1);
    clear(a2);
    columns([&](int j, int, double x, double y, double&) {
        a1[j] += x * x;
        a2[j] += y * y;
    });
    bad = __syncthreads_or(bad);
    total(a1, a2, two, ssx, ssy);
    const double nx = sqrt(ssx), ny = sqrt(ssy);
    const double r_x = nx / (double)pd.n, r_y = ny / (double)pd.m;
    // mean directions and v = mu_x - mu_y (Eq. for u, before normalisation),
    // v . v and v . s_x
    clear(a1);
    clear(a2);
    columns([&](int j, int, double x, double y, double& vc) {
        const double mx = nx > 0.0 ? x / nx : 0.0;
        const double my = ny > 0.0 ? y / ny : 0.0;
        vc = mx - my;
        a1[j] += vc * vc;
        a2[j] += vc * x;
    });
    total(a1, a2, two, vv, w);
    const int identity = (!align) || !(sqrt(vv) > 1e-12) || !(r_x > 0.0) || !(r_y > 0.0);
    // t = H s_x + s_y: the pooled total of Z = [X'; Y]
    const double coef = identity ? 0.0 : 2.0 * w / vv;
    clear(a1);
    columns([&](int j, int c, double x, double y, double& vc) {
        const double tc = (x - coef * vc) + y;
        if (c < nt) vp[c] = vc;
        tp[c] = tc;
        tq[c] = (float)tc;
        a1[j] += vc * tc;
        if (v32) v32[(int64_t)p * d_pad + c] = (float)vc;
    });
    total(a1, a2, one, vt, none);
    // f(r_x) in lane 0 and f(r_y) in lane 1 of the first wave
    const double f = wave == 0 ? log_g(lane & 1 ? r_y : r_x, (double)d, gd) : 0.0;
    const double fx = __shfl(f, 0, 64), fy = __shfl(f, 1, 64);
    if (threadIdx.x == 0) {
        const double scale = fabs(fx) + fabs(fy);
        PairState q;
        q.r_x = r_x;
        q.r_y = r_y;
        q.t_obs = fy - fx;  // log v(X') - log v(Y), v = 1/g_d(r)
        q.tau = 1e-10 * (scale > 1.0 ? scale : 1.0);
        q.vv = vv;
        q.f_x = fx;
        q.f_y = fy;
        q.vt = vt;
        q.identity = identity;
        q.status = (r_x > 0.0 && r_x < 1.0 && r_y > 0.0 && r_y < 1.0)
                       ? (bad ? HBT_ERR_NOT_UNIT : HBT_OK)
                       : HBT_ERR_DEGENERATE;
        q._pad2[0] = q._pad2[1] = 0;
        st[p] = q;
        cnt[p].count = 0;
        cnt[p].n_recheck = 0;
        cnt[p].sum_dt = 0.0;
        cnt[p].sum_dt2 = 0.0;
        hbt_result r;
        r.t_obs = q.t_obs;
        r.r_x = r_x;
        r.r_y = r_y;
        r.p = 0.0;
        r.tau = q.tau;
        r.mu_cos = 1.0 - 0.5 * vv;  // |mu_x - mu_y|^2 = 2 - 2 cos
        r.t_mean = 0.0;
        r.t_sd = 0.0;
        r.count = 0;
        r.B = 0;
        r.n_recheck = 0;
        r.n = pd.n;
        r.m = pd.m;
        r.status = q.status;
        r.h_identity = identity;
        res[p] = r;
    }
}

hipError_t launch_finalize(const PairDesc* pairs, int npairs, const double* partial,
                           const int32_t* chunk_bad, int d,
                           int d_pad, int align, int gd, double* sxy, PairState* st, double* v,
                           double* t64, float* t32, PairCount* cnt, hbt_result* res, uint32_t* ticket,
                           hipStream_t s, int p0, float* v32, bool phases) {
    if (npairs <= 0) return hipSuccess;
    auto go = [&](auto kern, dim3 grid) {
        hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, pairs, partial, chunk_bad, d, d_pad, align, gd, sxy, st, v, t64,
                           t32, cnt, res, p0, v32, ticket);
    };
    if (phases)
        go(k_finalize<kFinPhases>, dim3((d_pad + kFinCols - 1) / kFinCols, npairs));
    else if (npairs <= 8)
        go(k_finalize<kFinSplit>, dim3((d_pad + kFinCols - 1) / kFinCols, npairs));
    else
        go(k_finalize<kFinPair>, dim3(npairs));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// reflection + storage: one work-group per octet of 8 pooled rows
// Two values' e4m3 lo bytes: lo = z - hi (hi the stored, scaled bf16 of each,
// times inv to undo the plane scale; exact in FP32), rounded to nearest even
// as e4m3 of lo 2^kE4m3LoShift, at group rows ra, rb of the 32-row group whose
// first lo unit (of this column) plo points at.
__device__ __forceinline__ void store_e4m3_lo2(unsigned char* plo, int d_pad, int ra, int rb, float za,
                                               float zb, uint32_t hi2, float inva, float invb) {
    const float ha = __uint_as_float(hi2 << 16) * inva;
    const float hb = __uint_as_float(hi2 & 0xffff0000u) * invb;
    constexpr float up = (float)(1 << kE4m3LoShift);
    const uint32_t q = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32((za - ha) * up, (zb - hb) * up, 0, false);
    plo[(int64_t)f8_unit(ra) * d_pad * 16 + f8_byte(ra)] = (unsigned char)(q & 0xffu);
    plo[(int64_t)f8_unit(rb) * d_pad * 16 + f8_byte(rb)] = (unsigned char)((q >> 8) & 0xffu);
}

// ---------------------------------------------------------------------------
// Z storage formats:
//   HBT_F64    : double [Np][d_pad]
//   HBT_F32    : float  [Np][d_pad]
//   HBT_BF16X2 : two planes (hi, then lo at +zplane_elems) of bf16
//                [Np/8][d_pad][8]: the 8 values of a storage octet are
//                contiguous per column, the operand layout of the bf16 MFMA;
//                storage octet 4 g + o4 holds rows 32 g + bf16_plane_row(o4, k)
//                of the pair, scaled by bf16_plane_scale(o4, k) (k = 0..7).
//   HBT_BF16_E4M3: the HBT_BF16X2 hi plane, then at byte 2 zplane_elems the
//                e4m3 lo plane [Np/16][d_pad][16] (f8_unit, f8_byte).
//   HBT_I8X3   : three planes (q0, q1, q2 at +zplane_elems bytes each) of
//                int8 digits [Np/16][d_pad][16]; storage octet 4 g + o4
//                fills bytes 8 (o4 & 1) .. +7 of unit 2 g + o4 / 2 with rows
//                32 g + i8_plane_row(o4, k).
// A work-group (or wave) handles the 8 rows of one storage octet for every
// format; the row-major formats simply write each row in its place.
template <typename Tin, int PREC>
__global__ __launch_bounds__(256) void k_reflect(const PairDesc* __restrict__ pairs, int npairs,
                                                 const PairState* __restrict__ st,
                                                 const double* __restrict__ v, int d, int d_pad,
                                                 double* __restrict__ coef, void* zstore,
                                                 int64_t zplane_elems, float* __restrict__ z32) {
    __shared__ double cf[8];
    const int64_t oct = blockIdx.x;
    const int p = upper_index(npairs, oct * 8, [&](int k) { return pairs[k].zrow0; });
    const PairDesc pd = pairs[p];
    const int identity = st[p].identity;
    const double vv = st[p].vv;
    const double* vp = v + (int64_t)p * d_pad;
    const int lo8 = (int)(oct - pd.zrow0 / 8);  // storage octet within the pair
    const int g0 = 32 * (lo8 >> 2), o4 = lo8 & 3;
    const int N = pd.n + pd.m;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // coefficients 2 (v . x_i) / (v . v) of the X rows (eq:householder_fast)
    for (int r = wave; r < 8; r += 4) {
        const int i = g0 + (PREC == HBT_I8X3 ? i8_plane_row(o4, r) : bf16_plane_row(o4, r));
        double w = 0.0;
        if (!identity && i < pd.n) {
            const Tin* x = (const Tin*)pd.X + (int64_t)i * d;
            for (int c = lane; c < d; c += 64) w += vp[c] * (double)x[c];
            w = wave_sum_f64(w);
        }
        if (lane == 0) {
            const double k = (!identity && i < pd.n) ? 2.0 * w / vv : 0.0;
            cf[r] = k;
            if (i < pd.n) coef[pd.coef0 + i] = k;
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < d_pad; c += 256) {
        double z[8];
        const double vc = c < d ? vp[c] : 0.0;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = g0 + (PREC == HBT_I8X3 ? i8_plane_row(o4, r) : bf16_plane_row(o4, r));
            double val = 0.0;
            if (c < d) {
                if (i < pd.n)
                    val = (double)((const Tin*)pd.X)[(int64_t)i * d + c] - cf[r] * vc;
                else if (i < N)
                    val = (double)((const Tin*)pd.Y)[(int64_t)(i - pd.n) * d + c];
            }
            z[r] = val;
        }
        if (z32) {  // row-major FP32 copy for the point-to-centroid route
#pragma unroll
            for (int r = 0; r < 8; ++r)
                z32[(pd.zrow0 + g0 + bf16_plane_row(o4, r)) * (int64_t)d_pad + c] = (float)z[r];
        }
        if (PREC == HBT_I8X3) {
            uint32_t w[3][2] = {{0u, 0u}, {0u, 0u}, {0u, 0u}};
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                uint32_t q[3];
                i8_digits(z[r], q[0], q[1], q[2]);
#pragma unroll
                for (int k = 0; k < 3; ++k) w[k][r >> 2] |= q[k] << (8 * (r & 3));
            }
            uint2* dst = (uint2*)((char*)zstore + ((oct >> 1) * d_pad + c) * 16 + 8 * (oct & 1));
#pragma unroll
            for (int k = 0; k < 3; ++k)
                *(uint2*)((char*)dst + k * zplane_elems) = make_uint2(w[k][0], w[k][1]);
        } else if (PREC == HBT_BF16X2) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int r = 0; r < 8; r += 2) {
                const float a = (float)z[r] * bf16_plane_scale(o4, r);
                const float b = (float)z[r + 1] * bf16_plane_scale(o4, r + 1);
                const uint2 hl = split_bf16x2(a, b);
                hi[r / 2] = hl.x;
                lo[r / 2] = hl.y;
            }
            uint4* ph = (uint4*)zstore + oct * d_pad + c;
            *ph = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            *(ph + zplane_elems / 8) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        } else if (PREC == HBT_BF16_E4M3) {
            uint32_t hi[4];
            unsigned char* plo = (unsigned char*)zstore + 2 * zplane_elems + (((oct >> 2) * 2) * d_pad + c) * 16;
#pragma unroll
            for (int r = 0; r < 8; r += 2) {
                const float a = (float)z[r], b = (float)z[r + 1];
                hi[r / 2] = split_bf16x2(a * bf16_plane_scale(o4, r), b * bf16_plane_scale(o4, r + 1)).x;
                store_e4m3_lo2(plo, d_pad, bf16_plane_row(o4, r), bf16_plane_row(o4, r + 1), a, b, hi[r / 2],
                               bf16_plane_inv_scale(o4, r), bf16_plane_inv_scale(o4, r + 1));
            }
            *((uint4*)zstore + oct * d_pad + c) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        } else if (PREC == HBT_F32) {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                ((float*)zstore)[(pd.zrow0 + g0 + bf16_plane_row(o4, r)) * (int64_t)d_pad + c] = (float)z[r];
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r)
                ((double*)zstore)[(pd.zrow0 + g0 + bf16_plane_row(o4, r)) * (int64_t)d_pad + c] = z[r];
        }
    }
}

template <typename Tin>
static hipError_t launch_reflect_t(int precision, const PairDesc* pairs, int npairs,
                                   int64_t total_octets, const PairState* st, const double* v,
                                   int d, int d_pad, double* coef, void* z, int64_t ze, float* z32,
                                   hipStream_t s) {
    dim3 g((unsigned)total_octets), b(256);
    switch (precision) {
        case HBT_F64:
            hipLaunchKernelGGL((k_reflect<Tin, HBT_F64>), g, b, 0, s, pairs, npairs, st, v, d, d_pad,
                               coef, z, ze, z32);
            break;
        case HBT_F32:
            hipLaunchKernelGGL((k_reflect<Tin, HBT_F32>), g, b, 0, s, pairs, npairs, st, v, d, d_pad,
                               coef, z, ze, z32);
            break;
        case HBT_I8X3:
            hipLaunchKernelGGL((k_reflect<Tin, HBT_I8X3>), g, b, 0, s, pairs, npairs, st, v, d,
                               d_pad, coef, z, ze, z32);
            break;
        case HBT_BF16_E4M3:
            hipLaunchKernelGGL((k_reflect<Tin, HBT_BF16_E4M3>), g, b, 0, s, pairs, npairs, st, v, d,
                               d_pad, coef, z, ze, z32);
            break;
        default:
            hipLaunchKernelGGL((k_reflect<Tin, HBT_BF16X2>), g, b, 0, s, pairs, npairs, st, v, d,
                               d_pad, coef, z, ze, z32);
            break;
    }
    return hipGetLastError();
}

// The same reflection and storage for FP32 rows with d a multiple of 4 and
// 16-byte aligned rows (the condition shared with the vector column sums):
// one wave per octet, the octet's 8 rows held in registers (lane l: columns
// 256 j + 64 e + l, j < J, e < 4, each load instruction reading 256
// contiguous bytes of a row); the coefficients are FP64 wave reductions, and
// every store instruction then writes one contiguous run of columns (1 KB per
// plane for split BF16).
// Stores one storage octet of a pair: this lane's J x 4 columns of the 8
// rows row_of(0..7) (pair-relative pooled rows), z_r = x_r - k_r vc in FP64,
// in the precision's format.  soct is the octet's index in the whole storage.
template <int PREC, int J, typename Tin, typename RowOf>
__device__ __forceinline__ void store_octet(const Tin (&x)[8][J][4], const double (&k)[8],
                                            const double (&vc)[J][4], int64_t soct, int64_t zrow0,
                                            RowOf row_of, int o4, int d_pad, void* zstore,
                                            int64_t zplane_elems, float* __restrict__ z32) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int c = 256 * j + 64 * e + lane;
            if (256 * j + 64 * e >= d_pad) continue;  // wave-uniform: d_pad is a multiple of 64
            if (PREC == HBT_F64) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int64_t zr = zrow0 + row_of(r);
                    const double z = (double)x[r][j][e] - k[r] * vc[j][e];
                    ((double*)zstore)[zr * d_pad + c] = z;
                    if (z32) z32[zr * d_pad + c] = (float)z;
                }
                continue;
            }
            if (PREC == HBT_I8X3) {  // digits of the FP64 update
                uint32_t w[3][2] = {{0u, 0u}, {0u, 0u}, {0u, 0u}};
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    uint32_t q[3];
                    i8_digits((double)x[r][j][e] - k[r] * vc[j][e], q[0], q[1], q[2]);
#pragma unroll
                    for (int t = 0; t < 3; ++t) w[t][r >> 2] |= q[t] << (8 * (r & 3));
                }
                char* dst = (char*)zstore + ((soct >> 1) * d_pad + c) * 16 + 8 * (soct & 1);
#pragma unroll
                for (int t = 0; t < 3; ++t) *(uint2*)(dst + t * zplane_elems) = make_uint2(w[t][0], w[t][1]);
                continue;
            }
            // FP64 update, rounded to FP32 at once (the storage is FP32 or BF16 hi+lo)
            float zf[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) zf[r] = (float)((double)x[r][j][e] - k[r] * vc[j][e]);
            if (PREC == HBT_F32 || z32) {
#pragma unroll
                for (int r = 0; r < 8; ++r) {
                    const int64_t zr = zrow0 + row_of(r);
                    if (PREC == HBT_F32) ((float*)zstore)[zr * d_pad + c] = zf[r];
                    if (z32) z32[zr * d_pad + c] = zf[r];
                }
            }
            if (PREC == HBT_BF16X2) {
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int r = 0; r < 8; r += 2) {
                    const uint2 hl = split_bf16x2(zf[r] * bf16_plane_scale(o4, r), zf[r + 1] * bf16_plane_scale(o4, r + 1));
                    hi[r / 2] = hl.x;
                    lo[r / 2] = hl.y;
                }
                uint4* ph = (uint4*)zstore + soct * d_pad + c;
                *ph = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                *(ph + zplane_elems / 8) = make_uint4(lo[0], lo[1], lo[2], lo[3]);
            }
            if (PREC == HBT_BF16_E4M3) {
                uint32_t hi[4];
                unsigned char* plo = (unsigned char*)zstore + 2 * zplane_elems + (((soct >> 2) * 2) * d_pad + c) * 16;
#pragma unroll
                for (int r = 0; r < 8; r += 2) {
                    hi[r / 2] = split_bf16x2(zf[r] * bf16_plane_scale(o4, r), zf[r + 1] * bf16_plane_scale(o4, r + 1)).x;
                    store_e4m3_lo2(plo, d_pad, row_of(r) & 31, row_of(r + 1) & 31, zf[r], zf[r + 1], hi[r / 2],
                                   bf16_plane_inv_scale(o4, r), bf16_plane_inv_scale(o4, r + 1));
                }
                *((uint4*)zstore + soct * d_pad + c) = make_uint4(hi[0], hi[1], hi[2], hi[3]);
            }
        }
}

template <int PREC>
__device__ __forceinline__ int plane_row(int o4, int k) {
    return PREC == HBT_I8X3 ? i8_plane_row(o4, k) : bf16_plane_row(o4, k);
}

// The reflection on the 16-byte path: one wave per storage octet of the
// 32-row groups that hold X rows (x_octets(n) per pair, numbered from
// PairDesc::xoct0); the groups that hold only Y rows or padding are stored by
// k_colsum_store4.  ALL (rows that the 16-byte loads do not take): every octet of
// the storage.  Bound by memory; 64 pairs of 20 to 5000 rows of d = 299 in split
// BF16, work-groups of one octet that read its rows twice: 150 us, 67 so.
template <typename Tin, int PREC, int J, bool ALL>
__global__ __launch_bounds__(256) void k_reflect4(const PairDesc* __restrict__ pairs, int npairs,
                                                  int64_t total_octets,
                                                  const PairState* __restrict__ st,
                                                  const double* __restrict__ v, int d, int d_pad,
                                                  double* __restrict__ coef, void* zstore,
                                                  int64_t zplane_elems, float* __restrict__ z32,
                                                  int64_t oct0) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t oct = (int64_t)blockIdx.x * 4 + wave + oct0;
    if (oct >= total_octets) return;
    const int p = ALL ? upper_index(npairs, oct * 8, [&](int k) { return pairs[k].zrow0; })
                      : upper_index(npairs, oct, [&](int k) { return pairs[k].xoct0; });
    const PairDesc pd = pairs[p];
    const int identity = st[p].identity;
    const double vv = st[p].vv;
    const double* vp = v + (int64_t)p * d_pad;
    const int lo8 = (int)(oct - (ALL ? pd.zrow0 / 8 : pd.xoct0));  // storage octet within the pair
    const int g0 = 32 * (lo8 >> 2), o4 = lo8 & 3;
    const int N = pd.n + pd.m;
    auto row_of = [&](int r) { return g0 + plane_row<PREC>(o4, r); };
    auto col = [&](int j, int e) { return 256 * j + 64 * e + lane; };
    Tin x[8][J][4];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = row_of(r);  // wave-uniform; a padding row reads Y's last row and keeps zeros
        const Tin* row = i < pd.n ? (const Tin*)pd.X + (int64_t)i * d
                                  : (const Tin*)pd.Y + (int64_t)((i < N ? i : N - 1) - pd.n) * d;
        load_cols<J>(x[r], row, d, i < N);
    }
    double vc[J][4];
    const __amdgpu_buffer_rsrc_t vrs = row_rsrc(vp, 8 * d);  // columns past d read 0
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            vc[j][e] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(vrs, 8 * col(j, e), 0, 0));
    // coefficients 2 (v . x_i) / (v . v) of the X rows (eq:householder_fast)
    double k[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = row_of(r);
        k[r] = 0.0;
        if (!identity && i < pd.n) {  // wave-uniform
            double w = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) w += vc[j][e] * (double)x[r][j][e];
            k[r] = 2.0 * wave_sum_f64(w) / vv;
        }
    }
    // the update below converts the rows to FP64 again instead of keeping the
    // dot product's FP64 copies alive (twice the registers)
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int j = 0; j < J; ++j)
            asm volatile("" : "+v"(x[r][j][0]), "+v"(x[r][j][1]), "+v"(x[r][j][2]), "+v"(x[r][j][3]));
    if (lane < 8) {
        double kr = k[0];
#pragma unroll
        for (int r = 1; r < 8; ++r) kr = lane == r ? k[r] : kr;
        const int i = row_of(lane);
        if (i < pd.n) coef[pd.coef0 + i] = kr;
    }
    store_octet<PREC, J>(x, k, vc, pd.zrow0 / 8 + lo8, pd.zrow0, row_of, o4, d_pad, zstore,
                         zplane_elems, z32);
}

hipError_t launch_reflect_vec(int precision, const PairDesc* pairs, int npairs,
                              int64_t total_octets, const PairState* st, const double* v, int d,
                              int d_pad, double* coef, void* zstore, int64_t zplane_elems,
                              float* z32, hipStream_t s, int64_t oct0) {
    if (total_octets <= oct0) return hipSuccess;
    const int J = (d_pad + 255) / 256;
    const dim3 g((unsigned)((total_octets - oct0 + 3) / 4)), b(256);
#define HBT_R4(PR, JJ)                                                                         \
    hipLaunchKernelGGL((k_reflect4<float, PR, JJ, false>), g, b, 0, s, pairs, npairs, total_octets, st, v, d, \
                       d_pad, coef, zstore, zplane_elems, z32, oct0)
#define HBT_R4J(PR)                            \
    switch (J) {                               \
        case 1: HBT_R4(PR, 1); break;          \
        case 2: HBT_R4(PR, 2); break;          \
        case 3: HBT_R4(PR, 3); break;          \
        case 4: HBT_R4(PR, 4); break;          \
        default: return hipErrorInvalidValue;  \
    }
    switch (precision) {
        case HBT_F64: HBT_R4J(HBT_F64); break;
        case HBT_F32: HBT_R4J(HBT_F32); break;
        case HBT_I8X3: HBT_R4J(HBT_I8X3); break;
        case HBT_BF16_E4M3: HBT_R4J(HBT_BF16_E4M3); break;
        default: HBT_R4J(HBT_BF16X2); break;
    }
#undef HBT_R4J
#undef HBT_R4
    return hipGetLastError();
}

// Rows that the 16-byte path does not take: whole rows in registers where they
// fit (d <= 1024 in FP32, 512 in FP64), else k_reflect.
hipError_t launch_reflect(int input_dtype, int precision, const PairDesc* pairs, int npairs,
                          int64_t total_octets, const PairState* st, const double* v, int d,
                          int d_pad, double* coef, void* zstore, int64_t zplane_elems,
                          float* z32, hipStream_t s) {
    if (total_octets <= 0) return hipSuccess;
    const bool f64 = input_dtype == HBT_IN_F64;
    const int J = (d_pad + 255) / 256;
    if (J > (f64 ? 2 : 4))
        return f64 ? launch_reflect_t<double>(precision, pairs, npairs, total_octets, st, v, d, d_pad, coef, zstore,
                                              zplane_elems, z32, s)
                   : launch_reflect_t<float>(precision, pairs, npairs, total_octets, st, v, d, d_pad, coef, zstore,
                                             zplane_elems, z32, s);
    const dim3 g((unsigned)((total_octets + 3) / 4)), b(256);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, g, b, 0, s, pairs, npairs, total_octets, st, v, d, d_pad, coef, zstore, zplane_elems,
                           z32, (int64_t)0);
    };
    auto width = [&](auto prec) {
        constexpr int PR = decltype(prec)::value;
        switch (J) {
            case 1: f64 ? go(k_reflect4<double, PR, 1, true>) : go(k_reflect4<float, PR, 1, true>); break;
            case 2: f64 ? go(k_reflect4<double, PR, 2, true>) : go(k_reflect4<float, PR, 2, true>); break;
            case 3: go(k_reflect4<float, PR, 3, true>); break;
            default: go(k_reflect4<float, PR, 4, true>); break;
        }
    };
    switch (precision) {
        case HBT_F64: width(std::integral_constant<int, HBT_F64>{}); break;
        case HBT_F32: width(std::integral_constant<int, HBT_F32>{}); break;
        case HBT_I8X3: width(std::integral_constant<int, HBT_I8X3>{}); break;
        case HBT_BF16_E4M3: width(std::integral_constant<int, HBT_BF16_E4M3>{}); break;
        default: width(std::integral_constant<int, HBT_BF16X2>{}); break;
    }
    return hipGetLastError();
}

// Column sums and, in the same pass, the Z storage of the Y rows (16-byte
// path, group-sum calls).  X chunks are summed by colsum4_chunk.  A Y chunk is
// one 32-row group of the storage: wave w loads octet w (the 8 rows
// plane_row(w, .) of the group), adds its Y rows to the sums and stores the
// octet as it is (H leaves Y unchanged; rows past n + m are the zero
// padding), except in the group that also holds X rows, which the reflection
// stores.  Y's rows are then read once for both purposes.
template <int PREC, int J>
__global__ __launch_bounds__(256) void k_colsum_store4(const PairDesc* __restrict__ pairs,
                                                       int npairs, int d, int d_pad,
                                                       double* __restrict__ partial, void* zstore,
                                                       int64_t zplane_elems,
                                                       float* __restrict__ z32,
                                                       int32_t* __restrict__ chunk_bad, int c0,
                                                       const PairTables tab) {
    __shared__ double red[4][256 * J];
    write_tables(tab);
    const int c = blockIdx.x + c0;
    PairDesc pd;
    const SumChunk ch = chunk_of(tab, pairs, npairs, c, &pd);
    double* prow = partial + (int64_t)c * d;
    if (!ch.side) {  // work-group-uniform
        colsum4_chunk<J>(ch, pd, d, prow, red, chunk_bad + c);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int n = pd.n, N = n + pd.m;
    const int g0 = (n + ch.r0) & ~31;  // the chunk's group
    auto row_of = [&](int r) { return g0 + plane_row<PREC>(wave, r); };
    auto col = [&](int j, int e) { return 256 * j + 64 * e + lane; };
    float x[8][J][4];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = row_of(r);
        const bool y = i >= n && i < N;  // wave-uniform; other rows read Y's first row and keep zeros
        load_cols<J>(x[r], (const float*)pd.Y + (int64_t)(y ? i - n : 0) * d, d, y);
    }
    // each wave's sums go to LDS at once, so they are not live across the stores
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            double t = 0.0;
#pragma unroll
            for (int r = 0; r < 8; ++r) t += (double)x[r][j][e];
            red[wave][col(j, e)] = t;
        }
    bool bad = false;
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = row_of(r);
        if (i < n || i >= N) continue;  // wave-uniform: only this group's Y rows
        float ss = 0.0f;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) ss += x[r][j][e] * x[r][j][e];
        bad |= not_unit((double)wave_total_f32(ss));
    }
    // the stores convert the rows to FP64 again instead of keeping the sums'
    // FP64 copies alive (twice the registers)
#pragma unroll
    for (int r = 0; r < 8; ++r)
#pragma unroll
        for (int j = 0; j < J; ++j)
            asm volatile("" : "+v"(x[r][j][0]), "+v"(x[r][j][1]), "+v"(x[r][j][2]), "+v"(x[r][j][3]));
    if (g0 >= n) {  // wave-uniform
        double k0[8], v0[J][4];
#pragma unroll
        for (int r = 0; r < 8; ++r) k0[r] = 0.0;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) v0[j][e] = 0.0;
        store_octet<PREC, J>(x, k0, v0, pd.zrow0 / 8 + g0 / 8 + wave, pd.zrow0, row_of, wave, d_pad,
                             zstore, zplane_elems, z32);
    }
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) chunk_bad[c] = bad ? 1 : 0;
    for (int cc = threadIdx.x; cc < d; cc += 256)
        prow[cc] = (red[0][cc] + red[1][cc]) + (red[2][cc] + red[3][cc]);
}

hipError_t launch_colsum_store_vec(int precision, const PairDesc* pairs, int npairs, int nchunks,
                                   int d, int d_pad, double* partial, void* zstore,
                                   int64_t zplane_elems, float* z32, int32_t* chunk_bad,
                                   hipStream_t s, int c0, const PairTables& tab) {
    if (nchunks <= 0) return hipSuccess;
    const int J = (d_pad + 255) / 256;
    const dim3 g(nchunks), b(256);
#define HBT_C4(PR, JJ)                                                                         \
    hipLaunchKernelGGL((k_colsum_store4<PR, JJ>), g, b, 0, s, pairs, npairs, d, d_pad, partial, \
                       zstore, zplane_elems, z32, chunk_bad, c0, tab)
#define HBT_C4J(PR)                            \
    switch (J) {                               \
        case 1: HBT_C4(PR, 1); break;          \
        case 2: HBT_C4(PR, 2); break;          \
        case 3: HBT_C4(PR, 3); break;          \
        case 4: HBT_C4(PR, 4); break;          \
        default: return hipErrorInvalidValue;  \
    }
    switch (precision) {
        case HBT_F64: HBT_C4J(HBT_F64); break;
        case HBT_F32: HBT_C4J(HBT_F32); break;
        case HBT_I8X3: HBT_C4J(HBT_I8X3); break;
        case HBT_BF16_E4M3: HBT_C4J(HBT_BF16_E4M3); break;
        default: HBT_C4J(HBT_BF16X2); break;
    }
#undef HBT_C4J
#undef HBT_C4
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// hbt_align's output: X' = H X in the input dtype, one wave per row.  Rows of
// d <= 256 J are read once and kept in registers; J = 0, any d, reads them twice.
// Bound by the latency of a row's loads and its sum over the wave: n = 3000,
// d = 1024, float, 11.5 us reading them twice, 6.1 so.
// ---------------------------------------------------------------------------
template <typename Tin, int J>
__global__ __launch_bounds__(256) void k_reflect_out(const PairDesc* __restrict__ pair,
                                                     const PairState* __restrict__ st,
                                                     const double* __restrict__ v, int n, int d,
                                                     Tin* X_out, double* v_out) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = blockIdx.x * 4 + wave;
    if (v_out && blockIdx.x == 0)
        for (int c = threadIdx.x; c < d; c += 256) v_out[c] = v[c];
    if (i >= n) return;
    const Tin* x = (const Tin*)pair->X + (int64_t)i * d;
    Tin* y = X_out + (int64_t)i * d;
    const int identity = st->identity;
    double w = 0.0;
    // every lane has read its share of the row (inside the dot product) before
    // any write, so X_out may alias X
    if constexpr (J > 0) {
        Tin xr[J][4];
        double vc[J][4];
        load_cols<J>(xr, x, d, true);
        load_cols<J>(vc, v, d, true);
        if (!identity) {
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) w += vc[j][e] * (double)xr[j][e];
            w = wave_sum_f64(w);
        }
        const double k = identity ? 0.0 : 2.0 * w / st->vv;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int c = 256 * j + 64 * e + lane;
                if (c < d) y[c] = (Tin)((double)xr[j][e] - k * vc[j][e]);
            }
    } else {
        if (!identity) {
            for (int c = lane; c < d; c += 64) w += v[c] * (double)x[c];
            w = wave_sum_f64(w);
        }
        const double k = identity ? 0.0 : 2.0 * w / st->vv;
        for (int c = lane; c < d; c += 64) y[c] = (Tin)((double)x[c] - k * v[c]);
    }
}

hipError_t launch_reflect_out(int input_dtype, const PairDesc* pair, const PairState* st,
                              const double* v, int n, int d, void* X_out, double* v_out,
                              hipStream_t s) {
    auto go = [&](auto kern, auto* out) {
        hipLaunchKernelGGL(kern, dim3((n + 3) / 4), dim3(256), 0, s, pair, st, v, n, d, out, v_out);
    };
    const bool f64 = input_dtype == HBT_IN_F64;
    double* xd = (double*)X_out;
    float* xf = (float*)X_out;
    switch ((d + 255) / 256) {
        case 1: f64 ? go(k_reflect_out<double, 1>, xd) : go(k_reflect_out<float, 1>, xf); break;
        case 2: f64 ? go(k_reflect_out<double, 2>, xd) : go(k_reflect_out<float, 2>, xf); break;
        case 3: f64 ? go(k_reflect_out<double, 3>, xd) : go(k_reflect_out<float, 3>, xf); break;
        case 4: f64 ? go(k_reflect_out<double, 4>, xd) : go(k_reflect_out<float, 4>, xf); break;
        default: f64 ? go(k_reflect_out<double, 0>, xd) : go(k_reflect_out<float, 0>, xf); break;
    }
    return hipGetLastError();
}

}  // namespace hbt
