// Learned permutation-budget allocator: features of a pair from its
// alignment results, a 12 -> 64 -> 64 -> 2 ReLU network (forward, gradient,
// Adam), and the number of permutations implied by the network's estimate
// of the pair's permutation null distribution.
//
// The network predicts (mean, log sd) of the permuted statistics T_b of a
// pair (Sec. 3.1, Algorithm 1 Step 5) from quantities of Algorithm 1 Steps
// 1-4.  The exact permutation p-value (eq:pvalue) remains the decision: the
// prediction only sets how many splits a pair gets.
//
// Parameter vector theta (float), row-major blocks in this order:
//   shift[12], scale[12]      input standardisation x~ = (x - shift) * scale
//   oshift[2], oscale[2]      output standardisation out = oshift + oscale * y~
//   W1[64][12], b1[64]        hidden layer 1 (ReLU)
//   W2[64][64], b2[64]        hidden layer 2 (ReLU)
//   W3[2][64],  b3[2]         y~ (standardised (mean, log sd))
#include "hbt_launch.h"

namespace hbt {

constexpr int kF = HBT_MLP_FEATURES, kH = 64, kO = 2;
constexpr int oShift = 0, oScale = kF, oOShift = 2 * kF, oOScale = oOShift + kO, oW1 = oOScale + kO,
              oB1 = oW1 + kH * kF, oW2 = oB1 + kH,
              oB2 = oW2 + kH * kH, oW3 = oB2 + kH, oB3 = oW3 + kO * kH, kP = oB3 + kO;
static_assert(kP == HBT_MLP_PARAMS, "parameter layout");
static_assert(oW1 == HBT_MLP_TRAINABLE_OFFSET, "trainable offset");

// ---------------------------------------------------------------------------
// features (FP64 arithmetic, stored as float)
// ---------------------------------------------------------------------------
__global__ void k_features(int64_t npairs, const hbt_result* __restrict__ res, double d, int gd,
                           float* __restrict__ feat) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npairs) return;
    const hbt_result r = res[p];
    const double n = (double)r.n, m = (double)r.m, N = n + m;
    const double f[kF] = {log(n),
                          log(m),
                          r.r_x,
                          r.r_y,
                          (n * r.r_x + m * r.r_y) / N,  // pooled MRL after alignment
                          r.mu_cos,
                          log_g(r.r_x, d, gd),
                          log_g(r.r_y, d, gd),
                          r.t_obs,
                          n / N,
                          log1p(-r.r_x * r.r_x),
                          log1p(-r.r_y * r.r_y)};
#pragma unroll
    for (int k = 0; k < kF; ++k) feat[p * kF + k] = (float)f[k];
}

// training targets of a pair: (mean, log sd) of its permuted statistics
__global__ void k_null_targets(int64_t npairs, const hbt_result* __restrict__ res,
                               float* __restrict__ target) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npairs) return;
    target[p * kO] = (float)res[p].t_mean;
    target[p * kO + 1] = (float)log(res[p].t_sd);
}

hipError_t launch_null_targets(int64_t npairs, const hbt_result* res, float* target, hipStream_t s) {
    hipLaunchKernelGGL(k_null_targets, dim3((unsigned)((npairs + 255) / 256)), dim3(256), 0, s, npairs,
                       res, target);
    return hipGetLastError();
}

// Column statistics of a rows x cols matrix: shift[k] = mean, scale[k] =
// 1 / sd (invert) or sd (population sd); one work-group per column,
// fixed-order FP64 reductions.  A constant column gets scale 1.
__global__ __launch_bounds__(256) void k_col_norm(int64_t rows, int cols, const float* __restrict__ feat,
                                                  float* __restrict__ shift, float* __restrict__ scale,
                                                  int invert) {
    __shared__ double red[256];
    const int k = blockIdx.x;
    auto block_sum = [&](double x) {
        red[threadIdx.x] = x;
        __syncthreads();
        for (int o = 128; o > 0; o >>= 1) {
            if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
            __syncthreads();
        }
        const double s = red[0];
        __syncthreads();
        return s;
    };
    double s = 0.0;
    for (int64_t r = threadIdx.x; r < rows; r += 256) s += (double)feat[r * cols + k];
    const double mean = block_sum(s) / (double)rows;
    double q = 0.0;
    for (int64_t r = threadIdx.x; r < rows; r += 256) {
        const double x = (double)feat[r * cols + k] - mean;
        q += x * x;
    }
    const double sd = sqrt(block_sum(q) / (double)rows);
    if (threadIdx.x == 0) {
        shift[k] = (float)mean;
        scale[k] = sd > 0.0 ? (float)(invert ? 1.0 / sd : sd) : 1.0f;
    }
}

// ---------------------------------------------------------------------------
// network.  A work-group of eight waves takes a chunk of 64 rows: lane l of
// every wave is row l of the chunk, and wave w computes units 8 w .. 8 w + 7
// of a layer, so that a parameter is wave-uniform (a scalar load, used as the
// multiplier's scalar operand) and a chunk spreads over 512 lanes.  The
// activations pass between the waves through LDS.  Every unit's sum is one
// chain of FP32 fma over its inputs in ascending order, from the bias, so a
// row's outputs do not depend on the chunking.
// ---------------------------------------------------------------------------
constexpr int kRowsWg = 64;   // rows of a chunk
constexpr int kMlpWaves = 8;
constexpr int kUnits = kH / kMlpWaves;  // units of a layer per wave
// One layer's activations of a chunk, unit-major with 68 floats a unit: the
// lanes of a wave read one unit of 64 rows (consecutive words, the unit an
// immediate offset), or 16 units of 4 consecutive rows (words 68 u + r on 64
// distinct banks, an operand of the gradient's matrix product).
constexpr int kActLd = kRowsWg + 4;
typedef float Act[kH * kActLd];
__device__ __forceinline__ int act_at(int r, int u) { return u * kActLd + r; }

// Standardised inputs of a row, and this wave's units of z1 = relu(W1 x~ + b1)
// for it into z1s (0 for a lane without a row).  The loops over units are not
// unrolled: the parameters of one unit at a time fit the scalar registers.
__device__ __forceinline__ void layer1(const float* __restrict__ th, const float* x, int lane, int u0, bool live,
                                       float (&xs)[kF], Act& z1s) {
#pragma unroll
    for (int i = 0; i < kF; ++i) xs[i] = (x[i] - th[oShift + i]) * th[oScale + i];
#pragma unroll 2
    for (int u = u0; u < u0 + kUnits; ++u) {
        float s = th[oB1 + u];
#pragma unroll
        for (int i = 0; i < kF; ++i) s = fmaf(th[oW1 + u * kF + i], xs[i], s);
        z1s[act_at(lane, u)] = live && s > 0.0f ? s : 0.0f;
    }
}

// This wave's units of z2 = relu(W2 z1 + b2) for the lane's row, into z2s.
__device__ __forceinline__ void layer2(const float* __restrict__ th, const Act& z1s, int lane, int u0, bool live,
                                       Act& z2s) {
    float z1[kH];
#pragma unroll
    for (int i = 0; i < kH; ++i) z1[i] = z1s[act_at(lane, i)];
#pragma unroll 1
    for (int u = u0; u < u0 + kUnits; ++u) {
        float s = th[oB2 + u];
#pragma unroll
        for (int i = 0; i < kH; ++i) s = fmaf(th[oW2 + u * kH + i], z1[i], s);
        z2s[act_at(lane, u)] = live && s > 0.0f ? s : 0.0f;
    }
}

// Output o (0, 1) of the lane's row before the output standardisation.
__device__ __forceinline__ float layer3(const float* __restrict__ th, const Act& z2s, int lane, int o) {
    float s = th[oB3 + o];
#pragma unroll 16
    for (int j = 0; j < kH; ++j) s = fmaf(th[oW3 + o * kH + j], z2s[act_at(lane, j)], s);
    return s;
}

// Bound by launch and latency (4096 rows: 41 MFLOP).  One thread per row with
// the parameters in LDS took 31 us for 4096 rows (16 work-groups, each lane
// 5,000 fma one after the other); 64-row chunks over 64 work-groups 9.3 us.
__global__ __launch_bounds__(64 * kMlpWaves, 4) void k_mlp_forward(int64_t rows, const float* __restrict__ feat,
                                                     const float* __restrict__ theta,
                                                     float* __restrict__ out) {
    __shared__ Act z1s, z2s;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int u0 = kUnits * wave;
    const int64_t r = (int64_t)blockIdx.x * kRowsWg + lane;
    const bool live = r < rows;
    float xs[kF];
    layer1(theta, feat + (live ? r : rows - 1) * kF, lane, u0, live, xs, z1s);
    __syncthreads();
    layer2(theta, z1s, lane, u0, live, z2s);
    __syncthreads();
    if (wave < kO && live)
        out[r * kO + wave] = fmaf(theta[oOScale + wave], layer3(theta, z2s, lane, wave), theta[oOShift + wave]);
}

// The same outputs, bit for bit, with one thread per row and the parameters in LDS,
// for calls of many rows.  Bound by the FP32 rate (62 TFLOP/s at a million rows): no
// activation leaves its thread and no wave waits for another, but a work-group takes
// 256 rows, so few rows leave CUs idle.  131,072 rows 31 us (25.7 in chunks), 230,000
// 44.9 either way, 524,288 83.6 (94.7), a million 161 (179).
constexpr int kRowThreads = 256;
__global__ __launch_bounds__(kRowThreads) void k_mlp_forward_rows(int64_t rows, const float* __restrict__ feat,
                                                                  const float* __restrict__ theta,
                                                                  float* __restrict__ out) {
    __shared__ float th[kP];
    for (int k = threadIdx.x; k < kP; k += kRowThreads) th[k] = theta[k];
    __syncthreads();
    const int64_t r = (int64_t)blockIdx.x * kRowThreads + threadIdx.x;
    if (r >= rows) return;
    float xs[kF], z1[kH];
#pragma unroll
    for (int i = 0; i < kF; ++i) xs[i] = (feat[r * kF + i] - th[oShift + i]) * th[oScale + i];
#pragma unroll
    for (int u = 0; u < kH; ++u) {
        float s = th[oB1 + u];
#pragma unroll
        for (int i = 0; i < kF; ++i) s = fmaf(th[oW1 + u * kF + i], xs[i], s);
        z1[u] = s > 0.0f ? s : 0.0f;
    }
    float o[kO];
#pragma unroll
    for (int k = 0; k < kO; ++k) o[k] = th[oB3 + k];
    for (int u = 0; u < kH; ++u) {  // a unit of layer 2, and its part of the outputs
        float s = th[oB2 + u];
#pragma unroll
        for (int i = 0; i < kH; ++i) s = fmaf(th[oW2 + u * kH + i], z1[i], s);
        const float z2 = s > 0.0f ? s : 0.0f;
#pragma unroll
        for (int k = 0; k < kO; ++k) o[k] = fmaf(th[oW3 + k * kH + u], z2, o[k]);
    }
#pragma unroll
    for (int k = 0; k < kO; ++k) out[r * kO + k] = fmaf(th[oOScale + k], o[k], th[oOShift + k]);
}

// Gradient of L = (1/R) sum_r (1/2) |(out_r - target_r) / oscale|^2 (the
// squared error of y~ against standardised targets), one work-group per chunk
// of 64 rows (chunk b, b + gridDim, ... for more than kGradWgs of them):
// forward, the error signals at the pre-activations of the three layers
// (dout, d2, d1), then the chunk's sums over rows of the outer products, FP64:
// W1 and W2 on v_mfma_f64_16x16x4 (each product of two floats is exact), W3
// and the biases by plain sums.  The activations never leave LDS; part[b] gets
// the work-group's 5122 sums and its loss, and k_mlp_sum adds the work-groups
// in order.  20,000 rows (313 work-groups): 34 + 8 us (rows' activations written to memory and one
// thread per parameter summing all rows in turn: 81 + 5150 us).
constexpr int kPart = kP - oW1 + 1;  // the trained parameters' sums, then the loss
constexpr int kGradWgs = 512;
typedef double f64x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(64 * kMlpWaves, 4) void k_mlp_grad(int64_t rows, const float* __restrict__ feat,
                                                  const float* __restrict__ target,
                                                  const float* __restrict__ theta, double* __restrict__ part) {
    __shared__ Act z1s, z2s, d1s, d2s;
    __shared__ float xls[kRowsWg][kF + 4 + 1];  // x~ of the rows, columns 12..15 zero
    __shared__ float gs[kO][kRowsWg];
    __shared__ double ls[kRowsWg];
    const float* th = theta;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int u0 = kUnits * wave;
    const int q = lane >> 4, c = lane & 15;
    // waves w and w + 4 take rows 16 w .. 16 w + 15 of dW2, 32 columns each (2
    // blocks of 16); the first four also those rows of dW1, the others W3 and
    // the biases
    const int j0 = 16 * (wave & 3), half = wave >> 2;
    f64x4 g2[2], g1;
#pragma unroll
    for (int v = 0; v < 4; ++v) g1[v] = g2[0][v] = g2[1][v] = 0.0;
    double gx = 0.0;  // waves 4, 5: W3 of output wave - 4; 6: b1; 7: b2 (unit lane)
    double gb = 0.0;  // wave 6, lanes 0 and 1: b3; wave 7, lane 0: the loss
    const float inv = 1.0f / (float)rows;
    for (int64_t r0 = (int64_t)blockIdx.x * kRowsWg; r0 < rows; r0 += (int64_t)gridDim.x * kRowsWg) {
        const int64_t r = r0 + lane;
        const bool live = r < rows;  // rows past the end add zeros
        float xs[kF];
        __syncthreads();  // the previous chunk's readers are done
        layer1(th, feat + (live ? r : rows - 1) * kF, lane, u0, live, xs, z1s);
        if (wave == 0) {
#pragma unroll
            for (int i = 0; i < kF; ++i) xls[lane][i] = live ? xs[i] : 0.0f;
#pragma unroll
            for (int i = kF; i < 16; ++i) xls[lane][i] = 0.0f;
        }
        __syncthreads();
        layer2(th, z1s, lane, u0, live, z2s);
        __syncthreads();
        if (wave < kO) {
            // error of y~ against the standardised target (t - oshift) / oscale
            const float o = layer3(th, z2s, lane, wave);
            const float e = o - (target[(live ? r : rows - 1) * kO + wave] - th[oOShift + wave]) / th[oOScale + wave];
            gs[wave][lane] = live ? e * inv : 0.0f;
            if (wave == 0) ls[lane] = live ? (double)e * (double)e : 0.0;
            // (the second output's square is added below)
            else d1s[lane] = live ? e : 0.0f;
        }
        __syncthreads();
        const float g0 = gs[0][lane], g1f = gs[1][lane];
        if (wave == 0) ls[lane] = 0.5 * (ls[lane] + (double)d1s[lane] * (double)d1s[lane]);
        // d2_j = relu'(a2_j) (W3^T dout)_j
#pragma unroll 4
        for (int u = u0; u < u0 + kUnits; ++u) {
            const bool on = live && z2s[act_at(lane, u)] > 0.0f;
            d2s[act_at(lane, u)] = on ? fmaf(th[oW3 + u], g0, th[oW3 + kH + u] * g1f) : 0.0f;
        }
        __syncthreads();
        // d1 = relu'(a1) o (W2^T d2), unit by unit of layer 2
        float d1[kUnits];
#pragma unroll
        for (int u = 0; u < kUnits; ++u) d1[u] = 0.0f;
#pragma unroll 4
        for (int j = 0; j < kH; ++j) {
            const float d2 = d2s[act_at(lane, j)];
#pragma unroll
            for (int u = 0; u < kUnits; ++u) d1[u] = fmaf(th[oW2 + j * kH + u0 + u], d2, d1[u]);
        }
#pragma unroll
        for (int u = 0; u < kUnits; ++u)
            d1s[act_at(lane, u0 + u)] = z1s[act_at(lane, u0 + u)] > 0.0f ? d1[u] : 0.0f;  // z1 = 0 without a row
        __syncthreads();
        // sums over the chunk's rows: A (16 x 4) lane l -> row l%16, k l/16; B
        // lane l -> k l/16, column l%16
#pragma unroll 4
        for (int s = 0; s < kRowsWg / 4; ++s) {
            const int rr = 4 * s + q;
            const double a2 = (double)d2s[act_at(rr, j0 + c)];
#pragma unroll
            for (int k = 0; k < 2; ++k)
                g2[k] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2, (double)z1s[act_at(rr, 32 * half + 16 * k + c)], g2[k],
                                                             0, 0, 0);
        }
        if (half == 0) {
#pragma unroll 4
            for (int s = 0; s < kRowsWg / 4; ++s)
                g1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)d1s[act_at(4 * s + q, j0 + c)],
                                                          (double)xls[4 * s + q][c], g1, 0, 0, 0);
        } else if (wave < 6) {
            const float* go = gs[wave - 4];
#pragma unroll 8
            for (int k = 0; k < kRowsWg; ++k) gx += (double)go[k] * (double)z2s[act_at(k, lane)];
        } else {
            const Act& a = wave == 6 ? d1s : d2s;
#pragma unroll 8
            for (int k = 0; k < kRowsWg; ++k) gx += (double)a[act_at(k, lane)];
            if (wave == 6 && lane < kO) {
#pragma unroll 8
                for (int k = 0; k < kRowsWg; ++k) gb += (double)gs[lane][k];
            }
            if (wave == 7 && lane == 0) {
#pragma unroll 8
                for (int k = 0; k < kRowsWg; ++k) gb += ls[k];
            }
        }
    }
    double* o = part + (int64_t)blockIdx.x * kPart - oW1;  // indexed by the parameter
    // D lane l -> column l%16, register v -> row 4 v + l/16
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int j = j0 + 4 * v + q;
        if (half == 0 && c < kF) o[oW1 + j * kF + c] = g1[v];
#pragma unroll
        for (int k = 0; k < 2; ++k) o[oW2 + j * kH + 32 * half + 16 * k + c] = g2[k][v];
    }
    if (wave >= 4) o[(wave < 6 ? oW3 + (wave - 4) * kH : wave == 6 ? oB1 : oB2) + lane] = gx;
    if (wave == 6 && lane < kO) o[oB3 + lane] = gb;
    if (wave == 7 && lane == 0) o[kP] = gb;
}

// grad = the work-groups' sums added: 64 parameters per work-group, wave w
// adds the parts w, w + 4, ... in order (eight loads in flight), then the four
// waves' sums in order.
__global__ __launch_bounds__(256) void k_mlp_sum(int64_t rows, int nparts, const double* __restrict__ part,
                                                 float* __restrict__ grad, double* __restrict__ loss_out) {
    __shared__ double red[4][64];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int k = blockIdx.x * 64 + lane;
    double s = 0.0;
    if (k < kPart) {
        int b = wave;
        for (; b + 28 < nparts; b += 32) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = part[(int64_t)(b + 4 * u) * kPart + k];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t[u];
        }
        for (; b < nparts; b += 4) s += part[(int64_t)b * kPart + k];
    }
    red[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || k >= kPart) return;
    s = (red[0][lane] + red[1][lane]) + (red[2][lane] + red[3][lane]);
    if (k == kPart - 1) {
        if (loss_out) *loss_out = s / (double)rows;
    } else {
        grad[oW1 + k] = (float)s;
    }
}

// Adam (Kingma & Ba, Algorithm 1) on theta[oW1:]; c1 = 1 - beta1^t and
// c2 = 1 - beta2^t come from the host.
__global__ void k_adam(float* __restrict__ theta, const float* __restrict__ grad,
                       float* __restrict__ m, float* __restrict__ v, float lr, float b1, float b2,
                       float eps, float c1, float c2) {
    const int k = oW1 + blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= kP) return;
    const float g = grad[k];
    const float mk = b1 * m[k] + (1.0f - b1) * g;
    const float vk = b2 * v[k] + (1.0f - b2) * g * g;
    m[k] = mk;
    v[k] = vk;
    theta[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// ---------------------------------------------------------------------------
// budgets: p^ = 1 - Phi((T_obs - mean) / sd); outside the fallback band
// [p_lo, p_hi] the number of splits that separates p^ from the nearer edge by
// zq standard errors, clamped to [b_min, b_max]; inside it, b_max.
// ---------------------------------------------------------------------------
__global__ void k_budgets(int64_t npairs, const float* __restrict__ out,
                          const hbt_result* __restrict__ res, double lo, double hi, int64_t bmin,
                          int64_t bmax, double zq, int64_t* __restrict__ budget) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npairs) return;
    const double mu = (double)out[p * kO], sd = exp((double)out[p * kO + 1]);
    const double ph = 0.5 * erfc((res[p].t_obs - mu) / sd * 0.70710678118654752440);
    int64_t B = bmax;
    if (ph < lo || ph > hi) {
        const double edge = ph < lo ? lo : hi;
        const double gap = (ph - edge) * (ph - edge);
        const double need = zq * zq * ph * (1.0 - ph) / gap;
        if (need < (double)bmax) {
            const int64_t c = (int64_t)ceil(need);
            B = c < bmin ? bmin : c;
        }
    }
    budget[p] = B;
}

// Expected-cost rule: a pair whose p^ lies in the fallback band gets bmax
// (it would be rerun there anyway); any other pair gets the B among bmin,
// 2 bmin, 4 bmin, ... (below bmax) and bmax that minimises the expected
// splits B + bmax * P(its p lands in [lo, hi] after B splits) (a landing
// is rerun with bmax splits), the estimate (1 + count) / (B + 1) taken as
// normal with mean (1 + B p^) / (B + 1) and sd sqrt(B p^ (1 - p^)) / (B + 1);
// ties go to the smaller B.
__device__ double land_prob(double ph, double B, double lo, double hi) {
    const double mean = (1.0 + B * ph) / (B + 1.0);
    const double sd = sqrt(B * ph * (1.0 - ph)) / (B + 1.0);
    if (!(sd > 0.0)) return (mean >= lo && mean <= hi) ? 1.0 : 0.0;
    const double k = 0.70710678118654752440 / sd;
    // Phi((hi - mean) / sd) - Phi((lo - mean) / sd)
    return 0.5 * erfc((lo - mean) * k) - 0.5 * erfc((hi - mean) * k);
}

__global__ void k_budgets_cost(int64_t npairs, const float* __restrict__ out,
                               const hbt_result* __restrict__ res, double lo, double hi, int64_t bmin,
                               int64_t bmax, int64_t* __restrict__ budget) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npairs) return;
    const double mu = (double)out[p * kO], sd = exp((double)out[p * kO + 1]);
    const double ph = 0.5 * erfc((res[p].t_obs - mu) / sd * 0.70710678118654752440);
    int64_t B = bmax;
    if (ph < lo || ph > hi) {
        double best = (double)bmax;
        for (int64_t c = bmin; c < bmax; c *= 2) {
            const double cost = (double)c + (double)bmax * land_prob(ph, (double)c, lo, hi);
            if (cost < best) {
                best = cost;
                B = c;
            }
        }
    }
    budget[p] = B;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
static int grad_wgs(int64_t rows) {
    const int64_t c = (rows + kRowsWg - 1) / kRowsWg;
    return (int)(c < kGradWgs ? c : kGradWgs);
}

size_t mlp_train_ws_bytes(int64_t rows) { return (size_t)grad_wgs(rows) * kPart * sizeof(double) + 256; }

hipError_t launch_features(int64_t npairs, const hbt_result* res, int d, int gd, float* feat,
                           hipStream_t s) {
    hipLaunchKernelGGL(k_features, dim3((unsigned)((npairs + 255) / 256)), dim3(256), 0, s, npairs,
                       res, (double)d, gd, feat);
    return hipGetLastError();
}

hipError_t launch_feature_norm(int64_t rows, const float* feat, float* theta, hipStream_t s) {
    hipLaunchKernelGGL(k_col_norm, dim3(kF), dim3(256), 0, s, rows, kF, feat, theta + oShift,
                       theta + oScale, 1);
    return hipGetLastError();
}

hipError_t launch_target_norm(int64_t rows, const float* target, float* theta, hipStream_t s) {
    hipLaunchKernelGGL(k_col_norm, dim3(kO), dim3(256), 0, s, rows, kO, target, theta + oOShift,
                       theta + oOScale, 0);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(int64_t rows, const float* feat, const float* theta, float* out,
                              hipStream_t s) {
    if (rows > kRowsWg * 14 * (int64_t)device_cus()) {  // where the two are equal (figures at the kernel)
        hipLaunchKernelGGL(k_mlp_forward_rows, dim3((unsigned)((rows + kRowThreads - 1) / kRowThreads)),
                           dim3(kRowThreads), 0, s, rows, feat, theta, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((rows + kRowsWg - 1) / kRowsWg)), dim3(64 * kMlpWaves), 0, s,
                       rows, feat, theta, out);
    return hipGetLastError();
}

hipError_t launch_mlp_grad(int64_t rows, const float* feat, const float* target, const float* theta,
                           float* grad, double* loss, void* ws, hipStream_t s) {
    const int wgs = grad_wgs(rows);
    double* part = (double*)(((uintptr_t)ws + 7) & ~(uintptr_t)7);
    hipLaunchKernelGGL(k_mlp_grad, dim3(wgs), dim3(64 * kMlpWaves), 0, s, rows, feat, target, theta, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mlp_sum, dim3((kPart + 63) / 64), dim3(256), 0, s, rows, wgs, part, grad, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, float lr, float b1,
                       float b2, float eps, float c1, float c2, hipStream_t s) {
    const int nt = kP - oW1;
    hipLaunchKernelGGL(k_adam, dim3((nt + 255) / 256), dim3(256), 0, s, theta, grad, m, v, lr, b1, b2,
                       eps, c1, c2);
    return hipGetLastError();
}

hipError_t launch_budgets(int64_t npairs, const float* out, const hbt_result* res, double lo,
                          double hi, int64_t bmin, int64_t bmax, double zq, int64_t* budget,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_budgets, dim3((unsigned)((npairs + 255) / 256)), dim3(256), 0, s, npairs, out,
                       res, lo, hi, bmin, bmax, zq, budget);
    return hipGetLastError();
}

hipError_t launch_budgets_cost(int64_t npairs, const float* out, const hbt_result* res, double lo,
                               double hi, int64_t bmin, int64_t bmax, int64_t* budget, hipStream_t s) {
    hipLaunchKernelGGL(k_budgets_cost, dim3((unsigned)((npairs + 255) / 256)), dim3(256), 0, s, npairs,
                       out, res, lo, hi, bmin, bmax, budget);
    return hipGetLastError();
}

}  // namespace hbt
