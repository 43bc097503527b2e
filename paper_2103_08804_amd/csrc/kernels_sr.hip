// Natural-gradient (stochastic reconfiguration) step of Sec. III on the GPU.
//
// With the extended index sets i in [0, N] and j in [0, M], where sigma~_N = 1
// and T~_M = 1, every log-derivative is a product O_(i,j)(s) = sigma~_si T~_sj:
// (i < N, j = M) is O_{a_i} = sigma_i, (i = N, j < M) is O_{b_j} = tanh theta_j
// and (i < N, j < M) is O_{W_ij}.  Every P-vector contraction over samples,
//   out_(i,j) = sum_s sigma~_si conj(T~_sj) c_s,
// is then one [(N+1) x n] x [n x (M+1)] product with a per-sample complex
// coefficient c_s:  <O>^* (c = w), <O^* R> (c = w R), the matrix-free
// S v (c = w u, u = O v) and the fidelity gradient (c = 2(1-R) conj(R)/n).
// Partial sums run in FP32 over a chunk of samples and in FP64 across chunks.
#include <float.h>

#include <algorithm>

#include "../../include/chebrbm.h"
#include "device.hpp"
#include "internal.hpp"

namespace crbm {


// device scalar slots (SC_DONE0 and SC_DONE1: whether the solve had ended before an even and an odd CG
// iteration; SC_LATE0 and SC_LATE1: whether the iteration before left the stopping test to it, SC_LATE: whether the last
// one left it to the end; SC_WSUM the sum of the sample weights; SC_OMV <O>.p of the matrix-free product, two slots)
enum {
    SC_RM_RE = 0, SC_RM_IM, SC_R2, SC_GAMMA, SC_GCOT, SC_COEF,
    SC_DONE0 = 8, SC_DONE1, SC_WSUM = 11, SC_FF, SC_ITERS = 14, SC_FLAGS, SC_OMV = 18,
    SC_LATE0 = 20, SC_LATE1, SC_LATE,
    SC_COUNT = 32
};

// ------------------------------------------------------------------ P-index <-> (i, j)
__device__ __forceinline__ void p_to_ij(long k, int N, int M, int& i, int& j) {
    if (k < N) { i = (int)k; j = M; }
    else if (k < N + M) { i = N; j = (int)(k - N); }
    else { const long r = k - N - M; i = (int)(r / M); j = (int)(r % M); }
}
__device__ __forceinline__ long ij_to_p(int i, int j, int N, int M) {
    if (j == M) return i;                 // i < N
    if (i == N) return (long)N + j;
    return (long)N + M + (long)i * M + j;
}

// ------------------------------------------------------------------ scalar reductions
// red[2 blk] = (sum w Re R, sum w Im R), red[2 blk + 1] = (sum w |R|^2, sum w)
__global__ __launch_bounds__(256) void k_r_moments(const float2* __restrict__ R, const double* __restrict__ w, long n,
                                                   double2* __restrict__ red) {
    __shared__ double sh[4][4];
    double rx = 0, ry = 0, r2 = 0, ws_sum = 0;
    const double wdef = 1.0 / (double)n;
    for (long s = (long)blockIdx.x * 256 + threadIdx.x; s < n; s += (long)gridDim.x * 256) {
        const double ws = w ? w[s] : wdef;
        const double x = R[s].x, y = R[s].y;
        rx += ws * x; ry += ws * y; r2 += ws * (x * x + y * y); ws_sum += ws;
    }
    rx = wave_sum(rx); ry = wave_sum(ry); r2 = wave_sum(r2); ws_sum = wave_sum(ws_sum);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { sh[0][wv] = rx; sh[1][wv] = ry; sh[2][wv] = r2; sh[3][wv] = ws_sum; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0, b = 0, c = 0, d = 0;
        for (int k = 0; k < 4; ++k) { a += sh[0][k]; b += sh[1][k]; c += sh[2][k]; d += sh[3][k]; }
        red[2 * blockIdx.x] = make_double2(a, b);
        red[2 * blockIdx.x + 1] = make_double2(c, d);
    }
}

// Fit mode (0): gamma = arccos sqrt(|<R>|^2/<|R|^2>) and the force scale dgamma gamma cot gamma.
// Energy mode (1): R holds E_loc; the SC_GAMMA slot takes the variance <|E|^2> - |<E>|^2 and the
// force scale is -lr (passed as dgamma).
// One wave: each lane adds its share of the partials (one thread adding all 256 in turn took 37-47 us).
__device__ __forceinline__ void sum_r_partials(const double2* __restrict__ red, int n_blocks, double& a, double& b,
                                               double& c, double& d) {
    a = b = c = d = 0.0;
#pragma unroll 4
    for (int k = threadIdx.x; k < n_blocks; k += kWave) {
        a += red[2 * k].x; b += red[2 * k].y; c += red[2 * k + 1].x; d += red[2 * k + 1].y;
    }
    a = wave_sum(a); b = wave_sum(b); c = wave_sum(c); d = wave_sum(d);
}

__global__ __launch_bounds__(64) void k_r_final(const double2* __restrict__ red, int n_blocks, double dgamma, int mode,
                                                double* __restrict__ sc) {
    double a, b, c, d;
    sum_r_partials(red, n_blocks, a, b, c, d);
    if (threadIdx.x != 0) return;
    sc[SC_RM_RE] = a; sc[SC_RM_IM] = b; sc[SC_R2] = c;
    for (int k = SC_DONE0; k < SC_COUNT; ++k) sc[k] = 0.0;
    sc[SC_WSUM] = d;
    if (mode == 1) {
        sc[SC_GAMMA] = c - (a * a + b * b);
        sc[SC_GCOT] = 1.0;
        sc[SC_COEF] = dgamma;
        if (!isfinite(a) || !isfinite(b) || !isfinite(c)) sc[SC_FLAGS] = CRBM_FLAG_NONFINITE;
        return;
    }
    const double ratio = (a * a + b * b) / c;
    const double gamma = acos(fmin(1.0, sqrt(ratio)));
    const double gcot = (gamma < 1e-4) ? 1.0 - gamma * gamma / 3.0 : gamma / tan(gamma);
    sc[SC_GAMMA] = gamma; sc[SC_GCOT] = gcot; sc[SC_COEF] = dgamma * gcot;
    if (!(c > 0.0) || !isfinite(a) || !isfinite(b) || !isfinite(c)) sc[SC_FLAGS] = CRBM_FLAG_NONFINITE;
}

// gamma and beta = <R> of the fit as it stands (Sec. III: beta is taken once the steps are done):
// out = {gamma, Re <R>, Im <R>, <|R|^2>, flags}
__global__ __launch_bounds__(64) void k_fit_stats(const double2* __restrict__ red, int n_blocks,
                                                  double* __restrict__ out) {
    double a, b, c, d;
    sum_r_partials(red, n_blocks, a, b, c, d);
    if (threadIdx.x != 0) return;
    const double gamma = acos(fmin(1.0, sqrt((a * a + b * b) / c)));
    out[0] = gamma;
    out[1] = a;
    out[2] = b;
    out[3] = c;
    out[4] = (!(c > 0.0) || !isfinite(a) || !isfinite(b) || !isfinite(c)) ? (double)CRBM_FLAG_NONFINITE : 0.0;
}

// Exact-enumeration weights p(s) = |psi_s|^2 / sum_s' |psi_s'|^2 = exp(2 Re log psi_s - LSE) (the sampling
// distribution of Sec. III with every configuration listed once).  Pass 1: per block the largest
// 2 Re log psi and the sum of exp(2 Re log psi - that largest value).  Pass 2: every block merges the
// partials in block order (the same result in every block) and writes its share of the weights.
constexpr int kLseBlocks = kLseParts;
__global__ __launch_bounds__(256) void k_lse_partial(const float2* __restrict__ lp, long n, double2* __restrict__ part) {
    __shared__ double sh[4];
    double mx = -INFINITY;
    for (long s = (long)blockIdx.x * 256 + threadIdx.x; s < n; s += (long)gridDim.x * 256)
        mx = fmax(mx, 2.0 * (double)lp[s].x);
    for (int o = 32; o >= 1; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, kWave));
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
    double acc = 0.0;
    if (mx > -INFINITY)
        for (long s = (long)blockIdx.x * 256 + threadIdx.x; s < n; s += (long)gridDim.x * 256)
            acc += exp(2.0 * (double)lp[s].x - mx);
    acc = wave_sum(acc);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = make_double2(mx, sh[0] + sh[1] + sh[2] + sh[3]);
}
__global__ __launch_bounds__(256) void k_lse_weights(const float2* __restrict__ lp, long n,
                                                     const double2* __restrict__ part, int n_part,
                                                     double* __restrict__ w) {
    // every wave merges the partials, its lanes in parallel (one thread in turn took 35 us)
    double mx = -INFINITY;
    for (int k = threadIdx.x & 63; k < n_part; k += kWave) mx = fmax(mx, part[k].x);
    for (int o = 32; o >= 1; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, kWave));
    double z = 0.0;
    for (int k = threadIdx.x & 63; k < n_part; k += kWave)
        if (part[k].x > -INFINITY) z += part[k].y * exp(part[k].x - mx);
    z = wave_sum(z);
    const double L = mx + log(z);   // NaN or infinite when no amplitude is finite and non-zero
    for (long s = (long)blockIdx.x * 256 + threadIdx.x; s < n; s += (long)gridDim.x * 256)
        w[s] = exp(2.0 * (double)lp[s].x - L);
}

hipError_t launch_fit_stats(const float2* R, const double* w, long n, double2* red, double* out, hipStream_t stream) {
    const int nb = (int)std::min<long>((n + 255) / 256, 256);
    hipLaunchKernelGGL(k_r_moments, dim3(nb), dim3(256), 0, stream, R, w, n, red);
    hipLaunchKernelGGL(k_fit_stats, dim3(1), dim3(64), 0, stream, red, nb, out);
    return hipGetLastError();
}

hipError_t launch_enum_weights(const float2* lp, long n, double2* part, double* w, hipStream_t stream) {
    const int np = (int)std::min<long>((n + 255) / 256, kLseBlocks);
    hipLaunchKernelGGL(k_lse_partial, dim3(np), dim3(256), 0, stream, lp, n, part);
    const unsigned nb = (unsigned)std::min<long>((n + 255) / 256, 1024);
    hipLaunchKernelGGL(k_lse_weights, dim3(nb), dim3(256), 0, stream, lp, n, part, np, w);
    return hipGetLastError();
}

// ------------------------------------------------------------------ O^H c contraction
// out_c[i][j] = sum_s sigma~_i(s) y_c(s, j) with y_c(s, j) = c_c(s) conj(t~_j(s)), sigma~_N = 1 and
// t~_M = 1: per coefficient a real (N+1) x n by n x (M+1) complex product (rows i < N are the a
// parameters' O, row N the b parameters', the rest W's, up to conjugation and the sample weights).
// On the matrix cores: sigma~ is +-1 and exact in BF16, y (formed in binary32 as before) is the exact sum of three
// BF16 parts, so with v_mfma_f32_32x32x16_bf16 every product is exact and only the FP32 sums round.
// A wave owns 32 extended hidden units and SB blocks of 32 extended sites and walks a run of sample chunks, 16
// samples per step: lane l loads T of its unit l % 32 at the eight samples 8 (l / 32) .. + 7 (half a wave reads 256
// contiguous bytes), which is the B operand's own layout, so y needs no LDS; the A operand comes from sign bits stored
// by site (k_spin_cols), one word per 32 samples.  The next step's T is loaded before the current step is used.  Up to
// four waves share a workgroup and its coefficients.  Bound by reading T and writing the chunk planes (290 MB at the
// first size below, 60 us).  Chunk sums are written in FP32 and added across chunks in FP64.
// Against sigma~ as floats and y through LDS to v_mfma_f32_32x32x2f32, at 157 TFLOP/s the bound then: 65,536 samples,
// N = 100, M = 400: 195 to 83 us; 8,192 samples, N = 256, M = 512: 93 to 34 us.  Errors against 64 bits are the same
// (a matrix-free step at the first size: 4.0e-6 both).
// coef kinds: 0 -> c = w; 1 -> c = w R; 2 -> c = w (u - mean) (u double2 [n], mean a double pair);
//             3 -> c = 2 (1 - R) conj(R) / n; 4 -> c = w (R - u[0]) (u pointing at <R>: the centred
//             ratio, whose contraction <O^* (R - <R>)> = <O^* R> - <O^*><R> carries no cancellation of
//             the mean of O)
constexpr int OM_C = 32, OM_S = 32;   // units of a wave, multiple of samples of a chunk

typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// the value a binary32 takes after rounding to bfloat16 (nearest, ties to even)
__device__ __forceinline__ float round_to_bf16(float x) {
    uint32_t u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}

__device__ __forceinline__ float2 coef_of(int kind, long s, const double* w, double wdef, const float2* R,
                                          const double2* u, const double* mean, double two_over_n) {
    const float ws = w ? (float)w[s] : (float)wdef;
    switch (kind) {
        case 0: return make_float2(ws, 0.f);
        case 1: return cscale(R[s], ws);
        case 2: return make_float2((float)(u[s].x - mean[0]) * ws, (float)(u[s].y - mean[1]) * ws);
        case 4: return cscale(csub(R[s], make_float2((float)u[0].x, (float)u[0].y)), ws);
        default: {
            const float2 r = R[s];
            const float2 d = cmul(make_float2(1.f - r.x, -r.y), cconj(r));
            return cscale(d, (float)two_over_n);
        }
    }
}

// Sign bits of sigma~ by site, once per call: word [s / 32][i] (ot_sites(N) words a row), bit s % 32 set where
// sigma_i(s) = -1; the b row i = N, the rows past it and the samples past n are +1.  A wave takes 64 samples and 64 sites.
template <bool WORDS>
__global__ __launch_bounds__(256) void k_spin_cols(const int8_t* __restrict__ sig, long n, int N, int sites,
                                                   uint32_t* __restrict__ bits) {
    const int lane = threadIdx.x & 63;
    const long blk = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (blk * 64 >= n) return;
    const long s = blk * 64 + lane;
    const bool in = s < n;
    const int8_t* row = sig + (in ? s : 0) * N;
    const int c0 = 64 * blockIdx.y, len = min(64, N - c0);
    uint64_t mine = 0;
    if (WORDS) {   // rows start on 4 bytes and N is a multiple of 4
#pragma unroll 4
        for (int i = 0; i < len; i += 4) {
            const uint32_t x = in ? *reinterpret_cast<const uint32_t*>(row + c0 + i) : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint64_t m = __builtin_amdgcn_ballot_w64((x >> (8 * k + 7)) & 1u);
                if (lane == i + k) mine = m;
            }
        }
    } else {
#pragma unroll 4
        for (int i = 0; i < len; ++i) {
            const uint64_t m = __builtin_amdgcn_ballot_w64(in && row[c0 + i] < 0);
            if (lane == i) mine = m;
        }
    }
    if (c0 + lane < sites) {
        bits[2 * blk * sites + c0 + lane] = (uint32_t)mine;
        bits[(2 * blk + 1) * sites + c0 + lane] = (uint32_t)(mine >> 32);
    }
}

typedef __attribute__((__vector_size__(4 * sizeof(int)))) int ot_i32x4;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 ot_bf16x8;

// the eight BF16 spins (1 or -1) of sign bits 0..7 of x
__device__ __forceinline__ ot_i32x4 ot_spins(uint32_t x) {
    ot_i32x4 a;
#pragma unroll
    for (int d = 0; d < 4; ++d)
        a[d] = (int)(0x3F803F80u | ((x << (15 - 2 * d)) & 0x8000u) | ((x << (30 - 2 * d)) & 0x80000000u));
    return a;
}

// The three BF16 parts (by truncation, an exact sum) of eight binary32 values; an infinity keeps to its first part.
__device__ __forceinline__ void ot_split(const float (&y)[8], ot_i32x4 (&part)[3]) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        uint32_t p[3][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float v = y[2 * d + k];
            p[0][k] = __float_as_uint(v);
            const float r1 = fabsf(v) == INFINITY ? 0.f : v - __uint_as_float(p[0][k] & 0xFFFF0000u);
            p[1][k] = __float_as_uint(r1);
            p[2][k] = __float_as_uint(r1 - __uint_as_float(p[1][k] & 0xFFFF0000u));
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) part[q][d] = (int)__builtin_amdgcn_perm(p[q][1], p[q][0], 0x07060302u);
    }
}

// eight rows of T from byte offset off on (range-checked against the whole offset, which is in the vector register)
__device__ __forceinline__ void ot_rows(__amdgpu_buffer_rsrc_t r, int off, int row_bytes, float2 (&t)[8]) {
#pragma unroll
    for (int m = 0; m < 8; ++m)
        t[m] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off + m * row_bytes, 0, 0));
}

template <int SB>
__global__ __launch_bounds__(256, SB <= 2 ? 3 : 2) void k_ot(int N, int M, int sites, const uint32_t* __restrict__ bits,
                                            const float2* __restrict__ T,
                                            long n, long chunk, int n_chunks, int nk, int kind0, int kind1,
                                            const double* __restrict__ w, const float2* __restrict__ R,
                                            const double2* __restrict__ u, const double* __restrict__ mean,
                                            float* __restrict__ partial, const double* __restrict__ skip, int round_bf16,
                                            const double2* __restrict__ shift_b) {
    if (skip && *skip != 0.0) return;
    __shared__ float2 sC[256];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, half = lane >> 5, tile = blockDim.x;
    const int b0 = blockIdx.x * SB, c = blockIdx.z % nk;
    const int jw = (blockIdx.y * (blockDim.x >> 6) + wv) * OM_C, j = jw + (lane & 31);
    const bool live = jw <= M, ones = jw + OM_C > M;     // wave-uniform: some unit; units at or past M
    const double wdef = 1.0 / (double)n;
    const double two_over_n = 2.0 / (double)n;
    const long plane = (long)(N + 1) * (M + 1);
    const int row_bytes = M * (int)sizeof(float2), toff = 8 * half * row_bytes + j * (int)sizeof(float2);
    float2 shift = make_float2(0.f, 0.f);
    if (shift_b && j < M) shift = make_float2((float)shift_b[j].x, (float)shift_b[j].y);
    const bool shifted = shift_b != nullptr;
    const uint32_t* bw[SB];   // a block past the last reads the last one's spins and writes nothing
#pragma unroll
    for (int b = 0; b < SB; ++b) bw[b] = bits + min(32 * (b0 + b), sites - 32) + (lane & 31);
    // chunks ck = z, z + planes of the grid, ...: each summed in FP32 on its own
    for (int ck = blockIdx.z / nk; ck < n_chunks; ck += gridDim.z / nk) {
        const long s_begin = (long)ck * chunk;
        const long s_end = min(n, s_begin + chunk);
        f32x16 acc[SB][2];
#pragma unroll
        for (int b = 0; b < SB; ++b)
#pragma unroll
            for (int ri = 0; ri < 2; ++ri)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[b][ri][v] = 0.f;
        for (long t0 = s_begin; t0 < s_end; t0 += tile) {
            const long t_end = min(s_end, t0 + tile);
            __syncthreads();
            sC[tid] = t0 + tid < t_end ? coef_of(c == 0 ? kind0 : kind1, t0 + tid, w, wdef, R, u, mean, two_over_n)
                                       : make_float2(0.f, 0.f);
            __syncthreads();
            if (!live) continue;
            // the tile's rows of T; rows past it read as zero (columns past M read the next row and are dropped at the end)
            const __amdgpu_buffer_rsrc_t Tr = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float2*>(T + t0 * M), (short)0, (int)(t_end - t0) * row_bytes, 0x00020000);
            float2 t[8];
            uint32_t word[SB];
            ot_rows(Tr, toff, row_bytes, t);
#pragma unroll
            for (int b = 0; b < SB; ++b) word[b] = bw[b][(t0 >> 5) * sites];
            const int len = (int)(t_end - t0);
            for (int s0 = 0; s0 < len; s0 += 16) {
                ot_i32x4 a[SB];
#pragma unroll
                for (int b = 0; b < SB; ++b) a[b] = ot_spins(word[b] >> ((s0 & 16) + 8 * half));
                if ((s0 & 16) && s0 + 16 < len)
#pragma unroll
                    for (int b = 0; b < SB; ++b) word[b] = bw[b][((t0 + s0 + 16) >> 5) * sites];
                if (ones)
#pragma unroll
                    for (int m = 0; m < 8; ++m)
                        if (j >= M) t[m] = make_float2(1.f, 0.f);
                if (shifted)
#pragma unroll
                    for (int m = 0; m < 8; ++m) t[m] = csub(t[m], shift);
                if (round_bf16)
#pragma unroll
                    for (int m = 0; m < 8; ++m) t[m] = make_float2(round_to_bf16(t[m].x), round_to_bf16(t[m].y));
                if ((ones || shifted) && s0 + 16 > len)   // the rows past the tile are zero again
#pragma unroll
                    for (int m = 0; m < 8; ++m)
                        if (s0 + 8 * half + m >= len) t[m] = make_float2(0.f, 0.f);
                float yx[8], yy[8];
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    const float2 y = cmul(cconj(t[m]), sC[s0 + 8 * half + m]);
                    yx[m] = y.x;
                    yy[m] = y.y;
                    asm volatile("" : "+v"(yx[m]), "+v"(yy[m]));   // t is free before the next rows are asked for
                }
                ot_rows(Tr, toff + (s0 + 16) * row_bytes, row_bytes, t);
                __builtin_amdgcn_sched_barrier(0);   // issued here, in flight during the products
#pragma unroll
                for (int ri = 0; ri < 2; ++ri) {
                    ot_i32x4 part[3];
                    ot_split(ri == 0 ? yx : yy, part);
#pragma unroll
                    for (int q = 2; q >= 0; --q)
#pragma unroll
                        for (int b = 0; b < SB; ++b)
                            acc[b][ri] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((ot_bf16x8)a[b], (ot_bf16x8)part[q],
                                                                               acc[b][ri], 0, 0, 0);
                }
            }
        }
        // accumulator element v of lane l: row 8(v/4) + 4(l/32) + v%4 of the fragment, column l % 32;
        // the chunk's FP32 sums go to planes [chunk][c][Re/Im] straight from the accumulators
        int i0 = 32 * b0 + 4 * half;
        asm volatile("" : "+v"(i0));   // the 16 SB row offsets are formed here, not kept through the loop over chunks
        if (j <= M) {
#pragma unroll
            for (int ri = 0; ri < 2; ++ri) {
                float* out = partial + (((long)ck * nk + c) * 2 + ri) * plane + j;
#pragma unroll
                for (int b = 0; b < SB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int i = i0 + 32 * b + 8 * (v >> 2) + (v & 3);
                        if (i <= N) out[i * (M + 1)] = acc[b][ri][v];
                    }
            }
        }
    }
}

// out[c][P-index] = sum over chunks of the FP32 chunk sums (in FP64), with optional conjugation.  With
// shift_b: the chunks summed conj(T - c_j) for the units j < M, and conj(c_j) times the same coefficient
// vector's sum over sigma~_i (its column j = M) is added back here; for coefficient vector 0 (the weights)
// that sum is exactly 1 on the b row.
// A block adds 64 entries: wave v the chunks v, v + 4, .., the four waves' sums in order (a thread per entry walking
// all chunks left most of the device idle: 250 us at 10 x 10 with 256 chunks, now 52 us).
// tail (one coefficient vector, the matrix-free S v): out = sum + eps v, and the block's dot products.
struct OpTail {
    int on;
    double eps;
    const double2* v;    // the vector S acts on
    const double2* r;    // residual of the CG (null with F)
    const double2* F;    // right-hand side: the dots are |F - y|^2 and |v|^2 instead (null within the CG)
    double* dots;        // [blocks][4]: r^H r, v^H y, r^H y, y^H y (real parts)
};
// dot products of one wave's 64 entries (k < P valid) of y = (S + eps) v
__device__ __forceinline__ void tail_dots(const OpTail& t, long k, bool valid, double2 v, double2 y, int lane, long blk) {
    double d0 = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0;
    if (valid) {
        if (t.F) {
            const double2 f = zsub(t.F[k], y);
            d0 = f.x * f.x + f.y * f.y;
            d1 = v.x * v.x + v.y * v.y;
        } else {
            const double2 r = t.r[k];
            d0 = r.x * r.x + r.y * r.y;
            d1 = v.x * y.x + v.y * y.y;
            d2 = r.x * y.x + r.y * y.y;
            d3 = y.x * y.x + y.y * y.y;
        }
    }
    d0 = wave_sum(d0); d1 = wave_sum(d1); d2 = wave_sum(d2); d3 = wave_sum(d3);
    if (lane == 0) {
        double* o = t.dots + 4 * blk;
        o[0] = d0; o[1] = d1; o[2] = d2; o[3] = d3;
    }
}
__global__ __launch_bounds__(256) void k_ot_reduce(int N, int M, const float* __restrict__ partial, int n_chunks, int nk,
                                                   int conj0, double2* __restrict__ out0, double2* __restrict__ out1,
                                                   const double* __restrict__ skip, const double2* __restrict__ shift_b,
                                                   OpTail tail) {
    if (skip && *skip != 0.0) return;
    __shared__ double2 sa[4][64], sy[4][64];
    const int lane = threadIdx.x & 63, v = threadIdx.x >> 6;
    const long plane = (long)(N + 1) * (M + 1);
    const long o = (long)blockIdx.x * 64 + lane;
    const bool in = o < plane - 1;               // the last entry (i = N, j = M) is no parameter
    const int i = in ? (int)(o / (M + 1)) : 0, j = in ? (int)(o % (M + 1)) : M;
    const long k = in ? ij_to_p(i, j, N, M) : 0;
    for (int c = 0; c < nk; ++c) {
        const bool shifted = shift_b && j < M, summed = shifted && (i < N || c > 0);
        const long oy = (long)i * (M + 1) + M;
        double2 acc = make_double2(0.0, 0.0), y = make_double2(0.0, 0.0);
        if (in)
#pragma unroll 8
            for (int b = v; b < n_chunks; b += 4) {
                const float* pc = partial + ((long)b * nk + c) * 2 * plane;
                acc.x += (double)pc[o];
                acc.y += (double)pc[plane + o];
                if (summed) {
                    y.x += (double)pc[oy];
                    y.y += (double)pc[plane + oy];
                }
            }
        if (c > 0) __syncthreads();
        sa[v][lane] = acc;
        sy[v][lane] = y;
        __syncthreads();
        if (v != 0) continue;
        for (int b = 1; b < 4; ++b) { acc = zadd(acc, sa[b][lane]); y = zadd(y, sy[b][lane]); }
        if (shifted) {
            if (!summed) y = make_double2(1.0, 0.0);
            const double2 cj = make_double2((double)(float)shift_b[j].x, (double)(float)shift_b[j].y);
            acc = zadd(acc, zconjmul(cj, y));
        }
        if (c == 0 && conj0) acc.y = -acc.y;
        if (tail.on) {
            double2 vk = make_double2(0.0, 0.0);
            if (in) {
                vk = tail.v[k];
                acc = make_double2(acc.x + tail.eps * vk.x, acc.y + tail.eps * vk.y);
            }
            tail_dots(tail, k, in, vk, acc, lane, blockIdx.x);
        }
        if (in) (c == 0 ? out0 : out1)[k] = acc;
    }
}

// Sample chunks of at least n/256 and at least 256 samples (a multiple of the 32-sample tile), at most
// 256 of them, which the plan's reduction buffer holds (it has room for min(ceil(n / 256), 257)
// chunks of two coefficients, twice over); each chunk is summed in FP32 on its own.  Chunks of 128 samples while
// they leave at most 384 workgroups of one site block: a workgroup walks its chunk 16 samples after the other, which
// is then all that the launch waits for.  The rule takes the shape alone, so that the sums do not depend on the device.
// The grid holds as many workgroups as the device keeps resident at once (the kernel's occupancy
// times the CUs, so that no second, nearly empty round follows); each loops over its chunks.
// Sites: the blocks of 32 in as few equal groups of at most 4 as hold them (SB of the kernel), in more and smaller
// whole ones as long as these make no more than 3/2 workgroups per compute unit: a wave with fewer blocks forms fewer
// products per step (three blocks as two and one were slower).  Units: the blocks of 32 in as few equal groups of at most 4 waves.
// Gradient of N = 100, M = 400 (its four launches): 300 samples 17 us, 33 in chunks of 256 with four blocks a wave;
// 4,096 samples 28 against 36; N = 256, M = 512, 2,000 samples 33 against 36.
struct OtPlan { long chunk; int n_chunks, sb, site_groups, waves, unit_groups, grid_z; };
static void ot_chunking(int N, int M, long n, int nk, long& chunk, int& n_chunks) {
    chunk = (n + 255) / 256;
    chunk = ((chunk + OM_S - 1) / OM_S) * OM_S;
    if (chunk < 256) chunk = 256;
    const long unit_groups = ((M + 1 + OM_C - 1) / OM_C + 3) / 4;
    if ((ot_sites(N) / 32) * unit_groups * nk * ((n + 255) / 256) <= 192) chunk = 128;
    n_chunks = (int)((n + chunk - 1) / chunk);
}
static OtPlan ot_plan(int N, int M, long n, int nk, int n_cu) {
    OtPlan p;
    ot_chunking(N, M, n, nk, p.chunk, p.n_chunks);
    const int site_blocks = ot_sites(N) / 32, unit_blocks = (M + 1 + OM_C - 1) / OM_C;
    p.site_groups = (site_blocks + 3) / 4;
    p.sb = (site_blocks + p.site_groups - 1) / p.site_groups;
    p.unit_groups = (unit_blocks + 3) / 4;
    p.waves = (unit_blocks + p.unit_groups - 1) / p.unit_groups;
    for (int sb = 1; sb < p.sb; ++sb) {
        const long groups = (site_blocks + sb - 1) / sb;
        if (groups * sb != site_blocks || groups * p.unit_groups * nk * p.n_chunks > 3L * n_cu / 2) continue;
        p.sb = sb;
        p.site_groups = (int)groups;
    }
    const long slots = (long)n_cu * (4 * (p.sb <= 2 ? 3 : 2) / p.waves);
    long z = slots / ((long)p.site_groups * p.unit_groups * nk);
    if (z < 1) z = 1;
    if (z > p.n_chunks) z = p.n_chunks;
    // the same number of chunks for every workgroup where possible
    z = (p.n_chunks + ((p.n_chunks + z - 1) / z) - 1) / ((p.n_chunks + z - 1) / z);
    p.grid_z = (int)z * nk;
    return p;
}

// bits: the sign bits by site (spin_cols) of the n samples; partial: scratch of at least
// 2 nk (N + 1)(M + 1) floats per chunk
static hipError_t run_ot(int N, int M, const uint32_t* bits, const float2* T, long n, int kind0, int kind1, int nk,
                         const double* w, const float2* R, const double2* u, void* partial_buf, int conj0,
                         double2* out0, double2* out1, hipStream_t stream, const double* skip, Profiler* prof,
                         int n_cu, int round_bf16 = 0, const double2* shift_b = nullptr,
                         const double* mean = nullptr, const OpTail& tail = OpTail{}) {
    const OtPlan op = ot_plan(N, M, n, nk, n_cu);
    float* partial = static_cast<float*>(partial_buf);
    const dim3 grid(op.site_groups, op.unit_groups, op.grid_z), block(64 * op.waves);
    if (prof) prof->begin(PROF_OT, stream);
    switch (op.sb) {
#define CRBM_CASE(b)                                                                                                  \
    case b:                                                                                                           \
        hipLaunchKernelGGL(k_ot<b>, grid, block, 0, stream, N, M, ot_sites(N), bits, T, n, op.chunk, op.n_chunks, nk, \
                           kind0, kind1, w, R, u, mean, partial, skip, round_bf16, shift_b);                          \
        break;
        CRBM_CASE(1) CRBM_CASE(2) CRBM_CASE(3) CRBM_CASE(4)
#undef CRBM_CASE
    }
    if (prof) prof->end(stream);
    const long plane = (long)(N + 1) * (M + 1);
    hipLaunchKernelGGL(k_ot_reduce, dim3((unsigned)((plane + 63) / 64)), dim3(256), 0, stream, N, M, partial,
                       op.n_chunks, nk, conj0, out0, out1, skip, shift_b, tail);
    return hipGetLastError();
}

static void spin_cols(const int8_t* sig, long n, int N, uint32_t* bits, hipStream_t stream) {
    const dim3 grid((unsigned)(((n + 63) / 64 + 3) / 4), (unsigned)((ot_sites(N) + 63) / 64));
    if (N % 4 == 0 && (reinterpret_cast<uintptr_t>(sig) & 3) == 0)
        hipLaunchKernelGGL(k_spin_cols<true>, grid, dim3(256), 0, stream, sig, n, N, ot_sites(N), bits);
    else
        hipLaunchKernelGGL(k_spin_cols<false>, grid, dim3(256), 0, stream, sig, n, N, ot_sites(N), bits);
}

// sum of v over the workgroup (256 threads, four waves); thread 0 has the result
__device__ __forceinline__ double block_total(double v, double (&sh)[4]) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    return sh[0] + sh[1] + sh[2] + sh[3];
}

// ORc = <O^* (R - <R>)> = <O^* R> - <O^*><R>  (R = E_loc in energy mode):
// fit mode (0):    F_k = coef [<O_k^* R>/<R> - <O_k^*>] = coef ORc_k / <R>;
// energy mode (1): F_k = coef [<O_k^* E> - <O_k^*><E>] = coef ORc_k   (coef = -lr).
// means: Om holds conj(<O>) on entry and <O> on exit (else it is left as it is); ff[block] = |F|^2 of the block.
__device__ __forceinline__ double2 force_of(double2 orc, int mode, const double* __restrict__ sc) {
    const double2 rm = make_double2(sc[SC_RM_RE], sc[SC_RM_IM]);
    const double coef = sc[SC_COEF];
    const double2 d = mode == 1 ? orc : zdiv(orc, rm);
    return make_double2(coef * d.x, coef * d.y);
}
__global__ __launch_bounds__(256) void k_make_f(long P, int mode, int means, double2* __restrict__ Om,
                                                const double2* __restrict__ ORm, const double* __restrict__ sc,
                                                double2* __restrict__ F, double* __restrict__ ff) {
    __shared__ double sh[4];
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    double2 f = make_double2(0.0, 0.0);
    if (k < P) {
        f = force_of(ORm[k], mode, sc);
        F[k] = f;
        if (means) Om[k].y = -Om[k].y;
    }
    const double t = block_total(f.x * f.x + f.y * f.y, sh);
    if (threadIdx.x == 0) ff[blockIdx.x] = t;
}

// ------------------------------------------------------------------ weighted P-vector contractions in double
// With sample weights (exact enumeration: every configuration once, weighted by |psi|^2 / Z) the weights span
// many orders of magnitude and the configurations next to nodes of the state carry O_k of the same size
// inverted, so the sums over samples run in double here: Om_k = sum_s w_s conj(O_sk) and
// ORc_k = sum_s w_s conj(O_sk) (R_s - <R>).  One thread per parameter and run of samples (threads of one site
// row read consecutive hidden units of T), the runs added in order by a second pass, which also forms F: P is a
// few hundred, so without the split two workgroups walked all samples, each step waiting on its loads (P = 120,
// 1024 samples: 350 us, now 9 us and 4 us for the second pass).
constexpr int OT64_T = 128;
__global__ __launch_bounds__(OT64_T) void k_ot64(int N, int M, long P, const int8_t* __restrict__ sig,
                                                 const float2* __restrict__ T, const double* __restrict__ w,
                                                 const float2* __restrict__ R, long n, long run,
                                                 const double* __restrict__ sc, double2* __restrict__ part) {
    const long k = (long)blockIdx.x * OT64_T + threadIdx.x;
    if (k >= P) return;
    int i, j;
    p_to_ij(k, N, M, i, j);
    const double rx = sc[SC_RM_RE], ry = sc[SC_RM_IM];
    double ox = 0, oy = 0, qx = 0, qy = 0;
    const long s0 = (long)blockIdx.y * run, s1 = min(n, s0 + run);
#pragma unroll 8
    for (long s = s0; s < s1; ++s) {
        const double ws = w[s];
        const double sv = (i == N) ? 1.0 : (double)sig[s * N + i];
        double tx = 1.0, ty = 0.0;
        if (j < M) { const float2 t = T[s * M + j]; tx = t.x; ty = t.y; }
        const double cx = ws * sv * tx, cy = -ws * sv * ty;          // w conj(O)
        const double dx = (double)R[s].x - rx, dy = (double)R[s].y - ry;
        ox += cx; oy += cy;
        qx += cx * dx - cy * dy; qy += cx * dy + cy * dx;
    }
    part[(2L * blockIdx.y) * P + k] = make_double2(ox, oy);
    part[(2L * blockIdx.y + 1) * P + k] = make_double2(qx, qy);
}
// the runs added in order; Om = <O>, ORc, F and the block's |F|^2: 64 parameters a block, wave v the runs v, v + 4, ..
__global__ __launch_bounds__(256) void k_ot64_final(long P, int n_run, int mode, const double2* __restrict__ part,
                                                    const double* __restrict__ sc, double2* __restrict__ Om,
                                                    double2* __restrict__ ORc, double2* __restrict__ F,
                                                    double* __restrict__ ff) {
    __shared__ double2 so[4][64], sq[4][64];
    const int lane = threadIdx.x & 63, v = threadIdx.x >> 6;
    const long k = (long)blockIdx.x * 64 + lane;
    double2 o = make_double2(0.0, 0.0), q = make_double2(0.0, 0.0);
    if (k < P)
#pragma unroll 4
        for (int b = v; b < n_run; b += 4) {
            o = zadd(o, part[(2L * b) * P + k]);
            q = zadd(q, part[(2L * b + 1) * P + k]);
        }
    so[v][lane] = o;
    sq[v][lane] = q;
    __syncthreads();
    if (v != 0) return;
    double2 f = make_double2(0.0, 0.0);
    if (k < P) {
        for (int b = 1; b < 4; ++b) { o = zadd(o, so[b][lane]); q = zadd(q, sq[b][lane]); }
        f = force_of(q, mode, sc);
        Om[k] = make_double2(o.x, -o.y);
        ORc[k] = q;
        F[k] = f;
    }
    const double t = wave_sum(f.x * f.x + f.y * f.y);
    if (lane == 0) ff[blockIdx.x] = t;
}

// ------------------------------------------------------------------ dense S (FP32, VALU)
// Upper-triangle tiles (I <= J) of 64 x 64, mirrored into the lower triangle so that S is stored in full:
//   S[k][k'] = sum_s w conj(O_sk - m_k) (O_sk' - m_k') + (1 - sum_s w) conj(m_k) m_k',  m = <O>,
// which is <O^* O> - <O>^* <O> (Sec. III) with the operands centred before the sums: where |<O_k>|^2 is
// large against the variance (tanh theta near +-1), raw sums less the product of the means would lose that
// ratio's digits.  Binary32 operands, products and sums in double (the weighted sums serve exact enumeration
// with a dense solve, where a few configurations next to nodes of the state can make |S| large against the
// diagonal shift); S is written in binary32 and, for the Cholesky solve, also in double (S64).
// The samples run in gridDim.y runs, each into its own slice of `part` (added by k_sbuild_runs), where the few
// tiles of a small P would leave the device idle (P = 120, 1024 samples: 374 us on 3 workgroups, now 20 us on 96, and 4 us for the sum).
// The double matrix S64 is that of the solve: it takes the diagonal shift eps as well.
constexpr int SB_T = 64, SB_K = 16;

__device__ __forceinline__ void sbuild_store(long P, long k, long kp, bool mirror, double2 sum,
                                             const double2* __restrict__ Om, const double* __restrict__ sc,
                                             float2* __restrict__ S, double2* __restrict__ S64, double eps) {
    const double2 mm = zconjmul(Om[k], Om[kp]);
    const double rest = 1.0 - sc[SC_WSUM];
    const double2 d = make_double2(sum.x + rest * mm.x, sum.y + rest * mm.y);
    const float2 v = make_float2((float)d.x, (float)d.y);
    S[k * P + kp] = v;
    if (mirror) S[kp * P + k] = cconj(v);
    if (S64) {
        S64[k * P + kp] = k == kp ? make_double2(d.x + eps, d.y) : d;
        if (mirror) S64[kp * P + k] = make_double2(d.x, -d.y);
    }
}

__global__ __launch_bounds__(256) void k_sbuild(int N, int M, long P, const int8_t* __restrict__ sig,
                                                const float2* __restrict__ T, const double* __restrict__ w, long n,
                                                const double2* __restrict__ Om, float2* __restrict__ S, int ntile,
                                                const double* __restrict__ sc, double2* __restrict__ S64, double eps,
                                                long run, double2* __restrict__ part) {
    __shared__ float2 sa[SB_K][SB_T];
    __shared__ float2 sb[SB_K][SB_T];
    // map blockIdx.x -> (I, J), I <= J
    long rem = blockIdx.x;
    int I = 0;
    while (rem >= ntile - I) { rem -= ntile - I; ++I; }
    const int J = I + (int)rem;
    const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
    const long kA0 = (long)I * SB_T, kB0 = (long)J * SB_T;
    // columns loaded by this thread: column c = tid & 63, rows ss = tid >> 6 (+4 steps)
    const int lc = tid & 63;
    int ia, ja, ib, jb;
    const bool va = kA0 + lc < P, vb = kB0 + lc < P;
    p_to_ij(va ? kA0 + lc : 0, N, M, ia, ja);
    p_to_ij(vb ? kB0 + lc : 0, N, M, ib, jb);
    const double2 mA = va ? Om[kA0 + lc] : make_double2(0.0, 0.0), mB = vb ? Om[kB0 + lc] : make_double2(0.0, 0.0);
    const float2 mAf = make_float2((float)mA.x, (float)mA.y), mBf = make_float2((float)mB.x, (float)mB.y);
    const double wdef = 1.0 / (double)n;
    double2 acc[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[r][c] = make_double2(0.0, 0.0);

    const long s_end = min(n, (long)(blockIdx.y + 1) * run);
    for (long s0 = (long)blockIdx.y * run; s0 < s_end; s0 += SB_K) {
#pragma unroll
        for (int st = 0; st < SB_K / 4; ++st) {
            const int ss = (tid >> 6) + 4 * st;
            const long s = s0 + ss;
            float2 oa = make_float2(0.f, 0.f), ob = make_float2(0.f, 0.f);
            if (s < s_end) {
                const float ws = w ? (float)w[s] : (float)wdef;
                if (va) {
                    const float sv = (ia == N) ? 1.f : (float)sig[s * N + ia];
                    const float2 tv = (ja == M) ? make_float2(1.f, 0.f) : T[s * M + ja];
                    oa = cscale(cconj(csub(cscale(tv, sv), mAf)), ws);
                }
                if (vb) {
                    const float sv = (ib == N) ? 1.f : (float)sig[s * N + ib];
                    const float2 tv = (jb == M) ? make_float2(1.f, 0.f) : T[s * M + jb];
                    ob = csub(cscale(tv, sv), mBf);
                }
            }
            sa[ss][lc] = oa;
            sb[ss][lc] = ob;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < SB_K; ++kk) {
            float2 av[4], bv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) av[r] = sa[kk][ty + 16 * r];
#pragma unroll
            for (int c = 0; c < 4; ++c) bv[c] = sb[kk][tx + 16 * c];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const double ax = av[r].x, ay = av[r].y, bx = bv[c].x, by = bv[c].y;
                    acc[r][c].x = fma(ax, bx, fma(-ay, by, acc[r][c].x));
                    acc[r][c].y = fma(ax, by, fma(ay, bx, acc[r][c].y));
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const long k = kA0 + ty + 16 * r;
        if (k >= P) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const long kp = kB0 + tx + 16 * c;
            if (kp >= P) continue;
            if (part) part[((long)blockIdx.y * P + k) * P + kp] = acc[r][c];
            else sbuild_store(P, k, kp, I != J, acc[r][c], Om, sc, S, S64, eps);
        }
    }
}

// S of the sample runs' slices, added in order (upper tiles; the others are written from them)
__global__ __launch_bounds__(256) void k_sbuild_runs(long P, int n_run, const double2* __restrict__ part,
                                                     const double2* __restrict__ Om, const double* __restrict__ sc,
                                                     float2* __restrict__ S, double2* __restrict__ S64, double eps) {
    const long e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= P * P) return;
    const long k = e / P, kp = e % P;
    if (k / SB_T > kp / SB_T) return;
    double2 a = make_double2(0.0, 0.0);
#pragma unroll 8
    for (int z = 0; z < n_run; ++z) a = zadd(a, part[(long)z * P * P + e]);
    sbuild_store(P, k, kp, k / SB_T != kp / SB_T, a, Om, sc, S, S64, eps);
}

// ------------------------------------------------------------------ dense Hermitian product
// y = (S + eps I) x with S complex64 [P][P] read from its lower triangle only, x and y complex128.
// Tile (I, J), J <= I, of HV_T x HV_T entries gives S_IJ x_J to the rows of I and, for J < I, also
// S_IJ^H x_I to the rows of J (the upper triangle is never read, halving the bytes of a product).
// Each partial vector has its own slot, part[A][B] = the share of tile pair {A, B} in y_A, and a
// second pass adds the nT slots of every row in the same order (deterministic).
constexpr int HV_T = kHemvTile;

// PAIR (P even, so every row and tile starts on 16 bytes): a lane reads two adjacent columns per load,
// columns 2 c0 + 32 j' + {0, 1}; otherwise one column, c0 + 16 j.
template <bool PAIR>
__global__ __launch_bounds__(256) void k_hemv_tiles(long P, int nT, const float2* __restrict__ S,
                                                    const double2* __restrict__ x, double2* __restrict__ part,
                                                    const double* __restrict__ skip) {
    if (skip && *skip != 0.0) return;
    // lower-triangle tile (I, J) of this workgroup: t = I (I + 1) / 2 + J
    const long t = blockIdx.x;
    int I = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
    while ((long)I * (I + 1) / 2 > t) --I;
    while ((long)(I + 1) * (I + 2) / 2 <= t) ++I;
    const int J = (int)(t - (long)I * (I + 1) / 2);
    __shared__ double2 xI[HV_T], xJ[HV_T];
    __shared__ double2 cred[4][HV_T];
    const int tid = threadIdx.x;
    const long i0 = (long)I * HV_T, j0 = (long)J * HV_T;
    xI[tid] = i0 + tid < P ? x[i0 + tid] : make_double2(0.0, 0.0);
    xJ[tid] = j0 + tid < P ? x[j0 + tid] : make_double2(0.0, 0.0);
    __syncthreads();
    // a 16-lane group takes one row at a time, so that every load instruction of a group covers
    // 128 (256 with PAIR) contiguous bytes of the row
    const int lane = tid & 63, w = tid >> 6, g = lane >> 4, c0 = lane & 15;
    const int nrows = (int)(P - i0 < HV_T ? P - i0 : HV_T);
    const int ncols = (int)(P - j0 < HV_T ? P - j0 : HV_T);
    double cx[16], cy[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) { cx[j] = 0.0; cy[j] = 0.0; }
    for (int rr = 4 * w + g; rr < nrows; rr += 16) {
        const float2* Sr = S + (i0 + rr) * P + j0;
        const double2 xi = xI[rr];
        double rx = 0.0, ry = 0.0;
#pragma unroll
        for (int jp = 0; jp < (PAIR ? 8 : 16); ++jp) {
            float2 sv2[2];
            if constexpr (PAIR) {
                const int c = 2 * c0 + 32 * jp;
                // columns past P: read columns 0, 1 instead; x_J is zero there and the column share is unused
                const float4 v4 = *reinterpret_cast<const float4*>(Sr + (c < ncols ? c : 0));
                sv2[0] = make_float2(v4.x, v4.y);
                sv2[1] = make_float2(v4.z, v4.w);
            } else {
                const int c = c0 + 16 * jp;
                sv2[0] = Sr[c < ncols ? c : 0];
            }
#pragma unroll
            for (int h = 0; h < (PAIR ? 2 : 1); ++h) {
                const int j = PAIR ? 2 * jp + h : jp;
                const int c = PAIR ? 2 * c0 + 32 * jp + h : c0 + 16 * jp;
                const double sx = sv2[h].x, sy = sv2[h].y;
                const double2 xj = xJ[c];
                rx += sx * xj.x - sy * xj.y;
                ry += sx * xj.y + sy * xj.x;
                cx[j] += sx * xi.x + sy * xi.y;            // conj(S_rc) x_r
                cy[j] += sx * xi.y - sy * xi.x;
            }
        }
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) {
            rx += __shfl_xor(rx, o, 16);
            ry += __shfl_xor(ry, o, 16);
        }
        if (c0 == 0) part[((long)I * nT + J) * HV_T + rr] = make_double2(rx, ry);
    }
    if (J == I) return;                              // the diagonal tile was read in full
    // column shares: add the 4 row groups of the wave, then the 4 waves in order
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        cx[j] += __shfl_xor(cx[j], 16);
        cy[j] += __shfl_xor(cy[j], 16);
        cx[j] += __shfl_xor(cx[j], 32);
        cy[j] += __shfl_xor(cy[j], 32);
    }
    if (g == 0)
#pragma unroll
        for (int j = 0; j < 16; ++j) cred[w][PAIR ? 2 * c0 + 32 * (j >> 1) + (j & 1) : c0 + 16 * j] = make_double2(cx[j], cy[j]);
    __syncthreads();
    const double2 a = cred[0][tid], b = cred[1][tid], c = cred[2][tid], d = cred[3][tid];
    part[((long)J * nT + I) * HV_T + tid] = make_double2(((a.x + b.x) + c.x) + d.x, ((a.y + b.y) + c.y) + d.y);
}

// y_k = sum_B part[k / HV_T][B][k % HV_T] + eps x_k; 64 rows per workgroup, its 4 waves add a quarter
// of the slots each, combined in wave order; the first wave also forms the rows' dot products
__global__ __launch_bounds__(256) void k_hemv_reduce(long P, int nT, const double2* __restrict__ part,
                                                     double2* __restrict__ y, const double* __restrict__ skip,
                                                     OpTail tail) {
    if (skip && *skip != 0.0) return;
    __shared__ double2 q[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const long k = (long)blockIdx.x * 64 + lane;
    double sx = 0.0, sy = 0.0;
    if (k < P) {
        const long I = k / HV_T, r = k % HV_T;
        const double2* pr = part + I * nT * HV_T + r;
        const int per = (nT + 3) / 4;
        const int b0 = w * per, b1 = b0 + per < nT ? b0 + per : nT;
#pragma unroll 8
        for (int B = b0; B < b1; ++B) {
            const double2 v = pr[(long)B * HV_T];
            sx += v.x;
            sy += v.y;
        }
    }
    q[w][lane] = make_double2(sx, sy);
    __syncthreads();
    if (w != 0) return;
    double2 yk = make_double2(0.0, 0.0), xk = make_double2(0.0, 0.0);
    if (k < P) {
        const double2 a = q[0][lane], b = q[1][lane], c = q[2][lane], d = q[3][lane];
        xk = tail.v[k];
        yk = make_double2((((a.x + b.x) + c.x) + d.x) + tail.eps * xk.x, (((a.y + b.y) + c.y) + d.y) + tail.eps * xk.y);
        y[k] = yk;
    }
    tail_dots(tail, k, k < P, xk, yk, lane, blockIdx.x);
}

// ------------------------------------------------------------------ matrix-free S v
// u_s = sum_j T_sj G_sj + sum_i sigma_si v_a_i with G = theta-GEMM(b = v_b, W = v_W).  The product reads v as the
// split planes of v_W and v_b in binary32, and subtracts <O>.v from every u_s; whoever forms v writes these along
// with it (mf_publish), so that an iteration has no launch of its own for them.
struct MfView {
    int N, M, Np;            // M = 0: dense product, nothing to publish
    long rows;
    uint16_t* planes;
    float2* vb;
    const double2* Om;
    double2* omv;            // [blocks] partial sums of <O>.v
};
__device__ __forceinline__ void mf_publish(const MfView& f, long k, bool valid, double2 v, double (&shx)[4],
                                           double (&shy)[4]) {
    double2 t = make_double2(0.0, 0.0);
    if (valid) {
        t = zmul(f.Om[k], v);
        const float2 c = make_float2((float)v.x, (float)v.y);
        if (k >= f.N + f.M) {
            const long r = k - f.N - f.M;
            split_plane_store(f.planes, f.rows, f.Np, (int)(r / f.M), (int)(r % f.M), c);
        } else if (k >= f.N) {
            f.vb[k - f.N] = c;
        }
    }
    const double tx = block_total(t.x, shx), ty = block_total(t.y, shy);
    if (threadIdx.x == 0) f.omv[blockIdx.x] = make_double2(tx, ty);
}
__global__ __launch_bounds__(256) void k_mf_publish(long P, const double2* __restrict__ v, MfView f) {
    __shared__ double shx[4], shy[4];
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    mf_publish(f, k, k < P, k < P ? v[k] : make_double2(0.0, 0.0), shx, shy);
}

// ------------------------------------------------------------------ CG (double)
// x = 0, r = p = F; the first block adds the |F|^2 partials and opens the iteration
__global__ __launch_bounds__(256) void k_cg_init(long P, const double2* __restrict__ F, const double* __restrict__ ff,
                                                 int n_ff, double2* __restrict__ x, double2* __restrict__ r,
                                                 double2* __restrict__ p, double* __restrict__ sc, MfView f) {
    __shared__ double sh[4], shx[4], shy[4];
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    const double2 v = k < P ? F[k] : make_double2(0.0, 0.0);
    if (k < P) {
        x[k] = make_double2(0.0, 0.0);
        r[k] = v;
        p[k] = v;
    }
    if (f.M) mf_publish(f, k, k < P, v, shx, shy);
    if (blockIdx.x != 0) return;
    double a = 0.0;
    for (int b = threadIdx.x; b < n_ff; b += 256) a += ff[b];
    a = block_total(a, sh);
    if (threadIdx.x == 0) {
        sc[SC_FF] = a;
        sc[SC_DONE0] = (a == 0.0 || (int)sc[SC_FLAGS] != 0) ? 1.0 : 0.0;
        sc[SC_ITERS] = 0.0;
    }
}

// One iteration after Ap: with the dot products that the product's last kernel left per block (r^H r, p^H Ap,
// r^H Ap, |Ap|^2), alpha = r^H r / p^H Ap, x += alpha p, r -= alpha Ap, the new |r|^2 = r^H r - 2 alpha r^H Ap +
// alpha^2 |Ap|^2 (r^H r is formed from r itself in every iteration, so nothing accumulates), the convergence test
// and p = r + beta p.  Every block adds the partials in the same order and takes the same decision; block 0
// records it in the other of the two done slots than the one this iteration reads.
// The new |r|^2 cancels: its terms round to within kCgSlack of r^H r + alpha^2 |Ap|^2 (up to 30 roundings in a row in
// each dot product, and 2 alpha |r| |Ap| is at most the sum of the other two).  Where the tolerance lies within
// that bound the test is left to the next iteration, which has the norm of r itself before it changes anything (after
// the last one, to k_finish), and where the value does not exceed it p starts again from r: an iteration that takes
// nearly all of the residual away (a shift far above S) would otherwise be judged by rounding noise.
// Launches that a finished solve skips cost about 2 us each, so an iteration has 3 (dense) or 5 (matrix-free) of
// them; with the vector updates, dot products and operand packing apart it had 5 and 12.
constexpr double kCgSlack = 0x1p-47;
__global__ __launch_bounds__(256) void k_cg_step(long P, double2* __restrict__ x, double2* __restrict__ r,
                                                 double2* __restrict__ p, const double2* __restrict__ Ap,
                                                 const double* __restrict__ dots, int n_dots, double* __restrict__ sc,
                                                 double tol, int maxit, int it, MfView f) {
    __shared__ double s0[4], s1[4], s2[4], s3[4];
    const int now = SC_DONE0 + (it & 1), next = SC_DONE0 + ((it + 1) & 1);
    const int late = SC_LATE0 + (it & 1), late_next = SC_LATE0 + ((it + 1) & 1);
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (sc[now] != 0.0) {
        if (lead) sc[next] = 1.0;
        return;
    }
    double d0 = 0.0, d1 = 0.0, d2 = 0.0, d3 = 0.0;
    for (int b = threadIdx.x; b < n_dots; b += 256) {
        const double2 u = *reinterpret_cast<const double2*>(dots + 4 * b), v = *reinterpret_cast<const double2*>(dots + 4 * b + 2);
        d0 += u.x; d1 += u.y; d2 += v.x; d3 += v.y;
    }
    const double rr = block_total(d0, s0), pap = block_total(d1, s1), rap = block_total(d2, s2), aa = block_total(d3, s3);
    const double limit = tol * sqrt(sc[SC_FF]);
    if (sc[late] != 0.0 && sqrt(rr) <= limit) {      // converged in the iteration before
        if (lead) sc[next] = 1.0;
        return;
    }
    const double alpha = rr / pap, step2 = alpha * alpha * aa;
    const double rn = rr - 2.0 * alpha * rap + step2, slack = kCgSlack * (rr + step2);
    const bool bad = !isfinite(rn) || !(pap > 0.0);
    const bool conv = !bad && sqrt(fmax(rn + slack, 0.0)) <= limit;
    const bool decided = bad || conv || sqrt(fmax(rn - slack, 0.0)) > limit;
    const bool stop = bad || conv || it + 1 >= maxit;
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    double2 pk = make_double2(0.0, 0.0);
    if (k < P) {
        pk = p[k];
        const double2 ak = Ap[k];
        x[k] = make_double2(x[k].x + alpha * pk.x, x[k].y + alpha * pk.y);
        const double2 rk = make_double2(r[k].x - alpha * ak.x, r[k].y - alpha * ak.y);
        r[k] = rk;
        if (!stop) {
            const double beta = rn > slack ? rn / rr : 0.0;
            pk = make_double2(rk.x + beta * pk.x, rk.y + beta * pk.y);
            p[k] = pk;
        }
    }
    if (f.M && !stop) {
        __shared__ double shx[4], shy[4];
        mf_publish(f, k, k < P, pk, shx, shy);
    }
    if (lead) {
        if (bad || (stop && !conv && decided))
            sc[SC_FLAGS] = (double)((int)sc[SC_FLAGS] | (bad ? CRBM_FLAG_NONFINITE : CRBM_FLAG_NOT_CONVERGED));
        sc[SC_ITERS] = (double)(it + 1);
        sc[next] = stop ? 1.0 : 0.0;
        sc[late_next] = decided ? 0.0 : 1.0;
        if (stop) sc[SC_LATE] = decided ? 0.0 : 1.0;
    }
}

// a, b, W += dalpha  (skipped when the step was flagged non-finite); the first block adds the residual's, the
// solution's and F's partials, takes the stopping test that a last CG iteration left open, from the norm of its
// residual r, and writes the statistics
__global__ __launch_bounds__(256) void k_finish(int N, int M, float2* __restrict__ a, float2* __restrict__ b,
                                                float2* __restrict__ W, const double2* __restrict__ x,
                                                const double* __restrict__ dots, int n_dots,
                                                const double* __restrict__ ff, int n_ff,
                                                const double2* __restrict__ r, double tol,
                                                const double* __restrict__ sc, double* __restrict__ out) {
    __shared__ double s0[4], s1[4], s2[4], s3[4];
    const long P = (long)N + M + (long)N * M;
    if (out && blockIdx.x == 0) {
        double d0 = 0.0, d1 = 0.0, d2 = 0.0;
        for (int k = threadIdx.x; k < n_dots; k += 256) {
            const double2 u = *reinterpret_cast<const double2*>(dots + 4 * k);
            d0 += u.x; d1 += u.y;
        }
        for (int k = threadIdx.x; k < n_ff; k += 256) d2 += ff[k];
        const double res = block_total(d0, s0), xx = block_total(d1, s1), f2 = block_total(d2, s2);
        int flags = (int)sc[SC_FLAGS];
        if (sc[SC_LATE] != 0.0) {
            double d3 = 0.0;
            for (long k = threadIdx.x; k < P; k += 256) d3 += r[k].x * r[k].x + r[k].y * r[k].y;
            const double rr = block_total(d3, s3);
            if (!(sqrt(rr) <= tol * sqrt(sc[SC_FF]))) flags |= CRBM_FLAG_NOT_CONVERGED;
        }
        if (threadIdx.x == 0) {
            out[0] = sc[SC_GAMMA];
            out[1] = sc[SC_RM_RE];
            out[2] = sc[SC_RM_IM];
            out[3] = sqrt(f2);
            out[4] = f2 > 0.0 ? sqrt(res / f2) : 0.0;
            out[5] = sc[SC_ITERS];
            out[6] = (double)flags;
            out[7] = sqrt(xx);
        }
    }
    if (((int)sc[SC_FLAGS] & (CRBM_FLAG_NONFINITE | CRBM_FLAG_CHOLESKY_FAIL)) != 0) return;
    const long k = (long)blockIdx.x * 256 + threadIdx.x;
    if (k >= P) return;
    float2* dst = (k < N) ? &a[k] : (k < N + M) ? &b[k - N] : &W[k - N - M];
    *dst = make_float2(dst->x + (float)x[k].x, dst->y + (float)x[k].y);
}

// ------------------------------------------------------------------ driver
static inline unsigned nblk(long n, int t = 256) { return (unsigned)((n + t - 1) / t); }

// slots of W.dots: [4 nb] dot products, [nb] |F|^2, [2 nb] <O>.v partials, nb >= blocks of 64 entries
static long dots_blocks(long P) { return P / 64 + 8; }
long sr_dots_len(long P) { return 8 * dots_blocks(P); }

// y = (S + eps I) v with the dot products of its tail; skip: device flag of a finished solve, or null.  The
// matrix-free product expects v published (k_mf_publish).  n_dots: blocks that left dot products.
static hipError_t apply_op(const SrArgs& A, const SrWork& W, const double2* v, double2* y, const double2* F,
                           const double* skip, int* n_dots, const MfView& f, hipStream_t stream) {
    const long P = A.P;
    OpTail t{};
    t.on = 1;
    t.eps = A.eps;
    t.v = v;
    t.r = W.r;
    t.F = F;
    t.dots = W.dots;
    if (A.solver == CRBM_SOLVER_CG_MATFREE) {
        // u = O v per sample, the theta product of V fused with the sum over T (partials in the G scratch)
        hipError_t e = launch_theta_ov(W.bits, A.n, A.N, A.M, f.vb, v, A.T, W.wplanes,
                                       reinterpret_cast<double2*>(W.G), W.u, f.omv, (int)nblk(P),
                                       W.scal + SC_OMV, W.n_cu, stream, skip);
        if (e != hipSuccess) return e;
        *n_dots = (int)nblk((long)(A.N + 1) * (A.M + 1), 64);
        return run_ot(A.N, A.M, W.ot_bits, A.T, A.n, 2, 0, 1, A.weights, A.R, W.u, W.red, 0, y, nullptr, stream, skip,
                      nullptr, W.n_cu, 0, nullptr, W.scal + SC_OMV, t);
    }
    const int nT = hemv_tiles(P);
    const dim3 grid((unsigned)((long)nT * (nT + 1) / 2));
    if (P % 2 == 0)
        hipLaunchKernelGGL(k_hemv_tiles<true>, grid, dim3(256), 0, stream, P, nT, W.S, v, W.hv_part, skip);
    else
        hipLaunchKernelGGL(k_hemv_tiles<false>, grid, dim3(256), 0, stream, P, nT, W.S, v, W.hv_part, skip);
    *n_dots = (int)nblk(P, 64);
    hipLaunchKernelGGL(k_hemv_reduce, dim3(nblk(P, 64)), dim3(256), 0, stream, P, nT, W.hv_part, y, skip, t);
    return hipGetLastError();
}

hipError_t launch_cholesky_solve(long P, const float2* S, double eps, const double2* F, double2* A64, double2* x,
                                 double2* v, double2* y, double* sc, bool a64_holds_s, hipStream_t stream);

hipError_t launch_sr_step(const SrArgs& A, const SrWork& W, hipStream_t stream) {
    const long P = A.P;
    hipError_t e;
    // scalars gamma, beta, gamma cot gamma
    const int nb_r = (int)std::min<long>((A.n + 255) / 256, 256);
    hipLaunchKernelGGL(k_r_moments, dim3(nb_r), dim3(256), 0, stream, A.R, A.weights, A.n, W.red);
    hipLaunchKernelGGL(k_r_final, dim3(1), dim3(64), 0, stream, W.red, nb_r, A.dgamma, A.mode, W.scal);
    double* ff = W.dots + 4 * dots_blocks(P);
    int n_ff;
    // the sign bits by site serve the O^H c contraction only
    if (!A.weights || A.solver == CRBM_SOLVER_CG_MATFREE) spin_cols(A.samples, A.n, A.N, W.ot_bits, stream);
    // conj(<O>) and <O^* (R - <R>)>: FP32 chunk sums on the matrix cores, or in double with sample weights
    if (A.weights) {
        // runs of at least 16 samples, as many as the reduction buffer holds up to 64
        long z = std::min<long>(std::min<long>(64, (A.n + 15) / 16), W.red_len / (2 * P));
        z = std::max<long>(z, 1);
        const long run = (A.n + z - 1) / z;
        z = (A.n + run - 1) / run;
        W.prof->begin(PROF_OT, stream);
        hipLaunchKernelGGL(k_ot64, dim3(nblk(P, OT64_T), (unsigned)z), dim3(OT64_T), 0, stream, A.N, A.M, P, A.samples,
                           A.T, A.weights, A.R, A.n, run, W.scal, W.red);
        W.prof->end(stream);
        n_ff = (int)nblk(P, 64);
        hipLaunchKernelGGL(k_ot64_final, dim3(n_ff), dim3(256), 0, stream, P, (int)z, A.mode, W.red, W.scal, W.Om, W.ORm,
                           W.F, ff);
        e = hipGetLastError();
    } else {
        e = run_ot(A.N, A.M, W.ot_bits, A.T, A.n, 0, 4, 2, A.weights, A.R,
                   reinterpret_cast<const double2*>(W.scal + SC_RM_RE), W.red, 0, W.Om, W.ORm, stream, nullptr, W.prof,
                   W.n_cu);
        n_ff = (int)nblk(P);
        hipLaunchKernelGGL(k_make_f, dim3(n_ff), dim3(256), 0, stream, P, A.mode, 1, W.Om, W.ORm, W.scal, W.F, ff);
    }
    if (e != hipSuccess) return e;

    if (A.solver != CRBM_SOLVER_CG_MATFREE) {
        if (A.weights == nullptr) {
            // The contraction sees T' = T - c (c = <T> in binary32; rounded to BF16 with BF16 operands).
            // The subtracted means are those of the same operands, T' + c, summed as T' in the chunks
            // with c <sigma~> added in double: S stays the centred Gram matrix of one set of vectors
            // (positive semi-definite) and no sum carries |c|^2 against the spread of T.
            if (A.prec == CRBM_PREC_BF16) {
                // F from the same rounded operands: the step then solves the ridge problem of one set of
                // vectors, min |O~ x - D|^2 + eps |x|^2.  With F from the unrounded O, the part of
                // <O^* D> outside the span of the rounded O~ would be divided by eps.
                e = run_ot(A.N, A.M, W.ot_bits, A.T, A.n, 0, 4, 2, nullptr, A.R,
                           reinterpret_cast<const double2*>(W.scal + SC_RM_RE), W.red, 1, W.Om16, W.ORm, stream,
                           nullptr, nullptr, W.n_cu, 1, W.Om + A.N);
                if (e != hipSuccess) return e;
                hipLaunchKernelGGL(k_make_f, dim3(n_ff), dim3(256), 0, stream, P, A.mode, 0, W.Om, W.ORm, W.scal, W.F,
                                   ff);
            } else {
                e = run_ot(A.N, A.M, W.ot_bits, A.T, A.n, 0, 0, 1, nullptr, A.R, nullptr, W.red, 1, W.Om16, nullptr,
                           stream, nullptr, nullptr, W.n_cu, 0, W.Om + A.N);
                if (e != hipSuccess) return e;
            }
            const int nsplit = W.spart ? sbuild_splits(A.N, A.M, A.n, W.n_cu, W.nsplit_max, W.sb_fold,
                                                       A.prec == CRBM_PREC_BF16) : 1;
            const int nsb = sbuild_border_splits(A.N, A.M, A.n, W.n_cu, W.nsb_max);
            e = launch_sbuild_mfma(A.N, A.M, P, A.samples, A.T, A.n, W.Om, W.Om16, W.S, A.prec, W.sb_kt, W.pack,
                                   W.pack_bytes, W.sb_order, W.sb_order_len,
                                   W.spart, nsplit, W.bx, W.bx_part, nsb, W.sb_fold, W.prof, stream);
        } else {
            // weighted (enumeration) sums: FP32 contraction on the vector units, the samples in as many runs (of at
            // least 16) as four workgroups per compute unit and the slices allow
            const int nt = (int)((P + SB_T - 1) / SB_T);
            const long ntri = (long)nt * (nt + 1) / 2;
            long z = std::min<long>(std::min<long>(W.n_sw, (A.n + SB_K - 1) / SB_K), 4L * W.n_cu / ntri);
            z = std::max<long>(z, 1);
            const long run = ((A.n + z - 1) / z + SB_K - 1) / SB_K * SB_K;
            z = (A.n + run - 1) / run;
            double2* S64 = A.solver == CRBM_SOLVER_CHOLESKY ? W.S64 : nullptr;
            W.prof->begin(PROF_SBUILD, stream);
            hipLaunchKernelGGL(k_sbuild, dim3((unsigned)ntri, (unsigned)z), dim3(256), 0, stream, A.N, A.M, P, A.samples,
                               A.T, A.weights, A.n, W.Om, W.S, nt, W.scal, S64, A.eps, run, z > 1 ? W.swpart : nullptr);
            if (z > 1)
                hipLaunchKernelGGL(k_sbuild_runs, dim3(nblk(P * P)), dim3(256), 0, stream, P, (int)z, W.swpart, W.Om,
                                   W.scal, W.S, S64, A.eps);
            W.prof->end(stream);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
    }

    MfView f{};
    if (A.solver == CRBM_SOLVER_CG_MATFREE) {
        e = launch_matfree_start(A.samples, W.bits, A.n, A.N, A.M, A.W, W.wplanes, stream);
        if (e != hipSuccess) return e;
        f.N = A.N;
        f.M = A.M;
        f.Np = theta_np(A.N);
        f.rows = theta_rows(A.M);
        f.planes = W.wplanes;
        f.vb = W.vstage;
        f.Om = W.Om;
        f.omv = reinterpret_cast<double2*>(W.dots + 6 * dots_blocks(P));
    }
    int n_dots = 0;
    if (A.solver == CRBM_SOLVER_CHOLESKY) {
        W.prof->begin(PROF_CHOLESKY, stream);
        e = launch_cholesky_solve(P, W.S, A.eps, W.F, W.S64, W.x, W.r, W.p, W.scal, A.weights != nullptr, stream);
        W.prof->end(stream);
        if (e != hipSuccess) return e;
    } else {
        hipLaunchKernelGGL(k_cg_init, dim3(nblk(P)), dim3(256), 0, stream, P, W.F, ff, n_ff, W.x, W.r, W.p, W.scal, f);
        W.prof->begin(PROF_CG, stream);
        for (int it = 0; it < A.cg_maxit; ++it) {
            e = apply_op(A, W, W.p, W.Ap, nullptr, W.scal + SC_DONE0 + (it & 1), &n_dots, f, stream);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_cg_step, dim3(nblk(P)), dim3(256), 0, stream, P, W.x, W.r, W.p, W.Ap, W.dots, n_dots,
                               W.scal, A.cg_tol, A.cg_maxit, it, f);
        }
        W.prof->end(stream);
    }
    // true residual |F - (S + eps) x|^2 in double (of a Cholesky solve: against the FP32-stored S)
    if (f.M) hipLaunchKernelGGL(k_mf_publish, dim3(nblk(P)), dim3(256), 0, stream, P, W.x, f);
    e = apply_op(A, W, W.x, W.Ap, W.F, nullptr, &n_dots, f, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finish, dim3(nblk(P)), dim3(256), 0, stream, A.N, A.M, A.a, A.b, A.W, W.x, W.dots, n_dots, ff,
                       n_ff, W.r, A.cg_tol, W.scal, A.stats);
    return hipGetLastError();
}

// ------------------------------------------------------------------ fidelity gradient
__global__ __launch_bounds__(1024) void k_loss(const float2* __restrict__ R, long n, double* __restrict__ loss) {
    __shared__ double sh[16];
    double acc = 0;
    for (long s = threadIdx.x; s < n; s += blockDim.x) {
        const double x = 1.0 - (double)R[s].x, y = -(double)R[s].y;
        acc += x * x + y * y;
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x != 0) return;
    double t = 0.0;
    for (int k = 0; k < 16; ++k) t += sh[k];
    *loss = t / (double)n;
}

// the gradient from caller-chosen scratch: bits (ot_bits_bytes(n, N)) and the contraction's chunk planes
static hipError_t fidelity_grad_on(const GradArgs& A, uint32_t* bits, void* partial, int n_cu, Profiler* prof,
                                   hipStream_t stream) {
    if (A.grad) {
        spin_cols(A.samples, A.n, A.N, bits, stream);
        hipError_t e = run_ot(A.N, A.M, bits, A.T, A.n, 3, 0, 1, nullptr, A.R, nullptr, partial, 0, A.grad, nullptr,
                              stream, nullptr, prof, n_cu);
        if (e != hipSuccess) return e;
    }
    if (A.loss) hipLaunchKernelGGL(k_loss, dim3(1), dim3(1024), 0, stream, A.R, A.n, A.loss);
    return hipGetLastError();
}

hipError_t launch_fidelity_grad(const GradArgs& A, const SrWork& W, hipStream_t stream) {
    return fidelity_grad_on(A, W.ot_bits, W.red, W.n_cu, W.prof, stream);
}

// Bytes before the chunk planes: the sign bits, and at least a byte per extended site (16 at a time) and sample, which
// the spins took before they were bits: the sizes that callers are told, and what the static scratch accepts, stay.
static size_t grad_bits_bytes(long n, int N) {
    const size_t b = std::max(ot_bits_bytes(n, N), (size_t)n * (size_t)((N + 1 + 15) / 16 * 16));
    return (b + 255) / 256 * 256;
}

// Scratch of the gradient for n samples, laid out as [sign bits | 256-byte alignment | chunk planes of one
// coefficient, 2 (N + 1)(M + 1) floats per sample chunk].
size_t fidelity_grad_scratch_bytes(int N, int M, long n) {
    long chunk;
    int n_chunks;
    ot_chunking(N, M, n, 1, chunk, n_chunks);
    return grad_bits_bytes(n, N) + (size_t)n_chunks * 2 * (size_t)(N + 1) * (size_t)(M + 1) * sizeof(float);
}

hipError_t launch_fidelity_grad_scratch(const GradArgs& A, void* scratch, int n_cu, hipStream_t stream) {
    const size_t rows = grad_bits_bytes(A.n, A.N);
    return fidelity_grad_on(A, static_cast<uint32_t*>(scratch), static_cast<unsigned char*>(scratch) + rows, n_cu, nullptr, stream);
}

}  // namespace crbm
