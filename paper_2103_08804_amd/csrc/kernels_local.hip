// theta GEMM, per-sample local estimators and Chebyshev moments.
//
//   theta = sigma W + 1 b^T          (RBM of Sec. I), a [n x N] x [N x M] product on the matrix cores
//   E_loc(s) = sum_bonds [J/4 s_i s_j + [s_i != s_j] J/2 psi(s^{ij})/psi(s)]   (Sec. VI)
//   R(s)     = phi(s)/psi_{n+1}(s)  for the Chebyshev targets of Sec. III
//   mu_n(q)  = < f_q^* beta_n t~_n / psi_gs >                    (Sec. II, App. A)
//
// A pair swap changes theta by Delta_k = -2 s_i (W_ik - W_jk), and
//   cosh(theta_k + Delta_k)/cosh(theta_k) = cosh(Delta_k) + tanh(theta_k) sinh(Delta_k),
// so the amplitude ratio of a bond is a product of M complex factors; each
// lane multiplies its own factors and the wave adds their logarithms.
// Log-amplitude differences between RBMs are summed element by element so
// that the M log 2 constants cancel before any rounding of the total.
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace crbm {

// ------------------------------------------------------------------ theta GEMM
// theta = sigma W + b on the matrix cores.  sigma = +-1 is exact in BF16, and each
// binary32 W entry is split exactly into three BF16 parts by truncation,
//   W = hi + mid + lo   (8 + 8 + 8 significand bits),
// so three v_mfma_f32_32x32x16_bf16 products give sigma W with exact products and
// FP32 accumulation.  The B columns of a tile of 64 hidden units are the real and imaginary
// parts of W ordered [Re 0..31 | Im 0..31 | Re 32..63 | Im 32..63], so that both parts of a
// unit end in one lane; W is split into its parts in that order once per RBM (k_wsplit).
//
// sigma comes as one sign bit per site (written once per sample set, in the launch that splits W): a lane builds its A
// operand, the eight sites of its sample that a matrix-core step reads, from one byte in registers, so the spins pass
// through no LDS.  The W tile (three parts x 128 rows x up to 128 sites, 104 KB) is staged in LDS once per
// workgroup, which then walks its samples in tiles of 8 waves x 32 with no barrier; beyond 128 sites the tile is
// staged in pieces per sample tile, of 64 sites for theta and of 128 for the products that are fused with a sum.
// 65,536 samples, 10 x 10, M = 400: 64 us per product, bound by the writes of theta (122 us with both operands staged
// per 128-sample tile, the spins a byte a load).
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8_t;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16_t;

constexpr int TH_C = 128, TH_K = 32;           // plane rows of a unit tile; sites are padded to TH_K
constexpr int TH_W = 8, TH_S = 32 * TH_W;      // waves and samples of a workgroup's tile
constexpr int TH_KMAX = 128;                   // sites of W staged at a time

// Word e of bits[s][w]: bit b of word w set where sigma of site 32 w + b is negative; nw = ceil(N / 32) words a row
template <bool WORDS>
__device__ __forceinline__ void spin_word(const int8_t* __restrict__ sig, long n, int N, int nw,
                                          uint32_t* __restrict__ bits, long e) {
    if (e >= n * nw) return;
    const long s = e / nw;
    const int i0 = 32 * (int)(e % nw), cnt = N - i0 < 32 ? N - i0 : 32;
    const int8_t* row = sig + s * N + i0;
    uint32_t m = 0;
    if (WORDS) {   // rows start on 4 bytes and N is a multiple of 4: four sign bits per word
#pragma unroll
        for (int d = 0; d < 8; ++d)
            if (4 * d < cnt) {
                const uint32_t x = (reinterpret_cast<const uint32_t*>(row)[d] >> 7) & 0x01010101u;
                m |= ((x * 0x10204080u) >> 28) << (4 * d);
            }
    } else {
        for (int b = 0; b < cnt; ++b) m |= (row[b] < 0 ? 1u : 0u) << b;
    }
    bits[e] = m;
}
// whether four sign bits may be taken from each word of four spins
static bool spin_rows_aligned(const int8_t* sig, int N) { return N % 4 == 0 && (reinterpret_cast<uintptr_t>(sig) & 3) == 0; }

// ------------------------------------------------------------------ helpers
// f_q(sigma) = N^{-1/2} sum_r exp(-i q.r) sigma_r / 2 over the wave's spins
__device__ __forceinline__ float2 site_phase(int r, int kind, int Lx, double q0, double q1) {
    const int x = kind == 0 ? r : r % Lx;
    const int y = kind == 0 ? 0 : r / Lx;
    const double ph = q0 * x + q1 * y;
    double s, c;
    sincos(ph, &s, &c);
    return make_float2((float)c, (float)-s);
}

__device__ __forceinline__ float2 fq_wave(const WaveSpins& sp, int lane, const Geometry& g, double q0, double q1) {
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int site = q * kWave + lane;
        if (site < g.N) acc = cadd(acc, cscale(site_phase(site, g.kind, g.Lx, q0, q1), 0.5f * (float)sp.s[q]));
    }
    acc = wave_sum(acc);
    return cscale(acc, rsqrtf((float)g.N));
}

// sum_i a_i sigma_i over the wave
__device__ __forceinline__ float2 a_dot_sigma(const float2* a, const WaveSpins& sp, int lane, int N) {
    float2 acc = make_float2(0.f, 0.f);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int site = q * kWave + lane;
        if (site < N) acc = cadd(acc, cscale(a[site], (float)sp.s[q]));
    }
    return acc;
}

// ------------------------------------------------------------------ theta GEMM fused with sum log cosh
// For the moment ratios only the per-sample sums  L(s) = sum_k log cosh theta_k(s)  of an RBM are
// needed, not theta itself.  With both parts of a hidden unit in one lane, each lane forms, row by row,
//   log cosh z = s z + log((1 + w)/2),   s = sign(Re z),  w = exp(-2 s z),  |(1 + w)/2| <= 1,
// keeping s z as a sum and (1 + w)/2 as a product, multiplies the products over the tile's columns
// by a reduce-scatter over the lane bits and takes one complex log per sample row.
//
// The planes of W are [3][Mt 128][Np], Np = N rounded up to TH_K, zero padded; the product's
// workgroups only copy tiles of them.  With spins given (sig), the blocks past the planes' w_blocks write their sign
// bits, so that a call on new samples has no launch of its own for them (but see launch_wsplit).
template <bool WORDS>
__global__ __launch_bounds__(256) void k_wsplit(ThetaSet set, int N, int M, int Np, int Mt, uint16_t* __restrict__ planes,
                                                unsigned w_blocks, const int8_t* __restrict__ sig, long n, int nw,
                                                uint32_t* __restrict__ bits) {
    if (blockIdx.x >= w_blocks) {
        if (blockIdx.z == 0) spin_word<WORDS>(sig, n, N, nw, bits, (long)(blockIdx.x - w_blocks) * 256 + threadIdx.x);
        return;
    }
    const float2* W = set.W[blockIdx.z];
    planes += blockIdx.z * (3L * Mt * TH_C * Np);
    const long rows = (long)Mt * TH_C;
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= rows * Np) return;
    const int r = (int)(idx / Np), i = (int)(idx % Np);
    const int rr = r % TH_C, cb = rr / 32;
    const int k = (r / TH_C) * 64 + (cb >> 1) * 32 + rr % 32;
    float w = 0.f;
    if (i < N && k < M) {
        const float2 v = W[(long)i * M + k];
        w = (cb & 1) ? v.y : v.x;
    }
    split_store(planes, rows * Np, idx, w);
}
// W of the set into planes; the sign bits of the n samples sig into bits (sig null: they are there already).  Past 128
// sites and 1.5 MB of bits they have a launch of their own, as the first product after them was slower with the bits
// written by the launch before it (256 sites, M = 128, 131,072 samples: 212 us against 148 us, whole moments 876 us
// against 815 us; 200 sites, M = 512, 65,536 samples: 1,011 us against 998 us); up to there the launch less is what
// shows (256 sites, M = 512, 32,768 samples: 793 us against 800 us), and up to 128 sites there is no difference at
// 4 MB either (100 sites, M = 400, 262,144 samples: 1,788 us both ways).
constexpr long kSpinWords = 3L << 17;
static void launch_wsplit(const ThetaSet& set, int N, int M, uint16_t* planes, const int8_t* sig, long n, uint32_t* bits,
                          hipStream_t stream) {
    const int Np = theta_np(N), nw = spin_words(N);
    const unsigned w_blocks = (unsigned)((theta_rows(M) * Np + 255) / 256);
    const unsigned s_blocks = sig ? (unsigned)((n * nw + 255) / 256) : 0u;
    auto blocks = [&](unsigned w, unsigned spins, int count) {
        const dim3 grid(w + spins, 1, count);
        if (spin_rows_aligned(sig, N))
            hipLaunchKernelGGL(k_wsplit<true>, grid, dim3(256), 0, stream, set, N, M, Np, (M + 63) / 64, planes, w, sig, n, nw,
                               bits);
        else
            hipLaunchKernelGGL(k_wsplit<false>, grid, dim3(256), 0, stream, set, N, M, Np, (M + 63) / 64, planes, w, sig, n,
                               nw, bits);
    };
    if (N > TH_KMAX && sig && n * nw > kSpinWords) {
        blocks(0, s_blocks, 1);
        blocks(w_blocks, 0, set.count);
    } else {
        blocks(w_blocks, s_blocks, set.count);
    }
}

// Complex product and |a|^2 with their fused multiply-adds written out, so that the moments do not depend in the
// last bits on which of the two products of a sum the compiler fuses in one kernel or another.
__device__ __forceinline__ float2 cmul_fused(float2 a, float2 b) {
    return make_float2(__builtin_fmaf(a.x, b.x, -(a.y * b.y)), __builtin_fmaf(a.x, b.y, a.y * b.x));
}
__device__ __forceinline__ float norm2_fused(float2 a) { return __builtin_fmaf(a.x, a.x, a.y * a.y); }

// cosh_factor with sign 1
__device__ __forceinline__ void lc_factor(float2 z, float2& lin, float2& p) {
    const float sg = z.x >= 0.f ? 1.f : -1.f;
    const float ex = expf(-2.f * fabsf(z.x));
    const float2 cs = cos_sin(2.f * sg * z.y);
    lin.x += fabsf(z.x);
    lin.y += sg * z.y;
    p = cmul_fused(p, make_float2(0.5f * __builtin_fmaf(ex, cs.x, 1.f), (-0.5f * ex) * cs.y));
}

// combine two partial sums of log cosh: the linear parts add, the bounded factors multiply
__device__ __forceinline__ void lc_join(float2& lin, float2& pr, float2 lin2, float2 pr2) {
    lin = cadd(lin, lin2);
    pr = cmul_fused(pr, pr2);
}

// The tile product.  KC: sites staged at a time (the padded N up to 128).  Lane l of wave w ends with column
// l % 32 of each 32-column block cb in acc[cb], rows 8 (v / 4) + 4 (l / 32) + v % 4 of the wave's 32 samples.
template <int KC>
struct ThetaLds {
    static constexpr int ROW = KC * 2 + 16;    // bytes per plane row: 16 rows of a fragment read fall in distinct banks
    unsigned char w[3][TH_C * ROW];
};
// sites [k0, k0 + KC) of the three parts of unit tile ct; columns past Np are left as they are (never read)
template <int KC>
__device__ __forceinline__ void theta_stage(ThetaLds<KC>& lds, const uint16_t* __restrict__ planes, long rows, int Np,
                                            int ct, int k0) {
    const int len = Np - k0 < KC ? Np - k0 : KC, per = len / 8;
    for (int c = threadIdx.x; c < 3 * TH_C * per; c += 64 * TH_W) {
        const int pr = c / per, ch = c % per, part = pr / TH_C, rr = pr % TH_C;
        const uint16_t* src = planes + part * rows * Np + ((long)ct * TH_C + rr) * Np + k0 + ch * 8;
        *reinterpret_cast<i32x4_t*>(lds.w[part] + rr * ThetaLds<KC>::ROW + ch * 16) = *reinterpret_cast<const i32x4_t*>(src);
    }
}
// the eight BF16 spins (1 or -1) of sign bits 0..7 of x
__device__ __forceinline__ i32x4_t spin_frag(uint32_t x) {
    i32x4_t a;
#pragma unroll
    for (int d = 0; d < 4; ++d)
        a[d] = (int)(0x3F803F80u | ((x << (15 - 2 * d)) & 0x8000u) | ((x << (30 - 2 * d)) & 0x80000000u));
    return a;
}
template <int KC>
__device__ __forceinline__ void theta_steps(const ThetaLds<KC>& lds, const uint32_t* __restrict__ words, int len, int lane,
                                            floatx16_t (&acc)[4]) {
#pragma unroll
    for (int k2 = 0; k2 < KC; k2 += 32) {
        if (k2 >= len) break;
        const uint32_t word = words[k2 >> 5];
#pragma unroll
        for (int kq = k2; kq < k2 + 32; kq += 16) {
            const i32x4_t a = spin_frag(word >> ((kq & 31) + 8 * (lane >> 5)));
            const int koff = (kq + 8 * (lane >> 5)) * 2;
#pragma unroll
            for (int part = 0; part < 3; ++part)
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) {
                    const i32x4_t bw = *reinterpret_cast<const i32x4_t*>(
                        lds.w[part] + (cb * 32 + (lane & 31)) * ThetaLds<KC>::ROW + koff);
                    acc[cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16((bf16x8_t)a, (bf16x8_t)bw, acc[cb], 0, 0, 0);
                }
        }
    }
}
// acc = sigma W of the wave's 32 samples from sw on.  Np > KC: the W tile is staged piece by piece (every wave of
// the workgroup must call); else it has been staged before.
template <int KC>
__device__ __forceinline__ void theta_tile(ThetaLds<KC>& lds, const uint32_t* __restrict__ bits, long n, int Np,
                                           const uint16_t* __restrict__ planes, long rows, int ct, long sw,
                                           floatx16_t (&acc)[4]) {
    const int lane = threadIdx.x & 63, nw = Np / 32;
    const long s = sw + (lane & 31) < n ? sw + (lane & 31) : n - 1;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[cb][v] = 0.f;
    if (Np <= KC) {
        theta_steps<KC>(lds, bits + s * nw, Np, lane, acc);
        return;
    }
    for (int k0 = 0; k0 < Np; k0 += KC) {
        __syncthreads();
        theta_stage<KC>(lds, planes, rows, Np, ct, k0);
        __syncthreads();
        theta_steps<KC>(lds, bits + s * nw + k0 / 32, Np - k0, lane, acc);
    }
}
// The loop of a workgroup (x, ct) over its sample tiles: body(sw, acc) with the wave's first sample sw.
template <int KC, class F>
__device__ __forceinline__ void theta_walk(ThetaLds<KC>& lds, const uint32_t* __restrict__ bits, long n, int Np,
                                           const uint16_t* __restrict__ planes, long rows, int ct, F&& body) {
    const int wave = threadIdx.x >> 6;
    if (Np <= KC) {
        theta_stage<KC>(lds, planes, rows, Np, ct, 0);
        __syncthreads();
    }
    for (long t0 = (long)blockIdx.x * TH_S; t0 < n; t0 += (long)gridDim.x * TH_S) {
        const long sw = t0 + wave * 32;
        floatx16_t acc[4];
        if (Np > KC || sw < n) theta_tile<KC>(lds, bits, n, Np, planes, rows, ct, sw, acc);
        if (sw < n) body(sw, acc);
    }
}
// workgroups along the samples: one a compute unit over the unit tiles, two where the staged tile is at most 64 sites
// (theta then has both resident; the products that are fused with a sum hold one at a time for their registers, and
// take two rounds), at most one per sample tile
static unsigned theta_grid(long n, int Np, int Mt, int n_cu) {
    const long slots = (long)n_cu * (Np <= 64 ? 2 : 1), tiles = (n + TH_S - 1) / TH_S;
    long g = slots / Mt;
    if (g < 1) g = 1;
    return (unsigned)(g < tiles ? g : tiles);
}
// calls f(std::integral_constant<int, KC>) for the padded row length Np
template <class F>
static void theta_dispatch(int Np, F&& f) {
    if (Np <= 32) f(std::integral_constant<int, 32>{});
    else if (Np <= 64) f(std::integral_constant<int, 64>{});
    else if (Np <= 96) f(std::integral_constant<int, 96>{});
    else f(std::integral_constant<int, TH_KMAX>{});
}

// theta = sigma W + b, complex64 [n][M]: lane column j holds units 64 ct + j (blocks 0, 1) and
// 64 ct + 32 + j (blocks 2, 3), real and imaginary part together, so 32 lanes store 256 contiguous bytes.
// blockIdx.z: which of up to three RBMs on the same samples.
template <int KC>
__global__ __launch_bounds__(64 * TH_W, 2) void k_theta(const uint32_t* __restrict__ bits, long n, int Np, int M,
                                                     ThetaSet set, const uint16_t* __restrict__ planes, long plane_len,
                                                     int Mt) {
    __shared__ __attribute__((aligned(16))) ThetaLds<KC> lds;
    const int lane = threadIdx.x & 63, ct = blockIdx.y, z = blockIdx.z;
    const float2* b = set.b[z];
    float2* theta = set.out[z];
    const int ku0 = ct * 64 + (lane & 31), ku1 = ku0 + 32;
    const float2 b0 = ku0 < M ? b[ku0] : make_float2(0.f, 0.f);
    const float2 b1 = ku1 < M ? b[ku1] : make_float2(0.f, 0.f);
    theta_walk<KC>(lds, bits, n, Np, planes + z * plane_len, (long)Mt * TH_C, ct,
                   [&](long sw, const floatx16_t (&acc)[4]) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const long sm = sw + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            if (sm >= n) continue;
            if (ku0 < M) theta[sm * M + ku0] = make_float2(acc[0][v] + b0.x, acc[1][v] + b0.y);
            if (ku1 < M) theta[sm * M + ku1] = make_float2(acc[2][v] + b1.x, acc[3][v] + b1.y);
        }
    });
}

hipError_t launch_matfree_start(const int8_t* sig, uint32_t* bits, long n, int N, int M, const float2* W, uint16_t* planes,
                                hipStream_t stream) {
    ThetaSet set{};
    set.count = 1;
    set.W[0] = W;
    launch_wsplit(set, N, M, planes, sig, n, bits, stream);
    return hipGetLastError();
}

hipError_t launch_theta(const int8_t* sig, uint32_t* bits, long n, int N, int M, const ThetaSet& set, uint16_t* planes,
                        int n_cu, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int Np = theta_np(N);
    const int Mt = (M + 63) / 64;
    launch_wsplit(set, N, M, planes, sig, n, bits, stream);
    // W of more than 128 sites is staged in pieces anyway: pieces of 64 leave room for two workgroups per compute unit
    // (8,192 samples, N = 256, M = 512: 68 us against 98 us in pieces of 128); up to 128 sites it is staged once
    theta_dispatch(Np > TH_KMAX ? 64 : Np, [&](auto kc) {
        hipLaunchKernelGGL(k_theta<kc.value>, dim3(theta_grid(n, kc.value, Mt * set.count, n_cu), (unsigned)Mt, set.count),
                           dim3(64 * TH_W), 0, stream, bits, n, Np, M, set, planes, lc_plane_elems(N, M), Mt);
    });
    return hipGetLastError();
}

// a double moved between lanes by a DPP control
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// a of this lane and of lane ^ 16 added where lane bit 4 is clear, b of the two where it is set
__device__ __forceinline__ double swap_add(double a, double b) {
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) + __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}
// the same swap on binary32 values: x the value of the lane with bit 4 clear, y that of its partner
__device__ __forceinline__ float2 swap16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return make_float2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
// rows t and t + W, t < W: a lane keeps the second where hi and adds the other lane's (CTRL) sent row
template <int W, int CTRL>
__device__ __forceinline__ void scatter_step(double (&px)[16], double (&py)[16], bool hi) {
#pragma unroll
    for (int t = 0; t < W; ++t) {
        const double kx = hi ? px[t + W] : px[t], ky = hi ? py[t + W] : py[t];
        const double sx = hi ? px[t] : px[t + W], sy = hi ? py[t] : py[t + W];
        px[t] = kx + dpp_double<CTRL>(sx);
        py[t] = ky + dpp_double<CTRL>(sy);
    }
}

// O v of the matrix-free S product without writing G = sigma V_W + v_b: the theta product of V tile by
// tile, each unit's G_sk multiplied by T_sk in the epilogue and the tile's 64 units summed per sample in
// double (products in FP32 widened to double, as a separate pass over G would); a reduce-scatter over
// lane bits 4..0 leaves each row's sum in two lanes.  partial[ct][s] (double2, n per 64-unit tile).
// One tile's rows: the products of a row's two units per lane, then the reduce-scatter.  t: T of the lane's rows and
// units, loaded before the matrix product so that the loads are in flight during it (0 past n and M).
__device__ __forceinline__ void theta_ov_rows(const floatx16_t (&acc)[4], const float2 (&t)[2][16], long sw, long n, int ct,
                                              float2 b0, float2 b1, int lane, double2* __restrict__ partial) {
    double px[16], py[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const float gx = acc[0][v] + b0.x, gy = acc[1][v] + b0.y, hx = acc[2][v] + b1.x, hy = acc[3][v] + b1.y;
        px[v] = (double)t[0][v].x * gx - (double)t[0][v].y * gy;
        py[v] = (double)t[0][v].x * gy + (double)t[0][v].y * gx;
        px[v] += (double)t[1][v].x * hx - (double)t[1][v].y * hy;
        py[v] += (double)t[1][v].x * hy + (double)t[1][v].y * hx;
    }
    // reduce-scatter of the 16 rows over the 32 columns: lane bits 4, 3, 2, 1 halve the rows a lane
    // keeps, bit 0 adds the last pair; the lane ends with row index 8 b4 + 4 b3 + 2 b2 + b1.  Bit 4 by row swaps, which
    // leave both addends of a kept row in its lane, the others by lane moves within a row of 16: over LDS permutes, this
    // and the products took 40 of the kernel's 108 us (65,536 samples, N = 100, M = 400; now 71)
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        px[t] = swap_add(px[t], px[t + 8]);
        py[t] = swap_add(py[t], py[t + 8]);
    }
    scatter_step<4, 0x128>(px, py, (lane & 8) != 0);    // row_ror:8
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const bool hi = (lane & 4) != 0;
        const double kx = hi ? px[t + 2] : px[t], ky = hi ? py[t + 2] : py[t];
        const double sx = hi ? px[t] : px[t + 2], sy = hi ? py[t] : py[t + 2];
        px[t] = kx + __shfl_xor(sx, 4);
        py[t] = ky + __shfl_xor(sy, 4);
    }
    scatter_step<1, 0x4E>(px, py, (lane & 2) != 0);     // quad_perm [2, 3, 0, 1]
    px[0] += dpp_double<0xB1>(px[0]);                   // quad_perm [1, 0, 3, 2]
    py[0] += dpp_double<0xB1>(py[0]);
    if (lane & 1) return;
    const int v = 8 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1) + ((lane >> 1) & 1);
    const long sm = sw + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (sm < n) partial[(long)ct * n + sm] = make_double2(px[0], py[0]);
}

template <int KC>
__global__ __launch_bounds__(64 * TH_W, 2) void k_theta_ov(const uint32_t* __restrict__ bits, long n, int Np, int M,
                                                        const float2* __restrict__ vb,
                                                        const uint16_t* __restrict__ planes, int Mt,
                                                        const float2* __restrict__ T, double2* __restrict__ partial,
                                                        const double* __restrict__ skip) {
    if (skip && *skip != 0.0) return;     // a converged iterative solve skips the product
    __shared__ __attribute__((aligned(16))) ThetaLds<KC> lds;
    const int lane = threadIdx.x & 63, ct = blockIdx.y;
    const int ku0 = ct * 64 + (lane & 31), ku1 = ku0 + 32;
    const float2 b0 = ku0 < M ? vb[ku0] : make_float2(0.f, 0.f);
    const float2 b1 = ku1 < M ? vb[ku1] : make_float2(0.f, 0.f);
    if (Np <= KC) {
        theta_stage<KC>(lds, planes, (long)Mt * TH_C, Np, ct, 0);
        __syncthreads();
    }
    for (long t0 = (long)blockIdx.x * TH_S; t0 < n; t0 += (long)gridDim.x * TH_S) {
        const long sw = t0 + (threadIdx.x >> 6) * 32;
        float2 t[2][16];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const long sm = sw + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
            const bool in = sm < n;
            const float2* row = T + (in ? sm : 0) * M;
            t[0][v] = row[ku0 < M ? ku0 : 0];
            t[1][v] = row[ku1 < M ? ku1 : 0];
            if (!in || ku0 >= M) t[0][v] = make_float2(0.f, 0.f);
            if (!in || ku1 >= M) t[1][v] = make_float2(0.f, 0.f);
        }
        floatx16_t acc[4];
        if (Np > KC || sw < n) theta_tile<KC>(lds, bits, n, Np, planes, (long)Mt * TH_C, ct, sw, acc);
        if (sw < n) theta_ov_rows(acc, t, sw, n, ct, b0, b1, lane, partial);
    }
}

// u[s] = sum over the tiles of partial[ct][s] + sigma_s . v_a: one thread per sample on a bounded grid
// (v_a in LDS, the spins as sign bits), so that the launches a converged solve skips stay cheap
constexpr int kOvFinalBlocks = 1024;
__global__ __launch_bounds__(256) void k_ov_final(int N, long n, int Mt, const uint32_t* __restrict__ bits, int nw,
                                                  const double2* __restrict__ va, const double2* __restrict__ partial,
                                                  double2* __restrict__ u, const double2* __restrict__ omv, int n_omv,
                                                  double* __restrict__ mean_out, const double* __restrict__ skip) {
    if (skip && *skip != 0.0) return;
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x < 64) {   // <O>.v, in one fixed order
        double2 m = make_double2(0.0, 0.0);
        for (int b = lane; b < n_omv; b += kWave) m = zadd(m, omv[b]);
        m = wave_sum(m);
        if (lane == 0) { mean_out[0] = m.x; mean_out[1] = m.y; }
    }
    __shared__ double2 a[256];
    for (int i = threadIdx.x; i < N; i += 256) a[i] = va[i];
    __syncthreads();
    for (long s = (long)blockIdx.x * 256 + threadIdx.x; s < n; s += (long)gridDim.x * 256) {
        const uint32_t* row = bits + s * nw;
        double ax = 0.0, ay = 0.0;
        for (int w = 0; w < nw; ++w) {
            const uint32_t word = row[w];
            const int cnt = N - 32 * w < 32 ? N - 32 * w : 32;
#pragma unroll 8
            for (int b = 0; b < cnt; ++b) {
                const double sv = (word >> b) & 1u ? -1.0 : 1.0;
                ax += sv * a[32 * w + b].x;
                ay += sv * a[32 * w + b].y;
            }
        }
        for (int ct = 0; ct < Mt; ++ct) {
            const double2 p = partial[(long)ct * n + s];
            ax += p.x;
            ay += p.y;
        }
        u[s] = make_double2(ax, ay);
    }
}

hipError_t launch_theta_ov(const uint32_t* bits, long n, int N, int M, const float2* vb, const double2* va,
                           const float2* T, const uint16_t* planes, double2* partial, double2* u, const double2* omv,
                           int n_omv, double* mean_out, int n_cu, hipStream_t stream, const double* skip) {
    if (n <= 0) return hipSuccess;
    const int Np = theta_np(N);
    const int Mt = (M + 63) / 64;
    theta_dispatch(Np, [&](auto kc) {
        hipLaunchKernelGGL(k_theta_ov<kc.value>, dim3(theta_grid(n, Np, Mt, n_cu), (unsigned)Mt), dim3(64 * TH_W), 0,
                           stream, bits, n, Np, M, vb, planes, Mt, T, partial, skip);
    });
    const long fb = (n + 255) / 256;
    hipLaunchKernelGGL(k_ov_final, dim3((unsigned)(fb < kOvFinalBlocks ? fb : kOvFinalBlocks)), dim3(256), 0, stream,
                       N, n, Mt, bits, spin_words(N), va, partial, u, omv, n_omv, mean_out, skip);
    return hipGetLastError();
}

// the sums of one tile's rows: wave's accumulators (rows sw + ..) to partial[ct][row]
__device__ __forceinline__ void theta_lc_rows(const floatx16_t (&acc)[4], long sw, const int8_t* __restrict__ sig, long n,
                                              int N, int M, int ct, int ku0, int ku1, float2 b0, float2 b1,
                                              const float2* __restrict__ b, const float2* __restrict__ W, int lane,
                                              float2* __restrict__ partial) {
    float2 lin[16], pr[16];
    uint32_t poles = 0;   // bit 2 v + h: element (row v, unit h) within the band of a zero of cosh
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        lin[v] = make_float2(0.f, 0.f);
        pr[v] = make_float2(1.f, 0.f);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if ((h == 0 ? ku0 : ku1) >= M) continue;
            const float2 bb = h == 0 ? b0 : b1;
            const float2 z = make_float2(acc[2 * h][v] + bb.x, acc[2 * h + 1][v] + bb.y);
            if (near_pole(z)) poles |= 1u << (2 * v + h);
            else lc_factor(z, lin[v], pr[v]);
        }
    }
    // accumulator element v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4 of the wave's 32 samples
    while (poles) {
        const int bit = __ffs(poles) - 1;
        poles &= poles - 1;
        const int v = bit >> 1, ku = (bit & 1) ? ku1 : ku0;
        const long row = sw + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (row >= n) continue;
        float2 lcr, thr;
        pole_eval(theta_double(sig + row * N, N, M, ku, b, W), lcr, thr);
#pragma unroll
        for (int vv = 0; vv < 16; ++vv)
            if (vv == v) lin[vv] = cadd(lin[vv], lcr);
    }
    // reduce-scatter of the 16 rows over the 32 columns (lane bits 4..1), then the last pair (bit 0):
    // lane ends with row 8 b4 + 4 b3 + 2 b2 + b1 of its half
#pragma unroll
    for (int t = 0; t < 8; ++t) {   // bit 4: the swap leaves both addends of a kept row in its lane
        const float2 lx = swap16(lin[t].x, lin[t + 8].x), ly = swap16(lin[t].y, lin[t + 8].y);
        const float2 px = swap16(pr[t].x, pr[t + 8].x), py = swap16(pr[t].y, pr[t + 8].y);
        const bool hi = (lane & 16) != 0;   // there the lane's own factor is the second
        lin[t] = make_float2(lx.x + lx.y, ly.x + ly.y);
        pr[t] = cmul_fused(hi ? make_float2(px.y, py.y) : make_float2(px.x, py.x),
                           hi ? make_float2(px.x, py.x) : make_float2(px.y, py.y));
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bool hi = (lane & 8) != 0;
        const float2 kl = hi ? lin[t + 4] : lin[t], kp = hi ? pr[t + 4] : pr[t];
        const float2 sl = hi ? lin[t] : lin[t + 4], sp = hi ? pr[t] : pr[t + 4];
        lin[t] = kl;
        pr[t] = kp;
        lc_join(lin[t], pr[t], make_float2(dpp_move<0x128, 0xF>(sl.x), dpp_move<0x128, 0xF>(sl.y)),
                make_float2(dpp_move<0x128, 0xF>(sp.x), dpp_move<0x128, 0xF>(sp.y)));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const bool hi = (lane & 4) != 0;
        const float2 kl = hi ? lin[t + 2] : lin[t], kp = hi ? pr[t + 2] : pr[t];
        const float2 sl = hi ? lin[t] : lin[t + 2], sp = hi ? pr[t] : pr[t + 2];
        lin[t] = kl;
        pr[t] = kp;
        lc_join(lin[t], pr[t], make_float2(__shfl_xor(sl.x, 4), __shfl_xor(sl.y, 4)),
                make_float2(__shfl_xor(sp.x, 4), __shfl_xor(sp.y, 4)));
    }
    {
        const bool hi = (lane & 2) != 0;
        const float2 kl = hi ? lin[1] : lin[0], kp = hi ? pr[1] : pr[0];
        const float2 sl = hi ? lin[0] : lin[1], sp = hi ? pr[0] : pr[1];
        lin[0] = kl;
        pr[0] = kp;
        lc_join(lin[0], pr[0], make_float2(dpp_move<0x4E, 0xF>(sl.x), dpp_move<0x4E, 0xF>(sl.y)),
                make_float2(dpp_move<0x4E, 0xF>(sp.x), dpp_move<0x4E, 0xF>(sp.y)));
    }
    {
        const float2 pn = make_float2(dpp_move<0xB1, 0xF>(pr[0].x), dpp_move<0xB1, 0xF>(pr[0].y));
        lin[0] = cadd(lin[0], make_float2(dpp_move<0xB1, 0xF>(lin[0].x), dpp_move<0xB1, 0xF>(lin[0].y)));
        pr[0] = cmul_fused(pn, pr[0]);
    }
    if (lane & 1) return;
    const int v = 8 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 2 * ((lane >> 2) & 1) + ((lane >> 1) & 1);
    const long sm = sw + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
    if (sm >= n) return;
    const float n2 = norm2_fused(pr[0]);
    partial[(long)ct * n + sm] = make_float2(lin[0].x + 0.5f * logf(n2), lin[0].y + atan2f(pr[0].y, pr[0].x));
}

template <int KC>
__global__ __launch_bounds__(64 * TH_W, 2) void k_theta_lc(const int8_t* __restrict__ sig, const uint32_t* __restrict__ bits,
                                                        long n, int N, int Np, int M, const float2* __restrict__ b,
                                                        const float2* __restrict__ W,
                                                        const uint16_t* __restrict__ planes, int Mt,
                                                        float2* __restrict__ partial) {
    __shared__ __attribute__((aligned(16))) ThetaLds<KC> lds;
    const int lane = threadIdx.x & 63, ct = blockIdx.y;   // ct: 64-unit tile
    // lane column j = lane % 32: units k0u = 64 ct + j (acc 0, 1) and k1u = k0u + 32 (acc 2, 3)
    const int ku0 = ct * 64 + (lane & 31), ku1 = ku0 + 32;
    const float2 b0 = ku0 < M ? b[ku0] : make_float2(0.f, 0.f);
    const float2 b1 = ku1 < M ? b[ku1] : make_float2(0.f, 0.f);
    if (Np <= KC) {
        theta_stage<KC>(lds, planes, (long)Mt * TH_C, Np, ct, 0);
        __syncthreads();
    }
    for (long t0 = (long)blockIdx.x * TH_S; t0 < n; t0 += (long)gridDim.x * TH_S) {
        const long sw = t0 + (threadIdx.x >> 6) * 32;
        floatx16_t acc[4];
        if (Np > KC || sw < n) theta_tile<KC>(lds, bits, n, Np, planes, (long)Mt * TH_C, ct, sw, acc);
        if (sw < n) theta_lc_rows(acc, sw, sig, n, N, M, ct, ku0, ku1, b0, b1, b, W, lane, partial);
    }
}

// B[s] = beta exp(a.sigma + sum_tiles partial - Lg[s])  (Lg = NULL: the sums of psi_gs itself go to
// Lg_out instead), one thread per sample with a in LDS and the spins as sign bits (one wave per sample, 63 of its
// lanes waiting on the exponential and the sine of one, took 55 us for 131,072 samples of 100 sites, now 11 us);
// the tile partials and Lg are added in double
__global__ __launch_bounds__(256) void k_lc_final(int N, long n, int Mt, const uint32_t* __restrict__ bits, int nw,
                                                  const float2* __restrict__ a, const float2* __restrict__ partial,
                                                  const double2* __restrict__ Lg, const double2* __restrict__ beta,
                                                  double2* __restrict__ B, double2* __restrict__ Lg_out) {
    __shared__ float2 sa[256];
    sa[threadIdx.x] = threadIdx.x < N ? a[threadIdx.x] : make_float2(0.f, 0.f);
    __syncthreads();
    const long s = (long)blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    uint32_t word[8];
#pragma unroll
    for (int w = 0; w < 8; ++w) word[w] = w < nw ? bits[s * nw + w] : 0u;
    // a.sigma: the sites l, l + 64, .. in binary32, their sums over l in double
    double x = 0.0, y = 0.0;
    const int cnt = N < 64 ? N : 64;
    for (int l = 0; l < cnt; ++l) {
        float2 f = make_float2(0.f, 0.f);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float2 v = sa[64 * q + l];
            const float sg = ((l < 32 ? word[2 * q] : word[2 * q + 1]) >> (l & 31)) & 1u ? -1.f : 1.f;
            f = cadd(f, cscale(v, sg));
        }
        x += (double)f.x;
        y += (double)f.y;
    }
    for (int ct = 0; ct < Mt; ++ct) {
        const float2 pt = partial[(long)ct * n + s];
        x += pt.x;
        y += pt.y;
    }
    if (!Lg) {
        Lg_out[s] = make_double2(x, y);
        return;
    }
    const double2 g = Lg[s];
    const double dx = x - g.x, dy = y - g.y;
    const double m = exp(dx);
    double sn, cs;
    sincos(dy, &sn, &cs);
    B[s] = zmul(*beta, make_double2(m * cs, m * sn));
}

hipError_t launch_lc_sums(const int8_t* sig, uint32_t* bits, bool new_samples, long n, int N, int M, const float2* a,
                          const float2* b, const float2* W, uint16_t* planes, float2* partial, const double2* Lg,
                          const double2* beta, double2* B, double2* Lg_out, int n_cu, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const int Np = theta_np(N);
    const int Mt = (M + 63) / 64;
    ThetaSet set{};
    set.count = 1;
    set.W[0] = W;
    launch_wsplit(set, N, M, planes, new_samples ? sig : nullptr, n, bits, stream);
    theta_dispatch(Np, [&](auto kc) {
        hipLaunchKernelGGL(k_theta_lc<kc.value>, dim3(theta_grid(n, Np, Mt, n_cu), (unsigned)Mt), dim3(64 * TH_W), 0,
                           stream, sig, bits, n, N, Np, M, b, W, planes, Mt, partial);
    });
    hipLaunchKernelGGL(k_lc_final, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, N, n, Mt, bits,
                       spin_words(N), a, partial, Lg, beta, B, Lg_out);
    return hipGetLastError();
}

// ------------------------------------------------------------------ local estimators
// One sample per wave: log psi, tanh theta and O (lanes over the hidden units), the anti-aligned bonds, then the exchange
// sum over them, eight bonds at a time.
// a wave-uniform 64-bit value in scalar registers
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const uint32_t lo = (uint32_t)uniform((int)(uint32_t)v), hi = (uint32_t)uniform((int)(uint32_t)(v >> 32));
    return (uint64_t)hi << 32 | lo;
}

// Reduce-scatter of 8 bond shares (log |p|, p/|p|) over the wave: across lane bit 5 keep 4 of the 8,
// bit 4 keep 2, bit 3 keep 1, then add (multiply) within the 8 lanes, so that lanes 8 g .. 8 g + 7
// end with the whole of share g in lm[0], ph[0].
__device__ __forceinline__ void reduce_scatter8(float (&lm)[8], float2 (&ph)[8], int lane) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bool hi = (lane & 32) != 0;
        const float kl = hi ? lm[t + 4] : lm[t], sl = hi ? lm[t] : lm[t + 4];
        const float2 kp = hi ? ph[t + 4] : ph[t], sp = hi ? ph[t] : ph[t + 4];
        lm[t] = kl + __shfl_xor(sl, 32);
        ph[t] = cmul(kp, make_float2(__shfl_xor(sp.x, 32), __shfl_xor(sp.y, 32)));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const bool hi = (lane & 16) != 0;
        const float kl = hi ? lm[t + 2] : lm[t], sl = hi ? lm[t] : lm[t + 2];
        const float2 kp = hi ? ph[t + 2] : ph[t], sp = hi ? ph[t] : ph[t + 2];
        lm[t] = kl + __shfl_xor(sl, 16);
        ph[t] = cmul(kp, make_float2(__shfl_xor(sp.x, 16), __shfl_xor(sp.y, 16)));
    }
    {
        const bool hi = (lane & 8) != 0;
        const float kl = hi ? lm[1] : lm[0], sl = hi ? lm[0] : lm[1];
        const float2 kp = hi ? ph[1] : ph[0], sp = hi ? ph[0] : ph[1];
        lm[0] = kl + __shfl_xor(sl, 8);
        ph[0] = cmul(kp, make_float2(__shfl_xor(sp.x, 8), __shfl_xor(sp.y, 8)));
    }
#pragma unroll
    for (int o = 4; o >= 1; o >>= 1) {
        lm[0] += __shfl_xor(lm[0], o);
        ph[0] = cmul(ph[0], make_float2(__shfl_xor(ph[0].x, o), __shfl_xor(ph[0].y, o)));
    }
}

// (log |p|, p / |p|) of a lane's share p, from n2 = |p|^2, on the hardware log2 and reciprocal square
// root: n2 is a product of a few factors of modest size, far from the denormal range the library
// forms guard against (p = 0 gives log |p| = -inf and the phase 1).
__device__ __forceinline__ void share_polar(float2 prod, float n2, float& lm, float2& ph) {
    constexpr float kHalfLn2 = 0.34657359027997264f;
    lm = kHalfLn2 * __builtin_amdgcn_logf(n2);
    ph = n2 > 0.f ? cscale(prod, __builtin_amdgcn_rsqf(n2)) : make_float2(1.f, 0.f);
}

// One lane's share of the factor product of an anti-aligned bond (i, j).  With Delta_k = -2 s_i D_k,
// D = W_i - W_j, s_k = sign Re theta_k and w_k = exp(-2 s_k theta_k) (|w_k| <= 1),
//   cosh(theta_k + Delta_k) / cosh theta_k = [exp(s_k Delta_k) + w_k exp(-s_k Delta_k)] / (1 + w_k),
// whose numerator has no cancellation when |Delta| is large (the form cosh Delta + tanh theta sinh Delta
// subtracts two numbers of size exp|Delta| when Re theta and Re Delta have opposite signs).  The bond's
// table row holds (exp 2D, exp -2D); exp(s_k Delta_k) is exp 2D when s_k = -s_i.  The denominators are
// the same for every bond of the sample: qinv = prod 1/(1 + w_k) over this lane's units (each factor in
// [0.58, 1.72] off the zeros of cosh), multiplied into the lane's share so that its logarithm stays the
// logarithm of the lane's part of the ratio; units near a zero of cosh enter a per-sample constant
// instead (bond_term).  nm[e]: the lanes whose unit e has s_k < 0; si_neg: the first site's spin is -1.
template <int E>
__device__ __forceinline__ float2 bond_share(const float4 (&tq)[E], const float2 (&tw)[E], const uint64_t (&nm)[E],
                                             bool si_neg, float2 qinv) {
    const uint64_t flip = si_neg ? ~0ull : 0ull;
    float2 prod = make_float2(1.f, 0.f);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        // exp(s_k Delta_k) is exp 2D when s_k = -s_i
        const bool sel = __builtin_amdgcn_inverse_ballot_w64(nm[e] ^ flip);
        const float2 X = sel ? make_float2(tq[e].x, tq[e].y) : make_float2(tq[e].z, tq[e].w);
        const float2 Y = sel ? make_float2(tq[e].z, tq[e].w) : make_float2(tq[e].x, tq[e].y);
        const float2 num = make_float2(fmaf(tw[e].x, Y.x, fmaf(-tw[e].y, Y.y, X.x)),
                                       fmaf(tw[e].x, Y.y, fmaf(tw[e].y, Y.x, X.y)));
        prod = e == 0 ? num : cmul(prod, num);
    }
    return cmul(prod, qinv);
}

// The bond's row of the table for this lane's hidden units (padding lanes give the factor 1): every load is
// issued, lanes past M re-reading the row's last entry.  E = ceil(M / 64), so only the last group holds such lanes.
template <int E>
__device__ __forceinline__ void bond_row(const Geometry& g, int bnd, int lane, float4 (&tq)[E]) {
    const float4* tab = g.bond_tab + (long)bnd * g.M;
#pragma unroll
    for (int e = 0; e < E; ++e) tq[e] = tab[e < E - 1 ? e * kWave + lane : min(e * kWave + lane, g.M - 1)];
    if ((E - 1) * kWave + lane >= g.M) tq[E - 1] = make_float4(1.f, 0.f, 1.f, 0.f);
}

// The exchange term of bond (i, j) for the sample with spin s_i = si, given the whole factor product
// as (log |p|, phase): J/2 d1 psi(s^ij)/psi(s) with psi(s^ij)/psi(s) = exp(lm + Re da) phase
// exp(i Im da), da = -2 s_i (a_i - a_j) + cq (cq = -sum log(1 + w_k) over the units next to a zero of
// cosh, whose denominators are kept out of the shares), and d1 the diagonal factor of t_0 after the swap.
__device__ __forceinline__ float2 bond_term(const LocalArgs& A, const RbmView& pe, int i, int j, float si, float lm,
                                            float2 ph, float2 d0, float2 cq, bool with_fq, float inv_sqrt_n) {
    const Geometry& g = A.g;
    const float2 da = cadd(cscale(csub(pe.a[i], pe.a[j]), -2.f * si), cq);
    const float2 u = cscale(ph, rsqrtf(ph.x * ph.x + ph.y * ph.y));
    float sn, cs;
    sincosf(da.y, &sn, &cs);
    const float2 rho = cscale(cmul(u, make_float2(cs, sn)), expf(lm + da.x));
    float2 d1 = make_float2(1.f, 0.f);
    if (with_fq) {
        if (A.local_op) {
            // s_0 / 2 after the swap of sites i and j (s_j = -s_i)
            d1 = make_float2(i == 0 ? -0.5f * si : (j == 0 ? 0.5f * si : d0.x), 0.f);
        } else {
            // f_q(s^{ij}) = f_q(s) - N^{-1/2} s_i (e^{-iq.r_i} - e^{-iq.r_j})
            const float2 pd = csub(site_phase(i, g.kind, g.Lx, A.q0, A.q1), site_phase(j, g.kind, g.Lx, A.q0, A.q1));
            d1 = csub(d0, cscale(pd, inv_sqrt_n * si));
        }
    }
    return cscale(cmul(d1, rho), 0.5f * (float)g.J);
}

// This lane's share of sum_k [log cosh theta_k - log cosh phi_k] over its hidden units, theta and phi
// rows of two RBMs (parameters vt, vp) at sample s (spins srow): log cosh z = s z + log((1 + w)/2),
// w = exp(-2 s z), with the linear parts added and the factors of modulus <= 1 multiplied, so that one
// complex log serves E units (the M log 2 of log 2 cosh cancel between the two RBMs); units near a zero
// of cosh are re-evaluated in double and enter the linear part.
template <int E>
__device__ __forceinline__ float2 lc_diff(const float2* __restrict__ th, const float2* __restrict__ ph, long s, int M,
                                          int lane, const RbmView& vt, const RbmView& vp,
                                          const int8_t* __restrict__ srow, int N) {
    float2 lin = make_float2(0.f, 0.f), pt = make_float2(1.f, 0.f), pp = make_float2(1.f, 0.f);
    uint32_t poles = 0;   // bit 2 e + h
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = e * kWave + lane;
        if (k >= M) continue;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float2 z = h == 0 ? th[s * M + k] : ph[s * M + k];
            if (near_pole(z)) poles |= 1u << (2 * e + h);
            else if (h == 0) cosh_factor(z, 1.f, lin, pt);
            else cosh_factor(z, -1.f, lin, pp);
        }
    }
    while (poles) {
        const int bit = __ffs(poles) - 1;
        poles &= poles - 1;
        const int h = bit & 1, k = (bit >> 1) * kWave + lane;
        const RbmView& v = h == 0 ? vt : vp;
        float2 lcr, thr;
        pole_eval(theta_double(srow, N, M, k, v.b, v.W), lcr, thr);
        lin = h == 0 ? cadd(lin, lcr) : csub(lin, lcr);
    }
    // log pt - log pp = log|pt|/|pp| + i arg(pt conj(pp))
    const float2 q = make_float2(pt.x * pp.x + pt.y * pp.y, pt.y * pp.x - pt.x * pp.y);
    const float nt = pt.x * pt.x + pt.y * pt.y, np = pp.x * pp.x + pp.y * pp.y;
    return make_float2(lin.x + 0.5f * (logf(nt) - logf(np)), lin.y + atan2f(q.y, q.x));
}

// One sample of a wave: log psi, tanh theta, O of fit; for the RBM whose Hamiltonian action is taken
// the bond-factor data of bond_share (w_k of this lane's units, their signs neg, the lane's product qinv of
// the denominators and the constant cq of those next to a zero of cosh), the diagonal factor d0 of t_0 and
// the anti-aligned bonds (mask words, count).
template <int E>
__device__ __forceinline__ void local_sample(const LocalArgs& A, const float2* __restrict__ th1g,
                                             const float2* __restrict__ thng, int lane, long s,
                                             bool want_local, bool with_fq, int n_words, float2 (&tw)[E],
                                             uint64_t (&nm)[E], float2& qinv, float2& cq, float2& d0, int& n_anti,
                                             uint64_t* mask, uint64_t* sneg) {
    const Geometry& g = A.g;
    const int N = g.N, M = g.M;
    d0 = make_float2(1.f, 0.f);
    n_anti = 0;
    uint32_t neg = 0u;
    qinv = make_float2(1.f, 0.f);
    cq = make_float2(0.f, 0.f);
#pragma unroll
    for (int e = 0; e < E; ++e) { tw[e] = make_float2(0.f, 0.f); nm[e] = 0ull; }
    WaveSpins sp;
    sp.load(A.samples + s * N, N, lane);
    float2 t1[E], T1[E];
    float2 lc1 = make_float2(0.f, 0.f);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = e * kWave + lane;
        t1[e] = (k < M) ? th1g[s * M + k] : make_float2(0.f, 0.f);
    }
    // tanh theta of fit, and log psi of fit when asked for; units near a zero of cosh re-evaluated in double
    const int8_t* srow = A.samples + s * N;
    const bool want_t = A.tanh_out || A.O_out, want_1 = want_t || A.logpsi_out;
    uint32_t poles = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = e * kWave + lane;
        const bool p = want_1 && k < M && near_pole(t1[e]);
        poles |= p ? 1u << e : 0u;
        T1[e] = (want_t && k < M && !p) ? ctanhf(t1[e]) : make_float2(0.f, 0.f);
        if (A.logpsi_out && k < M && !p) lc1 = cadd(lc1, log2cosh(t1[e]));
    }
    while (poles) {
        const int e = __ffs(poles) - 1;
        poles &= poles - 1;
        float2 lcr, thr;
        pole_eval(theta_double(srow, N, M, e * kWave + lane, A.fit.b, A.fit.W), lcr, thr);
        lc1 = cadd(lc1, make_float2(lcr.x + 0.69314718055994531f, lcr.y));
#pragma unroll
        for (int ee = 0; ee < E; ++ee)
            if (ee == e) T1[ee] = thr;
    }
    if (A.logpsi_out) {
        const float2 lp = wave_sum(cadd(lc1, a_dot_sigma(A.fit.a, sp, lane, N)));
        if (lane == 0) A.logpsi_out[s] = lp;
    }
    if (A.tanh_out) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = e * kWave + lane;
            if (k < M) A.tanh_out[s * M + k] = T1[e];
        }
    }
    if (A.O_out) {
        float2* row = A.O_out + s * (long)g.P;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int site = c * kWave + lane;
            if (site < N) row[site] = make_float2((float)sp.s[c], 0.f);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = e * kWave + lane;
            if (k < M) row[N + k] = T1[e];
        }
        for (int i = 0; i < N; ++i) {
            const float si = (float)sp.get(i);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int k = e * kWave + lane;
                if (k < M) row[N + M + (long)i * M + k] = cscale(T1[e], si);
            }
        }
    }
    if (!want_local) return;
    // bond-factor data of psi_n (Chebyshev mode) or fit (energy mode): w_k = exp(-2 s_k theta_k) with
    // s_k = sign Re theta_k, qinv = 1 / prod (1 + w_k) over this lane's units, and for the units near a zero
    // of cosh cq = -sum log(1 + w_k) (wave total) with log(1 + w_k) = log 2 - s_k theta_k + log cosh theta_k,
    // theta_k in double
    {
        const float2* thp = A.cheb_mode ? thng : th1g;
        const RbmView& vp = A.cheb_mode ? A.psn : A.fit;
        uint32_t pw = 0;
        float2 q1 = make_float2(1.f, 0.f), cl = make_float2(0.f, 0.f);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = e * kWave + lane;
            if (k >= M) continue;
            const float2 z = thp[s * M + k];
            const float sg = z.x >= 0.f ? 1.f : -1.f;
            neg |= z.x >= 0.f ? 0u : 1u << e;
            const float ex = expf(-2.f * fabsf(z.x));
            const float2 cs = cos_sin(2.f * sg * z.y);
            tw[e] = make_float2(ex * cs.x, -ex * cs.y);
            if (near_pole(z)) pw |= 1u << e;
            else q1 = cmul(q1, make_float2(1.f + tw[e].x, tw[e].y));   // |1 + w| in [0.58, 2] off the band
        }
#pragma unroll
        for (int e = 0; e < E; ++e) nm[e] = __ballot((neg >> e) & 1u);
        const bool node = __ballot(pw != 0u) != 0ull;
        if (lane == 0) g.node_flag[s] = node ? 1 : 0;
        while (pw) {
            const int e = __ffs(pw) - 1;
            pw &= pw - 1;
            const double2 td = theta_double(srow, N, M, e * kWave + lane, vp.b, vp.W);
            float2 lcr, thr;
            pole_eval(td, lcr, thr);
            const float sg = ((neg >> e) & 1u) ? -1.f : 1.f;
            cl = cadd(cl, make_float2(lcr.x + 0.69314718055994531f - sg * (float)td.x, lcr.y - sg * (float)td.y));
        }
        qinv = cdiv(make_float2(1.f, 0.f), q1);
        cq = wave_sum(make_float2(-cl.x, -cl.y));
        cq = make_float2(uniform(cq.x), uniform(cq.y));   // wave-uniform: scalar registers
    }
    // diagonal factor of t_0: f_q (momentum q) or, with local_op, the local S^z_0 = s_0 / 2
    if (with_fq) d0 = A.local_op ? make_float2(0.5f * (float)sp.get(0), 0.f) : fq_wave(sp, lane, g, A.q0, A.q1);
    // anti-aligned bonds of the sample, and the spin of their first site
    for (int c = 0; c < n_words; ++c) {
        const int bnd = c * kWave + lane;
        bool anti = false, down = false;
        if (bnd < g.n_bonds) {
            const int2 ij = g.bonds[bnd];
            anti = srow[ij.x] != srow[ij.y];
            down = srow[ij.x] < 0;
        }
        const uint64_t m = __ballot(anti), d = __ballot(down);
        if (lane == 0) { mask[c] = m; sneg[c] = d; }
        n_anti += __popcll(m);
    }
}

// The exchange part of E_loc, sum over anti-aligned bonds of (J/2) d1 psi(s^ij)/psi(s), in double, for a
// sample at which psi (the RBM whose Hamiltonian action is taken) is next to a node (a unit next to a zero
// of cosh): there psi(s) ~ 0 while (H psi)(s) is of the size of E psi(s), so the bond terms are large and
// cancel, which binary32 factors cannot resolve.  theta, w = exp(-2 s theta) (s = sign Re theta), the unit factors
// [exp(s Delta) + w exp(-s Delta)] / (1 + w) of bond_share, a_i - a_j and f_q are taken in double, 1 + w through
// log cosh theta so that it holds next to a zero; the numerators of a lane are multiplied and their logarithm taken
// once per bond (a logarithm per unit took three times as long).  Every n_parts-th bond from the
// part-th on.  Used by k_local_nodes only, so that the main kernels keep their registers.
template <int E>
__device__ __forceinline__ double2 exchange_double(const LocalArgs& A, const RbmView& pe, long s, int lane,
                                                const uint64_t* mask, int n_words, bool with_fq, int part,
                                                int n_parts) {
    const Geometry& g = A.g;
    const int N = g.N, M = g.M;
    const int8_t* srow = A.samples + s * N;
    double2 w[E];
    double sg[E];
    double2 lq = make_double2(0.0, 0.0);   // -sum log(1 + w), log(1 + w) = log 2 - s theta + log cosh theta
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = e * kWave + lane;
        w[e] = make_double2(0.0, 0.0);
        sg[e] = 1.0;
        if (k >= M) continue;
        const double2 th = theta_double(srow, N, M, k, pe.b, pe.W);
        sg[e] = th.x >= 0.0 ? 1.0 : -1.0;
        const double ex = exp(-2.0 * fabs(th.x));
        double sn, cs;
        sincos(2.0 * sg[e] * th.y, &sn, &cs);
        w[e] = make_double2(ex * cs, -ex * sn);
        const double2 lc = log_cosh_double(th);
        lq.x -= lc.x + 0.6931471805599453 - fabs(th.x);
        lq.y -= lc.y - sg[e] * th.y;
    }
    const double inv_sqrt_n = 1.0 / sqrt((double)N);
    auto phase = [&](int r) {
        const int x = g.kind == 0 ? r : r % g.Lx, y = g.kind == 0 ? 0 : r / g.Lx;
        double sn, cs;
        sincos(A.q0 * x + A.q1 * y, &sn, &cs);
        return make_double2(cs, -sn);
    };
    double2 fq = make_double2(0.0, 0.0);
    if (with_fq && !A.local_op) {
        for (int r = lane; r < N; r += kWave) {
            const double2 p = phase(r);
            fq.x += 0.5 * srow[r] * p.x;
            fq.y += 0.5 * srow[r] * p.y;
        }
        fq = wave_sum(fq);
        fq = make_double2(fq.x * inv_sqrt_n, fq.y * inv_sqrt_n);
    }
    double2 acc = make_double2(0.0, 0.0);
    int turn = 0;
    for (int c = 0; c < n_words; ++c) {
        uint64_t m = uniform64(mask[c]);
        while (m) {
            const int bnd = c * kWave + __builtin_ctzll(m);
            m &= m - 1ull;
            const bool mine = turn == part;
            turn = turn + 1 == n_parts ? 0 : turn + 1;
            if (!mine) continue;
            const int2 ij = g.bonds[bnd];
            const double si = (double)srow[ij.x];
            double2 p = make_double2(1.0, 0.0);
            double up = 0.0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int k = e * kWave + lane;
                if (k >= M) continue;
                const float2 wi = pe.W[(long)ij.x * M + k], wj = pe.W[(long)ij.y * M + k];
                const double m2s = -2.0 * si * sg[e];                 // s Delta = m2s (W_i - W_j)
                const double dx = m2s * ((double)wi.x - (double)wj.x), dy = m2s * ((double)wi.y - (double)wj.y);
                const double t = exp(-2.0 * fabs(dx));                 // exp(|dx|) is taken out of both terms
                const double ep = dx < 0.0 ? t : 1.0, em = dx < 0.0 ? 1.0 : t;
                double sn, cs;
                sincos(dy, &sn, &cs);
                const double2 y = zmul(w[e], make_double2(em * cs, -em * sn));
                p = zmul(p, make_double2(ep * cs + y.x, ep * sn + y.y));
                up += fabs(dx);
            }
            double2 d = make_double2(0.5 * log(p.x * p.x + p.y * p.y) + lq.x + up, atan2(p.y, p.x) + lq.y);
            d = wave_sum(d);
            const float2 ai = pe.a[ij.x], aj = pe.a[ij.y];
            d.x -= 2.0 * si * ((double)ai.x - (double)aj.x);
            d.y -= 2.0 * si * ((double)ai.y - (double)aj.y);
            const double mag = exp(d.x);
            double sn, cs;
            sincos(d.y, &sn, &cs);
            double2 t = make_double2(0.5 * g.J * mag * cs, 0.5 * g.J * mag * sn);
            if (with_fq) {
                double2 d1;
                if (A.local_op) {
                    d1 = make_double2(ij.x == 0 ? -0.5 * si : (ij.y == 0 ? 0.5 * si : 0.5 * srow[0]), 0.0);
                } else {
                    const double2 pi_ = phase(ij.x), pj = phase(ij.y);
                    d1 = make_double2(fq.x - inv_sqrt_n * si * (pi_.x - pj.x), fq.y - inv_sqrt_n * si * (pi_.y - pj.y));
                }
                t = zmul(d1, t);
            }
            acc = zadd(acc, t);
        }
    }
    return acc;
}

// One sample's local energy (J/4 s_i s_j over all bonds plus the exchange part exch) and, in Chebyshev mode,
// R = phi / psi_{n+1}.
template <int E>
__device__ __forceinline__ void local_finish(const LocalArgs& A, const float2* __restrict__ th1g,
                                             const float2* __restrict__ thng, const float2* __restrict__ thmg,
                                             int lane, long s, float2 exch, float2 d0, int n_anti) {
    const Geometry& g = A.g;
    const int N = g.N, M = g.M;
    const float J = (float)g.J;
    const float2 eloc = cadd(exch, cscale(d0, 0.25f * J * (float)(g.n_bonds - 2 * n_anti)));
    if (A.eloc_out && lane == 0) A.eloc_out[s] = eloc;
    if (!A.cheb_mode || !A.R_out) return;
    WaveSpins sp;
    sp.load(A.samples + s * N, N, lane);
    const float2 asig1 = a_dot_sigma(A.fit.a, sp, lane, N);
    const float2 ht = cscale(csub(eloc, cmul(make_float2((float)A.E_c, 0.f), d0)), (float)(1.0 / A.W_scale));
    const int8_t* srow = A.samples + s * N;
    float2 dn = cadd(csub(a_dot_sigma(A.psn.a, sp, lane, N), asig1),
                     lc_diff<E>(thng, th1g, s, M, lane, A.psn, A.fit, srow, N));
    dn = wave_sum(dn);
    // beta enters through its logarithm, added to the log-amplitude difference before the exponential, so
    // that neither a small beta nor a large ratio of unnormalised states leaves the binary32 range on its own
    float2 R;
    if (A.order == 0) {
        R = cmul(ht, cexpf(cadd(dn, A.lbeta_n)));
    } else {
        float2 dm = cadd(csub(a_dot_sigma(A.psm.a, sp, lane, N), asig1),
                         lc_diff<E>(thmg, th1g, s, M, lane, A.psm, A.fit, srow, N));
        dm = wave_sum(dm);
        const float2 fm = (A.order != 1) ? make_float2(1.f, 0.f)
                        : A.local_op ? make_float2(0.5f * (float)sp.get(0), 0.f) : fq_wave(sp, lane, g, A.q0, A.q1);
        R = csub(cscale(cmul(ht, cexpf(cadd(dn, A.lbeta_n))), 2.f), cmul(fm, cexpf(cadd(dm, A.lbeta_nm1))));
    }
    if (lane == 0) A.R_out[s] = R;
}

// One sample per wave.  Its anti-aligned bonds are taken in batches of 8 with the shares kept in registers, (log |p|,
// p/|p|) each, and a reduce-scatter that leaves a bond to 8 lanes.  Bound by VALU issue.  The bonds come from the mask
// words by scalar instructions, the masks that select a bond's factors sit in scalar registers, and the rows of several
// bonds are in flight together, loaded without branches.  Four samples to a wave that read a bond's row once for all of
// them, as wide states (M > 192) had it, kept too few waves in flight for the table reads it saved: 65,536 samples,
// 10 x 10, M = 400: 3.71 to 2.65 ms; 8,192 samples, 16 x 16, M = 512: 1.28 to 0.74 ms.  Occupancy counts for more than rows in
// flight or a few spilled registers: two bonds in flight at six waves per SIMD (M <= 128) or four (M > 192) against
// four bonds at four and two: 704 against 838 us (147,456 images on 6 x 6, M = 72), 2.65 against 3.68 ms.
template <int E>
__global__ __launch_bounds__(256, E <= 2 ? 6 : E == 3 ? 5 : 4) void k_local(LocalArgs A, const float2* __restrict__ th1g,
                                                   const float2* __restrict__ thng, const float2* __restrict__ thmg) {
    __shared__ uint64_t s_mask[4][kMaxBonds / 64], s_neg[4][kMaxBonds / 64];
    __shared__ short s_anti[4][kMaxBonds];
    const int lane = threadIdx.x & 63, wv = uniform((int)(threadIdx.x >> 6));
    const long s = (long)blockIdx.x * 4 + wv;
    if (s >= A.n_samples) return;
    const Geometry& g = A.g;
    const bool want_local = A.eloc_out || A.R_out;
    const bool with_fq = A.cheb_mode && A.order == 0;
    const RbmView& pe = A.cheb_mode ? A.psn : A.fit;
    const int n_words = (g.n_bonds + 63) / 64;
    float2 TW[E];
    uint64_t NM[E];
    float2 qinv, cq;
    float2 d0;
    int n_anti;
    local_sample<E>(A, th1g, thng, lane, s, want_local, with_fq, n_words, TW, NM, qinv, cq, d0, n_anti,
                    s_mask[wv], s_neg[wv]);
    if (!want_local) return;
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // the anti-aligned bonds in bond order, for the lanes that finish them
    short* lst = s_anti[wv];
    int base = 0;
    for (int c = 0; c < n_words; ++c) {
        const uint64_t m = s_mask[wv][c];
        if ((m >> lane) & 1ull) lst[base + __popcll(m & ((1ull << lane) - 1ull))] = (short)(c * kWave + lane);
        base += __popcll(m);
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    const float inv_sqrt_n = rsqrtf((float)g.N);
    const int8_t* srow = A.samples + s * g.N;
    float2 acc = make_float2(0.f, 0.f);
    constexpr int NB = 2;   // bonds whose rows are in flight together
    int c = 0;
    uint64_t m = uniform64(s_mask[wv][0]), sg = uniform64(s_neg[wv][0]);
    for (int b0 = 0; b0 < n_anti; b0 += 8) {
        const int cnt = n_anti - b0 < 8 ? n_anti - b0 : 8;
        float lm[8];
        float2 ph[8];
#pragma unroll
        for (int h = 0; h < 8; h += NB) {
            float4 tq[NB][E];
            bool down[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                int bit = 0;
                if (h + b < cnt) {
                    while (!m) {
                        ++c;
                        m = uniform64(s_mask[wv][c]);
                        sg = uniform64(s_neg[wv][c]);
                    }
                    bit = (int)__builtin_ctzll(m);
                    m &= m - 1ull;
                }
                down[b] = (sg >> bit) & 1ull;
                bond_row<E>(g, c * kWave + bit, lane, tq[b]);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                lm[h + b] = 0.f;
                ph[h + b] = make_float2(1.f, 0.f);
                if (h + b < cnt) {
                    const float2 prod = bond_share<E>(tq[b], TW, NM, down[b], qinv);
                    share_polar(prod, prod.x * prod.x + prod.y * prod.y, lm[h + b], ph[h + b]);
                }
            }
        }
        reduce_scatter8(lm, ph, lane);
        const int bb = b0 + (lane >> 3);
        if (bb < n_anti) {
            const int2 ij = g.bonds[lst[bb]];
            const float2 t = bond_term(A, pe, ij.x, ij.y, (float)srow[ij.x], lm[0], ph[0], d0, cq, with_fq, inv_sqrt_n);
            if ((lane & 7) == 0) acc = cadd(acc, t);
        }
    }
    local_finish<E>(A, th1g, thng, thmg, lane, s, wave_sum(acc), d0, n_anti);
}

// Samples at which the local-energy RBM is next to a node (flagged by k_local): E_loc with
// the exchange sum in double (exchange_double) and, in Chebyshev mode, R, overwriting the binary32 values
// of the main kernel.  A workgroup takes kNodeSpan samples and gives each flagged one to all its waves, every
// kNodeWaves-th anti-aligned bond to a wave: flagged samples are few (some tens of 65,536 at 10 x 10, M = 400), and
// one wave per sample left the launch waiting on the longest chain of double logarithms (1.2 ms, now 0.47 ms).
constexpr int kNodeWaves = 8, kNodeSpan = 16;
template <int E>
__global__ __launch_bounds__(64 * kNodeWaves) void k_local_nodes(LocalArgs A, const float2* __restrict__ th1g,
                                                                 const float2* __restrict__ thng,
                                                                 const float2* __restrict__ thmg) {
    __shared__ uint64_t s_mask[kMaxBonds / 64];
    __shared__ double2 s_part[kNodeWaves];
    const int lane = threadIdx.x & 63, wv = uniform((int)(threadIdx.x >> 6));
    const Geometry& g = A.g;
    const long s0 = (long)blockIdx.x * kNodeSpan;
    const uint64_t flagged = __ballot(lane < kNodeSpan && s0 + lane < A.n_samples && g.node_flag[s0 + lane] != 0);
    const int n_words = (g.n_bonds + 63) / 64;
    const bool with_fq = A.cheb_mode && A.order == 0;
    for (uint64_t todo = flagged; todo; todo &= todo - 1ull) {
        const long s = s0 + __builtin_ctzll(todo);
        const int8_t* srow = A.samples + s * g.N;
        int n_anti = 0;
        __syncthreads();
        for (int c = 0; c < n_words; ++c) {
            const int bnd = c * kWave + lane;
            bool anti = false;
            if (bnd < g.n_bonds) {
                const int2 ij = g.bonds[bnd];
                anti = srow[ij.x] != srow[ij.y];
            }
            const uint64_t m = __ballot(anti);
            if (threadIdx.x == 0) s_mask[c] = m;
            n_anti += __popcll(m);
        }
        __syncthreads();
        const double2 x = exchange_double<E>(A, A.cheb_mode ? A.psn : A.fit, s, lane, s_mask, n_words, with_fq, wv,
                                             kNodeWaves);
        if (lane == 0) s_part[wv] = x;
        __syncthreads();
        if (wv != 0) continue;
        double2 t = s_part[0];
        for (int k = 1; k < kNodeWaves; ++k) t = zadd(t, s_part[k]);
        float2 d0 = make_float2(1.f, 0.f);
        if (with_fq) {
            WaveSpins sp;
            sp.load(srow, g.N, lane);
            d0 = A.local_op ? make_float2(0.5f * (float)sp.get(0), 0.f) : fq_wave(sp, lane, g, A.q0, A.q1);
        }
        local_finish<E>(A, th1g, thng, thmg, lane, s, make_float2((float)t.x, (float)t.y), d0, n_anti);
    }
}

// (exp 2D, exp -2D) per bond and hidden unit, D = W_i - W_j, from the binary32 weights in double
__global__ __launch_bounds__(256) void k_bond_table(const int2* __restrict__ bonds, int nb, int M,
                                                    const float2* __restrict__ W, float4* __restrict__ tab) {
    const long idx = (long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long)nb * M) return;
    const int b = (int)(idx / M), k = (int)(idx % M);
    const int2 ij = bonds[b];
    const float2 wi = W[(long)ij.x * M + k], wj = W[(long)ij.y * M + k];
    const double x = 2.0 * ((double)wi.x - (double)wj.x), y = 2.0 * ((double)wi.y - (double)wj.y);
    const double ep = exp(x), em = exp(-x);
    double sn, cs;
    sincos(y, &sn, &cs);
    tab[idx] = make_float4((float)(ep * cs), (float)(ep * sn), (float)(em * cs), (float)(-em * sn));
}

hipError_t launch_local_core(const LocalArgs& A, const float2* th1, const float2* thn, const float2* thm,
                             hipStream_t stream) {
    if (A.eloc_out || A.R_out) {
        // the bond factors of the RBM whose Hamiltonian action is taken
        const float2* W = A.cheb_mode ? A.psn.W : A.fit.W;
        const long cnt = (long)A.g.n_bonds * A.g.M;
        hipLaunchKernelGGL(k_bond_table, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, stream, A.g.bonds,
                           A.g.n_bonds, A.g.M, W, A.g.bond_tab);
    }
    const int E = (A.g.M + kWave - 1) / kWave;
    const dim3 block(256);
    const dim3 grid1((unsigned)((A.n_samples + 3) / 4));
    const dim3 gridn((unsigned)((A.n_samples + kNodeSpan - 1) / kNodeSpan));
    switch (E) {
#define CRBM_LOCAL(e) case e: hipLaunchKernelGGL(k_local<e>, grid1, block, 0, stream, A, th1, thn, thm); break;
        CRBM_LOCAL(1) CRBM_LOCAL(2) CRBM_LOCAL(3) CRBM_LOCAL(4) CRBM_LOCAL(5) CRBM_LOCAL(6) CRBM_LOCAL(7) CRBM_LOCAL(8)
#undef CRBM_LOCAL
        default: return hipErrorInvalidValue;
    }
    if (A.eloc_out || A.R_out) {
        switch (E) {
#define CRBM_NODES(e) \
    case e: hipLaunchKernelGGL(k_local_nodes<e>, gridn, dim3(64 * kNodeWaves), 0, stream, A, th1, thn, thm); break;
            CRBM_NODES(1) CRBM_NODES(2) CRBM_NODES(3) CRBM_NODES(4) CRBM_NODES(5) CRBM_NODES(6) CRBM_NODES(7)
            CRBM_NODES(8)
#undef CRBM_NODES
            default: return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

// ------------------------------------------------------------------ moments
// f[q][s] = f_q(s) (double) for a chunk of up to 8 momenta: one thread per sample, the sites' phases formed once
// per block in LDS (a sine and a cosine in double per sample and site took 86 us for 131,072 samples of 100
// sites, now 6 us)
struct QChunk { double q[8][2]; };

__global__ __launch_bounds__(256) void k_fq(Geometry g, const uint32_t* __restrict__ bits, int nw, long n_s, QChunk qc,
                                            int n_q, double2* __restrict__ f) {
    __shared__ double2 ph[256];
    const long s = (long)blockIdx.x * 256 + threadIdx.x;
    const double inv = 1.0 / sqrt((double)g.N);
    for (int iq = 0; iq < n_q; ++iq) {
        __syncthreads();
        if (threadIdx.x < g.N) {
            const int site = threadIdx.x;
            const int x = g.kind == 0 ? site : site % g.Lx;
            const int y = g.kind == 0 ? 0 : site / g.Lx;
            double sn, cs;
            sincos(qc.q[iq][0] * x + qc.q[iq][1] * y, &sn, &cs);
            ph[site] = make_double2(0.5 * cs, 0.5 * sn);
        }
        __syncthreads();
        if (s >= n_s) continue;
        double2 acc = make_double2(0.0, 0.0);
        for (int w = 0; w < nw; ++w) {
            const uint32_t word = bits[s * nw + w];
            const int cnt = g.N - 32 * w < 32 ? g.N - 32 * w : 32;
#pragma unroll 8
            for (int b = 0; b < cnt; ++b) {
                const double sg = (word >> b) & 1u ? -1.0 : 1.0;
                acc.x += sg * ph[32 * w + b].x;
                acc.y -= sg * ph[32 * w + b].y;
            }
        }
        f[(long)iq * n_s + s] = make_double2(acc.x * inv, acc.y * inv);
    }
}

// partial[blk][entry0 + iq*nn] = sum over the block's samples of w conj(f_q) B  (B = f_q when b_is_f)
__global__ __launch_bounds__(256) void k_moment_accum(const double2* __restrict__ f, const double2* __restrict__ B,
                                                      int b_is_f, const double* __restrict__ w, long n_s, int n_q,
                                                      int nn, int entry0, int total, long chunk,
                                                      double2* __restrict__ partial) {
    __shared__ double shx[4], shy[4];
    const long s_begin = (long)blockIdx.x * chunk;
    const long s_end = min(n_s, s_begin + chunk);
    const double wdef = 1.0 / (double)n_s;
    for (int iq = 0; iq < n_q; ++iq) {
        double ax = 0.0, ay = 0.0;
        for (long s = s_begin + threadIdx.x; s < s_end; s += blockDim.x) {
            const double ws = w ? w[s] : wdef;
            const double2 fs = f[(long)iq * n_s + s];
            const double2 t = zconjmul(fs, b_is_f ? fs : B[s]);
            ax += ws * t.x;
            ay += ws * t.y;
        }
        ax = wave_sum(ax);
        ay = wave_sum(ay);
        if ((threadIdx.x & 63) == 0) { shx[threadIdx.x >> 6] = ax; shy[threadIdx.x >> 6] = ay; }
        __syncthreads();
        if (threadIdx.x == 0)
            partial[(long)blockIdx.x * total + entry0 + iq * nn] =
                make_double2(shx[0] + shx[1] + shx[2] + shx[3], shy[0] + shy[1] + shy[2] + shy[3]);
        __syncthreads();
    }
}

// one wave per entry, its lanes over the blocks (one thread adding 256 of them in turn took 61 us, now 5 us)
__global__ __launch_bounds__(64) void k_moment_final(const double2* __restrict__ partial, int n_blocks, int total,
                                                     double2* __restrict__ mu) {
    double2 acc = make_double2(0.0, 0.0);
    for (int b = threadIdx.x; b < n_blocks; b += kWave) acc = zadd(acc, partial[(long)b * total + blockIdx.x]);
    acc = wave_sum(acc);
    if (threadIdx.x == 0) mu[blockIdx.x] = acc;
}

hipError_t launch_fq_chunk(const Geometry& g, const uint32_t* bits, long n_s, const double* q_host, int n_q,
                           double2* f, hipStream_t stream) {
    QChunk qc{};
    for (int k = 0; k < n_q && k < 8; ++k) { qc.q[k][0] = q_host[2 * k]; qc.q[k][1] = g.kind == 0 ? 0.0 : q_host[2 * k + 1]; }
    hipLaunchKernelGGL(k_fq, dim3((unsigned)((n_s + 255) / 256)), dim3(256), 0, stream, g, bits, spin_words(g.N), n_s, qc,
                       n_q, f);
    return hipGetLastError();
}

hipError_t launch_moment_accum(const double2* f, const double2* B, int b_is_f, const double* w, long n_s, int n_q,
                               int nn, int entry0, int total, double2* partial, int n_blocks, hipStream_t stream) {
    const long chunk = (n_s + n_blocks - 1) / n_blocks;
    hipLaunchKernelGGL(k_moment_accum, dim3(n_blocks), dim3(256), 0, stream, f, B, b_is_f, w, n_s, n_q, nn, entry0,
                       total, chunk, partial);
    return hipGetLastError();
}

hipError_t launch_moment_final(const double2* partial, int n_blocks, int total, double2* mu, hipStream_t stream) {
    hipLaunchKernelGGL(k_moment_final, dim3(total), dim3(64), 0, stream, partial, n_blocks, total, mu);
    return hipGetLastError();
}

}  // namespace crbm
