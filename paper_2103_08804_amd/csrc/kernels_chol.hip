// Dense Hermitian positive-definite solve (S + eps I) x = F in double precision
// by a Cholesky factorisation L L^H followed by two triangular solves.  Used for
// the natural-gradient system of Sec. III when P is a few thousand (the
// factorisation costs P^3/3 complex multiply-adds).
//
// Right-looking and blocked in panels of CH_NB = 64 columns, per panel k:
//   1. the diagonal block A_kk is factored in LDS by one workgroup;
//   2. the rows below solve L_ik L_kk^H = A_ik, four rows per wave (the lanes hold
//      the 64 unknowns of a row, the substitution runs along the columns);
//   3. the trailing lower triangle is updated, A_ij -= L_ik L_jk^H (i >= j), in
//      32 x 32 output tiles with both 32 x 64 panels staged in LDS.
// The triangular solves run by blocks of 64 rows, one launch per block.
// Everything is in double, in a fixed order.
#include "../../include/chebrbm.h"
#include "device.hpp"
#include "internal.hpp"

namespace crbm {

enum { SC_FLAGS_SLOT = 15 };   // must match the scalar layout of the step driver
constexpr int CH_NB = 64;      // panel width
constexpr int CH_T = 32;       // trailing-update tile

// the value of v in lane m (m wave-uniform), through scalar registers
__device__ __forceinline__ double lane_value(double v, int m) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, m), hi = __builtin_amdgcn_readlane((int)(b >> 32), m);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

// 1 / sqrt(d), d > 0 and finite: the hardware estimate and two Newton steps (the serial chain of a column waits
// on it)
__device__ __forceinline__ double inv_sqrt(double d) {
    // scaled by a power of four into [1, 4) so that the steps neither overflow nor underflow
    const int e = (ilogb(d) >> 1) << 1;
    const double m = ldexp(d, -e);
    double y = __builtin_amdgcn_rsq(m);
    y = fma(y * fma(-m * y, y, 1.0), 0.5, y);
    y = fma(y * fma(-m * y, y, 1.0), 0.5, y);
    return ldexp(y, -(e / 2));
}

// the lower triangle of the diagonal block [b0, b0 + nb)^2 into LDS by 256 threads, all loads issued together
__device__ __forceinline__ void stage_block(long P, const double2* __restrict__ A, long b0, int nb,
                                            double2 (&D)[CH_NB][CH_NB + 1]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double2 v[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int r = w + 4 * q;
        const bool in = r < nb && lane <= r;
        v[q] = A[(b0 + (in ? r : 0)) * P + b0 + (in ? lane : 0)];
        if (!in) v[q] = make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q)
        if (w + 4 * q < nb) D[w + 4 * q][lane] = v[q];
}

__device__ __forceinline__ bool chol_failed(const double* sc) {
    return ((int)sc[SC_FLAGS_SLOT] & CRBM_FLAG_CHOLESKY_FAIL) != 0;
}

// A64 = S + eps I (lower triangle used)
__global__ __launch_bounds__(256) void k_chol_load(long P, const float2* __restrict__ S, double eps,
                                                   double2* __restrict__ A) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= P * P) return;
    const long i = idx / P, j = idx % P;
    const float2 v = S[idx];
    A[idx] = make_double2((double)v.x + (i == j ? eps : 0.0), (double)v.y);
}

// 1. L_kk of the diagonal block [k0, k0 + nb)^2, one workgroup.  The columns are factored in groups of CH_PW by
//    the first wave alone, lane = row with the group's entries of the row in registers: the pivot and the
//    multipliers reach all lanes through scalar registers, so the serial chain of a column (square root,
//    reciprocal, scaling) holds no LDS round trip and no barrier.  Then all 16 waves subtract the group from the
//    columns right of it through LDS.  Bound by that chain: 36 us per block (55 us with a barrier and an LDS
//    round trip per column).
constexpr int CH_PW = 16;
__global__ __launch_bounds__(1024) void k_chol_diagblock(long P, long k0, int nb, double2* __restrict__ A,
                                                         double* __restrict__ sc) {
    __shared__ double2 L[CH_NB][CH_NB + 1];
    __shared__ int s_fail;
    if (chol_failed(sc)) return;
    const int tid = threadIdx.x, tx = tid & 31, ty = tid >> 5, lane = tid & 63;
    if (tid == 0) s_fail = 0;
    {
        double2 v[2][2];
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int i = ty + 32 * p, j = tx + 32 * q;
                const bool in = i < nb && j <= i;
                v[p][q] = A[(k0 + (in ? i : 0)) * P + k0 + (in ? j : 0)];
                if (!in) v[p][q] = make_double2(0.0, 0.0);
            }
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q) L[ty + 32 * p][tx + 32 * q] = v[p][q];
    }
    __syncthreads();
    for (int p0 = 0; p0 < nb; p0 += CH_PW) {
        const int pw = nb - p0 < CH_PW ? nb - p0 : CH_PW;
        if (tid < 64) {
            double2 a[CH_PW];
#pragma unroll
            for (int c = 0; c < CH_PW; ++c)
                a[c] = (c < pw && lane < nb && lane >= p0 + c) ? L[lane][p0 + c] : make_double2(0.0, 0.0);
            bool fail = false;
#pragma unroll
            for (int c = 0; c < CH_PW; ++c) {
                if (c >= pw || fail) continue;
                const double d = lane_value(a[c].x, p0 + c);
                if (!(d > 0.0) || !isfinite(d)) { fail = true; continue; }
                const double inv = inv_sqrt(d);
                a[c] = lane == p0 + c ? make_double2(sqrt(d), 0.0) : make_double2(a[c].x * inv, a[c].y * inv);
#pragma unroll
                for (int l = c + 1; l < CH_PW; ++l) {   // A_il -= L_ic conj(L_lc); lanes above row l are not kept
                    const double bx = lane_value(a[c].x, p0 + l), by = lane_value(a[c].y, p0 + l);
                    a[l].x -= a[c].x * bx + a[c].y * by;
                    a[l].y -= a[c].y * bx - a[c].x * by;
                }
            }
            if (fail && lane == 0) s_fail = 1;
#pragma unroll
            for (int c = 0; c < CH_PW; ++c)
                if (c < pw && lane < nb && lane >= p0 + c) L[lane][p0 + c] = a[c];
        }
        __syncthreads();
        if (s_fail) {
            if (tid == 0) sc[SC_FLAGS_SLOT] = (double)((int)sc[SC_FLAGS_SLOT] | CRBM_FLAG_CHOLESKY_FAIL);
            return;
        }
        const int q0 = p0 + pw;
        for (int i = q0 + ty; i < nb; i += 32)
            for (int l = q0 + tx; l <= i; l += 32) {
                double2 v = L[i][l];
#pragma unroll 4
                for (int c = p0; c < q0; ++c) {
                    const double2 x = L[i][c], y = L[l][c];
                    v.x -= x.x * y.x + x.y * y.y;
                    v.y -= x.y * y.x - x.x * y.y;
                }
                L[i][l] = v;
            }
        __syncthreads();
    }
    for (int i = ty; i < nb; i += 32)
        for (int j = tx; j <= i; j += 32) A[(k0 + i) * P + k0 + j] = L[i][j];
}

// 2. rows i >= k0 + nb: x L_kk^H = a with x = L_ik, a = A_ik; lane l owns column l of the row, a wave CH_PR rows.
//    x_m = (a_m - sum_{l<m} x_l conj(L_kk[m][l])) / L_kk[m][m]: once x_l is known (step l, lane l) it is
//    read by every lane, and lanes m > l subtract its term from their own a_m, in the order l = 0, 1, ...
//    The rows of a wave share the reads of L and hide each other's chains, and the block is staged once for
//    4 CH_PR rows (21 us per panel at P = 3320, as with one row per wave, on a quarter of the workgroups).
constexpr int CH_PR = 4;
__global__ __launch_bounds__(256) void k_chol_panel(long P, long k0, int nb, double2* __restrict__ A,
                                                    const double* __restrict__ sc) {
    __shared__ double2 L[CH_NB][CH_NB + 1];
    if (chol_failed(sc)) return;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane < nb ? lane : 0;
    const long i0 = k0 + nb + ((long)blockIdx.x * 4 + (tid >> 6)) * CH_PR;
    double2 x[CH_PR];
#pragma unroll
    for (int q = 0; q < CH_PR; ++q)
        x[q] = (lane < nb && i0 + q < P) ? A[(i0 + q) * P + k0 + lane] : make_double2(0.0, 0.0);
    stage_block(P, A, k0, nb, L);
    __syncthreads();
    if (i0 >= P) return;
    const double dinv = lane < nb ? 1.0 / L[ln][ln].x : 0.0;   // lane m divides by L_mm at step m
#pragma unroll 4
    for (int m = 0; m < nb; ++m) {
        const double2 c = lane > m ? L[ln][m] : make_double2(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < CH_PR; ++q) {
            if (lane == m) x[q] = make_double2(x[q].x * dinv, x[q].y * dinv);
            const double xr = lane_value(x[q].x, m), xi = lane_value(x[q].y, m);
            x[q].x -= xr * c.x + xi * c.y;              // x_m conj(L[lane][m])
            x[q].y -= xi * c.x - xr * c.y;
        }
    }
    if (lane < nb)
#pragma unroll
        for (int q = 0; q < CH_PR; ++q)
            if (i0 + q < P) A[(i0 + q) * P + k0 + lane] = x[q];
}

// 3. trailing update of the lower triangle: A_ij -= sum_l L_il conj(L_jl), i >= j >= k1 = k0 + nb.
//    Workgroup = one 32 x 32 tile (I >= J) of the trailing matrix; thread = 2 x 2 outputs.
__global__ __launch_bounds__(256) void k_chol_update(long P, long k0, int nb, double2* __restrict__ A,
                                                     const double* __restrict__ sc) {
    __shared__ double2 Li[CH_T][CH_NB + 1], Lj[CH_T][CH_NB + 1];
    if (chol_failed(sc)) return;
    const long k1 = k0 + nb;
    // tile index -> (I, J), J <= I, over T = ceil((P - k1) / 32) tiles per side
    long rem = blockIdx.x;
    long I = 0;
    while (rem > I) { rem -= I + 1; ++I; }
    const long J = rem;
    const long i0 = k1 + I * CH_T, j0 = k1 + J * CH_T;
    const int tid = threadIdx.x;
    for (int e = tid; e < CH_T * nb; e += 256) {
        const int r = e / nb, l = e % nb;
        Li[r][l] = (i0 + r < P) ? A[(i0 + r) * P + k0 + l] : make_double2(0.0, 0.0);
        Lj[r][l] = (j0 + r < P) ? A[(j0 + r) * P + k0 + l] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int ti = (tid >> 4) * 2, tj = (tid & 15) * 2;
    double2 acc[2][2] = {};
    for (int l = 0; l < nb; ++l) {
        const double2 a0 = Li[ti][l], a1 = Li[ti + 1][l], b0 = Lj[tj][l], b1 = Lj[tj + 1][l];
        const double2 a[2] = {a0, a1}, b[2] = {b0, b1};
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                acc[p][q].x += a[p].x * b[q].x + a[p].y * b[q].y;
                acc[p][q].y += a[p].y * b[q].x - a[p].x * b[q].y;
            }
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const long i = i0 + ti + p, j = j0 + tj + q;
            if (i < P && j <= i) {
                double2* dst = A + i * P + j;
                *dst = make_double2(dst->x - acc[p][q].x, dst->y - acc[p][q].y);
            }
        }
}

// L y = F, then L^H x = y, by blocks of 64 rows, one launch per block: every workgroup stages the diagonal
// block and its first wave substitutes in it (each unknown, once known, is read by every lane and the later
// lanes subtract its term), all workgroups alike; then the workgroup applies the block's unknowns to its own
// share of the rest: forward, the rows below (a thread per 16 columns of a row, four a row); backward, the
// columns to the left (a thread per 16 rows of a column).  The right-hand side of a block and the rest are
// updated in one vector, the solved unknowns go to another (workgroups of the next launch read the former).
// 27 us per block and direction pair at P = 3320 (49 us with the substitution and the update as launches of their own).
__global__ __launch_bounds__(256) void k_trsv_init(long P, const double2* __restrict__ F, double2* __restrict__ v,
                                                   const double* __restrict__ sc) {
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < P) v[k] = chol_failed(sc) ? make_double2(0.0, 0.0) : F[k];
}

// v: right-hand side (updated past the block), x: solution; x_b in LDS at the end
template <bool BACK>
__device__ __forceinline__ void trsv_block(long P, const double2* __restrict__ A, long b0, int nb,
                                           const double2* __restrict__ v, double2 (&D)[CH_NB][CH_NB + 1],
                                           double2 (&xb)[CH_NB]) {
    const int tid = threadIdx.x, lane = tid & 63, ln = lane < nb ? lane : 0;
    stage_block(P, A, b0, nb, D);
    __syncthreads();
    if (tid < 64) {
        double2 x = lane < nb ? v[b0 + lane] : make_double2(0.0, 0.0);
        const double dinv = lane < nb ? 1.0 / D[ln][ln].x : 0.0;   // lane m divides by L_mm at step m
#pragma unroll 4
        for (int t = 0; t < nb; ++t) {
            const int m = BACK ? nb - 1 - t : t;
            const double2 c = BACK ? (lane < m ? D[m][ln] : make_double2(0.0, 0.0))
                                   : (lane > m ? D[ln][m] : make_double2(0.0, 0.0));
            if (lane == m) x = make_double2(x.x * dinv, x.y * dinv);
            const double2 xm = make_double2(lane_value(x.x, m), lane_value(x.y, m));
            const double2 p = BACK ? zconjmul(c, xm) : zmul(c, xm);
            x.x -= p.x;
            x.y -= p.y;
        }
        xb[lane] = lane < nb ? x : make_double2(0.0, 0.0);
    }
    __syncthreads();
}

__global__ __launch_bounds__(256) void k_trsv_fwd(long P, const double2* __restrict__ A, long b0, int nb,
                                                  double2* __restrict__ v, double2* __restrict__ x,
                                                  const double* __restrict__ sc) {
    __shared__ double2 D[CH_NB][CH_NB + 1];
    __shared__ double2 xb[CH_NB];
    if (chol_failed(sc)) return;
    trsv_block<false>(P, A, b0, nb, v, D, xb);
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid < nb) x[b0 + tid] = xb[tid];
    const long k = b0 + nb + (long)blockIdx.x * 64 + (tid >> 2);
    double2 t = make_double2(0.0, 0.0);
    if (k < P)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int l = (tid & 3) + 4 * q;
            if (l < nb) t = zadd(t, zmul(A[k * P + b0 + l], xb[l]));
        }
    t.x += __shfl_xor(t.x, 1); t.y += __shfl_xor(t.y, 1);
    t.x += __shfl_xor(t.x, 2); t.y += __shfl_xor(t.y, 2);
    if (k < P && (tid & 3) == 0) v[k] = zsub(v[k], t);
}

// x (the forward solution) is the right-hand side here and is updated left of the block; the solution goes to out
__global__ __launch_bounds__(256) void k_trsv_back(long P, const double2* __restrict__ A, long b0, int nb,
                                                   double2* __restrict__ v, double2* __restrict__ out,
                                                   const double* __restrict__ sc) {
    __shared__ double2 D[CH_NB][CH_NB + 1];
    __shared__ double2 xb[CH_NB], part[4][64];
    if (chol_failed(sc)) return;
    trsv_block<true>(P, A, b0, nb, v, D, xb);
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (blockIdx.x == 0 && tid < nb) out[b0 + tid] = xb[tid];
    const long j = (long)blockIdx.x * 64 + lane;
    double2 t = make_double2(0.0, 0.0);
    if (j < b0)
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int r = 16 * w + q;
            if (r < nb) t = zadd(t, zconjmul(A[(b0 + r) * P + j], xb[r]));
        }
    part[w][lane] = t;
    __syncthreads();
    if (w == 0 && j < b0) v[j] = zsub(v[j], zadd(zadd(part[0][lane], part[1][lane]), zadd(part[2][lane], part[3][lane])));
}

// after a failed factorisation the solution is 0
__global__ __launch_bounds__(256) void k_trsv_failed(long P, double2* __restrict__ x, const double* __restrict__ sc) {
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < P && chol_failed(sc)) x[k] = make_double2(0.0, 0.0);
}

// v, y: [P] scratch
hipError_t launch_cholesky_solve(long P, const float2* S, double eps, const double2* F, double2* A64, double2* x,
                                 double2* v, double2* y, double* sc, bool a64_holds_s, hipStream_t stream) {
    if (P < 1 || P > kCholMaxP) return hipErrorInvalidValue;
    // a64_holds_s: A64 already holds S + eps I in double
    if (!a64_holds_s)
        hipLaunchKernelGGL(k_chol_load, dim3((unsigned)((P * P + 255) / 256)), dim3(256), 0, stream, P, S, eps, A64);
    for (long k0 = 0; k0 < P; k0 += CH_NB) {
        const int nb = (int)(P - k0 < CH_NB ? P - k0 : CH_NB);
        hipLaunchKernelGGL(k_chol_diagblock, dim3(1), dim3(1024), 0, stream, P, k0, nb, A64, sc);
        const long rows = P - k0 - nb;
        if (rows <= 0) break;
        hipLaunchKernelGGL(k_chol_panel, dim3((unsigned)((rows + 4 * CH_PR - 1) / (4 * CH_PR))), dim3(256), 0, stream, P,
                           k0, nb, A64, sc);
        const long T = (rows + CH_T - 1) / CH_T;
        hipLaunchKernelGGL(k_chol_update, dim3((unsigned)(T * (T + 1) / 2)), dim3(256), 0, stream, P, k0, nb, A64, sc);
    }
    const dim3 gp((unsigned)((P + 255) / 256));
    hipLaunchKernelGGL(k_trsv_init, gp, dim3(256), 0, stream, P, F, v, sc);
    const long nblk = (P + CH_NB - 1) / CH_NB;
    for (long blk = 0; blk < nblk; ++blk) {
        const long b0 = blk * CH_NB;
        const int nb = (int)(P - b0 < CH_NB ? P - b0 : CH_NB);
        const long g = (P - b0 - nb + 63) / 64;
        hipLaunchKernelGGL(k_trsv_fwd, dim3((unsigned)(g > 0 ? g : 1)), dim3(256), 0, stream, P, A64, b0, nb, v, y, sc);
    }
    for (long blk = nblk - 1; blk >= 0; --blk) {
        const long b0 = blk * CH_NB;
        const int nb = (int)(P - b0 < CH_NB ? P - b0 : CH_NB);
        const long g = (b0 + 63) / 64;
        hipLaunchKernelGGL(k_trsv_back, dim3((unsigned)(g > 0 ? g : 1)), dim3(256), 0, stream, P, A64, b0, nb, y, x, sc);
    }
    hipLaunchKernelGGL(k_trsv_failed, gp, dim3(256), 0, stream, P, x, sc);
    return hipGetLastError();
}

}  // namespace crbm
