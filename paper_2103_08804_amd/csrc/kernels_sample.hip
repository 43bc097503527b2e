// Parameter initialisation, chain initialisation and the Metropolis sweep.
//
// Sampling (Sec. III): configurations s are drawn from |psi_s|^2 / <psi|psi>
// by Metropolis chains.  One wavefront owns one chain: lane l keeps the
// hidden units k = 64 e + l (e < E) of theta in registers together with the
// cached Re log(2 cosh theta_k); the spins are bytes in LDS.  A proposal
// touches rows W_i (and W_j), recomputes Re log(2 cosh theta'_k) per element,
// reduces the change over the wave and accepts on u < |psi'/psi|^2; only the
// real part of the log-amplitude is needed for the acceptance, so the
// imaginary part (and its atan2) never enters the inner loop.  theta is
// rebuilt from the spins at the start of every call.
#include <algorithm>

#include "device.hpp"
#include "internal.hpp"
#include "sweep.hpp"

namespace crbm {

// ------------------------------------------------------------------ init_rbm
__global__ void k_init_rbm(float2* __restrict__ a, float2* __restrict__ b, float2* __restrict__ W, int N, int M,
                           uint64_t seed, float stddev) {
    const long P = (long)N + M + (long)N * M;
    const long k = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= P) return;
    const u32x4 r = draw(seed, (uint32_t)k, 0ull, 2u);
    const float u1 = ((float)(r.x >> 8) + 1.0f) * (1.0f / 16777216.0f);
    const float u2 = (float)(r.y >> 8) * (1.0f / 16777216.0f);
    const float rad = stddev * sqrtf(-2.0f * logf(u1));
    float sn, cs;
    sincospif(2.0f * u2, &sn, &cs);
    const float2 v = make_float2(rad * cs, rad * sn);
    if (k < N) a[k] = v;
    else if (k < N + M) b[k - N] = v;
    else W[k - N - M] = v;
}

hipError_t launch_init_rbm(float2* a, float2* b, float2* W, int N, int M, uint64_t seed, float stddev,
                           hipStream_t stream) {
    const long P = (long)N + M + (long)N * M;
    const int threads = 256;
    const long blocks = (P + threads - 1) / threads;
    hipLaunchKernelGGL(k_init_rbm, dim3((unsigned)blocks), dim3(threads), 0, stream, a, b, W, N, M, seed, stddev);
    return hipGetLastError();
}

// ------------------------------------------------------------------ init_chains
// One thread per chain; the configuration is built in LDS (N <= 256).
__global__ __launch_bounds__(64) void k_init_chains(int8_t* __restrict__ spins, int N, int n_chains, uint64_t seed,
                                                    int zero_mag) {
    __shared__ int8_t buf[64][256];
    const int c = blockIdx.x * 64 + threadIdx.x;
    if (c >= n_chains) return;
    int8_t* s = buf[threadIdx.x];
    if (!zero_mag) {
        for (int i = 0; i < N; ++i) s[i] = (draw(seed, (uint32_t)c, (uint64_t)i, 1u).x & 1u) ? 1 : -1;
    } else {
        for (int i = 0; i < N; ++i) s[i] = (i < N / 2) ? 1 : -1;
        for (int k = N - 1; k >= 1; --k) {
            const int m = draw_index(draw(seed, (uint32_t)c, (uint64_t)k, 1u).x, k + 1);
            const int8_t t = s[k];
            s[k] = s[m];
            s[m] = t;
        }
    }
    for (int i = 0; i < N; ++i) spins[(long)c * N + i] = s[i];
}

hipError_t launch_init_chains(int8_t* spins, int N, int n_chains, uint64_t seed, int zero_mag, hipStream_t stream) {
    const int blocks = (n_chains + 63) / 64;
    hipLaunchKernelGGL(k_init_chains, dim3(blocks), dim3(64), 0, stream, spins, N, n_chains, seed, zero_mag);
    return hipGetLastError();
}

// ------------------------------------------------------------------ Metropolis sweep
// Spins of a chain as stored bytes, from its LDS row; `words`: N and the address allow four sites per store.
__device__ __forceinline__ void store_spins(const int8_t* row, int8_t* __restrict__ out, int N, int lane, bool words) {
    if (words) {
        if (4 * lane < N) reinterpret_cast<int*>(out)[lane] = reinterpret_cast<const int*>(row)[lane];
        return;
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int site = q * kWave + lane;
        if (site < N) out[site] = row[site];
    }
}

// Rows i (and j) of W: unit groups e < E - G from L2 (whole groups, through one descriptor of W), the last G from
// the workgroup's copy s_w ([N][G 64], zeros past M).
template <int E, bool PAIR, int G>
__device__ __forceinline__ void sample_rows(__amdgpu_buffer_rsrc_t W, const float2* s_w, int M, int i, int j, int lane,
                                            float2 (&wi)[E], float2 (&wj)[E]) {
    const int row = M * (int)sizeof(float2);
#pragma unroll
    for (int e = 0; e < E - G; ++e) {
        const unsigned off = (unsigned)(e * kWave + lane) * (unsigned)sizeof(float2);
        wi[e] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(W, off, i * row, 0));
        if (PAIR) wj[e] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(W, off, j * row, 0));
    }
#pragma unroll
    for (int e = E - G; e < E; ++e) {
        wi[e] = s_w[i * (G * kWave) + (e - (E - G)) * kWave + lane];
        if (PAIR) wj[e] = s_w[j * (G * kWave) + (e - (E - G)) * kWave + lane];
    }
}

// One wave per chain, up to 16 chains to a workgroup, which keeps the last G of the E unit groups of W in LDS.
// 64 proposals are drawn at once, one per lane, and their liveness is kept as two wave-uniform words, the spins at
// sites i and j of each draw: an exchange of equal spins costs nothing, an accepted move toggles the bits of the draws
// that touch its sites, and the spin bytes are brought up to date only where a sweep or a batch ends.  The rows of the
// next live proposal are fetched while the current one is evaluated, and again only when the current one, once
// accepted, changed which one is next.  Few chains: bound by one move's chain of row read, transcendentals and wave
// total; a full chip: by VALU issue (15 instructions per unit and move, three of them transcendental).
// Before, a move read its rows from L2 and waited for them, and every null move took the scalar path.
// 1,024 chains, 256 sweeps, N = 40, M = 80: 3.89 to 1.39 ms; 4,096 chains, 128 sweeps, N = 100, M = 400: 12.64 to 8.09 ms.
template <int E, bool PAIR, int G>
__global__ __launch_bounds__(1024) void k_sample(SampleArgs A) {
    extern __shared__ float2 s_w[];               // [N][G 64] of W, then a 256-byte spin row per wave, then Re a
    const int lane = threadIdx.x & 63, wv = uniform((int)(threadIdx.x >> 6)), n_waves = blockDim.x >> 6;
    const int N = A.N, M = A.M;
    const float2* __restrict__ W = A.psi.W;
    constexpr int kCols = G * kWave, k0 = (E - G) * kWave;   // columns held here, the first of them
    int8_t* const row = reinterpret_cast<int8_t*>(s_w + N * kCols) + wv * 256;
    float* const s_a = reinterpret_cast<float*>(reinterpret_cast<int8_t*>(s_w + N * kCols) + n_waves * 256);
    // Each wave copies its rows in blocks of U whose loads are in flight together: a lone wave of few chains would wait
    // for one row after the other, longer than a sweep takes (1 chain, N = 40, M = 400, one sweep: 45 us, now 21).
    // U is small enough for the sweep's own registers, and lanes past M and rows past N read what is then dropped.
    const __amdgpu_buffer_rsrc_t Wr = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float2*>(W), (short)0, N * M * (int)sizeof(float2), 0x00020000);
    constexpr int U = G <= 2 ? 8 : 24 / G;
    for (int i0 = wv; i0 < N; i0 += U * n_waves) {
        float2 v[U][G];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < G; ++e)
                v[u][e] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(
                    Wr, (unsigned)(k0 + e * kWave + lane) * (unsigned)sizeof(float2),
                    min(i0 + u * n_waves, N - 1) * M * (int)sizeof(float2), 0));
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < G; ++e)
                if (i0 + u * n_waves < N)
                    s_w[(i0 + u * n_waves) * kCols + e * kWave + lane] = k0 + e * kWave + lane < M ? v[u][e] : make_float2(0.f, 0.f);
    }
    for (int i = threadIdx.x; i < N; i += blockDim.x) s_a[i] = A.psi.a[i].x;
    const int chain = uniform((int)(blockIdx.x * n_waves + wv));
    const bool have = chain < A.n_chains;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int site = q * kWave + lane;
        row[site] = have && site < N ? A.spins[(long)chain * N + site] : (int8_t)0;
    }
    __syncthreads();
    if (!have) return;

    // theta = b + sigma W; lanes past M keep theta = 0, and their cached L is
    // the same function of the same value, so they add exactly zero below
    float2 th[E], wi[E], wj[E];
    float L[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = e * kWave + lane;
        th[e] = (k < M) ? A.psi.b[k] : make_float2(0.f, 0.f);
    }
#pragma unroll 4
    for (int i = 0; i < N; ++i) {
        const float si = (float)row[i];
        sample_rows<E, false, G>(Wr, s_w, M, i, i, lane, wi, wj);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            th[e].x = fmaf(si, wi[e].x, th[e].x);
            th[e].y = fmaf(si, wi[e].y, th[e].y);
        }
    }
#pragma unroll
    for (int e = 0; e < E; ++e) L[e] = re_log2cosh_fast(th[e]);

    uint32_t accepted = 0;
    const long total = (long)A.n_sweeps * N;
    const bool words = ((N | (int)reinterpret_cast<uintptr_t>(A.samples_out)) & 3) == 0;
    int8_t* out = A.samples_out ? A.samples_out + (long)chain * N : nullptr;
    const long out_step = (long)A.n_chains * N;
    int sweep_end = N;                            // end of the current sweep, counted from the batch's first proposal
    for (long t0 = 0; t0 < total; t0 += 64) {
        const DrawBatch b = draw_batch(A.seed, (uint32_t)chain, A.step_offset + (uint64_t)t0, lane, N);
        const int count = (int)min((long)64, total - t0);
        const uint64_t in_range = count == 64 ? ~0ull : (1ull << count) - 1ull;
        uint64_t up_i = __ballot(row[b.i] > 0), up_j = PAIR ? __ballot(row[b.j] > 0) : 0ull;
        // the move changes Re(a . s) by -s_i d2
        const float d2 = PAIR ? 2.f * (s_a[b.i] - s_a[b.j]) : 2.f * s_a[b.i];
        uint64_t taken = 0, applied = 0;
        uint64_t rest = (PAIR ? up_i ^ up_j : ~0ull) & in_range;
        auto sweeps_done = [&](int l) {           // sweeps that end at or before draw l of this batch
            while (sweep_end <= l) {
                if (out) {
                    apply_moves<PAIR>(row, taken ^ applied, b, lane);
                    applied = taken;
                    store_spins(row, out, N, lane, words);
                    out += out_step;
                }
                sweep_end += N;
            }
        };
        if (rest) {
            int l = __builtin_ctzll(rest);
            int ci = __builtin_amdgcn_readlane(b.i, l), cj = __builtin_amdgcn_readlane(b.j, l);
            sample_rows<E, PAIR, G>(Wr, s_w, M, ci, cj, lane, wi, wj);
            do {
                sweeps_done(l);
                const float u = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(b.u), l));
                const float dd = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(d2), l));
                const bool up = (up_i >> l) & 1ull;
                const uint64_t after = (~0ull << l) << 1;
                // the differences are formed before the next rows are asked for, so that those take the same registers
                float2 d[E];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    d[e] = PAIR ? csub(wi[e], wj[e]) : wi[e];
                    asm volatile("" : "+v"(d[e].x), "+v"(d[e].y));
                }
                rest &= after;
                int next = rest ? __builtin_ctzll(rest) : l;
                int ni = __builtin_amdgcn_readlane(b.i, next), nj = __builtin_amdgcn_readlane(b.j, next);
                sample_rows<E, PAIR, G>(Wr, s_w, M, ni, nj, lane, wi, wj);
                const float m2si = up ? -2.f : 2.f;
                float Ln[E];
                const float dl = units_dlog<E>(m2si, d, th, L, Ln) + (up ? -dd : dd);
                if (u < __expf(2.f * dl)) {
#pragma unroll
                    for (int e = 0; e < E; ++e) { th[e] = d[e]; L[e] = Ln[e]; }
                    up_i ^= __builtin_amdgcn_ballot_w64(b.i == ci);
                    if (PAIR) {
                        up_i ^= __builtin_amdgcn_ballot_w64(b.i == cj);
                        up_j ^= __builtin_amdgcn_ballot_w64(b.j == ci) ^ __builtin_amdgcn_ballot_w64(b.j == cj);
                        rest = (up_i ^ up_j) & in_range & after;
                        const int actual = rest ? __builtin_ctzll(rest) : next;
                        if (actual != next) {
                            next = actual;
                            ni = __builtin_amdgcn_readlane(b.i, next);
                            nj = __builtin_amdgcn_readlane(b.j, next);
                            sample_rows<E, PAIR, G>(Wr, s_w, M, ni, nj, lane, wi, wj);
                        }
                    }
                    ++accepted;
                    taken |= 1ull << l;
                }
                l = next;
                ci = ni;
                cj = nj;
            } while (rest);
        }
        sweeps_done(count);
        sweep_end -= 64;
        apply_moves<PAIR>(row, taken ^ applied, b, lane);
        if (A.trace && lane == 0) {
            uint32_t* w = A.trace + (long)chain * A.trace_words + (t0 >> 5);
            w[0] = (uint32_t)taken;
            if (count > 32) w[1] = (uint32_t)(taken >> 32);
        }
    }

    store_spins(row, A.spins + (long)chain * N, N, lane, ((N | (int)reinterpret_cast<uintptr_t>(A.spins)) & 3) == 0);
    if (A.n_accept && lane == 0) A.n_accept[chain] = accepted;
    if (A.theta_out) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int k = e * kWave + lane;
            if (k < M) A.theta_out[(long)chain * M + k] = th[e];
        }
    }
    if (A.logpsi_out) {
        // full complex log psi of the final state
        float2 acc = make_float2(0.f, 0.f);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (e * kWave + lane < M) acc = cadd(acc, log2cosh(th[e]));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int site = q * kWave + lane;
            if (site < N) acc = cadd(acc, cscale(A.psi.a[site], (float)row[site]));
        }
        acc = wave_sum(acc);
        if (lane == 0) A.logpsi_out[chain] = acc;
    }
}

// LDS of one compute unit
constexpr size_t kSampleLds = 160 * 1024;

template <int E, bool PAIR, int G>
static hipError_t sample_groups(const SampleArgs& A, int waves, hipStream_t stream) {
    const size_t lds = (size_t)A.N * G * kWave * sizeof(float2) + 256 * (size_t)waves + sizeof(float) * (size_t)A.N;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void*)k_sample<E, PAIR, G>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSampleLds);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_sample<E, PAIR, G>), dim3((unsigned)(((long)A.n_chains + waves - 1) / waves)), dim3(kWave * waves), lds, stream, A);
    return hipGetLastError();
}

// Waves per workgroup: as many as give each compute unit one workgroup, at most 16 (the largest workgroup).
// Above that many chains (4,096 on 256 units) a compute unit takes several workgroups in turn, two at a time where registers and half the LDS
// allow it.  As many unit groups of W go to LDS as fit, out of 1, 2, 3 and all: at N = 100, M = 400 three of seven
// cut the L2 reads that a full chip was waiting on.  One group always fits (N <= 256: 128 KB).
template <int E, bool PAIR>
static hipError_t sample_width(const SampleArgs& A, int n_cu, hipStream_t stream) {
    const int full = 16 * n_cu;
    const int waves = A.n_chains >= full ? 16 : (A.n_chains + n_cu - 1) / n_cu;
    const size_t budget = A.n_chains > full ? kSampleLds / 2 : kSampleLds;
    const size_t group = (size_t)A.N * kWave * sizeof(float2), rest = 256 * (size_t)waves + sizeof(float) * (size_t)A.N;
    const int fit = std::max(1, (int)((budget - rest) / group));
    if (fit >= E) return sample_groups<E, PAIR, E>(A, waves, stream);
    if constexpr (E > 3) if (fit >= 3) return sample_groups<E, PAIR, 3>(A, waves, stream);
    if constexpr (E > 2) if (fit >= 2) return sample_groups<E, PAIR, 2>(A, waves, stream);
    return sample_groups<E, PAIR, 1>(A, waves, stream);
}

hipError_t launch_sample(const SampleArgs& args, int n_cu, hipStream_t stream) {
    const bool pair = args.proposal == 1;
    switch ((args.M + kWave - 1) / kWave) {
#define CRBM_CASE(e) \
    case e: return pair ? sample_width<e, true>(args, n_cu, stream) : sample_width<e, false>(args, n_cu, stream);
        CRBM_CASE(1) CRBM_CASE(2) CRBM_CASE(3) CRBM_CASE(4) CRBM_CASE(5) CRBM_CASE(6) CRBM_CASE(7) CRBM_CASE(8)
#undef CRBM_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace crbm
