// Metropolis proposals shared by the sweep and the batched moments.
//
// A proposal flips site i (or, for an exchange, sites i and j with
// s_i = -s_j) and is accepted on u < |psi'/psi|^2 (Sec. III).  Sites and
// uniform come from the chain's counter-based stream alone, so 64 proposals
// are drawn at once, one per lane, and the null moves among them (exchanges of
// equal spins) are known without being visited.  A chain's spins are bytes in
// LDS, brought up to date from the accepted draws of a batch.
#pragma once
#include "device.hpp"
#include "internal.hpp"

namespace crbm {

// Draws of 64 consecutive proposals t0 + l, one per lane l (counter t0 + l of stream `chain`,
// Philox tag 0): the generator runs on the vector unit once per 64 proposals, and a proposal
// takes its sites and uniform from its lane with readlane.
struct DrawBatch {
    int i, j;
    float u;
};

__device__ __forceinline__ DrawBatch draw_batch(uint64_t seed, uint32_t chain, uint64_t t0, int lane, int N) {
    uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
    // An empty statement that marks the key as rewritten here: the ten round keys are then derived at
    // each batch (20 scalar adds per 64 proposals) instead of being hoisted out of the sweep loop,
    // where they would hold 20 scalar registers for the whole launch and push others into spills.
    asm volatile("" : "+s"(k0), "+s"(k1));
    const uint64_t t = t0 + (uint64_t)lane;
    const u32x4 x = philox4x32_10(chain, (uint32_t)t, (uint32_t)(t >> 32), 0u, k0, k1);
    return {draw_index(x.x, N), draw_index(x.y, N), draw_unit(x.z)};
}

// The accepted draws of `moved` applied to the chain's spin bytes: a flip exchanges +1 (0x01) and -1 (0xFF), so each
// lane applies its own draw with atomic XORs, in any order.
template <bool PAIR>
__device__ __forceinline__ void apply_moves(int8_t* row, uint64_t moved, const DrawBatch& b, int lane) {
    if (!((moved >> lane) & 1ull)) return;
    unsigned* const w = reinterpret_cast<unsigned*>(row);
    atomicXor(&w[b.i >> 2], 0xFEu << (8 * (b.i & 3)));
    if (PAIR) atomicXor(&w[b.j >> 2], 0xFEu << (8 * (b.j & 3)));
}

// change of theta_k per unit of -2 s_i: W_ik (flip) or W_ik - W_jk (exchange); zero past M.
// E = ceil(M / 64), so only the last group can hold lanes past M.  MASK = false for rows that hold
// zeros past M themselves.
template <int E, bool PAIR, bool MASK = true>
__device__ __forceinline__ float2 row_delta(const float2 (&wi)[E], const float2 (&wj)[E], int e, int lane, int M) {
    float2 d = PAIR ? csub(wi[e], wj[e]) : wi[e];
    if (MASK && e == E - 1 && e * kWave + lane >= M) d = make_float2(0.f, 0.f);
    return d;
}

// theta' = theta + m2si d (in place of d) and the wave total of the change of Re log 2cosh theta.  Lanes past M
// hold theta = 0 and L = Re log 2cosh(0) from the same function, so they add exactly zero.
template <int E>
__device__ __forceinline__ float units_dlog(float m2si, float2 (&d)[E], const float2 (&th)[E], const float (&L)[E],
                                            float (&Ln)[E]) {
    float dsum = 0.f;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        d[e].x = fmaf(m2si, d[e].x, th[e].x);
        d[e].y = fmaf(m2si, d[e].y, th[e].y);
        Ln[e] = re_log2cosh_fast(d[e]);
        const float x = Ln[e] - L[e];
        dsum = e == 0 ? x : dsum + x;   // 0 + x would only change the sign of a zero
    }
    return wave_total(dsum);
}

}  // namespace crbm
