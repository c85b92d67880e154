// H psi of a Pauli sum H, amplitude by amplitude: the inner loops shared by
// the batch (batch.hip) and the single-state adjoint sweep (adjoint.hip).
#pragma once

#include "dev_core.hpp"

namespace qs {

// A Hermitian Pauli string h P with i^{#Y} folded into its coefficient, which
// is then real (an even number of Y) or i times a real number.
struct PauliTerm {
    uint64_t x, yz;   // flip mask, sign mask
    double c;         // the real number
};

constexpr int kTermGroup = 4;   // terms whose gathers are in flight together

// (re, im)[u] += sum_n c_n (-1)^{popc(j & yz_n)} psi_j, j = i ^ x_n, for the
// thread's amplitudes i = first + t + 256 u (t: thread number, the block's
// 256 U amplitudes start at the uniform index first, a multiple of 256 U), over
// the terms [begin, end), a multiple of kTermGroup (zero terms pad).  IM: the
// terms whose coefficient is i c.  All sums in FP64.
// Bound: the vector unit's FP64 rate (two conversions and two FMAs per term
// and amplitude, 4.6 cycles each per wavefront) together with the gathers,
// which the caches serve.  So what does not differ between a thread's
// amplitudes is done once for all U: the flipped thread number with its parity
// and address; and what does not differ between threads is scalar.
template <typename R, int U, bool IM>
__device__ __forceinline__ void add_pauli_terms(double (&re)[U], double (&im)[U], const C2<R> *__restrict__ psi,
                                                uint64_t first, uint32_t t, const PauliTerm *__restrict__ terms,
                                                int begin, int end)
{
    for (int n0 = begin; n0 < end; n0 += kTermGroup) {
        C2<R> v[kTermGroup][U];
#pragma unroll
        for (int k = 0; k < kTermGroup; k++) {
            const uint64_t x = terms[n0 + k].x;
            const uint32_t tl = t ^ (uint32_t)(x & 255u);
#pragma unroll
            for (int u = 0; u < U; u++) v[k][u] = (psi + ((first + 256u * u) ^ (x & ~255ULL)))[tl];
        }
#pragma unroll
        for (int k = 0; k < kTermGroup; k++) {
            const PauliTerm tm = terms[n0 + k];
            const uint32_t tl = t ^ (uint32_t)(tm.x & 255u);
            const uint32_t lane = (uint32_t)__popc(tl & (uint32_t)(tm.yz & 255u)) << 31;
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint64_t j = (first + 256u * u) ^ (tm.x & ~255ULL);
                const uint32_t s = lane ^ ((uint32_t)__popcll(j & tm.yz & ~255ULL) << 31);
                const double c = __longlong_as_double(__double_as_longlong(tm.c) ^ (long long)((uint64_t)s << 32));
                const double vx = v[k][u].x, vy = v[k][u].y;
                re[u] = IM ? fma(-c, vy, re[u]) : fma(c, vx, re[u]);
                im[u] = IM ? fma(c, vx, im[u]) : fma(c, vy, im[u]);
            }
        }
    }
}

}  // namespace qs
