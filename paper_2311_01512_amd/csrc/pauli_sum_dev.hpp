// H psi of a Pauli sum H, amplitude by amplitude: the inner loops shared by
// the batch (batch.hip) and the single-state adjoint sweep (adjoint.hip).
#pragma once

#include "common.hpp"

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
// the terms [begin, end).  IM: the terms whose coefficient is i c.  All sums in
// FP64.
// Bound: the vector unit's FP64 rate (two conversions and two FMAs per term
// and amplitude, 4.6 cycles each per wavefront) together with the gathers,
// which the caches serve.  So what does not differ between a thread's
// amplitudes is done once for all U: the flipped thread number with its parity
// and address; and what does not differ between threads is scalar.
template <typename R, int U, int G, bool IM>
__device__ __forceinline__ void add_pauli_group(double (&re)[U], double (&im)[U], const C2<R> *__restrict__ psi,
                                                uint64_t first, uint32_t t, const PauliTerm *__restrict__ terms)
{
    C2<R> v[G][U];
#pragma unroll
    for (int k = 0; k < G; k++) {
        const uint64_t x = terms[k].x;
        const uint32_t tl = t ^ (uint32_t)(x & 255u);
#pragma unroll
        for (int u = 0; u < U; u++) v[k][u] = (psi + ((first + 256u * u) ^ (x & ~255ULL)))[tl];
    }
#pragma unroll
    for (int k = 0; k < G; k++) {
        const PauliTerm tm = terms[k];
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

template <typename R, int U, bool IM>
__device__ __forceinline__ void add_pauli_terms(double (&re)[U], double (&im)[U], const C2<R> *__restrict__ psi,
                                                uint64_t first, uint32_t t, const PauliTerm *__restrict__ terms,
                                                int begin, int end)
{
    int n = begin;
    for (; n + kTermGroup <= end; n += kTermGroup)
        add_pauli_group<R, U, kTermGroup, IM>(re, im, psi, first, t, terms + n);
    for (; n < end; n++) add_pauli_group<R, U, 1, IM>(re, im, psi, first, t, terms + n);
}

// Terms of one launch, passed by value: those with real coefficients, then
// those with imaginary ones.
constexpr int kSumTerms = 64;
struct PauliTerms {
    int real, count;
    PauliTerm t[kSumTerms];
};

// The terms [begin, end) of a Pauli sum over N qubits (codes term-major, each
// 0..3) for one launch.
inline PauliTerms pauli_terms(const int *codes, const double *coeffs, int N, int begin, int end)
{
    PauliTerms p{};
    for (int odd = 0; odd < 2; odd++) {
        for (int n = begin; n < end; n++) {
            PauliTerm d{};
            int ny = 0;
            for (int k = 0; k < N; k++) {
                const int c = codes[(size_t)n * N + k];
                if (c == 1 || c == 2) d.x |= 1ULL << k;
                if (c == 2 || c == 3) d.yz |= 1ULL << k;
                if (c == 2) ny++;
            }
            if ((ny & 1) != odd) continue;
            d.c = (ny & 2) ? -coeffs[n] : coeffs[n];
            p.t[p.count++] = d;
        }
        if (!odd) p.real = p.count;
    }
    return p;
}

}  // namespace qs
