// At-least-t constraints of at most 128 literals in FP32: value and gradient
// through the distribution of the number of true literals.
//
// With p_i = (1 - l_i) / 2 the probability that literal i is true, X = the number
// of true literals of independent draws and X_-i that of the others,
//   WE = 2 P(X < t) - 1,   dWE / dl_i = P(X_-i = t - 1)
// (the same multilinear polynomial that Alg. 2 evaluates at the roots of unity:
// its transform there is the characteristic function of X; Eq. chain's
// leave-one-out products are that of X_-i).  Running products at k / 2
// frequencies cost about 7 operations per literal and frequency; the
// distribution is built by products of polynomials with nonnegative coefficients
// and the leave-one-out probabilities come back down the same tree, about
// S^2 / 2 + 3 S^2 operations for a lane's S literals and less above it, and no
// cancellation anywhere.
//
// Mapping: L lanes of S literals.  A lane multiplies its literals up in quads
// (two halves of S / 2 beyond 16), L = 4 lanes their distributions in pairs.  At
// the top nothing is multiplied: the functional that a side's polynomial is paired
// with is the other side's distribution read backwards from t - 1 (LDS, written
// shifted by the uniform t).  Going down, the functional of a part is that of
// the whole taken through its sibling's distribution: h'(j) = sum_m sib(m) h(j + m).
// If t is above half of k, the false literals are counted instead (t' = k - t +
// 1, the same probabilities), so t - 1 < L S / 2 and the top needs only half the
// coefficients.  Padding literals have p = 0.
// Measured against the running products (grouped launch of every bin): mixed n =
// 2000 instance (200 constraints of 10..100 literals among 8500 others) 196 -> 116 us
// at 1024 restarts, 55 -> 34 at 256; 200 constraints of 32 literals at 10000 points
// 284 -> 160.  In a launch of its own beside the others, without the few spills of
// its 24- and 32-literal shapes at four waves per SIMD: slower (mixed round 483 ->
// 627 us, one more launch per step).
#pragma once
#include <type_traits>

#include "eval_kernel.h"

namespace ffsat {

// Shapes (S, L), shape_for_count (host.cpp): up to 16 literals on one lane, 32 on
// two, 128 on four
#define FFSAT_COUNT_SHAPES(X)                                                                                 \
    X(0, 4, 1) X(1, 8, 1) X(2, 12, 1) X(3, 16, 1) X(4, 12, 2) X(5, 16, 2) X(6, 12, 4) X(7, 16, 4) X(8, 24, 4) \
    X(9, 32, 4)
// LDS of a wave: L = 2 64 columns of S rows, L = 4 32 columns of 2 S rows, and one
// row for what falls outside
template <int S, int L>
__host__ __device__ constexpr int count_lds_floats() { return L == 1 ? 0 : (L == 2 ? 64 * (S + 1) : 32 * (2 * S + 1)); }
constexpr int COUNT_LDS_MAX = 32 * (2 * 32 + 1);

__device__ __forceinline__ float lane_swap1(float v) { return dpp_f32<0xB1>(v); }   // quad_perm [1,0,3,2]

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): loops whose
// bodies are too many for the unroller
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// Keeps the compiler from carrying values derived from p across this point: the
// polynomials are built again where they are needed (21 operations a quad)
// instead of held in registers.
template <int S>
__device__ __forceinline__ void fresh(float (&p)[S])
{
#pragma unroll
    for (int i = 0; i < S; ++i) asm volatile("" : "+v"(p[i]));
}

// distribution of the count of literals p[B..B+3]
template <int B, int S>
__device__ __forceinline__ void quad_poly(const float (&p)[S], float (&d)[5])
{
    const float p0 = p[B], p1 = p[B + 1], p2 = p[B + 2], p3 = p[B + 3];
    const float q0 = 1.f - p0, q1 = 1.f - p1, q2 = 1.f - p2, q3 = 1.f - p3;
    const float a0 = q0 * q1, a1 = __builtin_fmaf(q0, p1, p0 * q1), a2 = p0 * p1;
    const float b0 = q2 * q3, b1 = __builtin_fmaf(q2, p3, p2 * q3), b2 = p2 * p3;
    d[0] = a0 * b0;
    d[1] = __builtin_fmaf(a0, b1, a1 * b0);
    d[2] = __builtin_fmaf(a0, b2, __builtin_fmaf(a1, b1, a2 * b0));
    d[3] = __builtin_fmaf(a1, b2, a2 * b1);
    d[4] = a2 * b2;
}
// h[0..3]: functional of the quad; g[i] = P(the other three = j) summed against h
template <int B, int S>
__device__ __forceinline__ void quad_down(const float (&p)[S], const float (&h)[4], float (&g)[4])
{
    const float p0 = p[B], p1 = p[B + 1], p2 = p[B + 2], p3 = p[B + 3];
    const float q0 = 1.f - p0, q1 = 1.f - p1, q2 = 1.f - p2, q3 = 1.f - p3;
    const float a0 = q0 * q1, a1 = __builtin_fmaf(q0, p1, p0 * q1), a2 = p0 * p1;
    const float b0 = q2 * q3, b1 = __builtin_fmaf(q2, p3, p2 * q3), b2 = p2 * p3;
    const float ha0 = __builtin_fmaf(b0, h[0], __builtin_fmaf(b1, h[1], b2 * h[2]));
    const float ha1 = __builtin_fmaf(b0, h[1], __builtin_fmaf(b1, h[2], b2 * h[3]));
    const float hb0 = __builtin_fmaf(a0, h[0], __builtin_fmaf(a1, h[1], a2 * h[2]));
    const float hb1 = __builtin_fmaf(a0, h[1], __builtin_fmaf(a1, h[2], a2 * h[3]));
    g[0] = __builtin_fmaf(q1, ha0, p1 * ha1);
    g[1] = __builtin_fmaf(q0, ha0, p0 * ha1);
    g[2] = __builtin_fmaf(q3, hb0, p3 * hb1);
    g[3] = __builtin_fmaf(q2, hb0, p2 * hb1);
}
// P[0 .. N + 4] = P[0 .. N] * d
template <int N, int M>
__device__ __forceinline__ void mul_quad(float (&P)[M], const float (&d)[5])
{
#pragma unroll
    for (int c = N + 4; c >= 0; --c) {
        float s = 0.f;
#pragma unroll
        for (int m = 4; m >= 0; --m)
            if (c - m >= 0 && c - m <= N) s = __builtin_fmaf(P[c - m], d[m], s);
        P[c] = s;
    }
}
// P = distribution of the count of literals p[B .. B + N - 1], N in {4, 8, 12, 16}
template <int B, int N, int S>
__device__ __forceinline__ void seg_poly(const float (&p)[S], float (&P)[N + 1])
{
    float d[5];
    quad_poly<B>(p, d);
#pragma unroll
    for (int c = 0; c < 5; ++c) P[c] = d[c];
    if constexpr (N >= 8) { quad_poly<B + 4>(p, d); mul_quad<4>(P, d); }
    if constexpr (N >= 12) { quad_poly<B + 8>(p, d); mul_quad<8>(P, d); }
    if constexpr (N >= 16) { quad_poly<B + 12>(p, d); mul_quad<12>(P, d); }
}
// One quad of seg_down: the literals B + U .. B + U + 3, pre the distribution of the U
// literals before them, R the functional of the first U + 4 literals (then of U).
template <int B, int U, int N, int S, typename Out>
__device__ __forceinline__ void quad_step(const float (&p)[S], const float (&pre)[U + 1], float (&R)[N], Out &&out)
{
    float h[4], g[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i <= U; ++i) s = __builtin_fmaf(pre[i], R[a + i], s);
        h[a] = U == 0 ? R[a] : s;
    }
    quad_down<B + U>(p, h, g);
#pragma unroll
    for (int i = 0; i < 4; ++i) out(B + U + i, g[i]);
    if constexpr (U > 0) {
        float d[5];
        quad_poly<B + U>(p, d);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            float s = 0.f;
#pragma unroll
            for (int m = 0; m < 5; ++m) s = __builtin_fmaf(d[m], R[q + m], s);
            R[q] = s;
        }
    }
}
// out(i, P(others = .) . R) for the literals p[B .. B + N - 1]; R is overwritten
template <int B, int N, int S, typename Out>
__device__ __forceinline__ void seg_down(float (&p)[S], float (&R)[N], Out &&out)
{
    if constexpr (N >= 16) { float pre[13]; seg_poly<B, 12>(p, pre); quad_step<B, 12>(p, pre, R, out); fresh(p); }
    if constexpr (N >= 12) { float pre[9]; seg_poly<B, 8>(p, pre); quad_step<B, 8>(p, pre, R, out); fresh(p); }
    if constexpr (N >= 8) { float pre[5]; seg_poly<B, 4>(p, pre); quad_step<B, 4>(p, pre, R, out); fresh(p); }
    float one[1] = {1.f};
    quad_step<B, 0>(p, one, R, out);
}
// the lane's whole distribution
template <int S>
__device__ __forceinline__ void lane_poly(const float (&p)[S], float (&P)[S + 1])
{
    if constexpr (S <= 16) {
        seg_poly<0, S>(p, P);
    } else {
        float A[S / 2 + 1], Bp[S / 2 + 1];
        seg_poly<0, S / 2>(p, A);
        seg_poly<S / 2, S / 2>(p, Bp);
        static_for<0, S + 1>([&](auto ic) {
            constexpr int c = ic, m0 = c > S / 2 ? c - S / 2 : 0, m1 = c < S / 2 ? c : S / 2;
            float s = 0.f;
#pragma unroll
            for (int m = m0; m <= m1; ++m) s = __builtin_fmaf(A[m], Bp[c - m], s);
            P[c] = s;
        });
    }
}
template <int S, typename Out>
__device__ __forceinline__ void lane_down(float (&p)[S], float (&R)[S], Out &&out)
{
    fresh(p);
    if constexpr (S <= 16) {
        seg_down<0, S>(p, R, out);
    } else {
        constexpr int N = S / 2;
        // half by half, the sibling's distribution built anew
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if (half) fresh(p);
            float sib[N + 1], h[N];
            if (half == 0) seg_poly<N, N>(p, sib);
            else seg_poly<0, N>(p, sib);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                float s = 0.f;
#pragma unroll
                for (int m = 0; m <= N; ++m) s = __builtin_fmaf(sib[m], R[j + m], s);
                h[j] = s;
            }
            fresh(p);
            if (half == 0) seg_down<0, N>(p, h, out);
            else seg_down<N, N>(p, h, out);
        }
    }
}

// R[j] = P(count of the other lanes = t - 1 - j), j < S, and P(X < t) on every lane
// of the group, for t - 1 < L S / 2.  sm: the wave's
// count_lds_floats<S, L>() floats.
template <int S, int L>
__device__ __forceinline__ float count_top(const float (&P)[S + 1], int t, int lane, float *sm, float (&R)[S])
{
    float lt = 0.f;
    if constexpr (L == 1) {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            R[j] = j == t - 1 ? 1.f : 0.f;   // uniform
            lt += j < t ? P[j] : 0.f;
        }
    } else if constexpr (L == 2) {
        // row r + 1, column lane: this lane's P at t - 1 - r; row 0 takes the rest
#pragma unroll
        for (int c = 0; c <= S; ++c) sm[max(t - c, 0) * 64 + lane] = P[c];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        float cdf = 0.f;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const float v = sm[(j + 1) * 64 + (lane ^ 1)];
            R[j] = j < t ? v : 0.f;   // uniform
        }
        // P(X < t) = sum_r P(other = t - 1 - r) P(own <= r)
#pragma unroll
        for (int j = 0; j < S; ++j) {
            cdf += P[j];
            lt = __builtin_fmaf(R[j], cdf, lt);
        }
    } else {
        static_assert(L == 4, "one, two or four lanes");
        const int q = lane & 1, g = lane >> 1;
        // the pair's distribution at c = 2 i + q: the sibling's coefficients at
        // a lane-dependent parity, y[d + 1] = sib(d + q)
        float y[S + 2], Z[S + 1];
        {
            float s0 = 0.f;
#pragma unroll
            for (int d = -1; d <= S; ++d) {
                const float s1 = d + 1 <= S ? lane_swap1(P[d + 1 <= S ? d + 1 : 0]) : 0.f;
                y[d + 1] = q ? s1 : s0;
                s0 = s1;
            }
        }
        static_for<0, S + 1>([&](auto ic) {
            constexpr int i = ic, m0 = 2 * i > S ? 2 * i - S : 0, m1 = 2 * i + 1 < S ? 2 * i + 1 : S;
            float s = 0.f;
#pragma unroll
            for (int m = m0; m <= m1; ++m) s = __builtin_fmaf(P[m], y[2 * i - m + 1], s);
            Z[i] = s;
        });
        __builtin_amdgcn_sched_barrier(0);
        // row r + 1, column pair: the pair's distribution at t - 1 - r
#pragma unroll
        for (int i = 0; i <= S; ++i) sm[max(t - 2 * i - q, 0) * 32 + g] = Z[i];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const float *o = sm + (g ^ 1) + 32;
        // h(r) = P(other pair = t - 1 - r): R(j) = sum_m sib(m) h(j + m), and
        // P(X < t) = sum_r h(r) P(own pair <= r)
        float sib[S + 1];
#pragma unroll
        for (int m = 0; m <= S; ++m) sib[m] = lane_swap1(P[m]);
#pragma unroll
        for (int j = 0; j < S; ++j) R[j] = 0.f;
        float run = 0.f;
        static_for<0, S>([&](auto ic) {
            constexpr int i = ic;
            const float v0 = o[2 * i * 32], v1 = o[(2 * i + 1) * 32];
            const float h0 = 2 * i < t ? v0 : 0.f, h1 = 2 * i + 1 < t ? v1 : 0.f;   // uniform
            const float zs = lane_swap1(Z[i]);
            lt = __builtin_fmaf(h0, run + (q ? zs : Z[i]), lt);
            run += Z[i] + zs;
            lt = __builtin_fmaf(h1, run, lt);
            constexpr int r0 = 2 * i, r1 = 2 * i + 1;
#pragma unroll
            for (int j = (r0 > S ? r0 - S : 0); j <= (r0 < S - 1 ? r0 : S - 1); ++j) R[j] = __builtin_fmaf(sib[r0 - j], h0, R[j]);
#pragma unroll
            for (int j = (r1 > S ? r1 - S : 0); j <= (r1 < S - 1 ? r1 : S - 1); ++j) R[j] = __builtin_fmaf(sib[r1 - j], h1, R[j]);
            if constexpr (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // LDS reads eight ahead, not all at once (registers)
        });
    }
    __builtin_amdgcn_wave_barrier();   // the next constraint writes the rows again
    return lt;
}

// The work of one wave (see eval_unit): unit = (chunk of sp.cpw constraints,
// restart block).
template <int S, int L>
__device__ __forceinline__ void count_unit(const EvalArgs<float> &a, const Span sp, const int unit,
                                           const float *__restrict__ xin, const ConDesc *__restrict__ con,
                                           const int32_t *__restrict__ lits, const float *__restrict__ wts, float *sm)
{
    constexpr int RPW = 64 / L;
    const int lane = threadIdx.x & 63;
    const int n_chunks = (sp.count + sp.cpw - 1) / sp.cpw;
    if (unit >= n_chunks * sp.n_rb) return;          // whole wave leaves together
    if (a.skip != nullptr && *a.skip == 0) return;   // uniform
    const int chunk = unit / sp.n_rb;
    const int rb = unit - chunk * sp.n_rb;
    const int j = lane & (L - 1);
    const int b = rb * RPW + lane / L;
    const bool bok = b < a.B;
    const int bb = bok ? b : a.B - 1;
    const int i0 = j * S;
    float facc = 0.f;
    int nunsat = 0;
    const int c_end = min((chunk + 1) * sp.cpw, sp.count);
#pragma unroll 1
    for (int ci = chunk * sp.cpw; ci < c_end; ++ci) {
        const ConDesc d = con[sp.first + ci];
        const int k = d.k;
        // at least t true, or (t past the middle) fewer than t false; p = 0 for padding
        const bool flip = 2 * d.chk > k + 1;
        const int t = flip ? k - d.chk + 1 : d.chk;
        const float half = flip ? 0.5f : -0.5f;
        float p[S];
        int nv;
        uint32_t negm, tmask;
        load_segment<L, S, float>(a, d, xin, lits, i0, bb, flip ? -1.f : 1.f, p, nv, negm, tmask);
#pragma unroll
        for (int i = 0; i < S; ++i) p[i] = __builtin_fmaf(half, p[i], 0.5f);
        float *const slot = a.slot + ((size_t)i0 * a.B + b);
        asm volatile("" : "+v"(negm));
        if (a.want_check) {
            const int cnt = group_sum_int<L>(__popc(tmask));
            const bool uns = cnt < d.chk && bok && j == 0;
            nunsat += uns ? 1 : 0;
            if (a.unsat_bits != nullptr && uns)
                atomicOr(&a.unsat_bits[(size_t)b * a.wm + (d.orig >> 5)], 1u << (d.orig & 31));
            if (a.U != nullptr) {
                const unsigned long long bal = __ballot(uns);
                if (lane == 0 && bal != 0ull) atomicAdd(&a.U[d.orig], (int)__popcll(bal));
            }
        }
        float R[S], below;
        {
            float P[S + 1];
            lane_poly<S>(p, P);
            below = count_top<S, L>(P, t, lane, sm, R);
        }
        const float we = (flip ? -1.f : 1.f) * __builtin_fmaf(2.f, below, -1.f);
        const float wc = wts[d.orig];
        if (j == 0) facc = __builtin_fmaf(wc, we, facc);
        if (a.con_val != nullptr && j == 0 && bok) a.con_val[(size_t)d.orig * a.B + b] = we;
        if (a.want_grad) {
            asm volatile("" : "+v"(nv));
            lane_down<S>(p, R, [&](int i, float g) {
                if (i < nv && bok) {
                    const float gv = ((negm >> i) & 1u) ? -g : g;
                    slot[(size_t)(d.off + i) * a.B] = wc * gv;
                }
            });
        }
    }
    if (j == 0 && bok) {
        const size_t row = (size_t)(sp.fpart_row0 + chunk) * a.B + b;
        a.fpart[row] = facc;
        if (a.want_check) a.cpart[row] = nunsat;
    }
}

}  // namespace ffsat
