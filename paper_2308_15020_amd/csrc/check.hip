// The exact check of a batch of rounded points by itself (Alg. 1's certificate
// line, Thm. 2), on one bit per variable and restart.
//
// The evaluation kernels gather 4 bytes per (literal, restart) to look at a
// sign: 1.3 GB for 420000 3-SAT clauses and 256 restarts.  Here the signs are
// packed first (k_signs: bit b % 64 of word b / 64 of row v: x_v < 0 at restart
// b, one pass over x, which also writes the caller's assignment bits), and a
// literal of 64 restarts is one 8-byte word.
//  * Constraints of at most CHECK_SHORT literals: one thread each, the true
//    literals of 64 restarts counted in bit planes (k_check_short).  The 64
//    results of a wave are a 64 x 64 bit matrix; transposed over the lanes it
//    gives each restart its violated constraints, as the output's words and as
//    a count.
//  * Longer ones: one wave each, a lane per literal; the transposed words of 64
//    literals give each restart its count (k_check_long).
// Measured at n = 100000, 420000 clauses of 3, 256 restarts: 39 us for the
// signs and the assignment bits (109 MB in and out: 2.8 TB/s, the assignment words
// are written 4 bytes at a time), 46 us for the clauses (5 million gathered words
// from L2); the check inside the evaluation kernels took 745 us.
#include "internal.h"

namespace ffsat {

// Words of a row of packed signs: a multiple of four beyond one word, so that
// the four waves of a block (one word each) share the row's 32-byte sector.
int sign_stride(int B)
{
    const int w = (B + 63) / 64;
    return w == 1 ? 1 : (w + 3) / 4 * 4;
}

// Wave = 32 variables x 64 restarts (word blockIdx.y * wpb + wave).
template <typename IO>
__global__ __launch_bounds__(256) void k_signs(int n, int B, int stride, const IO *__restrict__ x,
                                               uint64_t *__restrict__ signs, uint32_t *__restrict__ assign)
{
    const int lane = threadIdx.x & 63;
    const int word = (int)(blockIdx.y * (blockDim.x >> 6) + (threadIdx.x >> 6));
    if (word >= stride) return;
    const int b = word * 64 + lane;
    const int v0 = (int)blockIdx.x * 32;
    const int nv = min(32, n - v0);
    const bool ok = b < B;
    IO xv[32];
#pragma unroll
    for (int q = 0; q < 32; ++q) xv[q] = (ok && q < nv) ? x[(size_t)(v0 + q) * B + b] : IO(0);
    uint32_t own = 0, lo = 0, hi = 0;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
        const bool neg = xv[q] < IO(0);
        own |= neg ? 1u << q : 0u;
        const unsigned long long bal = __ballot(neg);
        lo = lane == q ? (uint32_t)bal : lo;
        hi = lane == q ? (uint32_t)(bal >> 32) : hi;
    }
    if (lane < nv) signs[(size_t)(v0 + lane) * stride + word] = ((uint64_t)hi << 32) | lo;
    if (assign != nullptr && ok) assign[(size_t)b * ((n + 31) / 32) + blockIdx.x] = own;
}

// Transposes the 64 x 64 bit matrix whose row i lane i holds.
__device__ __forceinline__ uint64_t transpose64(uint64_t u, int lane)
{
    constexpr uint64_t M[6] = {0x00000000ffffffffull, 0x0000ffff0000ffffull, 0x00ff00ff00ff00ffull,
                               0x0f0f0f0f0f0f0f0full, 0x3333333333333333ull, 0x5555555555555555ull};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int s = 32 >> i;
        const uint64_t y = __shfl_xor((unsigned long long)u, s, 64);
        u = (lane & s) == 0 ? (u & M[i]) | ((y & M[i]) << s) : (u & ~M[i]) | ((y >> s) & M[i]);
    }
    return u;
}

// Block = gpw * 64 constraints (original order) x 4 words of 64 restarts, one
// word per wave (blockDim.x / 64 waves).
__global__ __launch_bounds__(256) void k_check_short(CheckArgs a)
{
    __shared__ int32_t nu[64 * CHECK_GROUPS];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    const int word = (int)blockIdx.y * waves + wave;
    const int c0 = (int)blockIdx.x * 64 * a.gpw;
    for (int i = threadIdx.x; i < 64 * a.gpw; i += blockDim.x) nu[i] = 0;
    __syncthreads();
    const int b = word * 64 + lane;
    const bool on = word * 64 < a.B;
    // restarts of this word
    const uint64_t valid = !on ? 0 : (a.B - word * 64 >= 64 ? ~0ull : (1ull << (a.B - word * 64)) - 1);
    int viol = 0;
#pragma unroll 1
    for (int g = 0; on && g < a.gpw; ++g) {
        const int c = c0 + g * 64 + lane;
        if (c - lane >= a.m) break;   // uniform
        uint64_t uns = 0;
        int k = 0, off = 0, chk = 0;
        if (c < a.m) {
            const ConDesc d = a.con[a.pos[c]];
            k = d.k <= CHECK_SHORT ? d.k : 0;
            off = d.off;
            chk = d.chk;
        }
        uint64_t p[6] = {0, 0, 0, 0, 0, 0};   // bit planes of the counts (at most 32)
        for (int i = 0; __any(i < k); i += 4) {
            int32_t l[4];
            uint64_t t[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) l[q] = i + q < k ? a.lit[off + i + q] : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                t[q] = i + q < k ? a.signs[(size_t)(l[q] & 0x7fffffff) * a.stride + word] : 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint64_t cy = i + q < k ? (l[q] < 0 ? ~t[q] : t[q]) : 0;
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    const uint64_t n = p[j] & cy;
                    p[j] ^= cy;
                    cy = n;
                }
            }
        }
        if (k > 0) {
            uint64_t sat;
            if (chk < 0) {
                sat = chk == -2 ? p[0] : ~p[0];
            } else {
                // count >= chk, from the top plane down
                uint64_t gt = 0, eq = ~0ull;
#pragma unroll
                for (int j = 5; j >= 0; --j) {
                    const bool tb = (chk >> j) & 1;
                    gt |= tb ? 0 : eq & p[j];
                    eq &= tb ? p[j] : ~p[j];
                }
                sat = chk > 63 ? 0 : gt | eq;
            }
            uns = ~sat & valid;
        }
        if (a.U != nullptr && uns != 0) atomicAdd(&nu[g * 64 + lane], (int)__popcll(uns));
        if (a.unsat_bits != nullptr || a.rows != nullptr) {
            const uint64_t col = transpose64(uns, lane);
            viol += (int)__popcll(col);
            if (a.unsat_bits != nullptr && b < a.B) {
                // longer constraints' bits are 0 here, k_check_long sets them
                const int w = (c - lane) >> 5;
                uint32_t *o = a.unsat_bits + (size_t)b * a.wm + w;
                o[0] = (uint32_t)col;
                if (w + 1 < a.wm) o[1] = (uint32_t)(col >> 32);
            }
        }
    }
    if (a.rows != nullptr && b < a.B) a.rows[(size_t)blockIdx.x * a.B + b] = viol;
    if (a.U != nullptr) {
        __syncthreads();
        for (int i = threadIdx.x; i < 64 * a.gpw && c0 + i < a.m; i += blockDim.x) {
            if (gridDim.y == 1) a.U[c0 + i] = nu[i];
            else if (nu[i] != 0) atomicAdd(&a.U[c0 + i], nu[i]);
        }
    }
}

// Block = CHECK_LONG_PER constraints of the list x 4 words, one per wave.
__global__ __launch_bounds__(256) void k_check_long(CheckArgs a, const int32_t *__restrict__ list, int n_list, int row0)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int word = (int)(blockIdx.y * (blockDim.x >> 6)) + wave;
    const int b = word * 64 + lane;
    if (word * 64 >= a.B) return;   // whole wave
    int viol = 0;
    const int q0 = (int)blockIdx.x * CHECK_LONG_PER, q1 = min(n_list, q0 + CHECK_LONG_PER);
#pragma unroll 1
    for (int q = q0; q < q1; ++q) {
        const ConDesc d = a.con[list[q]];
        int cnt = 0;
        for (int i0 = 0; i0 < d.k; i0 += 256) {
            int32_t l[4];
            uint64_t t[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + 64 * j + lane;
                l[j] = i < d.k ? a.lit[d.off + i] : 0;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int i = i0 + 64 * j + lane;
                const uint64_t s = i < d.k ? a.signs[(size_t)(l[j] & 0x7fffffff) * a.stride + word] : 0;
                t[j] = i < d.k && l[j] < 0 ? ~s : s;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + 64 * j < d.k) cnt += (int)__popcll(transpose64(t[j], lane));   // uniform
        }
        const bool sat = d.chk >= 0 ? cnt >= d.chk : ((cnt & 1) == (d.chk == -2 ? 1 : 0));
        const bool uns = !sat && b < a.B;
        viol += uns ? 1 : 0;
        if (a.unsat_bits != nullptr && uns) atomicOr(&a.unsat_bits[(size_t)b * a.wm + (d.orig >> 5)], 1u << (d.orig & 31));
        const int all = (int)__popcll(__ballot(uns));
        if (a.U != nullptr && lane == 0 && all > 0) atomicAdd(&a.U[d.orig], all);
    }
    if (a.rows != nullptr && b < a.B) a.rows[(size_t)(row0 + blockIdx.x) * a.B + b] = viol;
}

template <typename IO>
static hipError_t signs_impl(int n, int B, const IO *x, uint64_t *signs, uint32_t *assign, hipStream_t s)
{
    const int stride = sign_stride(B), wpb = stride < 4 ? stride : 4;
    hipLaunchKernelGGL((k_signs<IO>), dim3((unsigned)((n + 31) / 32), (unsigned)(stride / wpb)), dim3(64 * wpb), 0, s, n, B,
                       stride, x, signs, assign);
    return hipGetLastError();
}
hipError_t launch_signs_f32(int n, int B, const float *x, uint64_t *signs, uint32_t *assign, hipStream_t s)
{
    return signs_impl<float>(n, B, x, signs, assign, s);
}
hipError_t launch_signs_f64(int n, int B, const double *x, uint64_t *signs, uint32_t *assign, hipStream_t s)
{
    return signs_impl<double>(n, B, x, signs, assign, s);
}

// Groups of 64 constraints per wave: as many as still leave about four waves
// per SIMD (a restart's words of neighbouring groups share a 32-byte sector).
static int check_groups(int m, int stride)
{
    const int64_t waves = (int64_t)((m + 63) / 64) * stride;
    return (int)(waves >= 4096 * CHECK_GROUPS ? CHECK_GROUPS : (waves + 4095) / 4096);
}

int check_rows(int m, int B, int n_long)
{
    const int per = 64 * check_groups(m, sign_stride(B));
    return (m + per - 1) / per + (n_long + CHECK_LONG_PER - 1) / CHECK_LONG_PER;
}

hipError_t launch_check(CheckArgs a, const int32_t *list, int n_long, hipStream_t s)
{
    const int wpb = a.stride < 4 ? a.stride : 4;
    a.gpw = check_groups(a.m, a.stride);
    const int blocks = (a.m + 64 * a.gpw - 1) / (64 * a.gpw), gy = a.stride / wpb;
    hipError_t e = hipSuccess;
    if (a.U != nullptr && gy > 1 && (e = launch_fill_i32(a.U, a.m, 0, s)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_check_short, dim3((unsigned)blocks, (unsigned)gy), dim3(64 * wpb), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess || n_long == 0) return e;
    hipLaunchKernelGGL(k_check_long, dim3((unsigned)((n_long + CHECK_LONG_PER - 1) / CHECK_LONG_PER), (unsigned)gy),
                       dim3(64 * wpb), 0, s, a, list, n_long, blocks);
    return hipGetLastError();
}

}  // namespace ffsat
