// Kernels of the message-passing initialiser: a learned proposal of restart
// points over the clause-variable incidence graph (3 rounds of messages,
// hidden width H, BF16 matrix-core products with FP32 accumulation).
//
//  * k_gemm: C = op(A) op(B) on the matrix cores (gfx950's
//    v_mfma_f32_32x32x16 bf16, 16 reduction terms per instruction): one
//    wave per 32x32 tile of C, operands read as FP32 (two 16-byte loads per
//    lane where the reduction dimension is contiguous and aligned) and
//    rounded to bfloat16 (round to nearest even) in registers, FP32
//    accumulators; optional split of the reduction dimension into fixed
//    slices (summed in a fixed order afterwards), bias + ReLU epilogue.
//  * k_gather: per-row weighted sums over the incidence (both directions),
//    used for the messages and for their transposes in the backward pass.
//  * head (tanh of a dot product), loss, column sums, Adam, proposals.
#include "mpnn_internal.h"

namespace ffsat {

typedef short __attribute__((ext_vector_type(8))) s16x8_t;
typedef __bf16 __attribute__((ext_vector_type(8))) bf16x8_t;
typedef float __attribute__((ext_vector_type(16))) f32x16_t;

__device__ __forceinline__ short to_bf16(float f)
{
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (short)(u >> 16);
}

// The 8 values of a lane's share of one 16-term block: p[0..7] when the
// block lies inside [.., lim) and contiguous rows may be read as two
// aligned 16-byte loads (vec), else element by element with stride st,
// zero past lim.
__device__ __forceinline__ void load8(const float *p, size_t st, int k, int lim, bool ok, bool vec, float (&v)[8])
{
    if (ok && vec && k + 8 <= lim) {
        const float4 x0 = *reinterpret_cast<const float4 *>(p);
        const float4 x1 = *reinterpret_cast<const float4 *>(p + 4);
        v[0] = x0.x; v[1] = x0.y; v[2] = x0.z; v[3] = x0.w;
        v[4] = x1.x; v[5] = x1.y; v[6] = x1.z; v[7] = x1.w;
    } else {
#pragma unroll
        for (int q = 0; q < 8; ++q) v[q] = (ok && k + q < lim) ? p[(size_t)q * st] : 0.f;
    }
}
__device__ __forceinline__ s16x8_t round8(const float (&v)[8])
{
    s16x8_t r;
#pragma unroll
    for (int q = 0; q < 8; ++q) r[q] = to_bf16(v[q]);
    return r;
}

// C[M][N] (ldc) = sum over k in this block's slice of opA[i][k] * opB[k][j]
//   opA[i][k] = TA ? A[k*lda + i] : A[i*lda + k]
//   opB[k][j] = TB ? B[j*ldb + k] : B[k*ldb + j]
// EPI 0: C (+ slice * slice_stride) = acc; EPI 1: C = relu(acc + bias[j]).
// One 32x32x16 instruction per 16 reduction terms: lane l supplies the 8
// terms k0 + 8*(l/32) + v (v = 0..7) of row l % 32 of opA and of column
// l % 32 of opB (the same k for both operands, so the sum covers the block
// whatever order the unit takes them in), and holds
// D[8*(q/4) + 4*(l/32) + q%4][l % 32], q = 0..15.  vec_a / vec_b: the
// contiguous operand (opA rows for !TA, opB columns for TB) may be read as
// 16-byte loads (base 16-byte aligned, leading dimension a multiple of 4;
// slices and blocks start at multiples of 16).
// Bound by the latency of the operand loads (a wave has one tile and few
// neighbours).  TN products, whose loads are single elements, issue those of
// four instructions together: at 8700 rows, H = 64 the weight product took 24 us
// in 17 slices of one instruction at a time and takes 8 us in 64 slices of
// four.  The forward product reads wide and is faster one at a time (9.9
// against 11.5 us).
// colsum (TN products, EPI 0): the blocks of the first row tile also add the
// columns of opB over the slice in FP32 and write them as row M of C (a
// layer's bias gradient beside its weight gradient; it took a pass of its own).
template <bool TA, bool TB, int EPI>
__device__ __forceinline__ void gemm_tile(const GemmArgs &g, const float *__restrict__ A, const float *__restrict__ B,
                                          const float *__restrict__ bias, const int block)
{
    const int M = g.M, N = g.N, K = g.K, lda = g.lda, ldb = g.ldb, ldc = g.ldc, vec_a = g.vec_a, vec_b = g.vec_b;
    const int colsum = g.colsum;
    const size_t slice_stride = g.slice_stride;
    float *C = g.C;
    const int bx = block % g.gx, by = block / g.gx % g.gy, bz = block / (g.gx * g.gy);
    const int l = threadIdx.x;
    const int i0 = bx * 32, j0 = by * 32;
    const int kb = bz * g.kslice;
    const int ke = min(K, kb + g.kslice);
    const int ai = i0 + (l & 31);
    const int bj = j0 + (l & 31);
    const int kh = 8 * (l >> 5);
    const bool aok = ai < M, bok = bj < N;
    f32x16_t acc;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.f;
    constexpr int GEMM_STEPS = TA ? 4 : 1;
    float cs = 0.f;
    for (int k0 = kb; k0 < ke; k0 += 16 * GEMM_STEPS) {
        float a[GEMM_STEPS][8], b[GEMM_STEPS][8];
#pragma unroll
        for (int u = 0; u < GEMM_STEPS; ++u) {
            const int k = k0 + 16 * u + kh;
            if (TA) load8(A + (size_t)k * lda + ai, (size_t)lda, k, ke, aok, false, a[u]);
            else load8(A + (size_t)ai * lda + k, 1, k, ke, aok, vec_a != 0, a[u]);
            if (TB) load8(B + (size_t)bj * ldb + k, 1, k, ke, bok, vec_b != 0, b[u]);
            else load8(B + (size_t)k * ldb + bj, (size_t)ldb, k, ke, bok, false, b[u]);
        }
#pragma unroll
        for (int u = 0; u < GEMM_STEPS; ++u) {
            if (TA && colsum) {
#pragma unroll
                for (int q = 0; q < 8; ++q) cs += b[u][q];
            }
            if (k0 + 16 * u < ke)   // uniform
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, round8(a[u])),
                                                              __builtin_bit_cast(bf16x8_t, round8(b[u])), acc, 0, 0, 0);
        }
    }
    const int j = j0 + (l & 31);
    if (TA && colsum) cs += __shfl_xor(cs, 32, 64);
    if (j >= N) return;
    if (TA && colsum && bx == 0 && l < 32) C[bz * slice_stride + (size_t)M * ldc + j] = cs;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int i = i0 + 8 * (q >> 2) + 4 * (l >> 5) + (q & 3);
        if (i >= M) continue;
        if constexpr (EPI == 0) {
            C[bz * slice_stride + (size_t)i * ldc + j] = acc[q];
        } else {
            const float y = acc[q] + bias[j];
            C[(size_t)i * ldc + j] = y > 0.f ? y : 0.f;
        }
    }
}

template <bool TA, bool TB, int EPI>
__global__ __launch_bounds__(64) void k_gemm(GemmArgs g, const float *__restrict__ A, const float *__restrict__ B,
                                             const float *__restrict__ bias)
{
    gemm_tile<TA, TB, EPI>(g, A, B, bias, (int)blockIdx.x);
}

// Two independent products in one launch (a layer's weight gradient and the
// gradient of its input; the two input layers): each fills a part of the chip
// for about the time of one round of loads.  At n = 2000, 8700 constraints, H = 64
// a weight product took 8.3 us and the input's 5.7 after it, both together 10.
template <bool TA, bool TB, int EPI, bool TA1, bool TB1, int EPI1>
__global__ __launch_bounds__(64) void k_gemm2(GemmArgs g, const float *__restrict__ A, const float *__restrict__ B,
                                              const float *__restrict__ bias, GemmArgs g1, const float *__restrict__ A1,
                                              const float *__restrict__ B1, const float *__restrict__ bias1, int blocks)
{
    const int block = (int)blockIdx.x;
    if (block < blocks) gemm_tile<TA, TB, EPI>(g, A, B, bias, block);
    else gemm_tile<TA1, TB1, EPI1>(g1, A1, B1, bias1, block - blocks);
}

// Reduction terms per slice when K is split `splits` ways: whole 16-term
// blocks of the matrix-core instruction.
static int gemm_kslice(int K, int splits)
{
    splits = splits < 1 ? 1 : splits;
    const int kslice = (K + splits - 1) / splits;
    return std::max(16, ((kslice + 15) / 16) * 16);
}

int gemm_slices(int K, int splits)
{
    const int kslice = gemm_kslice(K, splits);
    return std::max(1, (K + kslice - 1) / kslice);
}

GemmArgs gemm_args(bool ta, bool tb, int epi, int M, int N, int K, const float *A, int lda, const float *B, int ldb,
                   float *C, int ldc, const float *bias, int splits, size_t slice_stride)
{
    GemmArgs g{};
    g.M = M;
    g.N = N;
    g.K = K;
    g.A = A;
    g.lda = lda;
    g.B = B;
    g.ldb = ldb;
    g.C = C;
    g.ldc = ldc;
    g.bias = bias;
    g.slice_stride = slice_stride;
    g.kslice = epi == 1 ? ((K + 15) / 16) * 16 : gemm_kslice(K, splits);
    g.vec_a = !ta && ((uintptr_t)A % 16 == 0) && lda % 4 == 0;
    g.vec_b = tb && ((uintptr_t)B % 16 == 0) && ldb % 4 == 0;
    g.colsum = ta ? 1 : 0;
    g.gx = (M + 31) / 32;
    g.gy = (N + 31) / 32;
    g.blocks = M <= 0 || N <= 0 ? 0 : g.gx * g.gy * (epi == 0 ? gemm_slices(K, splits) : 1);
    return g;
}

hipError_t gemm_relu(const GemmArgs &g, hipStream_t s)
{
    if (g.blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_gemm<false, false, 1>), dim3((unsigned)g.blocks), dim3(64), 0, s, g, g.A, g.B, g.bias);
    return hipGetLastError();
}

template <bool TA, bool TB, int EPI, bool TA1, bool TB1, int EPI1>
static hipError_t launch_gemm2(const GemmArgs &g, const GemmArgs &g1, hipStream_t s)
{
    if (g.blocks + g1.blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL((k_gemm2<TA, TB, EPI, TA1, TB1, EPI1>), dim3((unsigned)(g.blocks + g1.blocks)), dim3(64), 0, s, g,
                       g.A, g.B, g.bias, g1, g1.A, g1.B, g1.bias, g.blocks);
    return hipGetLastError();
}
hipError_t gemm_relu2(const GemmArgs &g, const GemmArgs &g1, hipStream_t s)
{
    return launch_gemm2<false, false, 1, false, false, 1>(g, g1, s);
}
hipError_t gemm_back(const GemmArgs &weights, const GemmArgs &input, hipStream_t s)
{
    return launch_gemm2<true, false, 0, false, true, 0>(weights, input, s);
}
hipError_t gemm_weights2(const GemmArgs &g, const GemmArgs &g1, hipStream_t s)
{
    return launch_gemm2<true, false, 0, true, false, 0>(g, g1, s);
}

// Per job: out[i] = sum_{s < S} part[s * stride + i] (fixed order); entries
// from len on go to tail.  One launch for all of a backward pass: bound by the
// latency of one round of loads, which each gradient paid on its own (nine
// launches of 5.3 us, now one of 8).
__global__ __launch_bounds__(64) void k_sum_slices(SumJobs jobs)
{
    int q = 0;
    while (q + 1 < jobs.n && (int)blockIdx.x >= jobs.job[q + 1].block0) ++q;
    const SumJob &j = jobs.job[q];
    const int i = ((int)blockIdx.x - j.block0) * 64 + (int)threadIdx.x;
    if (i >= j.len + j.len_tail) return;
    float acc = 0.f;
#pragma unroll 16
    for (int s = 0; s < j.S; ++s) acc += j.part[(size_t)s * j.stride + i];
    if (i < j.len) j.out[i] = acc;
    else j.tail[i - j.len] = acc;
}

hipError_t sum_slices(SumJobs &jobs, hipStream_t s)
{
    int blocks = 0;
    for (int q = 0; q < jobs.n; ++q) {
        jobs.job[q].block0 = blocks;
        blocks += (jobs.job[q].len + jobs.job[q].len_tail + 63) / 64;
    }
    if (blocks > 0) hipLaunchKernelGGL(k_sum_slices, dim3((unsigned)blocks), dim3(64), 0, s, jobs);
    jobs.n = 0;
    return hipGetLastError();
}

// Weighted incidence sums, one wave per destination row, lanes over the H
// features.  Row r owns edges e = row_ptr[r] .. row_ptr[r+1] with source row
// src_of[e], weight w[e] and the sign of literal lit[e].
//  MODE 0 (messages):  dst[r][H + f] = sum over positive edges of w * src[src][f]
//                      dst[r][2H + f] = sum over negative edges
//                      dst[r][f] = own[r * ostride + f] (the row's own state)
//  MODE 1 (transposes): dst[r][f] = own[r * ostride + f] + sum_e w * src[src][(pos ?
//                      1 : 2) H + f] where y[r][f] > 0, else 0 (own: the row's
//                      own columns of the product's result, or null; y: the
//                      layer's output, whose ReLU is taken back here)
// The metadata of up to 64 edges is loaded lane-parallel (one edge per lane)
// and broadcast with readlane, so that the feature loads of eight consecutive
// edges do not wait on each other's index loads; the terms are added in edge
// order.
template <int MODE>
__global__ __launch_bounds__(256) void k_gather(int rows, int H, const int32_t *__restrict__ row_ptr,
                                                const int32_t *__restrict__ src_of, const int32_t *__restrict__ lit,
                                                const float *__restrict__ w, const float *__restrict__ src, int sstride,
                                                float *dst, int dstride, const float *__restrict__ own, int ostride,
                                                const float *__restrict__ y)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = blockIdx.x * (blockDim.x >> 6) + wave;
    if (r >= rows) return;
    const int lane = threadIdx.x & 63;
    const int e0 = row_ptr[r], e1 = row_ptr[r + 1];
    for (int f0 = 0; f0 < H; f0 += 64) {
        const int f = f0 + lane;
        const bool fin = f < H;
        const int fc = fin ? f : 0;
        const float ow = own != nullptr ? own[(size_t)r * ostride + fc] : 0.f;
        const float yv = MODE == 1 ? y[(size_t)r * H + fc] : 0.f;
        float ap = 0.f, an = 0.f;
        for (int eb = e0; eb < e1; eb += 64) {
            const int e = eb + lane;
            int so = 0, pos = 1;
            float we = 0.f;
            if (e < e1) {
                pos = lit[e] >= 0 ? 1 : 0;
                // element offset of the feature row this edge reads
                so = src_of[e] * sstride + (MODE == 0 ? 0 : (pos ? H : 2 * H));
                we = w[e];
            }
            const int cnt = min(64, e1 - eb);
            constexpr int NQ = 8;
            // past the last edge: a null edge (row 0, weight 0) is loaded and not added
            for (int q = 0; q < cnt; q += NQ) {
                float v[NQ], wq[NQ];
                int pq[NQ];
#pragma unroll
                for (int t = 0; t < NQ; ++t) {
                    const int o = __builtin_amdgcn_readlane(so, q + t);
                    pq[t] = __builtin_amdgcn_readlane(pos, q + t);
                    wq[t] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, we), q + t));
                    v[t] = src[(size_t)o + fc];
                }
#pragma unroll
                for (int t = 0; t < NQ; ++t) {
                    if (q + t < cnt) {   // uniform
                        if (MODE == 1 || pq[t]) ap += wq[t] * v[t];
                        else an += wq[t] * v[t];
                    }
                }
            }
        }
        if (!fin) continue;
        float *o = dst + (size_t)r * dstride + f;
        if (MODE == 0) {
            o[0] = ow;
            o[H] = ap;
            o[2 * H] = an;
        } else {
            const float g = ow + ap;
            o[0] = yv > 0.f ? g : 0.f;
        }
    }
}

hipError_t gather(int mode, int rows, int H, const int32_t *row_ptr, const int32_t *src_of, const int32_t *lit,
                  const float *w, const float *src, int sstride, float *dst, int dstride, const float *own, int ostride,
                  const float *y, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)((rows + 3) / 4));
    if (mode == 0)
        hipLaunchKernelGGL(k_gather<0>, grid, dim3(256), 0, s, rows, H, row_ptr, src_of, lit, w, src, sstride, dst, dstride,
                           own, ostride, y);
    else
        hipLaunchKernelGGL(k_gather<1>, grid, dim3(256), 0, s, rows, H, row_ptr, src_of, lit, w, src, sstride, dst, dstride,
                           own, ostride, y);
    return hipGetLastError();
}

// dZ = dX[:, :H] * (Y > 0): the own columns of a product's result taken back
// through a ReLU
__global__ void k_relu_back(int64_t total, int H, float *dZ, const float *__restrict__ Y, const float *__restrict__ dx,
                            int dxstride)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int64_t r = i / H;
    const float g = dx[(size_t)r * dxstride + (i - r * H)];
    dZ[i] = Y[i] > 0.f ? g : 0.f;
}

hipError_t relu_back(int rows, int H, float *dZ, const float *Y, const float *dx, int dxstride, hipStream_t s)
{
    const int64_t total = (int64_t)rows * H;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_relu_back, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, total, H, dZ, Y, dx, dxstride);
    return hipGetLastError();
}

// head: z_v = h_v . wo + bo, mu_v = tanh(z_v); one wave per variable
__global__ __launch_bounds__(256) void k_head(int n, int H, const float *__restrict__ hv, const float *__restrict__ wo,
                                              const float *__restrict__ bo, float *mu)
{
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int v = blockIdx.x * (blockDim.x >> 6) + wave;
    if (v >= n) return;
    const int lane = threadIdx.x & 63;
    float acc = 0.f;
    for (int f = lane; f < H; f += 64) acc += hv[(size_t)v * H + f] * wo[f];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if (lane == 0) mu[v] = tanhf(acc + bo[0]);
}

hipError_t head(int n, int H, const float *hv, const float *wo, const float *bo, float *mu, hipStream_t s)
{
    hipLaunchKernelGGL(k_head, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, n, H, hv, wo, bo, mu);
    return hipGetLastError();
}

// head backward and loss: dz_v = 2 (mu - t) / n * (1 - mu^2), dZ_v = dz_v wo
// through the last layer's ReLU (y its output), loss terms (mu - t)^2 / n and
// dz into per-variable buffers.
__global__ void k_head_back(int n, int H, const float *__restrict__ mu, const float *__restrict__ t,
                            const float *__restrict__ wo, const float *__restrict__ y, float *dz, float *lterm,
                            float *dZ)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)n * H) return;
    const int v = (int)(i / H);
    const int f = (int)(i - (int64_t)v * H);
    const float d = mu[v] - t[v];
    const float g = 2.f * d / (float)n * (1.f - mu[v] * mu[v]);
    dZ[i] = y[i] > 0.f ? g * wo[f] : 0.f;
    if (f == 0) {
        dz[v] = g;
        lterm[v] = d * d / (float)n;
    }
}

hipError_t head_back(int n, int H, const float *mu, const float *t, const float *wo, const float *y, float *dz,
                     float *lterm, float *dZ, hipStream_t s)
{
    const int64_t total = (int64_t)n * H;
    hipLaunchKernelGGL(k_head_back, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, n, H, mu, t, wo, y,
                       dz, lterm, dZ);
    return hipGetLastError();
}

// Sums over the variables, partials per slice of `per` variables: column f < H
// dz_v h_v[f] (the head's weights), column H dz_v (its bias), column H + 1 the
// loss terms.  A block's four waves take a quarter of the slice each and add
// their partials in wave order (one wave per slice of 256 variables took 57 us
// at 2000 variables, bound by its chain of loads; 5 us so).
__global__ __launch_bounds__(256) void k_head_sums(int n, int H, const float *__restrict__ dz,
                                                   const float *__restrict__ lterm, const float *__restrict__ hv, int per,
                                                   float *part)
{
    __shared__ float sm[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int f = blockIdx.x * 64 + lane;
    const int v0 = blockIdx.y * per, v1 = min(n, v0 + per);
    const int q = (per + 3) / 4;
    const int a = v0 + wave * q, b = min(v1, a + q);
    float acc = 0.f;
    if (f < H) {
#pragma unroll 8
        for (int v = a; v < b; ++v) acc += dz[v] * hv[(size_t)v * H + f];
    } else if (f < H + 2) {
        const float *p = f == H ? dz : lterm;
#pragma unroll 8
        for (int v = a; v < b; ++v) acc += p[v];
    }
    sm[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && f < H + 2)
        part[(size_t)blockIdx.y * (H + 2) + f] = ((sm[0][lane] + sm[1][lane]) + sm[2][lane]) + sm[3][lane];
}

// job: out[0..H] = gradients of the head's weights and bias, *loss (optional)
hipError_t head_sums(int n, int H, const float *dz, const float *lterm, const float *hv, float *part, float *out,
                     float *loss, SumJobs &jobs, hipStream_t s)
{
    int slices = std::max(1, std::min(HEAD_SLICES, (n + 31) / 32));
    const int per = (n + slices - 1) / slices;
    slices = std::max(1, (n + per - 1) / per);
    hipLaunchKernelGGL(k_head_sums, dim3((unsigned)((H + 2 + 63) / 64), (unsigned)slices), dim3(256), 0, s, n, H, dz, lterm,
                       hv, per, part);
    jobs.job[jobs.n++] = SumJob{part, (size_t)(H + 2), H + 1, loss ? 1 : 0, slices, 0, out, loss};
    return hipGetLastError();
}

// Adam (Kingma & Ba 2015) on FP32 master weights; step t starts at 1.
__global__ void k_adam(int64_t P, float *w, const float *__restrict__ g, float *m1, float *m2, float lr, float b1,
                       float b2, float eps, float c1, float c2)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    w[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

hipError_t adam(int64_t P, float *w, const float *g, float *m1, float *m2, float lr, float b1, float b2, float eps,
                int step, hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, s, P, w, g, m1, m2, lr, b1, b2, eps, c1,
                       c2);
    return hipGetLastError();
}

__device__ __forceinline__ uint64_t splitmix64_m(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

// x[v][b] = clip(mu_v + sigma u, -1, 1) for b < nl, else u; u uniform in
// [-1, 1) from SplitMix64 of seed + (i+1) * golden gamma, i = v*B + b.
__global__ void k_propose(int64_t total, int B, int nl, const float *__restrict__ mu, float sigma, uint64_t seed,
                          float *x)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const int b = (int)(i % B);
    const int64_t v = i / B;
    const uint64_t r = splitmix64_m(seed + (uint64_t)(i + 1) * 0x9e3779b97f4a7c15ull);
    const float u = (float)(r >> 40) * (2.0f / 16777216.0f) - 1.0f;
    if (b < nl) x[i] = fminf(fmaxf(mu[v] + sigma * u, -1.f), 1.f);
    else x[i] = u;
}

hipError_t propose(int64_t total, int B, int nl, const float *mu, float sigma, uint64_t seed, float *x, hipStream_t s)
{
    hipLaunchKernelGGL(k_propose, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, total, B, nl, mu, sigma, seed,
                       x);
    return hipGetLastError();
}

}  // namespace ffsat

namespace ffsat {

__global__ void k_fill_f32(int64_t n, float *p, float v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t fill_f32(int64_t n, float *p, float v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, p, v);
    return hipGetLastError();
}

}  // namespace ffsat
