// Grouped launches of the root-of-unity bins with FP64 arithmetic: those of the
// FP32 evaluation (k >= 128 by default; eval_group64_f32.hip) and those of the FP64
// evaluation (eval_group64_f64.hip), each in one grid over a host-built block
// table (build_groups, host.cpp): the ramp and tail of a launch are paid once
// instead of once per bin, and bins too small to fill the chip run together.
// (SEG, L): 14..32 at L = 16, 16, 20, 24 and 25..32 at L = 8; the FP64 evaluation also
// has the shorter shapes.  Compiled for 3 waves per SIMD (168 VGPRs): the
// variants of more than 28 positions spill a few per-constraint values, none in
// their frequency loops, and the grid runs faster than at the 2 waves their
// full register count would give (all k / 2 frequencies: 20%; with those chosen at
// the point 4.5%, 2725 against 2850 us an iteration of the large instance).  Bound
// by VALU issue: two thirds of the SIMD cycles issue one, 2.6 of the 3 waves resident;
// 1982 constraints of 128..512 literals, 256 restarts 4.62 ms -> 1.39.
#pragma once
#include "eval_kernel.h"

namespace ffsat {

#define FFSAT_GROUP64_SHAPES(X)                                                                           \
    X(0, 17, 16) X(1, 18, 16) X(2, 19, 16) X(3, 20, 16) X(4, 21, 16) X(5, 22, 16) X(6, 23, 16)           \
    X(7, 24, 16) X(8, 25, 16) X(9, 26, 16) X(10, 27, 16) X(11, 28, 16) X(12, 29, 16) X(13, 30, 16)       \
    X(14, 31, 16) X(15, 32, 16) X(16, 14, 16) X(17, 15, 16) X(18, 16, 16) X(19, 16, 8) X(20, 20, 8)      \
    X(21, 24, 8) X(22, 25, 8) X(23, 26, 8) X(24, 27, 8) X(25, 28, 8) X(26, 29, 8) X(27, 30, 8)          \
    X(28, 31, 8) X(29, 32, 8)
#define FFSAT_GROUP64_SHORT(X)                                                                            \
    X(30, 4, 1) X(31, 8, 1) X(32, 12, 1) X(33, 16, 1) X(34, 20, 1) X(35, 24, 1) X(36, 16, 2) X(37, 20, 2)  \
    X(38, 24, 2) X(39, 16, 4) X(40, 20, 4) X(41, 24, 4)

template <typename IO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_eval_group64(EvalArgs<IO> a, const IO *__restrict__ xin,
                                                      const ConDesc *__restrict__ con,
                                                      const int32_t *__restrict__ lits,
                                                      const float *__restrict__ wts,
                                                      const TypeT<double> *__restrict__ types,
                                                      const FreqT<double> *__restrict__ freqs,
                                                      const GroupEntry *__restrict__ ent,
                                                      const int2 *__restrict__ blk)
{
    extern __shared__ __align__(16) char group_lds[];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    __shared__ double stage[4 * wave_doubles<IO>(32)];   // FP32 points 40 KB: 3 blocks of 4 waves a CU, as the registers allow
    if (a.skip != nullptr && *a.skip == 0) return;   // before the block table: nothing else to wait for
    const int2 bw = blk[blockIdx.x];
    const GroupEntry e = ent[__builtin_amdgcn_readfirstlane(bw.x)];
    const Span sp{e.first, e.count, e.cpw, e.n_rb, e.fpart_row0};
    const int fg = e.fg;
    const int unit = fg > 1 ? bw.y : bw.y + wave;
    const int wg = fg > 1 ? wave : 0;
    double *own = stage + wave * wave_doubles<IO>(32);
    switch (e.variant) {
#define X(ID, S, LL)                                                                                          \
    case ID:                                                                                                  \
        eval_unit<IO, double, S, LL, true>(a, sp, unit, xin, con, lits, wts, types, freqs, fg, wg, group_lds, own); \
        break;
        FFSAT_GROUP64_SHAPES(X)
#undef X
#define X(ID, S, LL)                                                                                          \
    case ID:                                                                                                  \
        if constexpr (sizeof(IO) == 8)                                                                        \
            eval_unit<IO, double, S, LL, true>(a, sp, unit, xin, con, lits, wts, types, freqs, fg, wg, group_lds, own); \
        break;
        FFSAT_GROUP64_SHORT(X)
#undef X
    default: break;
    }
}

template <typename IO>
static hipError_t launch_group64(const EvalArgs<IO> &a, const GroupEntry *ent, const int2 *blk, int nblk, size_t lds,
                                 hipStream_t s)
{
    if (nblk <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_eval_group64<IO>, dim3((unsigned)nblk), dim3(256), lds, s, a, a.x, a.con, a.lit, a.w,
                       reinterpret_cast<const TypeT<double> *>(a.types),
                       reinterpret_cast<const FreqT<double> *>(a.freqs), ent, blk);
    return hipGetLastError();
}

}  // namespace ffsat
