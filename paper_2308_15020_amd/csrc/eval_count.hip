// One bin per launch of the count form (count_kernel.h).
#include "count_kernel.h"

namespace ffsat {

template <int S, int L>
__global__ __launch_bounds__(256) void k_eval_count(EvalArgs<float> a, const float *__restrict__ xin,
                                                    const ConDesc *__restrict__ con, const int32_t *__restrict__ lits,
                                                    const float *__restrict__ wts)
{
    __shared__ float sm[L == 1 ? 1 : 4 * count_lds_floats<S, L>()];
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int unit = (int)blockIdx.x * (int)(blockDim.x >> 6) + wave;
    const Span sp{a.first, a.count, a.cpw, a.n_rb, a.fpart_row0};
    count_unit<S, L>(a, sp, unit, xin, con, lits, wts, sm + wave * count_lds_floats<S, L>());
}

using CountFn = void (*)(EvalArgs<float>, const float *, const ConDesc *, const int32_t *, const float *);

static CountFn count_fn(int seg, int L)
{
#define X(ID, S, LL) \
    if (seg == S && L == LL) return &k_eval_count<S, LL>;
    FFSAT_COUNT_SHAPES(X)
#undef X
    return nullptr;
}

bool count_variant_exists(int seg, int L) { return count_fn(seg, L) != nullptr; }

hipError_t launch_count_bin(const Bin &bin, const EvalArgs<float> &a, hipStream_t s)
{
    const CountFn fn = count_fn(bin.seg, bin.L);
    if (!fn || bin.wpb < 1 || bin.wpb > 4) return hipErrorInvalidValue;
    const int64_t units = (int64_t)((a.count + a.cpw - 1) / a.cpw) * a.n_rb;
    if (units <= 0) return hipSuccess;
    hipLaunchKernelGGL(fn, dim3((unsigned)((units + bin.wpb - 1) / bin.wpb)), dim3(64 * bin.wpb), 0, s, a, a.x, a.con, a.lit,
                       a.w);
    return hipGetLastError();
}

}  // namespace ffsat
