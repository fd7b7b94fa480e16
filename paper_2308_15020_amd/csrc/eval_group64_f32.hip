// The grouped launch of the FP32 evaluation's FP64-arithmetic bins.
#include "group64_kernel.h"

namespace ffsat {

int group_variant64(int io, int seg, int L)
{
#define X(ID, S, LL) \
    if (seg == S && L == LL) return ID;
    FFSAT_GROUP64_SHAPES(X)
    if (io == IO_F32) return -1;
    FFSAT_GROUP64_SHORT(X)
#undef X
    return -1;
}

hipError_t launch_eval_group64_f32(const EvalArgs<float> &a, const GroupEntry *ent, const int2 *blk, int nblk,
                                   size_t lds, hipStream_t s)
{
    return launch_group64<float>(a, ent, blk, nblk, lds, s);
}

}  // namespace ffsat
