// The grouped launch of the FP64 evaluation's root-of-unity bins.
#include "group64_kernel.h"

namespace ffsat {

hipError_t launch_eval_group64_f64(const EvalArgs<double> &a, const GroupEntry *ent, const int2 *blk, int nblk,
                                   size_t lds, hipStream_t s)
{
    return launch_group64<double>(a, ent, blk, nblk, lds, s);
}

}  // namespace ffsat
