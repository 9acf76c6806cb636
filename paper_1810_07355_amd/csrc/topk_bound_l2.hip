// The bound and filter kernels of topk_bound.h for f32 rows, squared L2.
#include "topk_bound.h"

namespace onng {
namespace topk_detail {

const void *topk_bound_fn_l2(int nch, int rw, bool bound) {
    return topk_bound_fn<ONNG_F32, ONNG_L2SQ>(nch, rw, bound);
}

}  // namespace topk_detail
}  // namespace onng
