// The bound and filter kernels of topk_bound.h for u8 rows.
#include "topk_bound.h"

namespace onng {
namespace topk_detail {

const void *topk_bound_fn_u8(int nch, int rw, bool bound) {
    return topk_bound_fn<ONNG_U8, ONNG_L2SQ>(nch, rw, bound);
}

}  // namespace topk_detail
}  // namespace onng
