// Instantiations of the streamed window kernel.
#include "resident_streamed.h"

namespace bi {
namespace res {

const void *vmp_streamed(bool flip)
{
    return flip ? (const void *)streamed_kernel<BI_ALGO_VMP, true> : (const void *)streamed_kernel<BI_ALGO_VMP, false>;
}

const void *mmp_streamed(bool flip)
{
    return flip ? (const void *)streamed_kernel<BI_ALGO_MMP, true> : (const void *)streamed_kernel<BI_ALGO_MMP, false>;
}

}  // namespace res
}  // namespace bi
