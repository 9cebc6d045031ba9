// Instantiations of the streamed window kernel.
#include "resident_streamed.h"

namespace bi {
namespace res {

const void *vmp_streamed() { return (const void *)streamed_kernel<BI_ALGO_VMP>; }
const void *mmp_streamed() { return (const void *)streamed_kernel<BI_ALGO_MMP>; }

}  // namespace res
}  // namespace bi
