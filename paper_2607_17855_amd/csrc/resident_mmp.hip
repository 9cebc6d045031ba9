// MMP instantiations of the register-resident window kernel.
#include "resident_window.h"

namespace bi {
namespace res {

const void *mmp_kernel(int shape, bool one) { return window_of<BI_ALGO_MMP>(shape, one); }

}  // namespace res
}  // namespace bi
