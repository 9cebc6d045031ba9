// VMP instantiations of the register-resident window kernel.
#include "resident_window.h"

namespace bi {
namespace res {

const void *vmp_kernel(int shape, bool one) { return window_of<BI_ALGO_VMP>(shape, one); }

}  // namespace res
}  // namespace bi
