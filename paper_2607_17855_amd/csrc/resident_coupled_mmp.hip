// MMP instantiations of the register-resident window kernel for general
// B-dependency lists.
#include "resident_coupled.h"

namespace bi {
namespace res {

const void *mmp_coupled(int shape, bool one, bool lds_tab) { return coupled_of<BI_ALGO_MMP>(shape, one, lds_tab); }

}  // namespace res
}  // namespace bi
