// MMP instantiations of the register-resident window kernel (a file of its
// own, so the shapes of the three algorithms compile side by side).
#include "resident_kernel.h"

namespace bi {
namespace res {

const void *mmp_kernel(int shape, bool one)
{
    static const void *const tab[][2] = {
#define BI_X(r, c) {(const void *)window_kernel<BI_ALGO_MMP, r, c, false>, (const void *)window_kernel<BI_ALGO_MMP, r, c, true>},
        BI_RES_SHAPES(BI_X)
#undef BI_X
    };
    return tab[shape][one];
}

}  // namespace res
}  // namespace bi
