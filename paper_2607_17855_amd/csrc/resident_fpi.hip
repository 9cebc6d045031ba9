// FPI instantiations of the register-resident kernel (a file of its own, so
// the shapes of the three algorithms compile side by side).
#include "resident_kernel.h"

namespace bi {
namespace res {

const void *fpi_kernel(int shape)
{
    static const void *const tab[] = {
#define BI_X(r, c) (const void *)filter_kernel<r, c, true>,
        BI_RES_SHAPES(BI_X, BI_X)
#undef BI_X
    };
    return tab[shape];
}

}  // namespace res
}  // namespace bi
