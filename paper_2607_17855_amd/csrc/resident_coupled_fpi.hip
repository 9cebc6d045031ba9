// FPI instantiations of the register-resident kernel for general B-dependency
// lists.
#include "resident_kernel.h"

namespace bi {
namespace res {

const void *fpi_coupled(int shape)
{
    static const void *const tab[] = {
#define BI_X(r, c) (const void *)filter_kernel<r, c, false>,
        BI_RES_SHAPES(BI_X, BI_X)
#undef BI_X
    };
    return tab[shape];
}

}  // namespace res
}  // namespace bi
