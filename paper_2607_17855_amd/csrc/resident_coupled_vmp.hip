// VMP instantiations of the register-resident window kernel for general
// B-dependency lists.
#include "resident_coupled.h"

namespace bi {
namespace res {

template <int I, int R, int C, bool LT>
static const void *pick(bool one)
{
    static_assert(kShapes[I].rb == R && kShapes[I].cb == C, "shape");
    return one ? (const void *)coupled_kernel<BI_ALGO_VMP, R, C, true, LT>
               : (const void *)coupled_kernel<BI_ALGO_VMP, R, C, false, LT>;
}

const void *vmp_coupled(int shape, bool one, bool lds_tab)
{
    if (lds_tab) {
        switch (shape) {
#define BI_X(i, r, c) \
    case i: return pick<i, r, c, true>(one);
            BI_RES_COUPLED(BI_X)
#undef BI_X
        }
    } else {
        switch (shape) {
#define BI_X(i, r, c) \
    case i: return pick<i, r, c, false>(one);
            BI_RES_COUPLED_PACKED(BI_X)
#undef BI_X
        }
    }
    return nullptr;
}

}  // namespace res
}  // namespace bi
