// Table of the register-resident window kernels, shared by their two
// instantiating files (resident_vmp.hip, resident_mmp.hip: files of their own,
// so the algorithms compile side by side).
#pragma once

#include "resident_kernel.h"

namespace bi {
namespace res {

template <int ALGO>
const void *window_of(int shape, bool one)
{
    static const void *const tab[][2] = {
#define BI_X(r, c) {(const void *)window_kernel<ALGO, r, c, false>, (const void *)window_kernel<ALGO, r, c, true>},
#define BI_F(r, c) {nullptr, nullptr},
        BI_RES_SHAPES(BI_X, BI_F)
#undef BI_F
#undef BI_X
    };
    return tab[shape][one];
}

}  // namespace res
}  // namespace bi
