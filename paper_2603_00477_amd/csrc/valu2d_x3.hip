// VALU 2D kernel instances: float storage, double arithmetic.  The compensated
// mode runs on the matrix path; these redo its Dirichlet bands.
#include "valu2d_impl.h"

namespace stl {
const std::vector<KernelEntry> &valu2d_table_x3()
{
    static const std::vector<KernelEntry> table = {V2_BAND_S(float, double, STENCIL_F32_BF16X3)};
    return table;
}
}  // namespace stl
