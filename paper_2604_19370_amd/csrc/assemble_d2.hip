// assemble_d2.hip -- right-hand-side kernels for double state, degree 2.
#include "assemble.h"

namespace iga {
const void *asm_kernel_d2(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<double, 2>(fuel, src, stk, batch);
}
}  // namespace iga
