// assemble_d1.hip -- right-hand-side kernels for double state, degree 1.
#include "assemble.h"

namespace iga {
const void *asm_kernel_d1(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<double, 1>(fuel, src, stk, batch);
}
}  // namespace iga
