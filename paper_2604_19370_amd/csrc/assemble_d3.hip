// assemble_d3.hip -- right-hand-side kernels for double state, degree 3.
#include "assemble.h"

namespace iga {
const void *asm_kernel_d3(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<double, 3>(fuel, src, stk, batch);
}
}  // namespace iga
