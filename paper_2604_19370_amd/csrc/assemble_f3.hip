// assemble_f3.hip -- right-hand-side kernels for float state, degree 3.
#include "assemble.h"

namespace iga {
const void *asm_kernel_f3(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<float, 3>(fuel, src, stk, batch);
}
}  // namespace iga
