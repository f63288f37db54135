// assemble_f2.hip -- right-hand-side kernels for float state, degree 2.
#include "assemble.h"

namespace iga {
const void *asm_kernel_f2(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<float, 2>(fuel, src, stk, batch);
}
}  // namespace iga
