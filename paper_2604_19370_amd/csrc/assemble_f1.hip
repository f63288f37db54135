// assemble_f1.hip -- right-hand-side kernels for float state, degree 1.
#include "assemble.h"

namespace iga {
const void *asm_kernel_f1(bool fuel, bool src, bool stk, bool batch)
{
    return asm_kernel<float, 1>(fuel, src, stk, batch);
}
}  // namespace iga
