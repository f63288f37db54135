// sweep_line_f1.hip -- line-per-lane solves for float state, degree 1.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_f1(bool diry, bool band, bool batch)
{
    return line_kernel<float, 1>(diry, band, batch);
}
}  // namespace iga
