// sweep_line_f3.hip -- line-per-lane solves for float state, degree 3.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_f3(bool diry, bool band, bool batch)
{
    return line_kernel<float, 3>(diry, band, batch);
}
}  // namespace iga
