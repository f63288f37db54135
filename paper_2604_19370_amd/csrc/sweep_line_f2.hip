// sweep_line_f2.hip -- line-per-lane solves for float state, degree 2.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_f2(bool diry, bool band, bool batch)
{
    return line_kernel<float, 2>(diry, band, batch);
}
}  // namespace iga
