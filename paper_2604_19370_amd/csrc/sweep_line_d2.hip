// sweep_line_d2.hip -- line-per-lane solves for double state, degree 2.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_d2(bool diry, bool band, bool batch)
{
    return line_kernel<double, 2>(diry, band, batch);
}
}  // namespace iga
