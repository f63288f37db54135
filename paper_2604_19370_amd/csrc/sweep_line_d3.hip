// sweep_line_d3.hip -- line-per-lane solves for double state, degree 3.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_d3(bool diry, bool band, bool batch)
{
    return line_kernel<double, 3>(diry, band, batch);
}
}  // namespace iga
