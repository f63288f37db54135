// sweep_line_d1.hip -- line-per-lane solves for double state, degree 1.
#include "sweep_line.h"

namespace iga {
const void *line_kernel_d1(bool diry, bool band, bool batch)
{
    return line_kernel<double, 1>(diry, band, batch);
}
}  // namespace iga
