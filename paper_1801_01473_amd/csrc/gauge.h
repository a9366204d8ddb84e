// Entry shared by the gauge-force translation units.
#pragma once

#include "common.h"

namespace lqcd {

// F = (or +=) the gauge force with every staple multiplied out per link.
int gauge_force_direct(const KGeom& k, const double2* U, double beta, double c1, int accumulate,
                       double2* F, hipStream_t s);

}  // namespace lqcd
