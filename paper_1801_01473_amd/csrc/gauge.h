// Entries shared by the gauge-side translation units.
#pragma once

#include "common.h"

namespace lqcd {

// F = (or +=) the gauge force with every staple multiplied out per link.
int gauge_force_direct(const KGeom& k, const double2* U, double beta, double c1, int accumulate,
                       double2* F, hipStream_t s);

// Block partials of S_g / beta, gauge_action_blocks(k) of them.
unsigned gauge_action_blocks(const KGeom& k);
int gauge_action_partials(const KGeom& k, const double2* U, double c1, double* part,
                          hipStream_t s);

}  // namespace lqcd
