// device_math.hip -- functions of the device code that are pure integer or float
// arithmetic, built for the host (test infrastructure).
#include "gap_diag.hpp"

extern "C" int dm_wrap_cell(int c, int n) { return gap::wrap_cell(c, n); }
extern "C" int dm_spec_guess(float l) { return gap::spec_guess(l); }
