// pg_quotient.h -- the tracer's divisions by the majorant, on host and device.
#pragma once
#include <hip/hip_runtime.h>

#include <cfloat>
#include <cmath>

namespace pg {

// a / b, correctly rounded, with y = 1 / b correctly rounded: two Newton
// corrections of a y, each from an exact remainder (Markstein, "IA-64 and
// elementary functions", 2000, ch. 8).  Five operations instead of a division
// of its own.  y, a and the quotient have to be finite: where a y overflows, the
// corrections make it NaN (walked_majorant keeps b from there).
__host__ __device__ __forceinline__ double div_by(double a, double b, double y) {
    double q = a * y;
    q = fma(fma(-b, q, a), y, q);
    return fma(fma(-b, q, a), y, q);
}

// The majorant that the walks use.  One below the least positive float bounds only
// zeros (the extinctions are floats): nothing collides and every ray passes, as
// with 0.  From there up a step, at most 53 ln 2 / majorant, is far from overflow.
__host__ __device__ __forceinline__ double walked_majorant(double m) { return m < (double)FLT_TRUE_MIN ? 0.0 : m; }

}  // namespace pg
