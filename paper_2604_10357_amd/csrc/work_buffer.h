// work_buffer.h -- which form of the work buffer a float64 tangent pass takes
// (host logic only, no HIP: checked on the CPU).
#pragma once

#include <cstddef>

#include "../../include/tlfea.h"

namespace tlfea {

// Element rows are the faster form of a large mesh, but they may be larger than
// the point records (damped T10: 7.7 against 3.8 KB an element).  A buffer that
// holds the records of the mesh and not its rows stays as it is, and the pass
// with it: after a change of the material or the precision no call allocates
// where none of the forms before it needed more, and what was captured on the
// handle still names the same memory.
inline bool buffer_takes_rows(size_t rows, size_t records, size_t cap) {
  return cap >= rows || cap < records;
}

// Takes `need` bytes, or where the device does not have them the `smaller` form's:
// a mesh that fits with its point records runs with them.  take(bytes) returns a
// status.
template <class Take>
int take_buffer(size_t need, size_t smaller, Take&& take) {
  const int rc = take(need);
  return rc == TLFEA_ERR_NOMEM && smaller < need ? take(smaller) : rc;
}

}  // namespace tlfea
