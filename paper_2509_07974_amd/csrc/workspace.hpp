// Workspace of a one-call estimate (host only, no device code).
#pragma once

#include <cstddef>

namespace fpcf4 {

// get(bytes) allocates and returns a status.  Asks for `total` bytes and, if
// that answers `none` (no memory), for the `base` that a request runs in at
// least; *bytes is what was asked for last.  A catalogue whose operand copies
// do not fit beside it is then still served, by the slower kernels.
template <typename Status, typename Get>
Status reserve(std::size_t total, std::size_t base, Status none, Get get, std::size_t* bytes) {
  *bytes = total;
  Status st = get(total);
  if (st == none && base < total) {
    *bytes = base;
    st = get(base);
  }
  return st;
}

}  // namespace fpcf4
