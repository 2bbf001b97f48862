// Device memory that a call is faster with and can do without.  The runtime's functions are arguments: the CPU test passes its own.
#pragma once

#include <cstddef>

namespace reslim {

// allocate(&p, bytes): whether there is as much.  Where there is not: null, and the error that the runtime keeps is taken from it, so that no
// later call of this thread reports it.
template <class Allocate, class ForgetError>
inline void *optional_memory(size_t bytes, Allocate allocate, ForgetError forget_error) {
  void *p = nullptr;
  if (allocate(&p, bytes)) return p;
  forget_error();
  return nullptr;
}

}  // namespace reslim
