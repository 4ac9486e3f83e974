// kernels.hpp -- the compiled sweep kernels by precision, tile shape, kernel variant and cache
// policy.  Each function returns the kernel and its block size (nullptr: no such tile shape).  They
// are defined in files of their own (kernels_*.hip), which the build compiles side by side.
#pragma once

#include "../../include/skyr.h"
#include "shapes.hpp"

namespace skyr {

// step sweep of one field
const void* step_kernel(skyr_precision prec, int variant, int ext, int stream, int& threads);
// gradient / observables sweep of one field
const void* grad_kernel(skyr_precision prec, int variant, int ext, int& threads);
// step sweep of a batch's fields (cache policy STREAM_NONE or STREAM_STORES)
const void* batch_kernel(skyr_precision prec, int variant, int ext, int stream, int& threads);
// printed-form sweep of one field (ext: the extra potentials or the gradient flow; groups: the steps of
// every slab's march are whole groups of five)
const void* printed_kernel(skyr_precision prec, int mode, bool ext, int stream, bool groups, int& threads);

// per precision, in files of their own
template <typename T> const void* step_kernel_of(int variant, int ext, int stream, int& threads);
template <typename T> const void* batch_kernel_of(int variant, int ext, int stream, int& threads);

}  // namespace skyr
