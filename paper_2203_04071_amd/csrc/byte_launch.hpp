// Launch functions of the byte kernel (byte_kernels.hip; a translation unit of its own, so that its instantiations compile
// beside the others).
#pragma once
#include "lut_byte.hpp"

namespace adapt_api {

// R = 8, 4 or 2 pixels per row slot; extra: see lut_byte_kernel
hipError_t launch_byte(const adapt::ByteParams &p, unsigned grid, int R, bool extra, hipStream_t s);

}  // namespace adapt_api
