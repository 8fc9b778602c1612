// Launch functions of the byte kernel (byte_kernels.hip; a translation unit of its own, so that its instantiations compile
// beside the others).
#pragma once
#include "lut_byte.hpp"

namespace adapt_api {

// R = 8, 4 or 2 pixels per row slot; level 0 .. 4: see adapt::byte_epilogue
hipError_t launch_byte(const adapt::ByteParams &p, unsigned grid, int R, int level, hipStream_t s);

}  // namespace adapt_api
