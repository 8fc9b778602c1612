// Instantiations of the byte kernel (lut_byte.hpp) and their launch.
#include "byte_launch.hpp"

namespace adapt_api {

namespace {

template <int DOPS, int R>
void launch(const adapt::ByteParams &p, unsigned grid, int level, hipStream_t s) {
    if (level == 4) adapt::lut_byte_kernel<DOPS, R, 4><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else if (level == 3) adapt::lut_byte_kernel<DOPS, R, 3><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else if (level == 2) adapt::lut_byte_kernel<DOPS, R, 2><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else if (level == 1) adapt::lut_byte_kernel<DOPS, R, 1><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else adapt::lut_byte_kernel<DOPS, R, 0><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
}

template <int R>
void launch_r(const adapt::ByteParams &p, unsigned grid, int level, hipStream_t s) {
    if (p.copy_lines == 256) launch<4, R>(p, grid, level, s);
    else if (p.copy_lines == 128) launch<2, R>(p, grid, level, s);
    else launch<1, R>(p, grid, level, s);
}

}  // namespace

hipError_t launch_byte(const adapt::ByteParams &p, unsigned grid, int R, int level, hipStream_t s) {
    const bool at_once = R == 2 && p.copy_lines <= 64 && p.m_tiles == 1;       // (see lut_byte_kernel)
    if (at_once && level == 0) adapt::lut_byte_kernel<1, 2, 0, true><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else if (at_once && level == 4) adapt::lut_byte_kernel<1, 2, 4, true><<<grid, adapt::BYTE_THREADS, 0, s>>>(p);
    else if (R == 8) launch_r<8>(p, grid, level, s);
    else if (R == 4) launch_r<4>(p, grid, level, s);
    else launch_r<2>(p, grid, level, s);
    return hipGetLastError();
}

}  // namespace adapt_api
