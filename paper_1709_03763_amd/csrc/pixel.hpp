// Pixel index of a projection; plain C++ as well, so that it is checked on the
// host.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define SC_HOST_DEVICE __host__ __device__
#else
#define SC_HOST_DEVICE
#endif

namespace sc {

// v W + u of the pixel (u, v) that two whole FP32 numbers name.  In integers:
// FP32 holds whole numbers up to 2^24 only, and an image up to 2^28 pixels.
// Both factors fit 24 bits, which the masks say: one full-rate multiplication.
// A fused multiply-add in FP32 and one conversion, exact for images of up to
// 2^24 pixels alone, is one vector instruction of 86 a voxel test less: voxel
// pass of 400 operations 1.984 ms, with integers 2.003.
SC_HOST_DEVICE inline uint32_t pixel_index(float u, float v, uint32_t width)
{
    return ((uint32_t)v & 0xFFFFFFu) * (width & 0xFFFFFFu) + (uint32_t)u;
}

}  // namespace sc
