// Byte offset of a bilinear cell's corner in an image of 32-bit pixels.  Plain
// C++, so that it also compiles for the host alone.
#pragma once

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define EBSD_HD __host__ __device__
#else
#define EBSD_HD
#endif

namespace ebsd {

// Corner (xf, yf), whole numbers, of an image with rows of row_bytes bytes, for
// images of more than 2^24 pixels (up to 16384 x 16384 px): there an index in FP32
// is rounded, to a neighbour's pixel, and past the image's end in its last rows.
// Rows of at most 64 KiB and their number fit 24 bits, so the product is one
// full-rate instruction.
EBSD_HD inline unsigned cell_offset(float xf, float yf, unsigned row_bytes)
{
    return ((unsigned)yf & 0xffffffu) * (row_bytes & 0xffffffu) + 4u * (unsigned)xf;
}

}  // namespace ebsd
