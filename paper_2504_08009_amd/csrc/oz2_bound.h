// The product of the bound planes (Section 4.1) for its row and column maxima alone, in tiles of 64 or 128 (oz2_stage2_tiles.hip).
// oz2_bound_tile: 256 where the large kernel's product and a pass over it (oz2_launch_bound_gemm) are estimated the faster way.
#ifndef OZ2_BOUND_H
#define OZ2_BOUND_H

#include "oz2_internal.h"

int oz2_bound_tile(const Oz2Layout& lay, int64_t m, int64_t n, bool symmetric, int64_t cus);
hipError_t oz2_launch_bound_maxima(int tile, const Oz2Layout& lay, char* ws, int64_t m, int64_t n, bool symmetric,
                                   const Oz2ScanFinish& fin, hipStream_t st);

#endif
