// FP64 products whose MFMA fragments are loaded straight from memory
// (frag_kernels.hip).
#pragma once

#include "common.h"

namespace rtcc3 {

// Row tiles of a segmented product over a block table sorted so that the
// entries of a run share their B operands (4 ints per tile: the run's first
// entry, its entries, the index of its first tile, its tiles).  The rows of a
// run's entries are numbered through, kFragRows of them per tile.
constexpr int kFragRows = 64;
constexpr int kFragRun = 64;  // most entries of a run

// The FP64 form of a segmented product (GemmDesc::seg, alpha = 1), plain store
// or atomic accumulation, with C contiguous rows of N0 elements at stride sCn1.
void frag_seg(const GemmDesc& g, const int* row_tiles, int nrt, hipStream_t s);

}  // namespace rtcc3
