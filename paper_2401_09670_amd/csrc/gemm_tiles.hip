// The tiles of the MFMA GEMM for products of few row tiles (a source of their own: half of the kernels to compile).
#include "gemm_kernel.h"

namespace ds {

hipError_t launch_few_row_tile(int tile, const GemmParams& p, bool nt, int splits, hipStream_t stream) {
  return launch_any<kFirstFewRows>(tile, p, nt, splits, stream,
                                   std::make_integer_sequence<int, kNumTiles - kFirstFewRows>());
}

}  // namespace ds
