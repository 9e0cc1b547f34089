// The tiles of the MFMA GEMM that only products of a layer take (a source of their own: half of the kernels to compile).
#include "gemm_kernel.h"

namespace ds {

hipError_t launch_layer_tile(int tile, const GemmParams& p, bool nt, int splits, hipStream_t stream) {
  return launch_any<kFirstLayerTile>(tile, p, nt, splits, stream,
                                      std::make_integer_sequence<int, kNumTiles - kFirstLayerTile>());
}

}  // namespace ds
