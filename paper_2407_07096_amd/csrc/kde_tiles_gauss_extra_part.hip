// Exact kernel density tiles, epilogue mode kModeGaussExtraPart (the Gaussian sums with the edge
// sampler's outputs
// in launches with several workgroups per chunk).
#include "kde_tiles.h"

namespace stag {

stag_status launch_tiles_gauss_extra_part(const Operands& xo, const Operands& qo, double* partial, const TileExtra& ex,
                               hipStream_t st) {
  return tiles::launch_tiles<tiles::kModeGaussExtraPart>(xo, qo, partial, ex, st);
}

}  // namespace stag
