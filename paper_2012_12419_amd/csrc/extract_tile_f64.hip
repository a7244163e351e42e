// extract_tile_f64.hip -- greedy extraction on tiles from FP64 values
// (extract_tile.hpp).
#include "extract_tile.hpp"

namespace mdpvi {

bool extract_tile_shape_f64(const Model& M, TileShape* S) { return extract_tile_shape<double>(M, S); }
hipError_t launch_extract_tile_f64(const Model& M, const TileShape& S, const double* V, uint8_t* pi, float* gap,
                                   hipStream_t s) {
  return launch_extract_tile_t<double>(M, S, V, pi, gap, s);
}

}  // namespace mdpvi
