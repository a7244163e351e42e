// extract_tile_f32.hip -- greedy extraction on tiles from FP32 values
// (extract_tile.hpp).
#include "extract_tile.hpp"

namespace mdpvi {

bool extract_tile_shape_f32(const Model& M, TileShape* S) { return extract_tile_shape<float>(M, S); }
hipError_t launch_extract_tile_f32(const Model& M, const TileShape& S, const float* V, uint8_t* pi, float* gap,
                                   hipStream_t s) {
  return launch_extract_tile_t<float>(M, S, V, pi, gap, s);
}

}  // namespace mdpvi
