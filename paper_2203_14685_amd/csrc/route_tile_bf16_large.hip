// Tiled bf16 route kernel, 65 to 256 experts.
#include "route_tile_bf16.hpp"

namespace hetumoe {

hipError_t launch_route_tile_bf16_small(const RouteArgs& a, hipStream_t st);

hipError_t launch_route_tile_bf16(const RouteArgs& a, hipStream_t st) {
  if (a.E <= 64) return launch_route_tile_bf16_small(a, st);
  if (tile_two_per_cu(a) && a.E <= 96) return tile_by_gate(a, TileBf16Launch<6, 4, 2, 64, 1, true>{a, st});
  if (tile_two_per_cu(a) && a.E <= 128) return tile_by_gate(a, TileBf16Launch<8, 4, 2, 64, 1, true>{a, st});
  if (a.E <= 96) return tile_by_gate(a, TileBf16Launch<6, 4, 2, 128, 1, false>{a, st});
  if (a.E <= 128) return tile_by_gate(a, TileBf16Launch<8, 4, 4, 128, 1, false>{a, st});
  if (a.E <= 192) return tile_by_gate(a, TileBf16Launch<12, 2, 4, 64, 2, false>{a, st});
  if (a.zsplit == 1) return tile_by_gate(a, TileBf16Launch<16, 2, 8, 64, 1, true>{a, st});
  return tile_by_gate(a, TileBf16Launch<16, 2, 8, 64, 1, false>{a, st});
}

bool route_uses_tile_bf16(const RouteArgs& a) { return a.dtype == 1 && tile_shape(a); }

TileSplit route_tile_split(int S, int d, int E, int dtype) {
  // one block per CU of a whole gfx950; a constant, so that the workspace size and
  // with it a batch's logits are the same on every device and need no device query
  constexpr int kBlocks = 256;
  constexpr int kRange = 256;   // columns: whole stages of every tile shape
  if (E > kTileMaxE || route_mfma_rs_shape(dtype, E, d)) return {1, d > 0 ? d : 1};
  const int nb = (S + kTileTok - 1) / kTileTok;
  int z = nb > 0 ? kBlocks / nb : 1;
  z = z < 16 ? z : 16;
  z = z < d / kRange ? z : d / kRange;
  if (z < 2) return {1, d > 0 ? d : 1};
  const int cols = ((d + z - 1) / z + kRange - 1) / kRange * kRange;
  return {(d + cols - 1) / cols, cols};
}

}  // namespace hetumoe
