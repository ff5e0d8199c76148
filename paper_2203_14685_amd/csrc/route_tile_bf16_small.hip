// Tiled bf16 route kernel, up to 64 experts.
#include "route_tile_bf16.hpp"

namespace hetumoe {

hipError_t launch_route_tile_bf16_small(const RouteArgs& a, hipStream_t st) {
  if (tile_two_per_cu(a)) {
    if (a.E <= 16) return tile_by_gate(a, TileBf16Launch<1, 4, 1, 64, 1, true>{a, st});
    if (a.E <= 32) return tile_by_gate(a, TileBf16Launch<2, 4, 1, 64, 1, true>{a, st});
    if (a.E <= 48) return tile_by_gate(a, TileBf16Launch<3, 4, 1, 64, 1, true>{a, st});
    return tile_by_gate(a, TileBf16Launch<4, 4, 2, 64, 1, true>{a, st});
  }
  if (a.E <= 16) return tile_by_gate(a, TileBf16Launch<1, 4, 1, 128, 1, false>{a, st});
  if (a.E <= 32) return tile_by_gate(a, TileBf16Launch<2, 4, 2, 128, 1, false>{a, st});
  if (a.E <= 48) return tile_by_gate(a, TileBf16Launch<3, 4, 1, 128, 1, false>{a, st});
  return tile_by_gate(a, TileBf16Launch<4, 4, 4, 128, 1, false>{a, st});
}

}  // namespace hetumoe
