// Gate kernels for gfx950: step 1 of Algorithm 1 (logit projection, softmax,
// expert selection) and the capacity rule of Sec. 3.1 (each expert keeps at
// most C assignments, handed out rank-major then in token order).
//
// Launches, all on the caller's stream:
//   route   logits (the projection x.W of Eq. 1), selection (top-k list,
//           per-group top-1, hierarchical top-k, or hash), softmax weights, and
//           for every 64-token "wave block" a histogram of its (rank, expert)
//           pairs.  Variants:
//             route_mfma_rs_kernel  bf16, W held in registers (E in {16, 32, 64,
//                                128}, d in {512, 1024, 2048}, d * E up to
//                                128 K): persistent;
//             route_tile_bf16_kernel, route_tile_f32_kernel  any E up to 256 and
//                                any d: x and W staged per K stage; batches that
//                                leave CUs idle split K over blocks, and
//                                select_rows_kernel adds the partial logits and
//                                selects (it also serves given logits);
//             route_valu_kernel  more experts, or W not 16-byte aligned: one
//                                thread per token;
//             route_hash_kernel  the hash gate (no projection).
//   group_scan (large histograms only), assign: the slots of the capacity rule
//           (slots.hip).
#include <atomic>

#include "select.hpp"

namespace hetumoe {

// ---------------------------------------------------------------- hash route
// SplitMix64 (Steele, Lea & Flood, OOPSLA 2014): output number n of the
// generator seeded with `seed` is the mixing function applied to seed + n*gamma.
__device__ __forceinline__ uint64_t splitmix64_output(uint64_t seed, uint64_t n) {
  uint64_t z = seed + n * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__global__ __launch_bounds__(kBlock) void route_hash_kernel(RouteArgs a) {
  extern __shared__ int hist_lds[];  // [kWavesPerBlock][E]
  const int tid = threadIdx.x;
  const int w = tid / kWave;
  const int64_t s = static_cast<int64_t>(blockIdx.x) * kBlock + tid;
  const bool valid = s < a.S;
  if (valid) {
    const int32_t tid32 = a.token_ids[s];
    int e;
    if (a.hash_table) {
      // table lookup (balanced assignment); ids outside the table or table
      // entries outside [0, E) are out of contract and fold into [0, E)
      const int32_t v = (tid32 >= 0 && tid32 < a.hash_vocab) ? a.hash_table[tid32] : tid32;
      e = ((v % a.E) + a.E) % a.E;
    } else {
      const uint64_t t = static_cast<uint64_t>(static_cast<int64_t>(tid32));
      e = static_cast<int>(splitmix64_output(a.hash_seed, t + 1ull) % static_cast<uint64_t>(a.E));
    }
    a.ids[s] = e;
    a.weights[s] = 1.f;
  }
  const int wb = blockIdx.x * kWavesPerBlock + w;
  wave_block_hist(hist_lds + w * a.E, wb < a.nb, s, valid, wb, a);
}

// ---------------------------------------------------------------- launchers
int device_cu_count() {
  // calls may come from several host threads: the cache is atomic (every
  // thread that fills an entry writes the same value)
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

#ifndef HETUMOE_ROUTE_VALU_ONLY
static bool route_uses_tile(const RouteArgs& a) { return route_uses_tile_bf16(a) || route_uses_tile_f32(a); }
bool route_splits(const RouteArgs& a) { return !route_uses_mfma_rs(a) && route_uses_tile(a); }
bool route_fuses_extended(const RouteArgs& a) { return route_uses_mfma_rs(a) || route_uses_tile(a); }
#else
bool route_splits(const RouteArgs&) { return false; }
bool route_fuses_extended(const RouteArgs&) { return false; }
#endif

hipError_t launch_route(const RouteArgs& a, hipStream_t st) {
  if (a.nb == 0) return hipSuccess;
  if (a.kind == 2) {
    const unsigned blocks = static_cast<unsigned>((a.nb + kWavesPerBlock - 1) / kWavesPerBlock);
    route_hash_kernel<<<dim3(blocks), dim3(kBlock), static_cast<size_t>(kWavesPerBlock) * a.E * sizeof(int), st>>>(a);
    return hipGetLastError();
  }
#ifndef HETUMOE_ROUTE_VALU_ONLY
  // matrix-core projections (a build with HETUMOE_ROUTE_VALU_ONLY defined, used
  // only to time the vector-ALU route against them, skips these)
  if (route_uses_mfma_rs(a)) return launch_route_mfma_rs(a, device_cu_count(), st);
  if (route_uses_tile_bf16(a)) return launch_route_tile_bf16(a, st);
  if (route_uses_tile_f32(a)) return launch_route_tile_f32(a, st);
#endif
  return a.dtype == 1 ? launch_route_valu_bf16(a, st) : launch_route_valu_f32(a, st);
}

}  // namespace hetumoe
