// Tiled matrix-core route kernels: the logit projection x.W of Eq. 1 for any
// expert count up to 256 and any row length, with softmax and expert selection
// (Sec. 3.1) on the logits in LDS.  One block per 64-token wave block.
#pragma once

#include "select.hpp"

namespace hetumoe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kTileTok = 64;        // tokens per block: one wave block
constexpr int kTileMaxE = 256;      // experts served
constexpr int kTilePart = 2;        // kernel mode: one K range's partial sums, no selection
constexpr int kTileOob = 0x7ffffff0;  // offset past every buffer resource: loads return zeros

// gfx950's LDS transpose read (ds_read_b64_tr_b16): within each group of 16
// lanes, lane i receives element i % 4 of the four-element rows addressed by
// lanes i / 4 + 4 j, j = 0..3.
__device__ __forceinline__ uint2 lds_tr16(const uint16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p)));
}

// Where row k of 32 (a K step) lies in LDS: rows 8 g + 4 h + q, which one transpose
// read takes for g = 0..3 and q = 0..3, are 16 neighbours.  With a row stride of an
// odd multiple of 32 bytes any 8 neighbours' 32-byte pieces fill all 64 banks.
__device__ __forceinline__ int tr_row(int k) { return (k & ~31) | ((k & 4) << 2) | ((k >> 1) & 12) | (k & 3); }

__device__ __forceinline__ __amdgpu_buffer_rsrc_t tile_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ u32x4 tile_load(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}

// Row stride of the block's logits in LDS (floats): an odd multiple of 8, so
// that 8 tokens x 8 lanes reading consecutive experts touch 64 distinct banks.
constexpr int tile_lgs(int NT) { return 16 * NT + 8; }

// The block's logits (bias included) are in lg: noise and temperature, the
// caller's copy of the logits, selection by P lanes per token, histogram.
template <int THREADS, int KMAX, int MODE, int LGS>
__device__ __forceinline__ void tile_epilogue(const RouteArgs& a, float* lg, int* hist_lds) {
  constexpr int P = THREADS / kTileTok;
  constexpr int kWaves = THREADS / kWave;
  const int tid = threadIdx.x;
  const int E = a.E;
  const int64_t tok0 = static_cast<int64_t>(blockIdx.x) * kTileTok;
  for (int i = tid; i < a.k * E; i += THREADS) hist_lds[i] = 0;
  if (a.temperature > 0.f || a.logits) {
    // whole rows per wave: coalesced over the experts without a division
    const int lane = lane_id();
    for (int r = tid / kWave; r < kTileTok; r += kWaves) {
      const int64_t s = tok0 + r;
      if (s >= a.S) break;
      for (int e = lane; e < E; e += kWave) {
        float v = lg[r * LGS + e];
        if (a.temperature > 0.f) {
          if (a.noise) v += a.noise[s * E + e];
          v = v / a.temperature;
          lg[r * LGS + e] = v;
        }
        if (a.logits) a.logits[s * E + e] = v;
      }
    }
  }
  __syncthreads();
  const int t = tid / P, j = tid % P;
  const int64_t s = tok0 + t;
  select_row<P, KMAX, MODE>(lg + t * LGS, E, a.k, a.groups, a.normalize, j, s < a.S, a.ids + s * a.k,
                            a.weights + s * a.k, hist_lds);
  __syncthreads();
  for (int i = tid; i < a.k * E; i += THREADS) a.hist[static_cast<int64_t>(blockIdx.x) * a.k * E + i] = hist_lds[i];
}

// Where the block's partial sums of its K range go: its 64 rows of its plane.
__device__ __forceinline__ float* tile_plane(const RouteArgs& a) {
  return a.part + static_cast<int64_t>(blockIdx.y) * a.S * a.E + static_cast<int64_t>(blockIdx.x) * kTileTok * a.E;
}

// Instantiates Launch<KMAX, MODE> for the gate of `a`: sorted lists no longer
// than k needs (each logit's insertion walks all of them).
template <class Launch>
static hipError_t tile_by_gate(const RouteArgs& a, Launch launch) {
  if (a.part) return launch.template operator()<1, kTilePart>();
  if (a.kind == 1) return launch.template operator()<1, 1>();
  if (a.kind == 3) {
    if (a.k == 1) return launch.template operator()<1, 3>();
    if (a.k == 2) return launch.template operator()<2, 3>();
    if (a.k <= 4) return launch.template operator()<4, 3>();
    return launch.template operator()<8, 3>();
  }
  if (a.k == 1) return launch.template operator()<1, 0>();
  if (a.k == 2) return launch.template operator()<2, 0>();
  if (a.k <= 4) return launch.template operator()<4, 0>();
  return launch.template operator()<8, 0>();
}

// Shapes whose rows and W the tiled kernels can address and load in 16-byte
// pieces; W's rows may have any length, the matrix as a whole is read flat.
static inline bool tile_shape(const RouteArgs& a) {
  const int64_t elt = a.dtype == 1 ? 2 : 4;
  return a.kind != 2 && a.E <= kTileMaxE && a.d > 0 && a.d * elt % 16 == 0 &&
         a.d * elt * kTileMaxE < (int64_t(1) << 30) && (reinterpret_cast<uintptr_t>(a.x) % 16) == 0 &&
         (reinterpret_cast<uintptr_t>(a.wg) % 16) == 0;
}

}  // namespace hetumoe
