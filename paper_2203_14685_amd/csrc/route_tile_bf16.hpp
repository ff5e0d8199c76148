// Tiled bf16 route kernel (route_tile.hpp), instantiated per expert-tile count
// in route_tile_bf16_small.hip and route_tile_bf16_large.hip.
#pragma once

#include "route_tile.hpp"

namespace hetumoe {

// 64 tokens x E experts per block on v_mfma_f32_16x16x32_bf16 (M = tokens, N =
// experts, K = d), WM x WN waves, each 64 / WM tokens x 16 NT / WN experts.  Per
// stage of KC columns the block stages its rows of x as they are and the KC rows
// of W as they are: the KC x E piece of W is one contiguous piece of memory,
// read flat in 16-byte pieces whatever E is and written to padded LDS rows.  A
// fragments are 16-byte LDS reads of x, B fragments (8 consecutive K of one
// expert) transpose reads of W.  The next stage is loaded into registers while
// the current one is multiplied; columns past d and rows past the batch come
// from outside the buffer resources and are zeros.  Each kSum columns are summed on
// their own and then added to the running sum, so rounding grows with their number,
// not with d / 32.  Experts past E hold whatever LDS held: their columns are never
// read.  Sixteen waves and the longest stage that LDS holds twice: 8192 x 4096 x 128 with two K ranges 29 us (8 waves,
// stages of 64) -> 26, 32768 x 4096 x 128 whole gate 118 -> 97; the loads are not
// what bounds it (one or two stages ahead: the same), the operand reads from LDS
// are, the transpose reads above all.
// ONE: the launch has one K range, so no sum over ranges is held (at 16 tiles the
// registers it takes went to scratch), and at most 128 registers; with stages
// of 64 two blocks of eight waves share a CU then (tile_two_per_cu).  Same sums
// either way.
template <int NT, int WM, int WN, int KC, int DEPTH, bool ONE, int KMAX, int MODE>
__global__ __launch_bounds__(WM* WN * 64) __attribute__((amdgpu_waves_per_eu(ONE ? 4 : WM * WN / 4)))
void route_tile_bf16_kernel(RouteArgs a) {
  constexpr int THREADS = WM * WN * kWave;
  constexpr int MT = 4 / WM, NTW = NT / WN;  // 16 x 16 tiles per wave
  static_assert(MT * WM == 4 && NTW * WN == NT, "whole tiles per wave");
  constexpr int kSum = NT > 8 ? 64 : 128;              // columns summed on their own, whatever KC is
  constexpr int LDX = KC + 8;                          // row strides in LDS (bf16): x 16 bytes past
  constexpr int LDW = 16 * (NT + ((1 - NT) & 3));      // whole banks, W rows 32 bytes past 128
  constexpr int LGS = tile_lgs(NT);
  constexpr int XN = kTileTok * KC / 8;                // 16-byte pieces of x per stage
  constexpr int XP = (XN + THREADS - 1) / THREADS;     // and per thread
  constexpr int WP = (KC * 16 * NT / 8 + THREADS - 1) / THREADS;
  constexpr int kStage = (kTileTok * LDX + KC * LDW) * 2;
  constexpr int kLg = kTileTok * LGS * 4;
  __shared__ __align__(16) unsigned char raw[2 * kStage > kLg ? 2 * kStage : kLg];
  __shared__ int hist_lds[8 * 16 * NT];
  float* lg = reinterpret_cast<float*>(raw);  // after the K loop

  const int tid = threadIdx.x;
  const int w = tid / kWave, wm = w / WN, wn = w % WN;
  const int lane = lane_id();
  const int g = lane / 16, m = lane % 16;
  const int d = a.d, E = a.E;
  const int64_t tok0 = static_cast<int64_t>(blockIdx.x) * kTileTok;
  const int rows = static_cast<int>(min(static_cast<int64_t>(kTileTok), a.S - tok0));
  const __amdgpu_buffer_rsrc_t xsrc =
      tile_rsrc(reinterpret_cast<const uint16_t*>(a.x) + tok0 * d, static_cast<unsigned>(rows) * d * 2u);
  const __amdgpu_buffer_rsrc_t wsrc = tile_rsrc(a.wg, static_cast<unsigned>(d) * E * 2u);
  const int wcnt = KC * E / 8;  // pieces of W per stage

  // where each piece of W goes: row and column of its first element
  int wrow[WP], wcol[WP];
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int p = 8 * (tid + i * THREADS);
    wrow[i] = p / E;
    wcol[i] = p - wrow[i] * E;
  }
  u32x4 xq[DEPTH][XP], wq[DEPTH][WP];
  auto load = [&](u32x4 (&xr)[XP], u32x4 (&wr)[WP], int kc, int kend) {
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      const int p = tid + i * THREADS;
      const int t = p / (KC / 8), col = kc + 8 * (p % (KC / 8));
      xr[i] = tile_load(xsrc, (XN % THREADS == 0 || p < XN) && col < kend ? (t * d + col) * 2 : kTileOob);
    }
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      const int p = tid + i * THREADS;
      wr[i] = tile_load(wsrc, p < wcnt && kc < kend ? kc * E * 2 + p * 16 : kTileOob);
    }
  };
  auto stage = [&](const u32x4 (&xr)[XP], const u32x4 (&wr)[WP], int buf) {
    uint16_t* xs = reinterpret_cast<uint16_t*>(raw + buf * kStage);
    uint16_t* ws = xs + kTileTok * LDX;
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      const int p = tid + i * THREADS;
      if (XN % THREADS != 0 && p >= XN) continue;
      *reinterpret_cast<u32x4*>(&xs[(p / (KC / 8)) * LDX + 8 * (p % (KC / 8))]) = xr[i];
    }
    if (E % 8 == 0) {
#pragma unroll
      for (int i = 0; i < WP; ++i)
        if (tid + i * THREADS < wcnt) *reinterpret_cast<u32x4*>(&ws[tr_row(wrow[i]) * LDW + wcol[i]]) = wr[i];
    } else {
      // the pieces cross rows of W: element pairs where E is even, single elements
      // where it is odd
#pragma unroll
      for (int i = 0; i < WP; ++i) {
        if (tid + i * THREADS >= wcnt) continue;
        int r = wrow[i], c = wcol[i];
        if (E % 2 == 0) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            *reinterpret_cast<uint32_t*>(&ws[tr_row(r) * LDW + c]) = wr[i][q];
            c += 2;
            if (c >= E) { c = 0; ++r; }
          }
        } else {
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            ws[tr_row(r) * LDW + c] = static_cast<uint16_t>(wr[i][q / 2] >> (16 * (q & 1)));
            c += 1;
            if (c >= E) { c = 0; ++r; }
          }
        }
      }
    }
  };

  f32x4 rsum[MT][NTW], sum[MT][NTW], acc[MT][NTW];
  auto multiply = [&](int buf) {
    const uint16_t* xs = reinterpret_cast<const uint16_t*>(raw + buf * kStage);
    const uint16_t* ws = xs + kTileTok * LDX;
#pragma unroll
    for (int ks = 0; ks < KC / 32; ++ks) {
      u32x4 av[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
        av[mt] = *reinterpret_cast<const u32x4*>(&xs[((wm * MT + mt) * 16 + m) * LDX + 32 * ks + 8 * g]);
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        // lane m of group g addresses row 8 g + 4 h + m / 4, experts 4 (m % 4) ..
        // and receives rows 8 g + 4 h + 0..3 of expert m of the tile
        uint2 half[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
          half[h] = lds_tr16(&ws[(32 * ks + 16 * h + 4 * g + m / 4) * LDW + (wn * NTW + nt) * 16 + 4 * (m % 4)]);
        const u32x4 bv = {half[0].x, half[0].y, half[1].x, half[1].y};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av[mt]),
                                                                __builtin_bit_cast(bf16x8, bv), acc[mt][nt], 0, 0, 0);
      }
    }
  };
  auto flush = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        rsum[mt][nt] += acc[mt][nt];
        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };

  // Stage s + 1 goes to LDS and stage s + 1 + DEPTH is requested while stage s
  // is multiplied; one barrier per stage.  A range's sums start from zero and
  // ranges are added in order, so a block that takes all of them gives the same
  // logits as blocks that take one each.
  const int z0 = MODE == kTilePart ? blockIdx.y : 0;
  const int z1 = MODE == kTilePart || ONE ? z0 + 1 : a.zsplit;
  for (int z = z0; z < z1; ++z) {
    const int k0 = z * a.zcols, kend = min(d, k0 + a.zcols);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) rsum[mt][nt] = acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < DEPTH; ++q) load(xq[q], wq[q], k0 + q * KC, kend);
    stage(xq[0], wq[0], 0);
    load(xq[0], wq[0], k0 + DEPTH * KC, kend);
    __syncthreads();
    for (int kc = k0, buf = 0; kc < kend;) {
#pragma unroll
      for (int q = 1; q <= DEPTH; ++q) {
        const int set = q % DEPTH;
        stage(xq[set], wq[set], buf ^ 1);
        load(xq[set], wq[set], kc + (DEPTH + 1) * KC, kend);
        __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
        multiply(buf);
        if (kSum == KC || (kc - k0) % kSum + KC == kSum || kc + KC >= kend) flush();
        __syncthreads();
        buf ^= 1;
        kc += KC;
        if (kc >= kend) break;
      }
    }
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) sum[mt][nt] = z == z0 ? rsum[mt][nt] : sum[mt][nt] + rsum[mt][nt];
  }
  if constexpr (MODE == kTilePart) {
    float* plane = tile_plane(a);
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      const int e = (wn * NTW + nt) * 16 + m;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int t = (wm * MT + mt) * 16 + 4 * g + i;
          if (t < rows && e < E) plane[static_cast<int64_t>(t) * E + e] = sum[mt][nt][i];
        }
    }
  } else {
    // logits (+ bias): lane holds tokens 4 g + i, expert m of each tile
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      const int e = (wn * NTW + nt) * 16 + m;
      const float b = (a.bias && e < E) ? a.bias[e] : 0.f;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) lg[((wm * MT + mt) * 16 + 4 * g + i) * LGS + e] = sum[mt][nt][i] + b;
  }
    __syncthreads();
    tile_epilogue<THREADS, KMAX, MODE, LGS>(a, lg, hist_lds);
  }
}

// Whether a batch runs with stages short enough for two blocks per CU (ONE): where
// there are more blocks than CUs, one block's first loads and selection run beside
// another's products.  Up to 48 experts LDS holds two blocks with the long stages
// too, and the short ones gain only past 512 blocks.  Whole gate, us, long / short
// stages: 16448 x 768 x 80 33.6 / 26.2; 65536 x 256 x 96 44.0 / 32.3; 32768 x 4096 x 128
// 96.3 / 86.1; up to 48 experts 65536 x 256 x 16 30.3 / 25.4, 65536 x 8192 x 16 250 / 220,
// 33000 x 4096 x 48 78 / 63, 131072 x 3080 x 48 200 / 205, and in 512 blocks 32768 x 4096 x
// 48 1.09 times as long.
static inline bool tile_two_per_cu(const RouteArgs& a) {
  return a.zsplit == 1 && a.nb > (a.E > 48 ? 256 : 512);
}

template <int NT, int WM, int WN, int KC, int DEPTH, bool ONE>
struct TileBf16Launch {
  const RouteArgs& a;
  hipStream_t st;
  template <int KMAX, int MODE>
  hipError_t operator()() const {
    if constexpr (ONE && MODE == kTilePart) {
      return hipErrorInvalidValue;  // one range is never a part
    } else {
      route_tile_bf16_kernel<NT, WM, WN, KC, DEPTH, ONE, KMAX, MODE>
          <<<dim3(a.nb, MODE == kTilePart ? a.zsplit : 1), dim3(WM * WN * kWave), 0, st>>>(a);
      return hipGetLastError();
    }
  }
};

}  // namespace hetumoe
