// Tiled fp32 route kernel (route_tile.hpp) on v_mfma_f32_16x16x4_f32.
#include "route_tile.hpp"

namespace hetumoe {

// Experts of the tiles: tile nt, column n holds expert tile_expert<NT>(nt, n),
// so that a lane's experts of up to four tiles are adjacent in a row of W and
// come with one LDS read, 16 lanes reading contiguous bytes.
template <int NT>
__device__ __forceinline__ int tile_expert(int nt, int n) {
  if constexpr (NT % 4 == 0) return (nt / 4) * 64 + n * 4 + nt % 4;
  else return n * NT + nt;
}

// 64 tokens x E experts per block: 4 waves of 16 tokens times WN groups of experts
// times KS slices of K.
// A stage is KS * KC rows of W, one contiguous piece of memory read flat in
// 16-byte pieces and written to LDS rows of 16 NT floats; slice ks multiplies
// its KC of them.  x goes straight from memory to registers (at
// most WN waves share it): a lane holds 4 consecutive columns of its token per 16 columns, and the
// MFMA of step i takes column 4 g + i from lane group g, W's row of the same
// number.  Each stage is summed on its own and then added to the running sum,
// so rounding grows with KC and the stage count, not with d.
template <int NT, int WN, int KS, int KC, int KMAX, int MODE>
__global__ __launch_bounds__(4 * WN * KS * 64) void route_tile_f32_kernel(RouteArgs a) {
  constexpr int THREADS = 4 * WN * KS * kWave;
  constexpr int NTW = NT / WN;  // tiles per wave
  static_assert(NTW * WN == NT && (WN == 1 || NTW % 4 == 0), "whole groups of four tiles");
  constexpr int LDW = 16 * NT;
  constexpr int LGS = tile_lgs(NT);
  constexpr int ROWS = KS * KC;
  constexpr int XQ = KC / 16;
  constexpr int WP = (ROWS * LDW / 4 + THREADS - 1) / THREADS;
  constexpr int kStage = 2 * ROWS * LDW * 4;  // double buffered
  constexpr int kLg = (KS > 2 ? KS - 1 : 1) * kTileTok * LGS * 4;  // the slices' sums, then the logits
  __shared__ __align__(16) unsigned char raw[kStage > kLg ? kStage : kLg];
  __shared__ int hist_lds[8 * 16 * NT];
  float* wbuf[2] = {reinterpret_cast<float*>(raw), reinterpret_cast<float*>(raw) + ROWS * LDW};
  float* lg = reinterpret_cast<float*>(raw);  // after the K loop

  const int tid = threadIdx.x;
  const int w = tid / kWave, wt = w % 4, wn = w / 4 % WN, ks = w / (4 * WN);
  const int lane = lane_id();
  const int g = lane / 16, m = lane % 16;
  const int d = a.d, E = a.E;
  const int64_t tok0 = static_cast<int64_t>(blockIdx.x) * kTileTok;
  const int rows = static_cast<int>(min(static_cast<int64_t>(kTileTok), a.S - tok0));
  const __amdgpu_buffer_rsrc_t xsrc =
      tile_rsrc(reinterpret_cast<const float*>(a.x) + tok0 * d, static_cast<unsigned>(rows) * d * 4u);
  const __amdgpu_buffer_rsrc_t wsrc = tile_rsrc(a.wg, static_cast<unsigned>(d) * E * 4u);
  const int wcnt = ROWS * E / 4;  // pieces of W per stage

  int wrow[WP], wcol[WP];  // row and column of each piece's first element
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int p = 4 * (tid + i * THREADS);
    wrow[i] = p / E;
    wcol[i] = p - wrow[i] * E;
  }
  u32x4 xr[XQ], xn[XQ], wr[WP];
  auto load = [&](int k0, int kend) {
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int col = k0 + ks * KC + 16 * q + 4 * g;
      xn[q] = tile_load(xsrc, col < kend ? ((wt * 16 + m) * d + col) * 4 : kTileOob);
    }
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      const int p = tid + i * THREADS;
      wr[i] = tile_load(wsrc, p < wcnt && k0 < kend ? k0 * E * 4 + p * 16 : kTileOob);
    }
  };
  auto stage = [&](float* ws) {
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      if (tid + i * THREADS >= wcnt) continue;
      if (E % 4 == 0) {
        *reinterpret_cast<u32x4*>(&ws[wrow[i] * LDW + wcol[i]]) = wr[i];
      } else {  // the piece crosses rows of W
        int r = wrow[i], c = wcol[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          ws[r * LDW + c] = __uint_as_float(wr[i][q]);
          c += 1;
          if (c >= E) { c = 0; ++r; }
        }
      }
    }
  };

  // A range's sums start from zero and ranges are added in order, so a block
  // that takes all of them gives the same logits as blocks that take one each.
  f32x4 sum[NTW];
  const int z0 = MODE == kTilePart ? blockIdx.y : 0;
  const int z1 = MODE == kTilePart ? z0 + 1 : a.zsplit;
  for (int z = z0; z < z1; ++z) {
    const int kz = z * a.zcols, kend = min(d, kz + a.zcols);
    f32x4 rsum[NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) rsum[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    load(kz, kend);
    if (z > z0) __syncthreads();  // the last range's sums are consumed
    stage(wbuf[0]);
    int buf = 0;
    for (int k0 = kz; k0 < kend; k0 += ROWS) {
#pragma unroll
      for (int q = 0; q < XQ; ++q) xr[q] = xn[q];
      const float* ws = buf ? wbuf[1] : wbuf[0];
      __syncthreads();
      load(k0 + ROWS, kend);
      __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
      f32x4 acc[NTW];
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) acc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < XQ; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float* wrow_p = &ws[(ks * KC + 16 * q + 4 * g + i) * LDW];
          const uint32_t xu = xr[q][i];
          const float xv = __uint_as_float(xu);
          float b[NTW];
          if constexpr (NT % 4 == 0) {
#pragma unroll
            for (int u = 0; u < NTW / 4; ++u) {
              const f32x4 v = *reinterpret_cast<const f32x4*>(wrow_p + 64 * (wn * (NTW / 4) + u) + 4 * m);
              b[4 * u] = v.x; b[4 * u + 1] = v.y; b[4 * u + 2] = v.z; b[4 * u + 3] = v.w;
            }
          } else if constexpr (NT == 2) {
            const float2 v = *reinterpret_cast<const float2*>(wrow_p + 2 * m);
            b[0] = v.x; b[1] = v.y;
          } else {
            b[0] = wrow_p[m];
          }
#pragma unroll
          for (int nt = 0; nt < NTW; ++nt) acc[nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv, b[nt], acc[nt], 0, 0, 0);
        }
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) rsum[nt] += acc[nt];
      // the other buffer was last read a stage ago, before the barrier above
      if (k0 + ROWS < kend) stage(buf ? wbuf[0] : wbuf[1]);
      buf ^= 1;
    }
    // the K slices' sums meet in LDS; slice 0 adds them, the last slice first
    __syncthreads();
    if (ks > 0) {
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          lg[((ks - 1) * kTileTok + wt * 16 + 4 * g + i) * LGS + tile_expert<NT>(wn * NTW + nt, m)] = rsum[nt][i];
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = 0.f;
#pragma unroll
          for (int q = KS - 1; q > 0; --q) {
            const float o = lg[((q - 1) * kTileTok + wt * 16 + 4 * g + i) * LGS + tile_expert<NT>(wn * NTW + nt, m)];
            v = q == KS - 1 ? o : v + o;
          }
          rsum[nt][i] += v;
        }
    }
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) sum[nt] = z == z0 ? rsum[nt] : sum[nt] + rsum[nt];
  }
  if constexpr (MODE == kTilePart) {
    float* plane = tile_plane(a);
    if (ks != 0) return;
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      const int e = tile_expert<NT>(wn * NTW + nt, m);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int t = wt * 16 + 4 * g + i;
        if (t < rows && e < E) plane[static_cast<int64_t>(t) * E + e] = sum[nt][i];
      }
    }
  } else {
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        const int e = tile_expert<NT>(wn * NTW + nt, m);
        const float b = (a.bias && e < E) ? a.bias[e] : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) lg[(wt * 16 + 4 * g + i) * LGS + e] = sum[nt][i] + b;
      }
    }
    __syncthreads();
    tile_epilogue<THREADS, KMAX, MODE, LGS>(a, lg, hist_lds);
  }
}

template <int NT, int WN, int KS, int KC>
struct TileF32Launch {
  const RouteArgs& a;
  hipStream_t st;
  template <int KMAX, int MODE>
  hipError_t operator()() const {
    route_tile_f32_kernel<NT, WN, KS, KC, KMAX, MODE>
        <<<dim3(a.nb, MODE == kTilePart ? a.zsplit : 1), dim3(4 * WN * KS * kWave), 0, st>>>(a);
    return hipGetLastError();
  }
};

bool route_uses_tile_f32(const RouteArgs& a) { return a.dtype == 0 && tile_shape(a); }

hipError_t launch_route_tile_f32(const RouteArgs& a, hipStream_t st) {
  // sixteen waves, four per SIMD: with eight, a stage's LDS writes, reads and
  // products followed one another (16384 x 2048 x 64: 57 us, 50 us with sixteen)
  if (a.E <= 16) return tile_by_gate(a, TileF32Launch<1, 1, 4, 64>{a, st});
  if (a.E <= 32) return tile_by_gate(a, TileF32Launch<2, 1, 4, 64>{a, st});
  if (a.E <= 64) return tile_by_gate(a, TileF32Launch<4, 1, 4, 32>{a, st});
  if (a.E <= 128) return tile_by_gate(a, TileF32Launch<8, 2, 2, 32>{a, st});
  return tile_by_gate(a, TileF32Launch<16, 4, 1, 32>{a, st});
}

}  // namespace hetumoe
