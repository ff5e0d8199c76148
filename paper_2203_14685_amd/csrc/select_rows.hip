// Selection on logits in memory (Sec. 3.1): logits given by the caller, or the
// partial sums of a projection whose K was split over blocks.
#include "select.hpp"

namespace hetumoe {

// One block per 64-token wave block, P lanes per token.  The block's rows are
// one contiguous piece of [S, E]: a flat, coalesced pass adds the planes, the
// bias and the noise, divides by the temperature, stores the final logits when
// asked and keeps them in LDS, four (V4: 16-byte) pieces in flight per thread.
// Rows of more than kSelectTileE experts stay in memory: the selection reads
// them from there.
template <int P, int KMAX, int MODE, bool V4>  // MODE: 0 top-k, 1 kTop1, 3 hierarchical top-k
__global__ __launch_bounds__(kWave * P) void select_rows_kernel(SelectArgs a, int lgs) {
  extern __shared__ __align__(16) float lds[];  // [64][lgs] logits (lgs > 0), then [k][E] counts
  constexpr int kThreads = kWave * P;
  constexpr int kVec = V4 ? 4 : 1;
  constexpr int kU = 4;
  const int t = threadIdx.x / P, j = threadIdx.x % P;
  const int E = a.E;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kWave * E;
  int* hist_lds = reinterpret_cast<int*>(lds + kWave * lgs);
  for (int i = threadIdx.x; i < a.k * E; i += kThreads) hist_lds[i] = 0;
  if (lgs > 0 || a.fin != a.raw) {
    const int rows = static_cast<int>(min(static_cast<int64_t>(kWave), a.S - static_cast<int64_t>(blockIdx.x) * kWave));
    const int n = E / kVec;  // pieces per row
    const int dr = kThreads / n, dc = kThreads - dr * n;
    const int64_t plane = static_cast<int64_t>(a.S) * E;
    int r = threadIdx.x / n, c = threadIdx.x - r * n;
    while (r < rows) {
      int ru[kU], cu[kU];
      float v[kU][kVec], g[kU][kVec];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        ru[u] = r;
        cu[u] = c * kVec;
        r += dr;
        c += dc;
        if (c >= n) { c -= n; ++r; }
        const int64_t o = base + (ru[u] < rows ? ru[u] * E + cu[u] : 0);
        if constexpr (V4) {
          const float4 q = *reinterpret_cast<const float4*>(a.raw + o);
          v[u][0] = q.x; v[u][1] = q.y; v[u][2] = q.z; v[u][3] = q.w;
          if (a.noise) {
            const float4 z = *reinterpret_cast<const float4*>(a.noise + o);
            g[u][0] = z.x; g[u][1] = z.y; g[u][2] = z.z; g[u][3] = z.w;
          }
        } else {
          v[u][0] = a.raw[o];
          if (a.noise) g[u][0] = a.noise[o];
        }
      }
      for (int p = 1; p < a.planes; ++p) {
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int64_t o = p * plane + base + (ru[u] < rows ? ru[u] * E + cu[u] : 0);
          if constexpr (V4) {
            const float4 q = *reinterpret_cast<const float4*>(a.raw + o);
            v[u][0] += q.x; v[u][1] += q.y; v[u][2] += q.z; v[u][3] += q.w;
          } else {
            v[u][0] += a.raw[o];
          }
        }
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        if (ru[u] >= rows) continue;
#pragma unroll
        for (int q = 0; q < kVec; ++q) {
          if (a.bias) v[u][q] += a.bias[cu[u] + q];
          if (a.temperature > 0.f) v[u][q] = (a.noise ? v[u][q] + g[u][q] : v[u][q]) / a.temperature;
        }
        if (a.fin && a.fin != a.raw) {
          float* f = a.fin + base + ru[u] * E + cu[u];
          if constexpr (V4) *reinterpret_cast<float4*>(f) = float4{v[u][0], v[u][1], v[u][2], v[u][3]};
          else *f = v[u][0];
        }
        if (lgs > 0) {
          float* f = lds + ru[u] * lgs + cu[u];
          if constexpr (V4) *reinterpret_cast<float4*>(f) = float4{v[u][0], v[u][1], v[u][2], v[u][3]};
          else *f = v[u][0];
        }
      }
    }
  }
  __syncthreads();
  const int64_t s = static_cast<int64_t>(blockIdx.x) * kWave + t;
  const bool valid = s < a.S;
  // invalid tokens select on the block's first row (their results are not written)
  const float* lrow = lgs > 0 ? lds + (valid ? t : 0) * lgs : a.fin + base + static_cast<int64_t>(valid ? t : 0) * E;
  select_row<P, KMAX, MODE>(lrow, E, a.k, a.groups, a.normalize, j, valid, a.ids + s * a.k, a.weights + s * a.k,
                            hist_lds);
  __syncthreads();
  for (int i = threadIdx.x; i < a.k * E; i += kThreads)
    a.hist[static_cast<int64_t>(blockIdx.x) * a.k * E + i] = hist_lds[i];
}

template <int P, int KMAX, int MODE>
static hipError_t launch_rows_t(const SelectArgs& a, hipStream_t st) {
  // row stride in LDS: an odd multiple of P floats, so that the lanes of
  // neighbouring tokens read different banks; past kSelectTileE no tile
  const int lgs = a.E <= kSelectTileE ? P * ((a.E + P - 1) / P | 1) : 0;
  const size_t bytes = static_cast<size_t>(kWave) * lgs * 4 + static_cast<size_t>(a.k) * a.E * 4;
  const uintptr_t all = reinterpret_cast<uintptr_t>(a.raw) | reinterpret_cast<uintptr_t>(a.noise) |
                        reinterpret_cast<uintptr_t>(a.fin);
  const dim3 grid(static_cast<unsigned>(a.nb)), block(kWave * P);
  if (a.E % 4 == 0 && all % 16 == 0) select_rows_kernel<P, KMAX, MODE, true><<<grid, block, bytes, st>>>(a, lgs);
  else select_rows_kernel<P, KMAX, MODE, false><<<grid, block, bytes, st>>>(a, lgs);
  return hipGetLastError();
}

template <int P, int MODE>
static hipError_t launch_rows_m(const SelectArgs& a, hipStream_t st) {
  if (MODE == 1 || a.k == 1) return launch_rows_t<P, 1, MODE>(a, st);
  if (a.k == 2) return launch_rows_t<P, 2, MODE>(a, st);
  if (a.k <= 4) return launch_rows_t<P, 4, MODE>(a, st);
  return launch_rows_t<P, 8, MODE>(a, st);
}

template <int P>
static hipError_t launch_rows_p(const SelectArgs& a, hipStream_t st) {
  if (a.kind == 1) return launch_rows_m<P, 1>(a, st);
  if (a.kind == 3) return launch_rows_m<P, 3>(a, st);
  return launch_rows_m<P, 0>(a, st);
}

hipError_t launch_select_rows(const SelectArgs& a, hipStream_t st) {
  if (a.nb == 0) return hipSuccess;
  return a.E <= 32 ? launch_rows_p<4>(a, st) : launch_rows_p<16>(a, st);
}

}  // namespace hetumoe
