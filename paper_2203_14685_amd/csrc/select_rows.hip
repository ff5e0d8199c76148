// Selection on logits in memory (Sec. 3.1): logits given by the caller, or the
// partial sums of a projection whose K was split over blocks.
#include "select.hpp"

namespace hetumoe {

// One block per 64-token wave block, P lanes per token.  The block's rows are
// one contiguous piece of [S, E]: a flat, coalesced pass adds the planes, the
// bias and the noise, divides by the temperature, stores the final logits when
// asked and keeps them in LDS, four (V4: 16-byte) pieces in flight per thread.
// Rows of more than kSelectTileE experts stay in memory: the selection reads
// them from a.fin, written here unless they are a.raw as it is.
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
  // a.fin may be a.raw: a thread then overwrites only elements that no other thread
  // uses (past the last row it reads the block's first element and drops it)
  const bool changed = a.planes > 1 || a.bias || a.temperature > 0.f;
  const bool store = a.fin && (a.fin != a.raw || (changed && lgs == 0));
  if (lgs > 0 || store) {
    const int rows = static_cast<int>(min(static_cast<int64_t>(kWave), a.S - static_cast<int64_t>(blockIdx.x) * kWave));
    const int n = E / kVec;  // pieces per row
    const int dr = kThreads / n, dc = kThreads - dr * n;
    const int64_t plane = static_cast<int64_t>(a.S) * E;
    const float scale = exact_reciprocal(a.temperature);
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
          if (a.temperature > 0.f) {
            const float x = a.noise ? v[u][q] + g[u][q] : v[u][q];
            v[u][q] = scale != 0.f ? x * scale : x / a.temperature;
          }
        }
        if (store) {
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

// Top-k on rows of whole 16-byte pieces (E a multiple of 4, up to 256): P lanes
// per token, lane j holds the 4 experts from 4 j + 4 P u of each of NV vectors in
// registers, straight from memory (the P lanes of a token read 16 P contiguous
// bytes), so there is no tile in LDS and no barrier before the selection.
template <int P, int KMAX, int NV>
__global__ __launch_bounds__(kWave * P) void select_topk_kernel(SelectArgs a) {
  extern __shared__ __align__(16) int hist_lds[];  // [k][E]
  constexpr int kThreads = kWave * P;
  const int t = threadIdx.x / P, j = threadIdx.x % P;
  const int E = a.E;
  const int64_t s = static_cast<int64_t>(blockIdx.x) * kWave + t;
  const bool valid = s < a.S;
  const int64_t plane = static_cast<int64_t>(a.S) * E;
  const int64_t row = (valid ? s : a.S - 1) * E;  // nb > 0, so S > 0
  float4 v[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int e = 4 * (j + P * u);
    v[u] = e < E ? *reinterpret_cast<const float4*>(a.raw + row + e) : float4{0.f, 0.f, 0.f, 0.f};
  }
  for (int i = threadIdx.x; i < a.k * E; i += kThreads) hist_lds[i] = 0;
  for (int p = 1; p < a.planes; ++p) {
#pragma unroll
    for (int u = 0; u < NV; ++u) {
      const int e = 4 * (j + P * u);
      if (e >= E) continue;
      const float4 q = *reinterpret_cast<const float4*>(a.raw + p * plane + row + e);
      v[u].x += q.x; v[u].y += q.y; v[u].z += q.z; v[u].w += q.w;
    }
  }
  KeyList<KMAX> list;
  list.init();
  const float scale = exact_reciprocal(a.temperature);
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    const int e = 4 * (j + P * u);
    if (e < E) {
      if (a.bias) {
        v[u].x += a.bias[e]; v[u].y += a.bias[e + 1]; v[u].z += a.bias[e + 2]; v[u].w += a.bias[e + 3];
      }
      if (a.temperature > 0.f) {
        if (a.noise) {
          const float4 q = *reinterpret_cast<const float4*>(a.noise + row + e);
          v[u].x += q.x; v[u].y += q.y; v[u].z += q.z; v[u].w += q.w;
        }
        if (scale != 0.f) {
          v[u].x *= scale; v[u].y *= scale; v[u].z *= scale; v[u].w *= scale;
        } else {
          v[u].x /= a.temperature; v[u].y /= a.temperature; v[u].z /= a.temperature; v[u].w /= a.temperature;
        }
      }
      if (a.fin && a.fin != a.raw && valid) *reinterpret_cast<float4*>(a.fin + row + e) = v[u];
    }
    const float x[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) list.insert(e < E ? logit_key(x[q]) : kKeyEmpty, e + q);
  }
  int key[KMAX], id[KMAX];
  pop_all<P, KMAX, 0>(list, key, id);
  const float top = key_logit(key[0]);
  float z = 0.f;
  if (a.normalize) {
#pragma unroll
    for (int r = 0; r < KMAX; ++r)
      if (r < a.k) z += __expf(key_logit(key[r]) - top);
  } else {
#pragma unroll
    for (int u = 0; u < NV; ++u)
      if (4 * (j + P * u) < E)
        z += (__expf(v[u].x - top) + __expf(v[u].y - top)) + (__expf(v[u].z - top) + __expf(v[u].w - top));
    z = group_reduce<P>(z, OpAdd());
  }
  __syncthreads();  // the counts are zero
  write_choices<P, KMAX>(key, id, top, 1.f / z, a.k, E, j, valid, a.ids + s * a.k, a.weights + s * a.k, hist_lds);
  __syncthreads();
  for (int i = threadIdx.x; i < a.k * E; i += kThreads)
    a.hist[static_cast<int64_t>(blockIdx.x) * a.k * E + i] = hist_lds[i];
}

template <int P, int NV>
static hipError_t launch_topk_p(const SelectArgs& a, hipStream_t st) {
  const size_t bytes = static_cast<size_t>(a.k) * a.E * 4;
  const dim3 grid(static_cast<unsigned>(a.nb)), block(kWave * P);
  if (a.k == 1) select_topk_kernel<P, 1, NV><<<grid, block, bytes, st>>>(a);
  else if (a.k == 2) select_topk_kernel<P, 2, NV><<<grid, block, bytes, st>>>(a);
  else if (a.k <= 4) select_topk_kernel<P, 4, NV><<<grid, block, bytes, st>>>(a);
  else select_topk_kernel<P, 8, NV><<<grid, block, bytes, st>>>(a);
  return hipGetLastError();
}

static bool rows_aligned(const SelectArgs& a) {
  const uintptr_t all = reinterpret_cast<uintptr_t>(a.raw) | reinterpret_cast<uintptr_t>(a.noise) |
                        reinterpret_cast<uintptr_t>(a.fin);
  return a.E % 4 == 0 && all % 16 == 0;
}

template <int P, int KMAX, int MODE>
static hipError_t launch_rows_t(const SelectArgs& a, hipStream_t st) {
  // row stride in LDS: an odd multiple of P floats, so that the lanes of
  // neighbouring tokens read different banks; past kSelectTileE no tile
  const int lgs = a.E <= kSelectTileE ? P * ((a.E + P - 1) / P | 1) : 0;
  const size_t bytes = static_cast<size_t>(kWave) * lgs * 4 + static_cast<size_t>(a.k) * a.E * 4;
  const dim3 grid(static_cast<unsigned>(a.nb)), block(kWave * P);
  if (rows_aligned(a)) select_rows_kernel<P, KMAX, MODE, true><<<grid, block, bytes, st>>>(a, lgs);
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
  if (a.kind == 0 && a.E <= kSelectTileE && rows_aligned(a)) {
    if (a.E <= 16) return launch_topk_p<4, 1>(a, st);
    if (a.E <= 32) return launch_topk_p<8, 1>(a, st);
    if (a.E <= 64) return launch_topk_p<16, 1>(a, st);
    if (a.E <= 128) return launch_topk_p<16, 2>(a, st);
    if (a.E <= 192) return launch_topk_p<16, 3>(a, st);
    return launch_topk_p<16, 4>(a, st);
  }
  // Four lanes per token up to 32 experts, and up to 128 where more than one block
  // per CU would wait for its turn: sixteen lanes finish a block sooner, four leave
  // the chip more of them.  Whole gate on given logits, us, four / sixteen lanes:
  // 16448 x 60 (257 blocks), kTop1 k = 4 15.5 / 22.5; 262144 x 60 46.6 / 128; 262144 x
  // 100, hierarchical 44.3 / 91.7; one float at a time, 20000 x 127, k = 2 20.3 / 18.7,
  // 65536 x 127 25.3 / 27.3.
  const bool four = a.E <= 32 || (a.E <= 128 && a.nb > (a.E <= 64 || rows_aligned(a) ? 256 : 512));
  return four ? launch_rows_p<4>(a, st) : launch_rows_p<16>(a, st);
}

}  // namespace hetumoe
