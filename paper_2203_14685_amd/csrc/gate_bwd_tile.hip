// Tiled matrix-core products of the gate backward, dW = x^T dL and dx = dL W^T,
// for every expert count up to 256 and every row length: the fp32 gate
// (v_mfma_f32_16x16x4_f32) and the bf16 shapes that the register-sized kernels of
// gate_bwd.hip do not take.  bf16 products multiply x or W, exact in bf16, with
// dL split into three bf16 parts whose sum is dL, as there.
#include "common.hpp"
#include "kernels.hpp"

namespace hetumoe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int kOob = 0x7ffffff0;  // offset past every buffer resource: loads return zeros

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ u32x4 load16(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}
// A value that is the same in all lanes but computed by the vector ALU (a median, a
// block index's quotient): a buffer resource built on it without this is taken
// lane by lane, in a loop around each load that also waits for the loads before.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 load8(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
}
__device__ __forceinline__ uint32_t load4(__amdgpu_buffer_rsrc_t r, int off) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}
// gfx950's LDS transpose read: see route_tile.hpp
__device__ __forceinline__ uint2 tr16(const uint16_t* p) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p)));
}
__device__ __forceinline__ f32x4 mfma_b16(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                 0, 0, 0);
}

// v = hi + mid + lo: the upper 16 bits of v, of v - hi, and of what is left (24
// bits of mantissa in three pieces of 8, each remainder exact), as the upper
// halves of three words.
__device__ __forceinline__ void split_trunc(float v, uint32_t& h, uint32_t& m, uint32_t& l) {
  h = __float_as_uint(v) & 0xffff0000u;
  const float r1 = v - __uint_as_float(h);
  m = __float_as_uint(r1) & 0xffff0000u;
  l = __float_as_uint(r1 - __uint_as_float(m));
}
// The same for N values of which some may be infinite: hi is the value itself
// then, and mid and lo, which inf - inf made NaN, are 0 (one test for all N: 8192 x
// 4096, E = 256 144.5 us with and without it).  NaN stays NaN in all three.
template <int N>
__device__ __forceinline__ void split_trunc_n(const uint32_t* v, uint32_t* h, uint32_t* m, uint32_t* l) {
  float top = 0.f;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    split_trunc(__uint_as_float(v[q]), h[q], m[q], l[q]);
    top = fmaxf(top, fabsf(__uint_as_float(v[q])));
  }
  if (top == INFINITY) {
#pragma unroll
    for (int q = 0; q < N; ++q)
      if (fabsf(__uint_as_float(v[q])) == INFINITY) m[q] = l[q] = 0u;
  }
}
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

// Row stride in LDS (bf16 elements) of rows of 16 n: an odd multiple of 32 bytes,
// and where row t of 32 lies: the 16 rows that one transpose read takes (8 g + 4 h
// + q for g, q = 0..3) are neighbours, so any 8 of them fill all 64 banks.
constexpr int tr_stride(int n) { return 16 * (n | 1); }
__device__ __forceinline__ int tr_row(int t) { return ((t & 4) << 2) | ((t >> 1) & 12) | (t & 3); }

// ---------------------------------------------------------------- dW, bf16
// Block: CB = 64 WM columns of x times all experts (16 NT, NTW tiles per wave)
// over one token range, in stages of 32 tokens, double buffered with one barrier
// per stage.  A stage's x rows go to LDS as they are; its 32 x E piece of dL, one
// contiguous piece of memory, is read flat in 16-byte pieces and written as three
// bf16 planes in the same order, so no transposed copy of dL is needed from the
// kernel before and the workspace stays what the vector path asks for.  Both
// operands are transpose reads.  64 tokens are summed on their own, then added.
// Bound by its stages (8192 x 4096, E = 256: 67 us; without the staging 47, without
// the products 47, with neither and no reads 18): waves of 64 columns x 32 experts,
// four per SIMD, overlap them better than half as many of 64 x 64 (73 us).
template <int NT, int WM, int WN>
__global__ __launch_bounds__(WM* WN * 64) void dwg_tile_bf16_kernel(GateBwdArgs a) {
  constexpr int THREADS = WM * WN * kWave;
  constexpr int NTW = NT / WN;
  static_assert(NTW * WN == NT, "whole tiles per wave");
  constexpr int TK = 32;
  constexpr int CB = 64 * WM;
  constexpr int LDX = CB + 16;  // an odd multiple of 32 bytes
  constexpr int LDE = tr_stride(NT);
  constexpr int XP = (TK * CB / 8 + THREADS - 1) / THREADS;
  constexpr int LP = (TK * 16 * NT / 4 + THREADS - 1) / THREADS;
  __shared__ __align__(16) uint16_t xs[2][TK * LDX];
  __shared__ __align__(16) uint16_t pl[2][3 * TK * LDE];
  const int tid = threadIdx.x;
  const int w = tid / kWave, wm = w / WN, wn = w % WN;
  const int lane = lane_id(), g = lane / 16, m = lane % 16;
  const int d = a.d, E = a.E;
  const int ncb = (d + CB - 1) / CB;
  const int split = blockIdx.x / ncb;
  const int j0 = (blockIdx.x % ncb) * CB;
  const int64_t sb = static_cast<int64_t>(split) * a.split_tokens;
  const int64_t se = min(static_cast<int64_t>(a.S), sb + a.split_tokens);
  const int lcnt = TK * E / 4;

  int lrow[LP], lcol[LP];
#pragma unroll
  for (int i = 0; i < LP; ++i) {
    const int p = 4 * (tid + i * THREADS);
    lrow[i] = p / E;
    lcol[i] = p - lrow[i] * E;
  }
  u32x4 xr[XP], lr[LP];
  auto load = [&](int64_t s0) {
    const int rows = static_cast<int>(max(min(static_cast<int64_t>(TK), se - s0), static_cast<int64_t>(0)));
    const int64_t sx = rows > 0 ? s0 : sb;
    const __amdgpu_buffer_rsrc_t xsrc =
        rsrc_of(reinterpret_cast<const uint16_t*>(a.x) + sx * d, static_cast<unsigned>(rows) * d * 2u);
    const __amdgpu_buffer_rsrc_t lsrc = rsrc_of(a.dl + sx * E, static_cast<unsigned>(rows) * E * 4u);
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      const int p = tid + i * THREADS, t = p / (CB / 8), col = j0 + 8 * (p % (CB / 8));
      xr[i] = load16(xsrc, (t < TK && col < d) ? (t * d + col) * 2 : kOob);
    }
#pragma unroll
    for (int i = 0; i < LP; ++i) {
      const int p = tid + i * THREADS;
      lr[i] = load16(lsrc, p < lcnt ? p * 16 : kOob);
    }
  };
  auto stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      const int p = tid + i * THREADS, t = p / (CB / 8);
      if (XP * THREADS == TK * CB / 8 || t < TK)
        *reinterpret_cast<u32x4*>(&xs[buf][tr_row(t) * LDX + 8 * (p % (CB / 8))]) = xr[i];
    }
#pragma unroll
    for (int i = 0; i < LP; ++i) {
      if (tid + i * THREADS >= lcnt) continue;
      const uint32_t u[4] = {lr[i].x, lr[i].y, lr[i].z, lr[i].w};
      uint32_t h[4], md[4], lo[4];
      split_trunc_n<4>(u, h, md, lo);
      if (E % 4 == 0) {
        uint16_t* o = &pl[buf][tr_row(lrow[i]) * LDE + lcol[i]];
        *reinterpret_cast<uint2*>(o) = uint2{pack_hi(h[0], h[1]), pack_hi(h[2], h[3])};
        *reinterpret_cast<uint2*>(o + TK * LDE) = uint2{pack_hi(md[0], md[1]), pack_hi(md[2], md[3])};
        *reinterpret_cast<uint2*>(o + 2 * TK * LDE) = uint2{pack_hi(lo[0], lo[1]), pack_hi(lo[2], lo[3])};
      } else {  // the piece crosses rows of dL
        int r = lrow[i], c = lcol[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          uint16_t* o = &pl[buf][tr_row(r) * LDE + c];
          o[0] = static_cast<uint16_t>(h[q] >> 16);
          o[TK * LDE] = static_cast<uint16_t>(md[q] >> 16);
          o[2 * TK * LDE] = static_cast<uint16_t>(lo[q] >> 16);
          c += 1;
          if (c >= E) { c = 0; ++r; }
        }
      }
    }
  };

  f32x4 sum[4][NTW], acc[4][NTW];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) sum[mt][nt] = acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // of the two waves that a SIMD holds of an eight-wave block, one stages before it
  // multiplies and one after: one's conversions meet the other's products
  const bool early = (__builtin_amdgcn_readfirstlane(w) & 4) == 0;
  load(sb);
  stage(0);
  load(sb + TK);
  __syncthreads();
  int buf = 0;
  for (int64_t s0 = sb; s0 < se; s0 += TK) {
    if (early) {
      stage(buf ^ 1);  // zeros after the last
      load(s0 + 2 * TK);
      __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
    }
    u32x4 av[4];
#pragma unroll
    for (int mt = 0; mt < 4; ++mt) {
      uint2 hf[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
        hf[h] = tr16(&xs[buf][(16 * h + 4 * g + m / 4) * LDX + wm * 64 + 16 * mt + 4 * (m % 4)]);
      av[mt] = u32x4{hf[0].x, hf[0].y, hf[1].x, hf[1].y};
    }
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt)
#pragma unroll
      for (int p = 0; p < 3; ++p) {
        uint2 hf[2];
#pragma unroll
        for (int h = 0; h < 2; ++h)
          hf[h] = tr16(&pl[buf][(p * TK + 16 * h + 4 * g + m / 4) * LDE + (wn * NTW + nt) * 16 + 4 * (m % 4)]);
        const u32x4 bv = {hf[0].x, hf[0].y, hf[1].x, hf[1].y};
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) acc[mt][nt] = mfma_b16(av[mt], bv, acc[mt][nt]);
      }
    if (buf) {  // every second stage, and below after the last
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) {
          sum[mt][nt] += acc[mt][nt];
          acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (!early) {
      stage(buf ^ 1);
      load(s0 + 2 * TK);
    }
    __syncthreads();
    buf ^= 1;
  }
  // lane holds columns 16 mt + 4 g + i, expert m of each tile
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      const int e = (wn * NTW + nt) * 16 + m, j = j0 + wm * 64 + 16 * mt + 4 * g;
      if (e < E && j < d)
        *reinterpret_cast<f32x4*>(a.wpart + (static_cast<int64_t>(split) * E + e) * d + j) = sum[mt][nt] + acc[mt][nt];
    }
}

// ---------------------------------------------------------------- dx, bf16
// Block: 8 waves of 16 tokens x `passes` passes of 64 columns.  A wave keeps its
// tokens' dL in registers as three bf16 parts (KS steps of 32 experts); a pass's
// 64 rows of W, contiguous, are read flat and written to padded LDS rows, two
// passes in turn; experts past E are zero in both.  The product is taken
// transposed (W rows are the A operand) and regrouped by lane swaps so that one
// store covers 8 tokens x 128 bytes, as in dx_mfma_kernel.
// W fragments are read ahead of their products and nothing waits for stores: the
// whole gate backward of 8192 x 4096, E = 256, 152.3 -> 146.1 us (this kernel 59 -> 52).
constexpr int kDxWaves = 8;
constexpr int kDxThreads = kDxWaves * kWave;

// N values of a row of dL in groups of W: experts n G + off + 0 .. W - 1, n = 0, 1, ..
// (G = 4 W, one group per lane group); zeros past E and past the buffer.
template <int N, int W = 8>
__device__ __forceinline__ void dl_row(__amdgpu_buffer_rsrc_t src, int row, int off, int E, uint32_t* v) {
  if (E % 4 == 0) {
#pragma unroll
    for (int q = 0; q < N / 4; ++q) {
      const int e = (q * 4 / W) * 4 * W + off + (q * 4) % W;
      const u32x4 t = load16(src, e < E ? (row + e) * 4 : kOob);
      v[4 * q] = t.x; v[4 * q + 1] = t.y; v[4 * q + 2] = t.z; v[4 * q + 3] = t.w;
    }
  } else {
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const int e = (q / W) * 4 * W + off + q % W;
      v[q] = load4(src, e < E ? (row + e) * 4 : kOob);
    }
  }
}

template <int KS, bool ACC>
__global__ __launch_bounds__(kDxThreads) void dx_tile_bf16_kernel(GateBwdArgs a, int passes) {
  constexpr int KE = 32 * KS;
  constexpr int LDW = KE + 8;
  constexpr int WP = (64 * KE / 8 + kDxThreads - 1) / kDxThreads;
  __shared__ __align__(16) uint16_t wl[2][64 * LDW];
  const int tid = threadIdx.x;
  const int w = tid / kWave, lane = lane_id(), g = lane / 16, m = lane % 16;
  const int d = a.d, E = a.E;
  const int CB = 64 * passes;
  const int ncb = (d + CB - 1) / CB;
  const int64_t sblk = static_cast<int64_t>(uniform(blockIdx.x / ncb)) * (16 * kDxWaves);
  const int jb = uniform(blockIdx.x % ncb) * CB;

  u32x4 ph[KS], pm[KS], pq[KS];
  {
    const int rows = static_cast<int>(min(static_cast<int64_t>(16 * kDxWaves), a.S - sblk));
    const __amdgpu_buffer_rsrc_t lsrc = rsrc_of(a.dl + sblk * E, static_cast<unsigned>(rows) * E * 4u);
    uint32_t v[KS][8];
    dl_row<8 * KS>(lsrc, (16 * w + m) * E, 8 * g, E, &v[0][0]);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      uint32_t h[8], md[8], lo[8];
      split_trunc_n<8>(v[ks], h, md, lo);
      ph[ks] = u32x4{pack_hi(h[0], h[1]), pack_hi(h[2], h[3]), pack_hi(h[4], h[5]), pack_hi(h[6], h[7])};
      pm[ks] = u32x4{pack_hi(md[0], md[1]), pack_hi(md[2], md[3]), pack_hi(md[4], md[5]), pack_hi(md[6], md[7])};
      pq[ks] = u32x4{pack_hi(lo[0], lo[1]), pack_hi(lo[2], lo[3]), pack_hi(lo[4], lo[5]), pack_hi(lo[6], lo[7])};
    }
  }
  const int wcnt = 64 * E / 8;
  int wrow[WP], wcol[WP];
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int p = 8 * (tid + i * kDxThreads);
    wrow[i] = p / E;
    wcol[i] = p - wrow[i] * E;
  }
  u32x4 wr[WP];
  auto load_w = [&](int j0) {
    const int wrows = uniform(max(min(64, d - j0), 0));
    const __amdgpu_buffer_rsrc_t src =
        rsrc_of(reinterpret_cast<const uint16_t*>(a.wg) + static_cast<int64_t>(wrows > 0 ? j0 : 0) * E,
                static_cast<unsigned>(wrows) * E * 2u);
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      const int p = tid + i * kDxThreads;
      wr[i] = load16(src, p < wcnt ? p * 16 : kOob);
    }
  };
  auto stage_w = [&](uint16_t* ws) {
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      if (tid + i * kDxThreads >= wcnt) continue;
      if (E % 8 == 0) {
        *reinterpret_cast<u32x4*>(&ws[wrow[i] * LDW + wcol[i]]) = wr[i];
      } else if (E % 2 == 0) {
        int r = wrow[i], c = wcol[i];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          *reinterpret_cast<uint32_t*>(&ws[r * LDW + c]) = wr[i][q];
          c += 2;
          if (c >= E) { c = 0; ++r; }
        }
      } else {
        int r = wrow[i], c = wcol[i];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          ws[r * LDW + c] = static_cast<uint16_t>(wr[i][q / 2] >> (16 * (q & 1)));
          c += 1;
          if (c >= E) { c = 0; ++r; }
        }
      }
    }
  };
  load_w(jb);
  if (E < KE) {  // experts past E: zero once, never written after
    const int n = KE - E;
    for (int i = tid; i < 2 * 64 * n; i += kDxThreads) {
      const int r = i / n;
      wl[r / 64][(r % 64) * LDW + E + i % n] = 0;
    }
  }
  // tokens of this lane's two pieces: 8 h + (m & 7); columns 32 (m >> 3) + cofs ..
  const int pcol = 32 * (m >> 3) + 16 * (g & 1) + 8 * (g >> 1);
  const bool lo8 = m < 8;
  // dx through a resource that ends with the wave's last row: no branch, so the
  // wait for a stage's W counts the stores issued after it instead of waiting for
  // them (rows past the batch and columns past d load zeros and store nothing)
  const int64_t s0 = sblk + 16 * uniform(w);
  const int dxn = uniform(s0 < a.S ? static_cast<int>(min(static_cast<int64_t>(16), a.S - s0)) : 0);
  const __amdgpu_buffer_rsrc_t dxr =
      rsrc_of(reinterpret_cast<uint16_t*>(a.dx) + (dxn > 0 ? s0 * d : 0), static_cast<unsigned>(dxn) * d * 2u);
  const int t0 = m & 7;
  const bool early = (__builtin_amdgcn_readfirstlane(w) & 4) == 0;
  const int jend = min(jb + CB, d);
  stage_w(wl[0]);
  load_w(jb + 64 < jend ? jb + 64 : d);
  __syncthreads();
  int buf = 0;
  for (int j0 = jb; j0 < jend; j0 += 64) {
    const uint16_t* ws = wl[buf];
    if (early) {
      stage_w(wl[buf ^ 1]);
      load_w(j0 + 128 < jend ? j0 + 128 : d);
    }
    const int j = j0 + pcol;
    const int off[2] = {j < d && t0 < dxn ? (t0 * d + j) * 2 : kOob,
                        j < d && t0 + 8 < dxn ? ((t0 + 8) * d + j) * 2 : kOob};
    u32x4 din[2];
    if constexpr (ACC) {
      din[0] = load16(dxr, off[0]);
      din[1] = load16(dxr, off[1]);
    }
    // W fragments are read kAhead ahead of their three products (as far as the
    // registers go); left to itself the compiler waits for each read in turn
    constexpr int kAhead = KS > 6 && ACC ? 1 : 3, kFrags = 4 * KS;
    u32x4 bw[kAhead + 1];
    auto frag = [&](int f) {
      return *reinterpret_cast<const u32x4*>(&ws[(16 * (f / KS) + m) * LDW + 32 * (f % KS) + 8 * g]);
    };
    f32x4 acc[4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < kAhead; ++f) bw[f] = frag(f);
    __builtin_amdgcn_sched_group_barrier(0x100, kAhead, 0);
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
      f32x4 ah = {0.f, 0.f, 0.f, 0.f}, am = ah, al = ah;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int f = nt * KS + ks;
        if (f + kAhead < kFrags) {
          bw[(f + kAhead) % (kAhead + 1)] = frag(f + kAhead);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // one LDS read
        }
        ah = mfma_b16(bw[f % (kAhead + 1)], ph[ks], ah);
        am = mfma_b16(bw[f % (kAhead + 1)], pm[ks], am);
        al = mfma_b16(bw[f % (kAhead + 1)], pq[ks], al);
        __builtin_amdgcn_sched_group_barrier(0x8, 3, 0);  // three products
      }
      acc[nt] = ah + (am + al);
    }
    // lanes of even g keep tile 2p's columns and get their neighbour's, lanes of
    // odd g tile 2p + 1's: 8 columns of token m each, then half rows trade places
    float xv[8], yv[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float f0 = acc[0][i], f1 = acc[1][i], f2 = acc[2][i], f3 = acc[3][i];
      const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, f0), __builtin_bit_cast(int, f1),
                                                      false, false);
      const auto q = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(int, f2), __builtin_bit_cast(int, f3),
                                                      false, false);
      xv[i] = __builtin_bit_cast(float, static_cast<int>(r[0]));
      xv[4 + i] = __builtin_bit_cast(float, static_cast<int>(r[1]));
      yv[i] = __builtin_bit_cast(float, static_cast<int>(q[0]));
      yv[4 + i] = __builtin_bit_cast(float, static_cast<int>(q[1]));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float keep = h == 0 ? xv[i] : yv[i];
        const float moved = __builtin_bit_cast(
            float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, h == 0 ? yv[i] : xv[i]), 0x128, 0xF, 0xF, false));
        o[i] = (h == 0) == lo8 ? keep : moved;
      }
      if constexpr (ACC) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          o[2 * q] += bf16_lo(din[h][q]);
          o[2 * q + 1] += bf16_hi(din[h][q]);
        }
      }
      __builtin_amdgcn_raw_buffer_store_b128(
          u32x4{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3]), pack_bf16x2(o[4], o[5]), pack_bf16x2(o[6], o[7])},
          dxr, off[h], 0, 2 /* nt */);
    }
    if (!early) {
      stage_w(wl[buf ^ 1]);
      load_w(j0 + 128 < jend ? j0 + 128 : d);
    }
    __syncthreads();
    buf ^= 1;
  }
}

// ---------------------------------------------------------------- dW, fp32
// Experts of the tiles, as in the fp32 route kernel: a lane's experts of up to
// four tiles are adjacent in a row of dL.
template <int NT>
__device__ __forceinline__ int dl_expert(int nt, int n) {
  if constexpr (NT % 4 == 0) return (nt / 4) * 64 + n * 4 + nt % 4;
  else return n * NT + nt;
}

// Block: 2 x 4 waves of 16 MT columns times 16 NT experts (blockIdx.y: which) over one
// token range, in stages of 64 tokens, each half of the waves 32 of them.  x goes
// from memory to registers: a lane loads MT adjacent columns of token 4 t + g, and
// column MT m + mt is row m of tile mt.  dL's rows are staged in LDS, double
// buffered.  A half sums 64 tokens (two stages) on their own, then adds them; the
// halves meet in LDS.
template <int NT, int MT>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(MT == 2 ? 4 : 1))) void dwg_tile_f32_kernel(GateBwdArgs a) {
  constexpr int TH = 32, TK = 2 * TH, XQ = TH / 4;
  constexpr int EB = 16 * NT;
  constexpr int LP = TK * EB / 512;  // single values per thread: rows of EB out of E
  constexpr int kStage = 2 * TK * EB, kHalf = 4 * 16 * MT * EB;
  __shared__ __align__(16) float ds[kStage > kHalf ? kStage : kHalf];
  const int tid = threadIdx.x;
  const int w = tid / kWave, lane = lane_id(), g = lane / 16, m = lane % 16;
  const int hs = w / 4, wc = w % 4;
  const int d = a.d, E = a.E;
  constexpr int CW = 16 * MT, CB = 4 * CW;  // columns per wave and block
  const int ncb = (d + CB - 1) / CB;
  const int split = blockIdx.x / ncb;
  const int jw = (blockIdx.x % ncb) * CB + wc * CW;
  const int j = jw + MT * m;
  const int e0 = blockIdx.y * EB;
  const int64_t sb = static_cast<int64_t>(split) * a.split_tokens;
  const int64_t se = min(static_cast<int64_t>(a.S), sb + a.split_tokens);

  uint32_t xr[XQ][MT], xn[XQ][MT];
  uint32_t lr[LP];
  auto load = [&](int64_t s0) {
    const int rows = static_cast<int>(max(min(static_cast<int64_t>(TK), se - s0), static_cast<int64_t>(0)));
    const int64_t sx = rows > 0 ? s0 : sb;
    const __amdgpu_buffer_rsrc_t xsrc =
        rsrc_of(reinterpret_cast<const float*>(a.x) + sx * d, static_cast<unsigned>(rows) * d * 4u);
    const __amdgpu_buffer_rsrc_t lsrc = rsrc_of(a.dl + sx * E, static_cast<unsigned>(rows) * E * 4u);
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const int o = j < d ? ((hs * TH + 4 * q + g) * d + j) * 4 : kOob;
      if constexpr (MT == 4) {
        const u32x4 v = load16(xsrc, o);
        xn[q][0] = v.x; xn[q][1] = v.y; xn[q][2] = v.z; xn[q][3] = v.w;
      } else {
        const u32x2 v = load8(xsrc, o);
        xn[q][0] = v.x; xn[q][1] = v.y;
      }
    }
#pragma unroll
    for (int i = 0; i < LP; ++i) {
      const int p = tid + i * 512, t = p / EB, e = e0 + p % EB;
      lr[i] = load4(lsrc, e < E ? (t * E + e) * 4 : kOob);
    }
  };
  f32x4 sum[MT][NT], acc[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) sum[mt][nt] = acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto flush = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        sum[mt][nt] += acc[mt][nt];
        acc[mt][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
  };
  load(sb);
  int buf = 0;
  for (int64_t s0 = sb; s0 < se; s0 += TK) {
    // the buffer was last read two stages ago, before the previous barrier
#pragma unroll
    for (int i = 0; i < LP; ++i) ds[buf * TK * EB + tid + i * 512] = __uint_as_float(lr[i]);
#pragma unroll
    for (int q = 0; q < XQ; ++q)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) xr[q][mt] = xn[q][mt];
    __syncthreads();
    load(s0 + TK);
    __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the products
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
      const float* row = &ds[(buf * TK + hs * TH + 4 * q + g) * EB];
      float b[NT];
      if constexpr (NT % 4 == 0) {
#pragma unroll
        for (int u = 0; u < NT / 4; ++u) {
          const f32x4 v = *reinterpret_cast<const f32x4*>(row + 64 * u + 4 * m);
          b[4 * u] = v.x; b[4 * u + 1] = v.y; b[4 * u + 2] = v.z; b[4 * u + 3] = v.w;
        }
      } else if constexpr (NT == 2) {
        const float2 v = *reinterpret_cast<const float2*>(row + 2 * m);
        b[0] = v.x; b[1] = v.y;
      } else {
        b[0] = row[m];
      }
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const uint32_t xu = xr[q][mt];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(xu), b[nt], acc[mt][nt], 0, 0, 0);
      }
    }
    if (buf) flush();
    buf ^= 1;
  }
  flush();
  __syncthreads();  // the stages are consumed
  f32x4* half = reinterpret_cast<f32x4*>(ds);  // [4 waves][MT NT][64 lanes]
  if (hs == 1) {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) half[(wc * MT * NT + mt * NT + nt) * kWave + lane] = sum[mt][nt];
  }
  __syncthreads();
  if (hs == 1) return;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) sum[mt][nt] += half[(wc * MT * NT + mt * NT + nt) * kWave + lane];
  // lane (g, m) of tile (mt, nt): columns MT (4 g + i) + mt, so its tiles hold MT
  // adjacent columns for each i
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int e = e0 + dl_expert<NT>(nt, m);
    if (e >= E) continue;
    float* o = a.wpart + (static_cast<int64_t>(split) * E + e) * d;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = jw + MT * (4 * g + i);
      if (c >= d) continue;
      if constexpr (MT == 4)
        *reinterpret_cast<f32x4*>(o + c) = f32x4{sum[0][nt][i], sum[1][nt][i], sum[2][nt][i], sum[3][nt][i]};
      else
        *reinterpret_cast<float2*>(o + c) = float2{sum[0][nt][i], sum[1][nt][i]};
    }
  }
}

// ---------------------------------------------------------------- dx, fp32
// Block: 8 waves of 16 tokens x `passes` passes of PC columns.  A wave keeps its
// tokens' dL in registers (KQ groups of 16 experts: lane group g holds experts 16
// q + 4 g + i, which MFMA step (q, i) takes); a pass's rows of W are staged in
// LDS, two passes in turn, experts past E zero.  The product is transposed (W
// rows are the A operand): row 4 g + i of tile pair member u is column 8 g + 4 u
// + i, so a lane's two tiles hold 8 adjacent columns of token m.
template <int KQ, int PC, bool ACC>
__global__ __launch_bounds__(kDxThreads) void dx_tile_f32_kernel(GateBwdArgs a, int passes) {
  constexpr int KE = 16 * KQ;
  constexpr int LDW = KE + 4;
  constexpr int WP = (PC * KE / 4 + kDxThreads - 1) / kDxThreads;
  static_assert(PC % 32 == 0, "whole tile pairs");
  __shared__ __align__(16) float wl[2][PC * LDW];
  const int tid = threadIdx.x;
  const int w = tid / kWave, lane = lane_id(), g = lane / 16, m = lane % 16;
  const int d = a.d, E = a.E;
  const int CB = PC * passes;
  const int ncb = (d + CB - 1) / CB;
  const int64_t sblk = static_cast<int64_t>(uniform(blockIdx.x / ncb)) * (16 * kDxWaves);
  const int jb = uniform(blockIdx.x % ncb) * CB;
  uint32_t dv[KQ][4];
  {
    const int rows = static_cast<int>(min(static_cast<int64_t>(16 * kDxWaves), a.S - sblk));
    const __amdgpu_buffer_rsrc_t lsrc = rsrc_of(a.dl + sblk * E, static_cast<unsigned>(rows) * E * 4u);
    dl_row<4 * KQ, 4>(lsrc, (16 * w + m) * E, 4 * g, E, &dv[0][0]);
  }
  const int wcnt = PC * E / 4;
  int wrow[WP], wcol[WP];
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int p = 4 * (tid + i * kDxThreads);
    wrow[i] = p / E;
    wcol[i] = p - wrow[i] * E;
  }
  u32x4 wr[WP];
  auto load_w = [&](int j0) {
    const int rows = uniform(max(min(PC, d - j0), 0));
    const __amdgpu_buffer_rsrc_t src =
        rsrc_of(reinterpret_cast<const float*>(a.wg) + static_cast<int64_t>(rows > 0 ? j0 : 0) * E,
                static_cast<unsigned>(rows) * E * 4u);
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      const int p = tid + i * kDxThreads;
      wr[i] = load16(src, p < wcnt ? p * 16 : kOob);
    }
  };
  auto stage_w = [&](float* ws) {
#pragma unroll
    for (int i = 0; i < WP; ++i) {
      if (tid + i * kDxThreads >= wcnt) continue;
      if (E % 4 == 0) {
        *reinterpret_cast<u32x4*>(&ws[wrow[i] * LDW + wcol[i]]) = wr[i];
      } else {
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
  load_w(jb);
  if (E < KE) {  // experts past E: zero once, never written after
    const int n = KE - E;
    for (int i = tid; i < 2 * PC * n; i += kDxThreads) {
      const int r = i / n;
      wl[r / PC][(r % PC) * LDW + E + i % n] = 0.f;
    }
  }
  // dx without a branch, as in dx_tile_bf16_kernel (8192 x 2048, E = 64: 29.7 -> 28.1 us)
  const int64_t s0 = sblk + 16 * uniform(w);
  const int dxn = uniform(s0 < a.S ? static_cast<int>(min(static_cast<int64_t>(16), a.S - s0)) : 0);
  const __amdgpu_buffer_rsrc_t dxr =
      rsrc_of(reinterpret_cast<float*>(a.dx) + (dxn > 0 ? s0 * d : 0), static_cast<unsigned>(dxn) * d * 4u);
  const int arow = 8 * (m / 4) + m % 4;  // column of A row m in tile 0 of a pair; tile 1 is 4 on
  const bool early = (__builtin_amdgcn_readfirstlane(w) & 4) == 0;
  int buf = 0;
  const int jend = min(jb + CB, d);
  stage_w(wl[0]);
  load_w(jb + PC < jend ? jb + PC : d);
  __syncthreads();
  for (int j0 = jb; j0 < jend; j0 += PC) {
    const float* ws = wl[buf];
    if (early) {
      stage_w(wl[buf ^ 1]);
      load_w(j0 + 2 * PC < jend ? j0 + 2 * PC : d);
    }
#pragma unroll
    for (int pr = 0; pr < PC / 32; ++pr) {
      const int j = j0 + 32 * pr + 8 * g;
      const bool ok = m < dxn && j < d;  // d and j: multiples of 4
      const int off[2] = {ok ? (m * d + j) * 4 : kOob, ok && j + 4 < d ? (m * d + j + 4) * 4 : kOob};
      u32x4 in[2];
      if constexpr (ACC) {
        in[0] = load16(dxr, off[0]);
        in[1] = load16(dxr, off[1]);
      }
      f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int q = 0; q < KQ; ++q) {
        f32x4 wv[2];
#pragma unroll
        for (int u = 0; u < 2; ++u)
          wv[u] = *reinterpret_cast<const f32x4*>(&ws[(32 * pr + arow + 4 * u) * LDW + 16 * q + 4 * g]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const float wf = wv[u][i];
            acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf, __uint_as_float(dv[q][i]), acc[u], 0, 0, 0);
          }
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if constexpr (ACC) acc[u] += __builtin_bit_cast(f32x4, in[u]);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[u]), dxr, off[u], 0, 0);
      }
    }
    if (!early) {
      stage_w(wl[buf ^ 1]);
      load_w(j0 + 2 * PC < jend ? j0 + 2 * PC : d);
    }
    __syncthreads();
    buf ^= 1;
  }
}

// ---------------------------------------------------------------- launchers
template <int NT, int WM, int WN>
static void launch_dwg_b16(const GateBwdArgs& a, hipStream_t st) {
  const int64_t blocks = static_cast<int64_t>((a.d + 64 * WM - 1) / (64 * WM)) * a.nsplit;
  dwg_tile_bf16_kernel<NT, WM, WN><<<dim3(static_cast<unsigned>(blocks)), dim3(WM * WN * kWave), 0, st>>>(a);
}

template <int NT, int MT>
static void launch_dwg_f32(const GateBwdArgs& a, hipStream_t st) {
  const int64_t blocks = static_cast<int64_t>((a.d + 64 * MT - 1) / (64 * MT)) * a.nsplit;
  dwg_tile_f32_kernel<NT, MT>
      <<<dim3(static_cast<unsigned>(blocks), (a.E + 16 * NT - 1) / (16 * NT)), dim3(512), 0, st>>>(a);
}

void launch_dwg_tile(const GateBwdArgs& a, hipStream_t st) {
  if (a.dtype == 1) {
    if (a.E <= 16) launch_dwg_b16<1, 4, 1>(a, st);
    else if (a.E <= 32) launch_dwg_b16<2, 4, 1>(a, st);
    else if (a.E <= 64) launch_dwg_b16<4, 4, 2>(a, st);
    else if (a.E <= 128) launch_dwg_b16<8, 4, 4>(a, st);
    else if (a.E <= 192) launch_dwg_b16<12, 2, 6>(a, st);
    else launch_dwg_b16<16, 2, 8>(a, st);
    return;
  }
  if (a.E <= 16) launch_dwg_f32<1, 4>(a, st);
  else if (a.E <= 32) launch_dwg_f32<2, 4>(a, st);
  else launch_dwg_f32<4, 2>(a, st);
}

// Passes per dx block of PC columns: as few as give `target` blocks, so that a
// block's dL registers and first W rows serve the more columns the larger the
// batch is.
static int dx_passes(const GateBwdArgs& a, int PC, int64_t tb, int target) {
  const int all = (a.d + PC - 1) / PC;
  int passes = 16;
  while (passes > 1 && tb * ((all + passes - 1) / passes) < target) passes /= 2;
  return passes < all ? passes : all;
}

template <int KS>
static void launch_dx_b16(const GateBwdArgs& a, int64_t tb, hipStream_t st) {
  const int passes = dx_passes(a, 64, tb, KS > 4 ? 256 : 512);
  const dim3 grid(static_cast<unsigned>(tb * ((a.d + 64 * passes - 1) / (64 * passes)))), block(kDxThreads);
  if (a.accumulate) dx_tile_bf16_kernel<KS, true><<<grid, block, 0, st>>>(a, passes);
  else dx_tile_bf16_kernel<KS, false><<<grid, block, 0, st>>>(a, passes);
}

template <int KQ, int PC>
static void launch_dx_f32(const GateBwdArgs& a, int64_t tb, hipStream_t st) {
  const int passes = dx_passes(a, PC, tb, 512);
  const dim3 grid(static_cast<unsigned>(tb * ((a.d + PC * passes - 1) / (PC * passes)))), block(kDxThreads);
  if (a.accumulate) dx_tile_f32_kernel<KQ, PC, true><<<grid, block, 0, st>>>(a, passes);
  else dx_tile_f32_kernel<KQ, PC, false><<<grid, block, 0, st>>>(a, passes);
}

void launch_dx_tile(const GateBwdArgs& a, hipStream_t st) {
  const int64_t tb = (static_cast<int64_t>(a.S) + 16 * kDxWaves - 1) / (16 * kDxWaves);
  if (a.dtype == 1) {
    if (a.E <= 32) launch_dx_b16<1>(a, tb, st);
    else if (a.E <= 64) launch_dx_b16<2>(a, tb, st);
    else if (a.E <= 96) launch_dx_b16<3>(a, tb, st);
    else if (a.E <= 128) launch_dx_b16<4>(a, tb, st);
    else if (a.E <= 192) launch_dx_b16<6>(a, tb, st);
    else launch_dx_b16<8>(a, tb, st);
    return;
  }
  if (a.E <= 16) launch_dx_f32<1, 64>(a, tb, st);
  else if (a.E <= 32) launch_dx_f32<2, 64>(a, tb, st);
  else if (a.E <= 64) launch_dx_f32<4, 64>(a, tb, st);
  else if (a.E <= 128) launch_dx_f32<8, 64>(a, tb, st);
  else if (a.E <= 192) launch_dx_f32<12, 32>(a, tb, st);
  else launch_dx_f32<16, 32>(a, tb, st);
}

}  // namespace hetumoe
