// Streaming expert selection and the wave-block histogram shared by the route
// kernels (gate step of Algorithm 1; Eq. 1, Sec. 3.1 kTop1).
//
// Order of experts everywhere: larger logit first, then lower expert index.
// Softmax sums are formed online (running maximum, rescaled sum) with the
// hardware exponential (__expf: v_exp_f32 on x*log2(e)); its relative error is
// about |x| * 6e-8 plus one ulp, far inside the 1e-5 weight tolerance.
#pragma once

#include "common.hpp"
#include "kernels.hpp"

namespace hetumoe {

constexpr int kEmpty = 0x7fffffff;

// ---------------------------------------------------------------- top-k
template <int KMAX>
struct TopkState {
  float tv[KMAX];
  int ti[KMAX];
  float m;     // running max of the logits seen
  float ssum;  // sum of exp(logit - m) over the logits seen
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < KMAX; ++i) { tv[i] = -INFINITY; ti[i] = kEmpty; }
    m = -INFINITY;
    ssum = 0.f;
  }
  // Sorted insertion: the carried pair moves down while it beats the entry it
  // meets.  An empty entry always loses, so every reported id is a real expert
  // even for non-finite logits.
  __device__ __forceinline__ void insert(float v, int e) {
    float cv = v;
    int ci = e;
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      const bool beats = better(cv, ci, tv[i], ti[i]);
      const float ov = tv[i];
      const int oi = ti[i];
      tv[i] = beats ? cv : ov;
      ti[i] = beats ? ci : oi;
      cv = beats ? ov : cv;
      ci = beats ? oi : ci;
    }
  }
  __device__ __forceinline__ void push(float v, int e) {
    if (v > m) { ssum = ssum * __expf(m - v) + 1.f; m = v; }
    else { ssum += __expf(v - m); }
    insert(v, e);
  }
  // (v, i) ranks before (pv, pi): larger logit, then lower index; empty entries last.
  __device__ __forceinline__ static bool better(float v, int i, float pv, int pi) {
    return i != kEmpty && (pi == kEmpty || v > pv || (v == pv && i < pi));
  }
  // Merge with the state of lane (lane ^ mask): afterwards both hold the best
  // KMAX of the union.  The best KMAX of two sorted lists A, B are
  // better-of(A[i], B[KMAX-1-i]), a bitonic sequence; log2(KMAX) half-cleaner
  // stages sort it.
  __device__ __forceinline__ void merge_xor(int mask) {
    float cv[KMAX];
    int ci[KMAX];
#pragma unroll
    for (int i = 0; i < KMAX; ++i) {
      const float pv = xor_partner(tv[KMAX - 1 - i], mask);
      const int pi = xor_partner(ti[KMAX - 1 - i], mask);
      const bool mine = better(tv[i], ti[i], pv, pi);
      cv[i] = mine ? tv[i] : pv;
      ci[i] = mine ? ti[i] : pi;
    }
#pragma unroll
    for (int st = KMAX / 2; st >= 1; st /= 2) {
#pragma unroll
      for (int i = 0; i < KMAX; ++i) {
        if ((i & st) == 0) {
          const bool keep = better(cv[i], ci[i], cv[i + st], ci[i + st]);
          const float v0 = cv[i], v1 = cv[i + st];
          const int i0 = ci[i], i1 = ci[i + st];
          cv[i] = keep ? v0 : v1;
          ci[i] = keep ? i0 : i1;
          cv[i + st] = keep ? v1 : v0;
          ci[i + st] = keep ? i1 : i0;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < KMAX; ++i) { tv[i] = cv[i]; ti[i] = ci[i]; }
    const float pm = xor_partner(m, mask);
    const float ps = xor_partner(ssum, mask);
    const float nm = fmaxf(m, pm);
    // a side that has seen nothing has m = -inf and ssum = 0: contributes 0
    const float a = (ssum > 0.f) ? ssum * __expf(m - nm) : 0.f;
    const float b = (ps > 0.f) ? ps * __expf(pm - nm) : 0.f;
    ssum = a + b;
    m = nm;
  }
  // Writes ids and weights of the first k entries.
  __device__ __forceinline__ void finish(int k, int normalize, int32_t* ids, float* weights) const {
    const float top = tv[0];
    float z = 0.f;
    if (normalize) {
#pragma unroll
      for (int r = 0; r < KMAX; ++r)
        if (r < k) z += __expf(tv[r] - top);
    } else {
      z = ssum * __expf(m - top);  // m == top for finite logits
    }
    const float inv = 1.f / z;
#pragma unroll
    for (int r = 0; r < KMAX; ++r) {
      if (r < k) {
        ids[r] = ti[r];
        weights[r] = (r == 0 ? 1.f : __expf(tv[r] - top)) * inv;
      }
    }
  }
};

// ---------------------------------------------------------------- kTop1
// Best expert of a run of experts inside one group, with the group softmax sum
// relative to that best logit.
struct GroupBest {
  float bv;    // best (= max) logit
  int bi;      // its expert
  float gsum;  // sum of exp(logit - bv)
  __device__ __forceinline__ void init() { bv = -INFINITY; bi = kEmpty; gsum = 0.f; }
  __device__ __forceinline__ void push(float v, int e) {
    if (bi == kEmpty) { bv = v; bi = e; gsum = 1.f; }
    else if (v > bv) { gsum = gsum * __expf(bv - v) + 1.f; bv = v; bi = e; }
    else { gsum += __expf(v - bv); }
  }
  __device__ __forceinline__ void merge_xor(int mask) {
    const float pv = xor_partner(bv, mask);
    const int pi = xor_partner(bi, mask);
    const float ps = xor_partner(gsum, mask);
    if (pi == kEmpty) return;
    if (bi == kEmpty) { bv = pv; bi = pi; gsum = ps; return; }
    const bool partner_wins = pv > bv || (pv == bv && pi < bi);
    const float nb = partner_wins ? pv : bv;
    gsum = gsum * __expf(bv - nb) + ps * __expf(pv - nb);
    bv = nb;
    bi = partner_wins ? pi : bi;
  }
};

// kTop1 streaming over all experts in index order: k contiguous groups of G;
// each finished group writes its best expert and weight 1 / sum exp(l - max).
struct Ktop1State {
  int G, g;
  GroupBest cur;
  __device__ __forceinline__ void init(int G_) { G = G_; g = 0; cur.init(); }
  __device__ __forceinline__ void push(float v, int e, int32_t* ids, float* weights) {
    cur.push(v, e);
    if (e == (g + 1) * G - 1) {
      ids[g] = cur.bi;
      weights[g] = 1.f / cur.gsum;
      ++g;
      cur.init();
    }
  }
};

// ---------------------------------------------------------------- selection on a compile-time slice
// Selection for one token by P consecutive lanes of a wave, for kernels that know
// E at compile time (all P lanes must call this together; the lane that writes
// an (id, weight) pair also counts it in hist_lds[r][id]): lane j's SL =
// E / P logits are read from LDS at once (`lslice` points at them; 8-byte
// aligned for SL = 2, 16-byte aligned from SL = 4 on) and held in registers;
// the maximum comes first and the softmax sum of the slice relative to it
// second, so no step waits on the one before it.
template <int SL>
__device__ __forceinline__ void load_slice(const float* lslice, float (&v)[SL]) {
  if constexpr (SL % 4 == 0) {
#pragma unroll
    for (int i = 0; i < SL; i += 4) {
      const float4 q = *reinterpret_cast<const float4*>(lslice + i);
      v[i] = q.x; v[i + 1] = q.y; v[i + 2] = q.z; v[i + 3] = q.w;
    }
  } else if constexpr (SL == 2) {
    const float2 q = *reinterpret_cast<const float2*>(lslice);
    v[0] = q.x; v[1] = q.y;
  } else {
#pragma unroll
    for (int i = 0; i < SL; ++i) v[i] = lslice[i];
  }
}

template <int SL>
__device__ __forceinline__ float slice_max(const float (&v)[SL]) {
  float mx = v[0];
#pragma unroll
  for (int i = 1; i < SL; ++i) mx = fmaxf(mx, v[i]);
  return mx;
}

template <int SL>
__device__ __forceinline__ float slice_expsum(const float (&v)[SL], float mx) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < SL; ++i) s += __expf(v[i] - mx);
  return s;
}

// Top-k state of a slice: sorted insertion in expert order (an equal logit
// never displaces a lower expert), with the slice's softmax sum.
template <int KMAX, int SL>
__device__ __forceinline__ void topk_of_slice(const float (&v)[SL], int e0, TopkState<KMAX>& tk) {
  tk.init();
  tk.m = slice_max(v);
  tk.ssum = slice_expsum(v, tk.m);
#pragma unroll
  for (int i = 0; i < SL; ++i) tk.insert(v[i], e0 + i);
}

// P lanes per token, each with SL = E / P logits of its row at lrow + j * SL.
template <int P, int KMAX, bool KTOP1, int SL>
__device__ __forceinline__ void select_token_c(const float* lrow, int k, int normalize, int j, bool valid,
                                               int32_t* ids, float* weights, int* hist_lds) {
  constexpr int E = P * SL;
  const int e0 = j * SL;
  if constexpr (!KTOP1) {
    float v[SL];
    load_slice<SL>(lrow + e0, v);
    TopkState<KMAX> tk;
    topk_of_slice<KMAX, SL>(v, e0, tk);
#pragma unroll
    for (int msk = 1; msk < P; msk <<= 1) tk.merge_xor(msk);
    if (valid && j == 0) {
      tk.finish(k, normalize, ids, weights);
#pragma unroll
      for (int r = 0; r < KMAX; ++r)
        if (r < k) atomicAdd(&hist_lds[r * E + tk.ti[r]], 1);
    }
  } else {
    // k divides E, a power of two, and so P: L = P / k lanes per group; lane j's
    // experts lie in group j / L
    const int L = P / k;
    float v[SL];
    load_slice<SL>(lrow + e0, v);
    GroupBest gb;
    gb.bv = v[0];
    gb.bi = e0;
#pragma unroll
    for (int i = 1; i < SL; ++i) {
      const bool up = v[i] > gb.bv;  // strict: the lower expert keeps a tie
      gb.bv = up ? v[i] : gb.bv;
      gb.bi = up ? e0 + i : gb.bi;
    }
    gb.gsum = slice_expsum(v, gb.bv);
    for (int msk = 1; msk < L; msk <<= 1) gb.merge_xor(msk);
    if (valid && j % L == 0) {
      const int grp = j / L;
      ids[grp] = gb.bi;
      weights[grp] = 1.f / gb.gsum;
      atomicAdd(&hist_lds[grp * E + gb.bi], 1);
    }
  }
}

// ---------------------------------------------------------------- selection on a row of any length
// One token by P consecutive lanes: lane j takes experts j, j + P, ... (the
// lanes read neighbouring LDS words, and P need not divide E) and keeps the KMAX
// best of them sorted; then, k times, the lanes take the best head of their
// lists and its lane drops it.  Logits are compared as integer keys of the same
// order (-0 as +0, NaN below -inf, an empty entry below all): one med3, one
// compare and two selects per entry and inserted logit, where float comparisons
// with an index tie-break took about 14, and a max and a min over the lanes per
// choice in place of sorted-list merges.
constexpr int kKeyEmpty = static_cast<int>(0x80000000u);
constexpr int kKeyNan = kKeyEmpty + 1;

__device__ __forceinline__ int logit_key(float v) {
  const int b = __float_as_int(v + 0.f);  // -0 becomes +0
  return v != v ? kKeyNan : b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float key_logit(int key) { return __int_as_float(key ^ ((key >> 31) & 0x7fffffff)); }

struct OpMinI {
  __device__ __forceinline__ int operator()(int a, int b) const { return a < b ? a : b; }
};

// The KMAX best of a lane's logits, best first; equal keys in expert order
// (experts come in increasing order, and an equal key displaces nothing).
template <int KMAX>
struct KeyList {
  int key[KMAX], id[KMAX];
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int i = 0; i < KMAX; ++i) { key[i] = kKeyEmpty; id[i] = kEmpty; }
  }
  __device__ __forceinline__ void insert(int v, int e) {
    bool up = v > key[KMAX - 1];  // v goes to entry i or above
#pragma unroll
    for (int i = KMAX - 1; i > 0; --i) {
      const bool above = v > key[i - 1];
      id[i] = above ? id[i - 1] : up ? e : id[i];
      key[i] = max(min(key[i - 1], v), key[i]);  // the middle one of the three
      up = above;
    }
    id[0] = up ? e : id[0];
    key[0] = max(key[0], v);
  }
  // lane j of P takes experts lo + j, lo + j + P, ... below hi
  template <int P>
  __device__ __forceinline__ void scan(const float* lrow, int lo, int hi, int j) {
    init();
    for (int e = lo + j; e < hi; e += 4 * P) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = lrow[min(e + u * P, hi - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) insert(e + u * P < hi ? logit_key(v[u]) : kKeyEmpty, e + u * P);
    }
  }
  // The best of the P lanes' first entries, dropped from its list.  LEFT: the
  // entries still wanted after it.
  template <int P, int LEFT>
  __device__ __forceinline__ void pop(int& best, int& expert) {
    best = group_reduce<P>(key[0], OpMaxI());
    expert = group_reduce<P>(key[0] == best ? id[0] : kEmpty, OpMinI());
    const bool mine = id[0] == expert;
#pragma unroll
    for (int i = 0; i < LEFT; ++i) {  // LEFT < KMAX
      key[i] = mine ? key[i + 1] : key[i];
      id[i] = mine ? id[i + 1] : id[i];
    }
  }
};

// Sum of exp(logit - top) over the experts [lo, hi), by all P lanes.  BEST: expert
// `best`, whose logit top is, counts exp(0) = 1 also where it is infinite.
template <int P, bool BEST>
__device__ __forceinline__ float row_expsum(const float* lrow, int lo, int hi, int j, float top, int best = 0) {
  float s = 0.f;
  for (int e = lo + j; e < hi; e += 4 * P) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = lrow[min(e + u * P, hi - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      s += e + u * P >= hi ? 0.f : BEST && e + u * P == best ? 1.f : __expf(v[u] - top);
  }
  return group_reduce<P>(s, OpAdd());
}

// All KMAX best of the P lanes, in order, on every lane.
template <int P, int KMAX, int R>
__device__ __forceinline__ void pop_all(KeyList<KMAX>& list, int (&key)[KMAX], int (&id)[KMAX]) {
  list.template pop<P, KMAX - 1 - R>(key[R], id[R]);
  if constexpr (R + 1 < KMAX) pop_all<P, KMAX, R + 1>(list, key, id);
}

// Choice r of the first k is written by lane r % P, which also counts it.
template <int P, int KMAX>
__device__ __forceinline__ void write_choices(const int (&key)[KMAX], const int (&id)[KMAX], float top, float inv, int k,
                                              int E, int j, bool valid, int32_t* ids, float* weights, int* hist_lds) {
#pragma unroll
  for (int r = 0; r < KMAX; ++r) {
    if (r < k && valid && j == r % P) {
      ids[r] = id[r];
      weights[r] = (r == 0 ? 1.f : __expf(key_logit(key[r]) - top)) * inv;
      atomicAdd(&hist_lds[r * E + id[r]], 1);
    }
  }
}

// 1 / t where that is exact (t a power of two with a normal reciprocal), so that
// x * (1 / t) is x / t rounded once, else 0.
__device__ __forceinline__ float exact_reciprocal(float t) {
  const uint32_t u = __float_as_uint(t);
  const uint32_t exp = u >> 23;
  return (u & 0x007fffffu) == 0 && exp >= 1 && exp <= 252 ? __uint_as_float((254 - exp) << 23) : 0.f;
}

// MODE: 0 top-k, 1 kTop1, 3 hierarchical top-k.  All P lanes call this
// together.
template <int P, int KMAX, int MODE>
__device__ __forceinline__ void select_row(const float* lrow, int E, int k, int groups, int normalize, int j,
                                           bool valid, int32_t* ids, float* weights, int* hist_lds) {
  if constexpr (MODE == 1) {
    const int G = E / k;
    for (int grp = 0; grp < k; ++grp) {
      const int lo = grp * G, hi = lo + G;
      KeyList<1> best;
      best.template scan<P>(lrow, lo, hi, j);
      int key, id;
      best.template pop<P, 0>(key, id);
      const float top = key_logit(key);
      // the sum that tests every term for `best` only where it matters (65536 x 192, k
      // = 2, whole gate: tested always 39.6 us, so 38.2)
      const float z = fabsf(top) == INFINITY ? row_expsum<P, true>(lrow, lo, hi, j, top, id)
                                             : row_expsum<P, false>(lrow, lo, hi, j, top);
      if (valid && j == grp % P) {
        ids[grp] = id;
        weights[grp] = 1.f / z;
        atomicAdd(&hist_lds[grp * E + id], 1);
      }
    }
  } else {
    int lo = 0, hi = E;
    if constexpr (MODE == 3) {
      // the group of the best expert over all
      KeyList<1> first;
      first.template scan<P>(lrow, 0, E, j);
      int key, id;
      first.template pop<P, 0>(key, id);
      const int Gs = E / groups;
      lo = id / Gs * Gs;
      hi = lo + Gs;
    }
    KeyList<KMAX> list;
    list.template scan<P>(lrow, lo, hi, j);
    int key[KMAX], id[KMAX];
    pop_all<P, KMAX, 0>(list, key, id);
    const float top = key_logit(key[0]);
    float z = 0.f;
    if (normalize) {
#pragma unroll
      for (int r = 0; r < KMAX; ++r)
        if (r < k) z += __expf(key_logit(key[r]) - top);
    } else {
      z = row_expsum<P, false>(lrow, 0, E, j, top);
    }
    write_choices<P, KMAX>(key, id, top, 1.f / z, k, E, j, valid, ids, weights, hist_lds);
  }
}

// Hierarchical top-k (Sec. 3.1, H Topk) on a compile-time slice: the best expert
// over all E (with the full softmax sum), its group of Gs contiguous experts,
// then the k best experts of that group.  Weights: softmax over the k chosen
// (normalize) or the full softmax at each of them.
template <int P, int KMAX, int SL>
__device__ __forceinline__ void select_token_htopk_c(const float* lrow, int k, int Gs, int normalize, int j,
                                                     bool valid, int32_t* ids, float* weights, int* hist_lds) {
  constexpr int E = P * SL;
  const int e0 = j * SL;
  float v[SL];
  load_slice<SL>(lrow + e0, v);
  TopkState<1> t1;
  topk_of_slice<1, SL>(v, e0, t1);
#pragma unroll
  for (int msk = 1; msk < P; msk <<= 1) t1.merge_xor(msk);
  const int best = t1.ti[0] == kEmpty ? 0 : t1.ti[0];
  const int lo = (best / Gs) * Gs, hi = lo + Gs;
  TopkState<KMAX> tk;
  tk.init();
  // experts outside the group go in as empty entries, which never displace
  // anything (no branch per logit)
#pragma unroll
  for (int i = 0; i < SL; ++i) {
    const int ee = e0 + i;
    const bool in = ee >= lo && ee < hi;
    tk.insert(in ? v[i] : -INFINITY, in ? ee : kEmpty);
  }
#pragma unroll
  for (int msk = 1; msk < P; msk <<= 1) tk.merge_xor(msk);
  // the group holds the overall best: the full softmax sum relative to it
  tk.m = t1.m;
  tk.ssum = t1.ssum;
  if (valid && j == 0) {
    tk.finish(k, normalize, ids, weights);
#pragma unroll
    for (int r = 0; r < KMAX; ++r)
      if (r < k) atomicAdd(&hist_lds[r * E + tk.ti[r]], 1);
  }
}

// ---------------------------------------------------------------- wave-block histogram
// hist[wb][r][e] = number of tokens of wave block wb whose rank-r choice is e.
// Every wave of the block calls this (it synchronises the block); `active` waves
// own a wave block, `s` is the calling lane's token.  The ids are read back from
// global memory, where the same thread wrote them.
__device__ __forceinline__ void wave_block_hist(int* lds_w, bool active, int64_t s, bool valid, int wb,
                                                const RouteArgs& a) {
  const int lane = lane_id();
  for (int r = 0; r < a.k; ++r) {
    if (active)
      for (int i = lane; i < a.E; i += kWave) lds_w[i] = 0;
    __syncthreads();
    if (active && valid) atomicAdd(&lds_w[a.ids[s * a.k + r]], 1);
    __syncthreads();
    if (active)
      for (int i = lane; i < a.E; i += kWave)
        a.hist[(static_cast<int64_t>(wb) * a.k + r) * a.E + i] = lds_w[i];
    __syncthreads();
  }
}

}  // namespace hetumoe
