// Capacity slots (Sec. 3.1): each expert keeps at most C assignments, handed out
// rank-major, then in token order.  The route kernels leave, for every 64-token
// wave block, how many of its tokens chose each expert at each rank: a row of Q =
// k E counts.
//   assign      a block per wave block: adds up the rows before its own (all of
//               them, or one per group after group_scan) for the first slot of
//               each run, then a wave per rank places the tokens: ballots on the
//               bits of the expert id give a token's place among those with the
//               same expert (ordered, no atomics) -> slots, slot_src.
//   group_scan  larger histograms first: running sums of the rows within groups
//               of F, in place, so that assign reads one row per group.
// Neither moves the histogram across columns: rows are read and written whole, as
// the route kernels wrote them.  (A scan per expert over all rows, a launch of its
// own, touches 16 bytes of every row per block: 7.7 us at 32768 tokens, E = 64, k
// = 4, plus 5.1 us for the assignment.)
#include "common.hpp"
#include "kernels.hpp"

namespace hetumoe {

constexpr int kGroupThreads = 256;

// In place: row b becomes the sum of its group's rows up to b.
__global__ __launch_bounds__(kGroupThreads) void group_scan_kernel(int32_t* hist, int nb, int Q, int F) {
  const int q = blockIdx.y * kGroupThreads + threadIdx.x;
  if (q >= Q) return;
  const int b0 = blockIdx.x * F, b1 = min(nb, b0 + F);
  int32_t* col = hist + q;
  int run = 0;
  for (int b = b0; b < b1; b += 16) {
    int v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = b + u < b1 ? col[static_cast<int64_t>(b + u) * Q] : 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      run += v[u];
      if (b + u < b1) col[static_cast<int64_t>(b + u) * Q] = run;
    }
  }
}

// Rank r of the 64 tokens of wave block wb by one wave; `offs`: the wave block's
// first slots of that rank, one per expert.
__device__ __forceinline__ void assign_rank(const AssignArgs& a, int wb, int r, const int* offs) {
  const int lane = lane_id();
  const int64_t s = static_cast<int64_t>(wb) * kWave + lane;
  const bool valid = s < a.S;
  const int64_t q = s * a.k + r;
  // ids are in [0, E); invalid lanes use E, so bits of 0..E are compared
  const int e = valid ? a.ids[q] : a.E;
  const int nbits = 32 - __clz(a.E);
  uint64_t same = ~0ull;
  for (int bit = 0; bit < nbits; ++bit) {
    const bool on = (e >> bit) & 1;
    const uint64_t bal = __ballot(on);
    same &= on ? bal : ~bal;
  }
  if (valid) {
    const int pos = offs[e] + popc_below(same);
    const bool kept = static_cast<unsigned>(pos) < static_cast<unsigned>(a.C);
    a.slots[q] = kept ? pos : -1;
    if (kept) a.slot_src[static_cast<int64_t>(e) * a.C + pos] = static_cast<int>(q);
  }
}

// T threads, WB wave blocks per block.  The histogram's rows are counts, or
// (GROUPED) running sums in groups of F, a multiple of WB.  G = T / Q groups of
// threads take the rows they add in turn, a thread one column (columns tid, tid +
// T, ... where Q > T).
template <int T, int WB, bool GROUPED>
__global__ __launch_bounds__(T) void assign_kernel(AssignArgs a, int F) {
  extern __shared__ int lds[];  // tot [Q], offs [WB][Q], then partial sums [2][T] where T / Q > 1
  const int tid = threadIdx.x;
  const int k = a.k, E = a.E, nb = a.nb, Q = k * E;
  const int wb0 = blockIdx.x * WB;
  int* tot = lds;
  int* offs = lds + Q;
  int* part = lds + (WB + 1) * Q;
  const int groups = GROUPED ? (nb + F - 1) / F : nb;
  const int own = GROUPED ? wb0 / F : wb0;  // rows (groups) before the block's own
  const int G = Q < T ? T / Q : 1;
  const int g = Q < T ? tid / Q : 0;
  // rows wb0 - 1 (GROUPED: unless the group starts here), wb0, ...: what a wave
  // block's offsets add to the sums before the block's own row (group)
  auto extra = [&](int q, int (&x)[WB]) {
#pragma unroll
    for (int i = 0; i < WB; ++i) {
      const int b = wb0 + i - 1;
      x[i] = (GROUPED ? (wb0 + i) % F != 0 : i > 0) && b < nb ? a.hist[static_cast<int64_t>(b) * Q + q] : 0;
    }
#pragma unroll
    for (int i = 1; i < WB; ++i) x[i] += GROUPED ? 0 : x[i - 1];
  };
  int ex[WB];
  if (tid < Q && Q <= T) extra(tid, ex);
  for (int q = tid - g * Q * (Q < T); q < Q && g < G; q += T) {
    const int32_t* col = a.hist + q;
    int t = 0, p = 0;
    for (int i0 = g; i0 < groups; i0 += 8 * G) {
      int v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = i0 + u * G;
        const int row = GROUPED ? min(i * F + F, nb) - 1 : i;  // a group's sum is its last row
        v[u] = i < groups ? col[static_cast<int64_t>(row) * Q] : 0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        t += v[u];
        p += i0 + u * G < own ? v[u] : 0;
      }
    }
    if (G > 1) {
      part[tid] = t;
      part[T + tid] = p;
    } else {
      tot[q] = t;
      offs[q] = p;
    }
  }
  __syncthreads();
  // few columns leave many partial sums per column: halved until eight are left (all
  // of them added by one thread: hash gate, 65536 tokens, E = 8 8.9 us, so 8.2)
  int parts = G;
  while (parts > 8) {
    const int half = (parts + 1) / 2;
    if (g + half < parts) {
      part[tid] += part[tid + half * Q];
      part[T + tid] += part[T + tid + half * Q];
    }
    parts = half;
    __syncthreads();
  }
  int first = 0;  // column tid (Q <= T): sum of the rows before the block's own
  if (tid < Q && Q <= T) {
    if (G > 1) {
      int t = 0;
      for (int i = 0; i < parts; ++i) {
        t += part[i * Q + tid];
        first += part[T + i * Q + tid];
      }
      tot[tid] = t;
    } else {
      first = offs[tid];
    }
  }
  __syncthreads();
  for (int q = tid; q < Q; q += T) {
    int p = Q <= T ? first : offs[q];
    for (int q2 = q - E; q2 >= 0; q2 -= E) p += tot[q2];  // rank-major: earlier ranks first
    if (Q > T) extra(q, ex);
#pragma unroll
    for (int i = 0; i < WB; ++i) offs[i * Q + q] = p + ex[i];
  }
  __syncthreads();
  for (int pr = tid / kWave; pr < WB * k; pr += T / kWave) {
    const int i = pr / k, r = pr - i * k;
    assign_rank(a, wb0 + i, r, offs + i * Q + r * E);
  }
  if (blockIdx.x == 0) {
    for (int e = tid; e < E; e += T) {
      int d = 0;
      for (int r = 0; r < k; ++r) d += tot[r * E + e];
      a.counts[e] = min(d, a.C);
      if (a.demand) a.demand[e] = d;
    }
  }
  // every block marks its share of each expert's empty slots, as many threads side
  // by side per expert as there are
  const int share = (a.C + gridDim.x - 1) / gridDim.x;
  const int c0 = blockIdx.x * share, c1 = min(a.C, c0 + share);
  const int per = T >= E ? T / E : 1;
  for (int e = tid / per; e < E; e += T / per) {
    int kept = 0;
    for (int r = 0; r < k; ++r) kept += tot[r * E + e];
    for (int c = max(kept, c0) + tid % per; c < c1; c += per) a.slot_src[static_cast<int64_t>(e) * a.C + c] = -1;
  }
}

template <int T, int WB>
static void launch_assign_t(const AssignArgs& a, int F, hipStream_t st) {
  const int Q = a.k * a.E;
  const size_t lds = static_cast<size_t>((WB + 1) * Q + (Q <= T / 2 ? 2 * T : 0)) * sizeof(int);
  // an empty batch still has counts and slots to write
  const dim3 grid(static_cast<unsigned>(a.nb > 0 ? (a.nb + WB - 1) / WB : 1)), block(T);
  if (F > 1) assign_kernel<T, WB, true><<<grid, block, lds, st>>>(a, F);
  else assign_kernel<T, WB, false><<<grid, block, lds, st>>>(a, 1);
}

hipError_t launch_assign(const AssignArgs& a, hipStream_t st) {
  const int64_t Q = static_cast<int64_t>(a.k) * a.E;
  // Whole gate on given logits, us.  Four wave blocks per block once there are 512
  // (four / one): S = 32768, E = 64, k = 1 15.5 / 17.8; 16384, 128, 4 18.4 / 17.5.
  // Sixteen once four would leave more blocks than the chip holds at a time, sooner
  // at k = 1, where a block of four places its tokens with four of sixteen waves
  // (sixteen / four): hash gate, 524288 tokens, E = 8 21 / 33, 200000, E = 64 14.4 / 20.0;
  // 131072, E = 256 16.9 / 19.1.
  const int WB = a.nb > (a.k == 1 ? 1024 : 2048) && Q <= 512 ? 16 : a.nb >= 512 && Q <= 2048 ? 4 : 1;
  // Counts as they are while a block adds up to 32 K of them, else groups of at
  // least 16 rows first (one launch / two): 16384, 64, 2 (32 K) 13.4 / 14.8; 16384,
  // 64, 3 (48 K) 16.4 / 15.2; 16384, 64, 4 (64 K) 17.7 / 15.7; 32768, 64, 4 (128 K)
  // 28.2 / 21.3.
  constexpr int64_t kBlockReads = 32768;
  int F = 1;
  if (Q * a.nb > kBlockReads) {
    F = 16;
    while (Q * a.nb / F > kBlockReads && F < 1024) F *= 2;
    const dim3 grid(static_cast<unsigned>((a.nb + F - 1) / F), static_cast<unsigned>((Q + kGroupThreads - 1) / kGroupThreads));
    group_scan_kernel<<<grid, dim3(kGroupThreads), 0, st>>>(a.hist, a.nb, static_cast<int>(Q), F);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
  }
  // a few counts only: small blocks start sooner
  if (Q <= 256 && a.k <= 4 && Q * a.nb <= 4096) launch_assign_t<256, 1>(a, F, st);
  else if (WB == 1) launch_assign_t<1024, 1>(a, F, st);
  // few sums to add after group_scan: half the threads start and meet sooner (512 /
  // 1024: hash gate, 65536 tokens, E = 64 10.2 / 10.8; given logits 100000 x 24, k = 2
  // 15.4 / 16.7); the counts themselves need them all (32768 x 64, k = 1 12.9 / 11.2)
  else if (WB == 4 && F > 1 && Q <= 64 && a.k <= 4) launch_assign_t<512, 4>(a, F, st);
  else if (WB == 4) launch_assign_t<1024, 4>(a, F, st);
  else launch_assign_t<1024, 16>(a, F, st);
  return hipGetLastError();
}

}  // namespace hetumoe
