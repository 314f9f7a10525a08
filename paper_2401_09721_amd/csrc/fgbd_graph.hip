// Neighbour selection and edge weights of the scan-line graph (Sec. 2.2).
//
// k_merge: one thread per point i.  For each direction it looks up i's sorted
// position r (rank array from the last radix pass), reads the items at
// r-w..r+w inside the cloud's range of positions (the last pass stores each
// item's packed coordinates in place of its code, so no coordinate is
// gathered), and
// keeps the K smallest distinct (squared distance, index) pairs in a
// register-resident sorted list (packed so one integer compare orders by
// distance then index).  It writes the fixed-K CSR row, and each block adds
// its FP64 sum of edge lengths and its edge count into its cloud's exact
// integer sums for sigma_g; every block works on one cloud.
//
// k_weights: every block reads its cloud's sigma_g (the mean edge length of
// eq. 4's bandwidth rule) from those sums,
// then computes row-normalised Gaussian weights of eq. 4 in FP64 with the row's
// smallest squared distance subtracted in the exponent (same ratio, no
// underflow of the whole row), stored as float.  Squared-distance gaps are
// integers, so exp(-gap / sigma_g^2) comes from a per-block table for small
// gaps.  Both kernels are grid-stride over XCD-contiguous shares of points.
#include "fgbd_internal.h"

namespace fgbd {

namespace {

// Squared distance between two points from their packed coordinates
// (x | y << b | z << 2b, b = grid bits <= 10), the form in which the last radix
// pass stores the sorted items.  Every factor is below 2^11 in magnitude, so
// the products run on the full-rate 24-bit multiplier.
// a * b + c on the 24-bit multiplier (operands within +-2^23).  Written out
// because the compiler otherwise folds a 24-bit product and an add into a
// 64-bit multiply-add.
__device__ __forceinline__ int mad_i24(int a, int b, int c) {
  int d;
  asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
struct Pt {
  int x, y, z;
};
__device__ __forceinline__ Pt unpack_pt(uint32_t c, int bits) {
  return {(int)__builtin_amdgcn_ubfe(c, 0u, (uint32_t)bits), (int)__builtin_amdgcn_ubfe(c, (uint32_t)bits, (uint32_t)bits),
          (int)(c >> (2 * bits))};
}
__device__ __forceinline__ uint32_t pt_dist2(const Pt &pi, uint32_t cj, int bits) {
  const int dx = (int)__builtin_amdgcn_ubfe(cj, 0u, (uint32_t)bits) - pi.x;
  const int dy = (int)__builtin_amdgcn_ubfe(cj, (uint32_t)bits, (uint32_t)bits) - pi.y;
  const int dz = (int)(cj >> (2 * bits)) - pi.z;
  return (uint32_t)mad_i24(dx, dx, mad_i24(dy, dy, __mul24(dz, dz)));
}

template <int KM, typename Key>
__device__ __forceinline__ void topk_insert_t(Key (&lst)[KM], int K, Key c) {
  if (c >= lst[K - 1]) return;
  bool dup = false;
#pragma unroll
  for (int k = 0; k < KM; ++k) dup |= (k < K) & (lst[k] == c);
  if (dup) return;
#pragma unroll
  for (int k = KM - 1; k > 0; --k) {
    if (k < K) {
      const Key prev = lst[k - 1];
      lst[k] = prev > c ? prev : (lst[k] > c ? c : lst[k]);
    }
  }
  lst[0] = lst[0] > c ? c : lst[0];
}

// |a - b| - 1, all ones exactly when a == b (keys below 2^31 or all ones).
__device__ __forceinline__ uint32_t absdiff_m1(uint32_t a, uint32_t b) {
  uint32_t d;
  asm("v_sad_u32 %0, %1, %2, -1" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// Branch-free insertion into a sorted list of KM distinct keys (keys below
// 2^31; all ones = empty): the candidate is carried down the list, each slot
// keeping the smaller of (slot, carried) and passing the larger on, and the
// largest falls off the end.  A candidate equal to a slot is turned into the
// all-ones sentinel when it meets that slot (earlier slots are smaller, so it
// meets it before any swap), which leaves the list unchanged: the carried
// value is max(slot, carried, |slot - carried| - 1), and the third term is
// all ones only for equal keys and below the larger key otherwise.  Three
// instructions per slot.  The first K slots are then the K smallest
// distinct keys for any K <= KM.
template <int KM>
__device__ __forceinline__ void topk_insert_minmax(uint32_t (&lst)[KM], uint32_t c) {
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    const uint32_t l = lst[k];
    const uint32_t e = absdiff_m1(l, c);
    lst[k] = min(l, c);
    c = max(max(l, c), e);
  }
}

// Median of three unsigned words in one instruction (the compiler forms it
// only from patterns with constants).  Vector registers only.
__device__ __forceinline__ uint32_t med3_u32(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t d;
  asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

// The same insertion with one median per slot: a candidate equal to a slot
// is first turned into the all-ones sentinel (eight equality tests whose
// results combine on the scalar unit), then slot k takes the median of the
// old slots k - 1 and k and the candidate, which shifts the list up from the
// candidate's place and drops the largest.
template <int KM>
__device__ __forceinline__ void topk_insert_med3(uint32_t (&lst)[KM], uint32_t c) {
  bool dup = false;
#pragma unroll
  for (int k = 0; k < KM; ++k) dup |= lst[k] == c;
  c = dup ? ~0u : c;
  uint32_t nw[KM];
  nw[0] = min(lst[0], c);
#pragma unroll
  for (int k = 1; k < KM; ++k) nw[k] = med3_u32(lst[k - 1], c, lst[k]);
#pragma unroll
  for (int k = 0; k < KM; ++k) lst[k] = nw[k];
}

// Sorts 8 keys ascending (a 19-comparator network of depth 6).
__device__ __forceinline__ void sort8(uint32_t (&v)[8]) {
  constexpr int net[19][2] = {{0, 2}, {1, 3}, {4, 6}, {5, 7}, {0, 4}, {1, 5}, {2, 6}, {3, 7}, {0, 1}, {2, 3},
                              {4, 5}, {6, 7}, {2, 4}, {3, 5}, {1, 4}, {3, 6}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int c = 0; c < 19; ++c) {
    const uint32_t x = v[net[c][0]], y = v[net[c][1]];
    v[net[c][0]] = min(x, y);
    v[net[c][1]] = max(x, y);
  }
}

// Window items r-WT..r+WT; positions outside lo..hi load a clamped position
// (branch-free, all loads in flight together) and are then marked empty.
template <int WT>
__device__ __forceinline__ void load_window(const uint64_t *__restrict__ srt, int r, int lo, int hi,
                                            uint64_t (&w)[2 * WT + 1]) {
#pragma unroll
  for (int s = 0; s <= 2 * WT; ++s) {
    const int pos = r + s - WT;
    w[s] = srt[min(max(pos, lo), hi)];
  }
#pragma unroll
  for (int s = 0; s <= 2 * WT; ++s) {
    const int pos = r + s - WT;
    if (pos < lo || pos > hi) w[s] = ~0ull;
  }
}

constexpr int kKeyIndexBits = 24;    // most index bits of the 31-bit keys (clouds of up to 2^24 points)
constexpr uint32_t kSqrtMax = 127;   // edge lengths up to its root come from a table

struct MergeArgs {
  DirTable dt;
  SegArgs sa;
  int64_t stride;  // items per direction (capacity)
  int32_t window, K;
  int32_t wide_rows;  // col and dist2 are aligned for 16-byte stores
  int32_t index_bits;   // of the sorted items (see Sorted); the wide kernels only
  uint64_t index_mask;
  int32_t *sort_done;   // host-mapped, NULL: not watched (see Run::sort_big)
  int32_t sort_seq;
};
// The sort before this launch has ended, so its flag is final: tells the host
// (an event recorded between the sort and the merge left the GPU idle for 5.7
// us on every call).
__device__ __forceinline__ void report_sort(const MergeArgs &a) {
  if (a.sort_done && blockIdx.x == 0 && threadIdx.x == 0)
    __hip_atomic_store(a.sort_done, a.sort_seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Exact (64-bit key) selection for one point, runtime window over positions
// lo..hi: used for every point of a cloud of more than 2^24 points and for
// the rare point whose 32-bit selection kept a clamped distance.
template <int KM>
__device__ void select_exact(const MergeArgs &a, int i, int lo, int hi, int window,
                             const uint64_t *__restrict__ sorted, const uint32_t *__restrict__ rank,
                             uint64_t (&lst)[KM]) {
#pragma unroll
  for (int k = 0; k < KM; ++k) lst[k] = ~0ull;
  for (int d = 0; d < a.dt.num_dirs; ++d) {
    const int r = (int)rank[(size_t)d * a.stride + i];
    const uint64_t *srt = sorted + (size_t)d * a.stride;
    const Pt pi = unpack_pt((uint32_t)(srt[r] >> 32), a.dt.bits);
    const int l = max(r - window, lo);
    const int h = min(r + window, hi);
    for (int rr = l; rr <= h; ++rr) {
      if (rr == r) continue;
      const uint64_t it = srt[rr];
      topk_insert_t<KM, uint64_t>(lst, a.K, ((uint64_t)pt_dist2(pi, (uint32_t)(it >> 32), a.dt.bits) << 32) | (uint32_t)it);
    }
  }
}

// Exact selection with a compile-time window on keys (d2 << 32 | index) held
// as doubles: positive doubles order as their bits do (d2 stays far below the
// exponent of infinity), and FP64 minimum and maximum are single full-width
// instructions, where a 64-bit integer exchange takes five.  Denormal keys
// (d2 below 2^20) pass through unchanged; the instructions are written out so
// that the compiler adds no quieting of its own.
__device__ __forceinline__ double min_f64(double a, double b) {
  double d;
  asm("v_min_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double max_f64(double a, double b) {
  double d;
  asm("v_max_f64 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ double key_f64(uint32_t hi, uint32_t lo) {
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
constexpr uint64_t kNoKey = 0x7fefffffffffffffull;  // the largest finite double: an empty slot
// The candidate goes down the sorted list, each slot keeping the smaller;
// one equal to a slot, or past every lane's last slot, changes nothing.
template <int KM>
__device__ __forceinline__ void insert_f64(double (&lst)[KM], double c) {
  if (__builtin_amdgcn_ballot_w64(c < lst[KM - 1]) == 0) return;  // uniform
  bool dup = false;
#pragma unroll
  for (int k = 0; k < KM; ++k) dup |= lst[k] == c;
  c = dup ? __builtin_bit_cast(double, kNoKey) : c;
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    const double l = lst[k];
    lst[k] = min_f64(l, c);
    c = max_f64(l, c);
  }
}
// Every direction's window is one batch of loads, as in k_merge.  Used where
// the 31-bit keys would not do: clouds of more than 2^24 points, a kept
// distance past their field (redone one candidate at a time, the few waves
// that hold one held up the whole launch: 115 us for 180k points with K = 16
// in 12 directions, 47 with this and the wider field), and rows that keep
// every candidate, line wraps among them (the paper's graph on 300k points:
// 25 -> 17 us).
template <int KM, int WT>
__device__ __forceinline__ void select_f64(const MergeArgs &a, int i, int lo, int hi,
                                           const uint64_t *__restrict__ sorted, const uint32_t *__restrict__ rank,
                                           uint64_t (&out)[KM]) {
  double lst[KM];
#pragma unroll
  for (int k = 0; k < KM; ++k) lst[k] = __builtin_bit_cast(double, kNoKey);
  constexpr int G = WT == 1 ? 4 : (WT == 2 ? 2 : 1);  // directions whose loads are in flight together
  const int L = a.dt.num_dirs;
  for (int d0 = 0; d0 < L; d0 += G) {
    int r[G];
    uint64_t w[G][2 * WT + 1];
#pragma unroll
    for (int g = 0; g < G; ++g) r[g] = (int)rank[(size_t)min(d0 + g, L - 1) * a.stride + i];
#pragma unroll
    for (int g = 0; g < G; ++g) load_window<WT>(sorted + (size_t)min(d0 + g, L - 1) * a.stride, r[g], lo, hi, w[g]);
    const Pt pi = unpack_pt((uint32_t)(w[0][WT] >> 32), a.dt.bits);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (d0 + g >= L) break;  // uniform
#pragma unroll
      for (int s = 0; s <= 2 * WT; ++s) {
        if (s == WT) continue;
        const uint32_t d2 = pt_dist2(pi, (uint32_t)(w[g][s] >> 32), a.dt.bits);
        insert_f64<KM>(lst, w[g][s] == ~0ull ? __builtin_bit_cast(double, kNoKey) : key_f64(d2, (uint32_t)w[g][s]));
      }
    }
  }
#pragma unroll
  for (int k = 0; k < KM; ++k) {
    const uint64_t u = __builtin_bit_cast(uint64_t, lst[k]);
    out[k] = u == kNoKey ? ~0ull : u;
  }
}

// One thread per point.  WT > 0 (compile-time window, clouds of at most 2^24
// points; a block of a larger cloud takes the 64-bit selection): the
// point's ranks in all directions go to LDS in one batch of loads; each
// direction's 2*WT+1 window items (the centre gives the point's own code) are
// then loaded as one batch and consumed (prefetching the next direction's
// window would raise the register count from 83 to 109 and the occupancy from
// six to four waves per SIMD, which measured slower); candidates are 31-bit
// keys (min(d2, max) << index bits | j - cloud start), exact whenever no kept entry has a clamped
// distance, else the point is redone with 64-bit keys.  With w = 4 each
// direction's 8 candidates are first sorted by a network: the first
// direction's (distinct points, empty list) are the list, and later ones are
// inserted in ascending order until no lane of the wave has one left that
// could enter its list.
// S > 1 (small clouds): S neighbouring lanes share a point, each selecting
// from every S-th direction, then exchange their lists (each inserts the
// other's): a wave's chain of window loads and insertions is S times shorter,
// which is what a launch of few waves per SIMD takes its time for (16k points:
// 24 us with S = 1, 15 with S = 4; 70k: 27 and 24; up to kMergeSmall points).
// ALL64: every point takes the 64-bit selection.
template <int KM, int WT, int S = 1, bool ALL64 = false>
__global__ __launch_bounds__(kBlock) void k_merge(MergeArgs a, const uint64_t *__restrict__ sorted,
                                                  const uint32_t *__restrict__ rank, int32_t *__restrict__ col,
                                                  int32_t *__restrict__ dist2,
                                                  unsigned long long *__restrict__ edge_acc) {
  __shared__ double s_red[4 * 3];  // block_sum_f64<3>: three doubles per wave
  __shared__ int s_rank[WT > 0 ? kMaxDirs : 1][kBlock];
  // edge lengths sqrt(d2) of the small squared distances, each computed once
  // per block (the same correctly rounded values as computing them inline)
  __shared__ double s_sqrt[kSqrtMax + 1];
  double acc[3] = {0.0, 0.0, 0.0};  // edge lengths, edges, far edges
  const int L = a.dt.num_dirs;
  const int K = a.K;
  const int bits = a.dt.bits;
  const int t = threadIdx.x;
  for (int v = t; v <= (int)kSqrtMax; v += kBlock) s_sqrt[v] = sqrt((double)v);
  const SegBlock sb = seg_block(a.sa, kGridMerge);
  const int lo = (int)sb.begin, hi = (int)sb.end - 1;
  // the 31-bit keys hold a cloud-local index in up to 24 bits: a cloud of more
  // than 2^24 points takes the 64-bit selection (uniform over the block)
  const bool fast = sb.end - sb.begin <= (int64_t)(1 << kKeyIndexBits);
  // the index takes as many bits as the cloud needs and the squared distance
  // the rest (7 bits for 2^24 points, 11 for 2^20), so that few rows hold a
  // distance that does not fit
  const int ib = max(1, 32 - __clz((int)min(sb.end - sb.begin, (int64_t)(1 << kKeyIndexBits)) - 1));
  const uint32_t d2_max = (1u << (31 - ib)) - 1u;
  const uint32_t gap = (uint32_t)far_gap(sb.end - sb.begin);  // an edge spanning more indices is far
  __syncthreads();
  const Share sh = seg_share(sb, kBlock / S);
  const int sub = S > 1 ? t % S : 0;
  for (int64_t base = sh.first; base < sh.end; base += sh.step) {
    const int i = (int)(base + t / S);
    if (i >= sh.end) continue;
    uint64_t lst[KM];
    if constexpr (ALL64) {
      select_f64<KM, WT>(a, i, lo, hi, sorted, rank, lst);
    } else if (WT > 0 && !fast) {
      if constexpr (WT > 0) select_f64<KM, WT>(a, i, lo, hi, sorted, rank, lst);
    } else if constexpr (WT > 0) {
      // the first 8 directions' ranks load unconditionally (a direction
      // index past L - 1 re-reads the last one) so all loads are in flight
      // together; a conditional load per direction would be waited for
      // before the next is issued
      int rv[8];
      if constexpr (S == 1) {
#pragma unroll
        for (int d = 0; d < 8; ++d) rv[d] = (int)rank[(size_t)min(d, L - 1) * a.stride + i];
#pragma unroll
        for (int d = 0; d < 8; ++d) s_rank[d][t] = rv[d];
        for (int d = 8; d < L; ++d) s_rank[d][t] = (int)rank[(size_t)d * a.stride + i];
      } else {  // the lane's own directions, sub, sub + S, ...
        constexpr int U = (kMaxDirs + S - 1) / S;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int v = (int)rank[(size_t)min(u * S + sub, L - 1) * a.stride + i];
          s_rank[u][t] = v;
          if (u == 0) rv[0] = v;
        }
      }
      uint32_t key[KM];
#pragma unroll
      for (int k = 0; k < KM; ++k) key[k] = ~0u;
      // the point's own packed coordinates (the same item in every order)
      const Pt pi = unpack_pt((uint32_t)(sorted[(size_t)(S > 1 ? min(sub, L - 1) : 0) * a.stride + rv[0]] >> 32), bits);
      for (int d0 = 0; d0 < L; d0 += S) {
        // (with S > 1, a lane past the last direction repeats that one: its
        // candidates are in the list already)
        const int d = S > 1 ? min(d0 + sub, L - 1) : d0;
        const uint64_t *srt = sorted + (size_t)d * a.stride;
        const int r = s_rank[S > 1 ? d0 / S : d][t];
        uint64_t cur[2 * WT + 1];
        uint32_t kc[2 * WT];
        // Wave-uniform: when every window of the wave lies inside the
        // cloud, the items load from one base address with no clamping and
        // no empty slots.
        if (__builtin_amdgcn_ballot_w64(r - WT < lo || r + WT > hi) == 0) {
          const uint64_t *wp = srt + (r - WT);
#pragma unroll
          for (int s = 0; s <= 2 * WT; ++s)
            if (s != WT) cur[s] = wp[s];
#pragma unroll
          for (int s = 0; s < 2 * WT; ++s) {
            const uint64_t it = cur[s < WT ? s : s + 1];
            const uint32_t d2 = pt_dist2(pi, (uint32_t)(it >> 32), bits);
            kc[s] = (min(d2, d2_max) << ib) | ((uint32_t)it - (uint32_t)lo);
          }
        } else {
          load_window<WT>(srt, r, lo, hi, cur);
#pragma unroll
          for (int s = 0; s < 2 * WT; ++s) {
            const uint64_t it = cur[s < WT ? s : s + 1];
            const uint32_t d2 = pt_dist2(pi, (uint32_t)(it >> 32), bits);
            kc[s] = it == ~0ull ? ~0u : ((min(d2, d2_max) << ib) | ((uint32_t)it - (uint32_t)lo));
          }
        }
        if constexpr (WT == 4) {
          sort8(kc);
          if (d0 == 0) {
#pragma unroll
            for (int k = 0; k < 8 && k < KM; ++k) key[k] = kc[k];
            continue;
          }
          // Sorted candidates: once no lane's next one is below its last
          // slot, none of the rest can enter any list (the slots only
          // decrease).
#pragma unroll
          for (int s = 0; s < 8; ++s) {
            if (__builtin_amdgcn_ballot_w64(kc[s] < key[KM - 1]) == 0) break;
            topk_insert_med3<KM>(key, kc[s]);
          }
        } else {
#pragma unroll
          for (int s = 0; s < 2 * WT; ++s) topk_insert_minmax<KM>(key, kc[s]);
        }
      }
      if constexpr (S > 1) {  // the lists of the point's other lanes
#pragma unroll
        for (int o = 1; o < S; o <<= 1) {
          uint32_t other[KM];
#pragma unroll
          for (int k = 0; k < KM; ++k) other[k] = (uint32_t)__shfl_xor((int)key[k], o, kWave);
#pragma unroll
          for (int k = 0; k < KM; ++k) {
            if (__builtin_amdgcn_ballot_w64(other[k] < key[KM - 1]) == 0) break;
            topk_insert_med3<KM>(key, other[k]);
          }
        }
      }
      bool clamped = false;
#pragma unroll
      for (int k = 0; k < KM; ++k) clamped |= (k < K) & (key[k] != ~0u) & ((key[k] >> ib) == d2_max);
      if (clamped) {
        select_f64<KM, WT>(a, i, lo, hi, sorted, rank, lst);
      } else {
#pragma unroll
        for (int k = 0; k < KM; ++k)
          lst[k] = key[k] == ~0u ? ~0ull : ((uint64_t)(key[k] >> ib) << 32) | ((key[k] & ((1u << ib) - 1u)) + (uint32_t)lo);
      }
    } else {
      select_exact<KM>(a, i, lo, hi, a.window, sorted, rank, lst);
    }
    int cv[KM], dv[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      const bool ok = lst[k] != ~0ull;
      const uint32_t d2 = (uint32_t)(lst[k] >> 32);
      cv[k] = ok ? (int32_t)(uint32_t)lst[k] : -1;

      dv[k] = ok ? (int32_t)d2 : 0;
      if (ok && k < K && sub == 0) {
        acc[0] += d2 <= kSqrtMax ? s_sqrt[d2] : sqrt((double)d2);
        acc[1] += 1.0;
        acc[2] += (uint32_t)abs(cv[k] - i) > gap ? 1.0 : 0.0;
      }
    }
    if constexpr (KM == 16 && S == 1) {
      if (K == 16 && a.wide_rows) {
        store_row<16>(col, (int64_t)i, 16, cv);
        store_row<16>(dist2, (int64_t)i, 16, dv);
        continue;
      }
    }
    if (S == 4 && KM == 8 && K == 8) {  // two of the eight slots per lane
      int c0 = cv[0], c1 = cv[1], e0 = dv[0], e1 = dv[1];
#pragma unroll
      for (int q = 1; q < 4; ++q) {
        c0 = sub == q ? cv[2 * q] : c0;
        c1 = sub == q ? cv[2 * q + 1] : c1;
        e0 = sub == q ? dv[2 * q] : e0;
        e1 = sub == q ? dv[2 * q + 1] : e1;
      }
      reinterpret_cast<int2 *>(col + (size_t)i * 8)[sub] = make_int2(c0, c1);
      reinterpret_cast<int2 *>(dist2 + (size_t)i * 8)[sub] = make_int2(e0, e1);
    } else if (S > 1) {
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        if (k < K && k % S == sub) {
          col[(size_t)i * K + k] = cv[k];
          dist2[(size_t)i * K + k] = dv[k];
        }
      }
    } else if (KM == 8 && K == 8) {
      int4 *cr = reinterpret_cast<int4 *>(col + (size_t)i * 8);
      int4 *dr = reinterpret_cast<int4 *>(dist2 + (size_t)i * 8);
      cr[0] = make_int4(cv[0], cv[1], cv[2], cv[3]);
      cr[1] = make_int4(cv[4], cv[5], cv[6], cv[7]);
      dr[0] = make_int4(dv[0], dv[1], dv[2], dv[3]);
      dr[1] = make_int4(dv[4], dv[5], dv[6], dv[7]);
    } else {
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        if (k < K) {
          col[(size_t)i * K + k] = cv[k];
          dist2[(size_t)i * K + k] = dv[k];
        }
      }
    }
  }
  report_sort(a);
  block_sum_f64<3>(acc, s_red);
  if (threadIdx.x == 0) {
    unsigned long long *e = edge_acc + ((size_t)sb.s * kEdgeSlots + sb.lb % kEdgeSlots) * kEdgeVals;
    const double whole = floor(acc[0]);  // acc[0] >= 0; the fraction below is exact
    atomicAdd(&e[0], (unsigned long long)whole);
    atomicAdd(&e[1], (unsigned long long)llrint((acc[0] - whole) * kEdgeFrac));
    atomicAdd(&e[2], (unsigned long long)acc[1]);
    atomicAdd(&e[3], (unsigned long long)acc[2]);
  }
}

// Selection for grids above 2^10 (codes wider than 32 bits) with keys
// (squared distance << index bits | index - cloud start) held as doubles, as
// in select_f64: a squared distance is below 3/4 of 2^(2b+2), so while
// 2b + 2 and the cloud's index bits make at most 63 the keys are positive
// finite doubles.  The candidates' coordinates are packed in the sorted items
// when the sort could hold them there (PACKED), else gathered from the input;
// a direction's eight candidates are one batch of loads, sorted by a network,
// and inserted until no lane's next one can enter.  BIG: squared distances of
// more than 32 bits (b > 15).  700k points at b = 11: 458 us with the general
// kernel below, 86 with this (139 with one 8-byte load per item: a capture
// that is not in raster order touches a line per lane with every load).
// 31-bit keys as in k_merge, the few points whose distances do not fit them
// selected again by the whole wave, took 88.
struct WidePt {
  int x, y, z;
};
template <bool BIG>
__device__ __forceinline__ uint64_t wide_dist2(const WidePt &p, const WidePt &q) {
  const int dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
  if constexpr (BIG) return (uint64_t)((int64_t)dx * dx + (int64_t)dy * dy + (int64_t)dz * dz);
  // (b <= 15: differences below 2^15 in magnitude, the sum below 3 * 2^30)
  return (uint32_t)mad_i24(dx, dx, mad_i24(dy, dy, __mul24(dz, dz)));
}
// The window without its centre.  When every window of the wave lies inside
// the cloud (uniform; returns true), the items load from one base address,
// two to a 16-byte load; else each position is clamped into lo..hi.
template <int WT>
__device__ __forceinline__ bool load_sides(const uint64_t *__restrict__ srt, int r, int lo, int hi,
                                           uint64_t (&w)[2 * WT]) {
  const bool inside = __builtin_amdgcn_ballot_w64(r - WT < lo || r + WT > hi) == 0;
  if (inside) {
    const uint64_t *wp = srt + (r - WT);
#pragma unroll
    for (int s = 0; s < 2 * WT; ++s) w[s] = wp[s < WT ? s : s + 1];
  } else {
#pragma unroll
    for (int s = 0; s < 2 * WT; ++s) w[s] = srt[min(max(r + (s < WT ? s : s + 1) - WT, lo), hi)];
  }
  return inside;
}
// Sorts 8 keys ascending (the network of sort8).
__device__ __forceinline__ void sort8_f64(double (&v)[8]) {
  constexpr int net[19][2] = {{0, 2}, {1, 3}, {4, 6}, {5, 7}, {0, 4}, {1, 5}, {2, 6}, {3, 7}, {0, 1}, {2, 3},
                              {4, 5}, {6, 7}, {2, 4}, {3, 5}, {1, 4}, {3, 6}, {1, 2}, {3, 4}, {5, 6}};
#pragma unroll
  for (int c = 0; c < 19; ++c) {
    const double x = v[net[c][0]], y = v[net[c][1]];
    v[net[c][0]] = min_f64(x, y);
    v[net[c][1]] = max_f64(x, y);
  }
}
template <int KM, bool PACKED, bool BIG>
__global__ __launch_bounds__(kBlock) void k_merge_wide4(MergeArgs a, const int32_t *__restrict__ xyz,
                                                        const uint64_t *__restrict__ sorted,
                                                        const uint32_t *__restrict__ rank, int32_t *__restrict__ col,
                                                        int32_t *__restrict__ dist2,
                                                        unsigned long long *__restrict__ edge_acc,
                                                        fgbd_result *__restrict__ res) {
  constexpr int WT = 4;
  __shared__ double s_red[4 * 3];
  __shared__ double s_sqrt[kSqrtMax + 1];
  __shared__ int s_rank[kMaxDirs][kBlock];  // the point's ranks, read in one batch
  const int t = threadIdx.x;
  for (int v = t; v <= (int)kSqrtMax; v += kBlock) s_sqrt[v] = sqrt((double)v);
  __syncthreads();
  double acc[3] = {0.0, 0.0, 0.0};  // edge lengths, edges, far edges
  const int L = a.dt.num_dirs, K = a.K, bits = a.dt.bits, ib = a.index_bits;
  const int top = (1 << bits) - 1;
  const SegBlock sb = seg_block(a.sa, kGridMerge);
  const int lo = (int)sb.begin, hi = (int)sb.end - 1;
  const int kb = 32 - __clz(max((int)(sb.end - sb.begin) - 1, 1));  // index bits of the keys
  const uint32_t gap = (uint32_t)far_gap(sb.end - sb.begin);
  auto unpack = [&](uint64_t v) {  // (PACKED items)
    if constexpr (!BIG) {  // b <= 15: ib + b is at least 32, so y and z lie in the upper word
      const uint32_t vl = (uint32_t)v, vh = (uint32_t)(v >> 32);
      return WidePt{(int)(__builtin_amdgcn_alignbit(vh, vl, (uint32_t)ib) & (uint32_t)top),
                    (int)__builtin_amdgcn_ubfe(vh, (uint32_t)(ib + bits - 32), (uint32_t)bits),
                    (int)(vh >> (ib + 2 * bits - 32))};
    }
    const uint64_t p = v >> ib;
    return WidePt{(int)((uint32_t)p & (uint32_t)top), (int)((uint32_t)(p >> bits) & (uint32_t)top),
                  (int)(uint32_t)(p >> (2 * bits))};
  };
  auto input = [&](uint32_t j) {
    return WidePt{xyz[3 * (size_t)j + 0], xyz[3 * (size_t)j + 1], xyz[3 * (size_t)j + 2]};
  };
  const double none = __builtin_bit_cast(double, kNoKey);
  int clamped = 0;
  const Share sh = seg_share(sb, kBlock);
  for (int64_t base = sh.first; base < sh.end; base += sh.step) {
    const int i = (int)(base + threadIdx.x);
    if (i >= sh.end) continue;
    double lst[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) lst[k] = none;
    const WidePt pi = input((uint32_t)i);
    {
      int rv[8];
#pragma unroll
      for (int d = 0; d < 8; ++d) rv[d] = (int)rank[(size_t)min(d, L - 1) * a.stride + i];
#pragma unroll
      for (int d = 0; d < 8; ++d) s_rank[d][t] = rv[d];
      for (int d = 8; d < L; ++d) s_rank[d][t] = (int)rank[(size_t)d * a.stride + i];
    }
    for (int d = 0; d < L; ++d) {
      const uint64_t *srt = sorted + (size_t)d * a.stride;
      const int r = s_rank[d][t];
      uint64_t w[2 * WT];
      const bool inside = load_sides<WT>(srt, r, lo, hi, w);
      WidePt q[2 * WT];
#pragma unroll
      for (int s = 0; s < 2 * WT; ++s) q[s] = PACKED ? unpack(w[s]) : input((uint32_t)(w[s] & a.index_mask));
      double c[2 * WT];
#pragma unroll
      for (int s = 0; s < 2 * WT; ++s) {
        const uint32_t j = ((uint32_t)w[s] & (uint32_t)a.index_mask) - (uint32_t)lo;
        const uint64_t d2 = wide_dist2<BIG>(q[s], pi);
        // (d2 << kb | j, by halves: kb is 1 to 31)
        if constexpr (BIG)
          c[s] = __builtin_bit_cast(double, d2 << kb | j);
        else
          c[s] = key_f64((uint32_t)d2 >> (32 - kb), (uint32_t)d2 << kb | j);
      }
      if (!inside) {
        // positions outside the cloud's range are no candidates
#pragma unroll
        for (int s = 0; s < 2 * WT; ++s) {
          const int pos = r + (s < WT ? s : s + 1) - WT;
          if (pos < lo || pos > hi) c[s] = none;
        }
      }
      sort8_f64(c);
      if (d == 0) {
#pragma unroll
        for (int k = 0; k < 8 && k < KM; ++k) lst[k] = c[k];
        continue;
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if (__builtin_amdgcn_ballot_w64(c[s] < lst[KM - 1]) == 0) break;
        insert_f64<KM>(lst, c[s]);
      }
    }
    int cv[KM], dv[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      const uint64_t u = __builtin_bit_cast(uint64_t, lst[k]);
      const bool ok = u != kNoKey && k < K;
      const uint64_t d2 = u >> kb;
      cv[k] = ok ? (int32_t)(((uint32_t)u & ((1u << kb) - 1u)) + (uint32_t)lo) : -1;
      dv[k] = ok ? (d2 > 0x7fffffffull ? 0x7fffffff : (int32_t)d2) : 0;
      if (ok) {
        clamped |= d2 > 0x7fffffffull;
        acc[0] += d2 <= kSqrtMax ? s_sqrt[d2] : sqrt((double)d2);
        acc[1] += 1.0;
        acc[2] += (uint32_t)abs(cv[k] - i) > gap ? 1.0 : 0.0;
      }
    }
    if (K == KM && a.wide_rows) {
      store_row<KM>(col, (int64_t)i, KM, cv);
      store_row<KM>(dist2, (int64_t)i, KM, dv);
    } else {
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        if (k < K) {
          col[(size_t)i * K + k] = cv[k];
          dist2[(size_t)i * K + k] = dv[k];
        }
      }
    }
  }
  if (__builtin_amdgcn_ballot_w64(clamped != 0) != 0 && lane_id() == 0)
    atomicOr(&res[sb.s].status, FGBD_ST_DIST_CLAMPED);
  report_sort(a);
  block_sum_f64<3>(acc, s_red);
  if (threadIdx.x == 0) {
    unsigned long long *e = edge_acc + ((size_t)sb.s * kEdgeSlots + sb.lb % kEdgeSlots) * kEdgeVals;
    const double whole = floor(acc[0]);
    atomicAdd(&e[0], (unsigned long long)whole);
    atomicAdd(&e[1], (unsigned long long)llrint((acc[0] - whole) * kEdgeFrac));
    atomicAdd(&e[2], (unsigned long long)acc[1]);
    atomicAdd(&e[3], (unsigned long long)acc[2]);
  }
}

// The general selection for grids above 2^10: any window and K, clouds whose
// indices do not fit beside the distance.  Each candidate's coordinates come
// from the input; squared distances are 64-bit and the K nearest are kept by
// (squared distance, index) in a sorted list of pairs.  One thread per point,
// runtime window.  dist2 saturates at 2^31 - 1 (FGBD_ST_DIST_CLAMPED), which
// only a neighbour more than 46340 voxels away can reach.
template <int KM>
__global__ __launch_bounds__(kBlock) void k_merge_wide(MergeArgs a, const int32_t *__restrict__ xyz,
                                                       const uint64_t *__restrict__ sorted,
                                                       const uint32_t *__restrict__ rank, int32_t *__restrict__ col,
                                                       int32_t *__restrict__ dist2,
                                                       unsigned long long *__restrict__ edge_acc,
                                                       fgbd_result *__restrict__ res) {
  __shared__ double s_red[4 * 3];
  double acc[3] = {0.0, 0.0, 0.0};  // edge lengths, edges, far edges
  const int L = a.dt.num_dirs;
  const int K = a.K;
  const SegBlock sb = seg_block(a.sa, kGridMerge);
  const int lo = (int)sb.begin, hi = (int)sb.end - 1;
  const uint32_t gap = (uint32_t)far_gap(sb.end - sb.begin);
  int clamped = 0;
  const Share sh = seg_share(sb, kBlock);
  for (int64_t base = sh.first; base < sh.end; base += sh.step) {
    const int i = (int)(base + threadIdx.x);
    if (i >= sh.end) continue;
    const int64_t px = xyz[3 * (size_t)i + 0], py = xyz[3 * (size_t)i + 1], pz = xyz[3 * (size_t)i + 2];
    uint64_t kd[KM];
    uint32_t kj[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      kd[k] = ~0ull;
      kj[k] = ~0u;
    }
    for (int d = 0; d < L; ++d) {
      const uint64_t *srt = sorted + (size_t)d * a.stride;
      const int r = (int)rank[(size_t)d * a.stride + i];
      const int l = max(r - a.window, lo), h = min(r + a.window, hi);
      for (int rr = l; rr <= h; ++rr) {
        if (rr == r) continue;
        const uint32_t j = (uint32_t)(srt[rr] & a.index_mask);
        const int64_t dx = xyz[3 * (size_t)j + 0] - px, dy = xyz[3 * (size_t)j + 1] - py,
                      dz = xyz[3 * (size_t)j + 2] - pz;
        uint64_t cd = (uint64_t)(dx * dx + dy * dy + dz * dz);
        uint32_t cj = j;
        // insert (cd, cj) into the list ordered by (distance, index), once
        bool dup = false;
#pragma unroll
        for (int k = 0; k < KM; ++k) dup |= kd[k] == cd && kj[k] == cj;
        if (dup) continue;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
          const bool less = cd < kd[k] || (cd == kd[k] && cj < kj[k]);
          const uint64_t td = kd[k];
          const uint32_t tj = kj[k];
          kd[k] = less ? cd : td;
          kj[k] = less ? cj : tj;
          cd = less ? td : cd;
          cj = less ? tj : cj;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < KM; ++k) {
      if (k >= K) continue;
      const bool ok = kj[k] != ~0u;
      int32_t dv = 0;
      if (ok) {
        dv = kd[k] > 0x7fffffffull ? 0x7fffffff : (int32_t)kd[k];
        clamped |= kd[k] > 0x7fffffffull;
        acc[0] += sqrt((double)kd[k]);
        acc[1] += 1.0;
        acc[2] += (uint32_t)abs((int)kj[k] - i) > gap ? 1.0 : 0.0;
      }
      col[(size_t)i * K + k] = ok ? (int32_t)kj[k] : -1;
      dist2[(size_t)i * K + k] = dv;
    }
  }
  if (__builtin_amdgcn_ballot_w64(clamped != 0) != 0 && lane_id() == 0)
    atomicOr(&res[sb.s].status, FGBD_ST_DIST_CLAMPED);
  report_sort(a);
  block_sum_f64<3>(acc, s_red);
  if (threadIdx.x == 0) {
    unsigned long long *e = edge_acc + ((size_t)sb.s * kEdgeSlots + sb.lb % kEdgeSlots) * kEdgeVals;
    const double whole = floor(acc[0]);
    atomicAdd(&e[0], (unsigned long long)whole);
    atomicAdd(&e[1], (unsigned long long)llrint((acc[0] - whole) * kEdgeFrac));
    atomicAdd(&e[2], (unsigned long long)acc[1]);
    atomicAdd(&e[3], (unsigned long long)acc[2]);
  }
}

// Renumbering of a cloud along scan order 0, for clouds whose kept edges
// mostly span more than far_gap input indices (an input order far from
// spatial, where every gather of the noise estimate and the sweeps would touch
// its own cache line): row r of col_w / dist2_w is the row of the point at
// position r of scan order 0, each neighbour replaced by its own position, and
// rgb_w[r] is that point's colour.  The rows keep their neighbours and their
// order (the selection broke ties by input index).  Runs on the merge grid; a
// cloud left as it is returns at once.
template <int KT>
__global__ __launch_bounds__(kBlock) void k_relabel(SegArgs sa, int32_t k_rt, Segs *__restrict__ order,
                                                    const unsigned long long *__restrict__ edge_acc,
                                                    const uint64_t *__restrict__ sorted0, uint64_t index_mask,
                                                    const uint32_t *__restrict__ rank0,
                                                    const int32_t *__restrict__ col, const int32_t *__restrict__ dist2,
                                                    const float *__restrict__ rgb, int32_t *__restrict__ col_w,
                                                    int32_t *__restrict__ dist2_w, float *__restrict__ rgb_w) {
  const int K = KT > 0 ? KT : k_rt;
  const SegBlock sb = seg_block(sa, kGridMerge);
  __shared__ unsigned long long s_u[kEdgeVals];
  if (threadIdx.x < kWave) {  // the cloud's edge and far-edge counts over its slots
    static_assert(kEdgeSlots == kWave, "one slot per lane");
    const unsigned long long *e = edge_acc + ((size_t)sb.s * kEdgeSlots + threadIdx.x) * kEdgeVals;
    unsigned long long all = e[2], far = e[3];
    for (int o = 32; o > 0; o >>= 1) {
      all += __shfl_xor(all, o, kWave);
      far += __shfl_xor(far, o, kWave);
    }
    if (threadIdx.x == 0) {
      s_u[0] = all;
      s_u[1] = far;
    }
  }
  __syncthreads();
  if (s_u[0] == 0 || 4ull * s_u[1] <= s_u[0]) return;  // uniform over the block
  if (sb.lb == 0 && threadIdx.x == 0) order->relabel[sb.s] = 1;
  const Share sh = seg_share(sb, kBlock);
  for (int64_t base = sh.first; base < sh.end; base += sh.step) {
    const int64_t r = base + threadIdx.x;
    if (r >= sh.end) continue;
    const int64_t i = (uint32_t)(sorted0[r] & index_mask);  // the point at position r
    rgb_w[3 * r + 0] = rgb[3 * i + 0];
    rgb_w[3 * r + 1] = rgb[3 * i + 1];
    rgb_w[3 * r + 2] = rgb[3 * i + 2];
    if (KT == 8) {
      const int4 *cr = reinterpret_cast<const int4 *>(col + i * 8);
      const int4 *dr = reinterpret_cast<const int4 *>(dist2 + i * 8);
      const int4 c0 = cr[0], c1 = cr[1];
      int cv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
      for (int k = 0; k < 8; ++k) cv[k] = cv[k] >= 0 ? (int)rank0[cv[k]] : -1;
      int4 *cw = reinterpret_cast<int4 *>(col_w + r * 8);
      int4 *dw = reinterpret_cast<int4 *>(dist2_w + r * 8);
      cw[0] = make_int4(cv[0], cv[1], cv[2], cv[3]);
      cw[1] = make_int4(cv[4], cv[5], cv[6], cv[7]);
      dw[0] = dr[0];
      dw[1] = dr[1];
    } else {
      for (int k = 0; k < K; ++k) {
        const int c = col[i * K + k];
        col_w[r * K + k] = c >= 0 ? (int)rank0[c] : -1;
        dist2_w[r * K + k] = dist2[i * K + k];
      }
    }
  }
}

// Runs on the merge grid: block b belongs to the same cloud as merge block b.
template <int KT>
__global__ __launch_bounds__(kBlock) void k_weights(SegArgs sa, int32_t k_rt, int32_t vec,
                                                    const int32_t *__restrict__ col,
                                                    const int32_t *__restrict__ dist2,
                                                    const unsigned long long *__restrict__ edge_acc,
                                                    double sigma_g_fixed,
                                                    fgbd_result *__restrict__ res, float *__restrict__ p) {
  __shared__ double s_red[8];
  __shared__ double s_exp[kExpTable];
  const int K = KT > 0 ? KT : k_rt;
  const SegBlock sb = seg_block(sa, kGridMerge);
  const double sg = cloud_sigma_g(edge_acc + (size_t)kEdgeSlots * kEdgeVals * sb.s, sigma_g_fixed,
                                  reinterpret_cast<unsigned long long *>(s_red));
  if (sb.lb == 0 && threadIdx.x == 0) res[sb.s].sigma_g = sg;
  fill_exp_table(sg, s_exp);
  __syncthreads();
  constexpr int KB = row_cap(KT);
  const Share sh = seg_share(sb, kBlock);
  for (int64_t base = sh.first; base < sh.end; base += sh.step) {
    const int64_t i = base + threadIdx.x;
    if (i >= sh.end) continue;
    int cv[KB], dv[KB];
    load_row<KT>(col, i, K, vec, -1, cv);
    load_row<KT>(dist2, i, K, vec, 0, dv);
    float pw[KB];
    row_weights<KB>(cv, dv, sg, s_exp, pw);
    store_row<KT>(p, i, K, pw);
  }
}

}  // namespace

hipError_t launch_merge(const Run &r, const int32_t *xyz, const Sorted &srt, int32_t *col, int32_t *dist2,
                        fgbd_result *res) {
  const uint64_t *sorted = srt.items;
  MergeArgs a;
  a.dt = r.dt;
  a.sa = r.sa;
  a.stride = r.pl.stride;
  a.window = r.prm.window;
  a.wide_rows = common_align(col, dist2) >= 16;
  a.K = r.prm.k;
  const int k = r.prm.k, window = r.prm.window;
  const int nb = r.pl.grid[kGridMerge];
  const uint32_t *rank = r.b.rank;
  unsigned long long *part = r.b.edge_acc;
  hipStream_t st = r.stream;
  a.index_bits = srt.index_bits;
  a.index_mask = srt.index_mask();
  a.sort_done = r.sort_big ? r.sort_big + 1 : nullptr;
  a.sort_seq = r.sort_seq;
  if (r.dt.passes > kSortPasses) {  // codes above 32 bits
    int kb = 1;  // index bits of the largest cloud the call may hold
    while (((int64_t)1 << kb) < r.pl.n_cap) ++kb;
    // keys of at most 63 bits; other windows and longer rows are left to the
    // general kernel (700k points at b = 11, K = 8: 86 us here, 458 there)
    if (window == 4 && k <= 16 && 2 * r.dt.bits + 2 + kb <= 63 && kb < 32) {
      using Fn = void (*)(MergeArgs, const int32_t *, const uint64_t *, const uint32_t *, int32_t *, int32_t *,
                          unsigned long long *, fgbd_result *);
      // [K > 8][packed][b > 15]
      static const Fn table[2][2][2] = {
          {{k_merge_wide4<8, false, false>, k_merge_wide4<8, false, true>},
           {k_merge_wide4<8, true, false>, k_merge_wide4<8, true, true>}},
          {{k_merge_wide4<16, false, false>, k_merge_wide4<16, false, true>},
           {k_merge_wide4<16, true, false>, k_merge_wide4<16, true, true>}}};
      table[k > 8][srt.index_bits > 0][r.dt.bits > 15]<<<nb, kBlock, 0, st>>>(a, xyz, sorted, rank, col, dist2, part,
                                                                               res);
      return hipGetLastError();
    }
    if (k <= 8)
      k_merge_wide<8><<<nb, kBlock, 0, st>>>(a, xyz, sorted, rank, col, dist2, part, res);
    else if (k <= 16)
      k_merge_wide<16><<<nb, kBlock, 0, st>>>(a, xyz, sorted, rank, col, dist2, part, res);
    else
      k_merge_wide<32><<<nb, kBlock, 0, st>>>(a, xyz, sorted, rank, col, dist2, part, res);
    return hipGetLastError();
  }
  // the compile-time-window kernels take 64-bit keys for a cloud of more
  // than 2^24 points (their 31-bit keys hold a cloud-local index); a graph
  // that keeps every candidate keeps line wraps, whose distances need the
  // 64-bit keys
  const bool small = merge_lanes(r.pl.n_cap, r.prm) > 1;
  const bool keeps_all = 2 * window * r.dt.num_dirs <= k;
  using Fn = void (*)(MergeArgs, const uint64_t *, const uint32_t *, int32_t *, int32_t *, unsigned long long *);
  Fn fn = k_merge<32, 0>;
  if (k <= 8 && window == 4)
    fn = small ? k_merge<8, 4, kMergeLanes> : k_merge<8, 4>;
  else if (k <= 8 && window == 1)
    fn = keeps_all ? k_merge<8, 1, 1, true> : k_merge<8, 1>;
  else if (k <= 8 && window == 2)
    fn = keeps_all ? k_merge<8, 2, 1, true> : k_merge<8, 2>;
  else if (k <= 8)
    fn = k_merge<8, 0>;
  else if (k <= 16 && window == 4)
    fn = small ? k_merge<16, 4, kMergeLanes> : k_merge<16, 4>;
  else if (k <= 16)
    fn = k_merge<16, 0>;
  fn<<<nb, kBlock, 0, st>>>(a, sorted, rank, col, dist2, part);
  return hipGetLastError();
}

hipError_t launch_relabel(const Run &r, const Sorted &sorted, const int32_t *col, const int32_t *dist2,
                          const float *rgb) {
  if (!r.relabel_ok) return hipSuccess;
  const int nb = r.pl.grid[kGridMerge];
  if (r.prm.k == 8)
    k_relabel<8><<<nb, kBlock, 0, r.stream>>>(r.sa, 8, r.b.segs, r.b.edge_acc, sorted.items, sorted.index_mask(),
                                              r.b.rank, col, dist2, rgb, r.b.col_w, r.b.dist2_w, r.b.rgb_w);
  else
    k_relabel<0><<<nb, kBlock, 0, r.stream>>>(r.sa, r.prm.k, r.b.segs, r.b.edge_acc, sorted.items,
                                              sorted.index_mask(), r.b.rank, col, dist2, rgb, r.b.col_w, r.b.dist2_w,
                                              r.b.rgb_w);
  return hipGetLastError();
}

hipError_t launch_weights(const Run &r, const int32_t *col, const int32_t *dist2, fgbd_result *res, float *p) {
  const int nb = r.pl.grid[kGridMerge];
  const size_t align = common_align(col, dist2, p);
  const int k = r.prm.k, vec = row_vec(k, align);
  using Fn = void (*)(SegArgs, int32_t, int32_t, const int32_t *, const int32_t *, const unsigned long long *, double,
                      fgbd_result *, float *);
  static const Fn table[kNumRowKinds] = {k_weights<8>, k_weights<6>, k_weights<16>, k_weights<-8>, k_weights<-16>,
                                         k_weights<-32>};
  table[row_kind(k, align)]<<<nb, kBlock, 0, r.stream>>>(r.sa, k, vec, col, dist2, r.b.edge_acc, r.prm.sigma_g, res, p);
  return hipGetLastError();
}

}  // namespace fgbd
