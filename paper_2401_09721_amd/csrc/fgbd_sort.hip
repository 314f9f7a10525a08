// Scan-line codes and the radix sort of Sec. 2.2 (the paper orders the
// points of each code with a radix sort).  One launch covers all L directions
// (grid.y = direction).  Items are 64-bit: code << 32 | point index, so each
// pass moves 8 bytes per item and ties (duplicate points) keep index order:
// the LSD passes are stable, and the top-digit route restores it.  That route,
// at the end of this file (one pass on the top 10 bits, then each window's
// buckets sorted in LDS), takes every code that leaves room for the index in
// 64 bits; the LSD passes below sort the others, and any code while the
// context has found very large ranges.
//
// Per 8-bit digit pass (4 passes for 32-bit codes):
//   upsweep   per tile digit histogram            -> hist[dir][tile][digit]
//   scan      exclusive prefix over (digit, tile)  -> global offsets, in place
//   downsweep stable rank inside the tile (wave-level match of digits with
//             64-bit ballots, per-wave counters in LDS), stage in LDS in digit
//             order, then write runs of equal digits to their global offsets.
// Pass 0 computes the codes from the int32 coordinates on the fly; the last
// pass also writes rank[dir][index] = sorted position, which the neighbour
// search uses to find each point's place in every order, and stores each
// sorted item with the point's packed coordinates (x | y << b | z << 2b) in
// place of its code.
//
// Grids above 2^10 (b = 11..21) give codes of up to 63 bits.  Items then carry
// the code 32 bits at a time: passes 0-3 sort by the low 32 bits, pass 3
// re-keys every item with the high bits of its code (made again from the
// point's coordinates), and passes 4.. sort by those (LSD over digit groups:
// the order is by the whole code).  The last pass then stores only the index
// (packed coordinates no longer fit beside it) and the neighbour search reads
// coordinates from the input.
//
// Several clouds are sorted in the same launches, each inside its own range
// of positions: tiles never straddle two clouds, the scan runs over all tiles
// of each digit and also stores the total after the last tile, and with P the
// scanned counts of digit c, the cloud's count of c is P[next cloud's first
// tile] - P[its first tile], so each tile's output offset for digit c is
//   start[s] + (digits < c in cloud s) + (P[this tile] - P[cloud's first tile]).
#include <type_traits>

#include "fgbd_internal.h"

namespace fgbd {

namespace {

struct SortArgs {
  DirTable dt;
  SegArgs sa;
  int64_t stride;     // items per direction (capacity)
  int32_t row;        // hist row length (tile capacity + 1: the row total)
  int32_t shift;      // digit shift of this pass inside the item's 32 code bits
  int32_t pass;
  int32_t passes;     // passes of the sort (4, or more for codes above 32 bits)
  int32_t fold;       // pass 0 only: the first blocks also do the call's setup
  SetupArgs su;
  int32_t ib;         // top-digit pass: index bits of the items (32, or fewer for codes above 32 bits)
  int4 *win;          // top-digit pass: the range of each local-sort window (see k_msd_downsweep)
  int32_t nwin;       // windows per direction (the tiles' own numbering)
};

// The tile's cloud and point range; false for a tile beyond the last one.
struct TileInfo {
  int s;
  int begin, end;  // points of the tile
  int first;       // first tile of the cloud
  int next_first;  // first tile of the next cloud (= tile count after the last)
  int seg_start;   // first point of the cloud
};
__device__ __forceinline__ bool tile_info(const SegArgs &sa, int tile, TileInfo &ti) {
  if (sa.n_fixed >= 0) {
    const int n = sa.n_fixed;
    if (tile * kSortTile >= n) return false;
    ti.s = 0;
    ti.first = 0;
    ti.next_first = (n + kSortTile - 1) / kSortTile;
    ti.seg_start = 0;
    ti.begin = tile * kSortTile;
    ti.end = min(ti.begin + kSortTile, n);
    return true;
  }
  const Segs *sg = sa.segs;
  if (tile >= sg->ntiles) return false;
  const int s = seg_lookup(sg->tile_first, sa.B, tile);
  ti.s = s;
  ti.first = sg->tile_first[s];
  ti.next_first = sg->tile_first[s + 1];
  ti.seg_start = sg->start[s];
  ti.begin = ti.seg_start + (tile - ti.first) * kSortTile;
  ti.end = min(ti.begin + kSortTile, (int)sg->start[s + 1]);
  return true;
}

// (direction, tile) of a block (grid.x = tiles, grid.y = directions):
// workgroups go to the 8 XCDs round robin, so block b runs on XCD b % 8; each
// XCD gets one contiguous range of the tile-major sequence (tile, direction),
// so it works on a contiguous range of tiles in every direction.  The L
// directions of one tile run back to back on one XCD, so pass 0 reads the
// tile's coordinates from memory once and from L2 after, and the runs that
// consecutive tiles write side by side for each digit meet in one L2 before
// they are written back.
__device__ __forceinline__ void xcd_tile(int &d, int &tile) {
  const int nb = (int)(gridDim.x * gridDim.y);
  const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int x = b % kXcds, k = b / kXcds;
  const int g = x * (nb / kXcds) + min(x, nb % kXcds) + k;
  d = g % (int)gridDim.y;
  tile = g / (int)gridDim.y;
}

// The last pass instead gives each XCD one contiguous range of the
// direction-major sequence (direction, tile): with 8 directions each XCD
// sorts one direction, so its scattered rank writes land in one array of
// 4 bytes per point (measured slightly faster than the tile-major ranges).
__device__ __forceinline__ void xcd_tile_last(int &d, int &tile) {
  const int nb = (int)(gridDim.x * gridDim.y);
  const int b = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  const int x = b % kXcds, k = b / kXcds;
  const int g = x * (nb / kXcds) + min(x, nb % kXcds) + k;
  d = g / (int)gridDim.x;
  tile = g % (int)gridDim.x;
}

__device__ __forceinline__ int num_tiles(const SortArgs &a) {
  return a.sa.n_fixed >= 0 ? (a.sa.n_fixed + kSortTile - 1) / kSortTile : a.sa.segs->ntiles;
}

// The scan-line code of one direction (the same integers as scan_code), with
// the direction's constants read once per block: inside the item loops a
// reload from the argument segment would wait on the LDS atomics too.
struct CodeGen {
  int ia, ih, im, uh, um, wm, bits;
  int sa, sh, sm;  // where the axes a, h, m sit in packed coordinates
  uint32_t oh, om;
};
__device__ __forceinline__ CodeGen code_gen(const DirTable &dt, int d) {
  const DirInfo di = dt.d[d];
  const uint32_t top = (1u << dt.bits) - 1u;
  CodeGen c;
  c.ia = di.a;
  c.ih = di.h;
  c.im = di.m;
  c.uh = di.uh;
  c.um = di.um;
  c.oh = di.uh > 0 ? (uint32_t)di.uh * top : 0u;
  c.om = di.um > 0 ? (uint32_t)di.um * top : 0u;
  c.wm = dt.bits + di.wm_extra;
  c.bits = dt.bits;
  c.sa = di.a * dt.bits;
  c.sh = di.h * dt.bits;
  c.sm = di.m * dt.bits;
  return c;
}
__device__ __forceinline__ uint32_t gen_code(const CodeGen &c, int gx, int gy, int gz) {
  const int ga = c.ia == 0 ? gx : (c.ia == 1 ? gy : gz);
  const int gh = c.ih == 0 ? gx : (c.ih == 1 ? gy : gz);
  const int gm = c.im == 0 ? gx : (c.im == 1 ? gy : gz);
  const uint32_t eh = (uint32_t)(gh - c.uh * ga) + c.oh;
  const uint32_t em = (uint32_t)(gm - c.um * ga) + c.om;
  return (((eh << c.wm) + em) << c.bits) | (uint32_t)ga;
}

// The code's bits above 32 (codes of grids above 2^10).
__device__ __forceinline__ uint32_t gen_code_hi(const CodeGen &c, int gx, int gy, int gz) {
  const int ga = c.ia == 0 ? gx : (c.ia == 1 ? gy : gz);
  const int gh = c.ih == 0 ? gx : (c.ih == 1 ? gy : gz);
  const int gm = c.im == 0 ? gx : (c.im == 1 ? gy : gz);
  const uint64_t eh = (uint32_t)(gh - c.uh * ga) + c.oh;
  const uint64_t em = (uint32_t)(gm - c.um * ga) + c.om;
  return (uint32_t)((((eh << c.wm) + em) << c.bits | (uint32_t)ga) >> 32);
}

// The inverse of gen_code, packed as x | y << b | z << 2b (b = grid bits).
__device__ __forceinline__ uint32_t decode_packed(const CodeGen &c, uint32_t code) {
  const uint32_t top = (1u << c.bits) - 1u;
  const int ga = (int)(code & top);
  const int em = (int)((code >> c.bits) & ((1u << c.wm) - 1u));
  const int eh = (int)(code >> (c.bits + c.wm));
  const int gm = em + c.um * ga - (int)c.om;
  const int gh = eh + c.uh * ga - (int)c.oh;
  return ((uint32_t)ga << c.sa) | ((uint32_t)gh << c.sh) | ((uint32_t)gm << c.sm);
}

// 64-bit shifts by launch constants on 32-bit halves: the instruction that
// shifts 64 bits at once runs at a quarter of the rate.
__device__ __forceinline__ uint32_t shr64_lo(uint64_t v, int s) {  // the low word of v >> s, 0 <= s < 64
  const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
  return s < 32 ? __builtin_amdgcn_alignbit(hi, lo, (uint32_t)s) : hi >> (s - 32);
}
__device__ __forceinline__ uint64_t shl64(uint32_t v, int s) {  // (uint64_t)v << s, 0 <= s < 64
  const uint32_t lo = s < 32 ? v << s : 0u;
  const uint32_t hi = s < 32 ? __builtin_amdgcn_alignbit(0u, v, (uint32_t)(32 - s) & 31u) : v << (s - 32);
  return (uint64_t)(s == 0 ? 0u : hi) << 32 | lo;
}

// The inverse for codes of any width that sit above ib index bits of an item:
// packed coordinates at the same place, the index kept.
__device__ __forceinline__ uint64_t decode_packed_wide(const CodeGen &c, uint64_t item, int ib) {
  const uint32_t top = (1u << c.bits) - 1u;
  const int ga = (int)(shr64_lo(item, ib) & top);
  const int em = (int)(shr64_lo(item, ib + c.bits) & ((1u << c.wm) - 1u));
  const int eh = (int)shr64_lo(item, ib + c.bits + c.wm);
  const int gm = em + c.um * ga - (int)c.om;
  const int gh = eh + c.uh * ga - (int)c.oh;
  return shl64((uint32_t)ga, ib + c.sa) | shl64((uint32_t)gh, ib + c.sh) | shl64((uint32_t)gm, ib + c.sm) |
         ((uint32_t)item & ((1u << ib) - 1u));
}

// The coordinates of a thread's items, kWave apart from position base, all in
// flight together: positions past the tile's end are clamped to its last
// point, as a load in a branch is waited for there (16 latencies one after
// the other were a quarter of the top-digit downsweep's time).
__device__ __forceinline__ void load_points(const int32_t *__restrict__ xyz, const TileInfo &ti, int base,
                                            int (&g)[kSortItems][3]) {
  const char *tile = reinterpret_cast<const char *>(point_at(xyz, ti.begin));
  const uint32_t at = (uint32_t)(base - ti.begin), last = (uint32_t)(ti.end - ti.begin) - 1u;
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    // (bytes: with the offset in elements the three loads were not one)
    const uint32_t off = 12u * min(at + (uint32_t)(j * kWave), last);
    const int32_t *p = reinterpret_cast<const int32_t *>(tile + off);
#pragma unroll
    for (int c = 0; c < 3; ++c) g[j][c] = p[c];
  }
}
// Non-zero for a point outside the 2^bits grid.
__device__ __forceinline__ int outside_grid(const int (&g)[3], int bits) {
  return (int)((uint32_t)(g[0] | g[1] | g[2]) & ~0u << bits);
}

// All blocks clear the first sweep's sums and the noise moment accumulators;
// block 0 builds the segment table:
// offsets clamped into a valid form (start[0] = 0, non-decreasing, at most
// n_cap), radix tiles per cloud, and each per-cloud grid's block ranges
// first(s) = floor(start[s] (G - B) / n) + s (at least one block per cloud).
__device__ __forceinline__ void setup_work(const SetupArgs &a, int block) {
  Segs *__restrict__ sg = a.sg;
  unsigned long long *__restrict__ sums1 = a.sums1;
  fgbd_result *__restrict__ res = a.res;
  __shared__ int64_t s_raw[kMaxSeg + 1];
  __shared__ int32_t s_start[kMaxSeg + 1], s_tf[kMaxSeg + 1];
  __shared__ int32_t s_bad;
  const int t = threadIdx.x;
  const int stride = a.blocks * (int)blockDim.x;
  for (int i = block * blockDim.x + t; i < 3 * a.sums_count; i += stride) sums1[i] = 0ull;
  for (int i = block * blockDim.x + t; i < a.noise_count; i += stride) a.noise_acc[i] = 0ull;
  for (int i = block * blockDim.x + t; i < a.edge_count; i += stride) a.edge_acc[i] = 0ull;
  if (block != 0) return;  // uniform over the block
  if (t < kMaxSeg) {
    sg->relabel[t] = 0;
    sg->sweep_barrier[t][0] = 0u;
  }
  const int B = a.B;
  if (t <= B) s_raw[t] = a.offsets ? a.offsets[t] : (t == 0 ? 0 : a.n_host);
  __syncthreads();
  if (t == 0) {
    int bad = s_raw[0] != 0;
    int64_t prev = 0;
    int32_t tiles = 0;
    s_start[0] = 0;
    for (int s = 1; s <= B; ++s) {
      int64_t v = s_raw[s];
      v = v < prev ? prev : v;
      v = v > a.n_cap ? a.n_cap : v;
      bad |= v != s_raw[s];
      s_start[s] = (int32_t)v;
      s_tf[s - 1] = tiles;
      tiles += (int32_t)((v - prev + kSortTile - 1) / kSortTile);
      prev = v;
    }
    s_tf[B] = tiles;
    s_bad = bad;
    sg->B = B;
    sg->n = s_start[B];
    sg->ntiles = tiles;
    sg->status = bad ? FGBD_ST_BAD_OFFSETS : 0;
  }
  __syncthreads();
  if (t <= B) {
    sg->start[t] = s_start[t];
    sg->tile_first[t] = s_tf[t];
    const int64_t n = s_start[B];
#pragma unroll
    for (int g = 0; g < kNumGrids; ++g) {
      const int G = a.grid[g];
      sg->blk_first[g][t] = t == B ? G : (n > 0 ? (int32_t)((int64_t)s_start[t] * (G - B) / n) + t : t);
    }
  }
  if (t < B && res && a.zero_result) {
    fgbd_result *r = res + t;
    r->sigma_est = 0.0;
    r->sigma_g = 0.0;
    r->loss = 0.0;
    r->q = 0;
    r->n_fslr = 0;
    r->n_eff = 0;
    r->status = (s_bad ? FGBD_ST_BAD_OFFSETS : 0) | (a.zero_result == 2 ? FGBD_ST_NO_PATCH : 0);
    r->sweeps = 0;
    r->m = 0;
  }
}

__global__ __launch_bounds__(256) void k_setup(SetupArgs a) { setup_work(a, (int)blockIdx.x); }

// Per-tile digit counts.  Pass 0 makes the codes from the coordinates;
// later passes read only the byte array of this pass's digits that the
// previous downsweep wrote beside the items (16 digits per thread, one
// 16-byte load).  The counts go to 8 LDS sub-histograms picked by lane
// (rows 257 words apart), so lanes of one atomic instruction that share a
// digit, or a bank, mostly hit different words; the 8 are summed at the end.
__global__ __launch_bounds__(kSortThreads) void k_sort_upsweep(SortArgs a, const int32_t *__restrict__ xyz,
                                                               const uint8_t *__restrict__ digits,
                                                               uint32_t *__restrict__ hist) {
  constexpr int kSub = 8, kSubStride = 257;
  __shared__ uint32_t s_hs[kSub * kSubStride];
  if (a.fold) {  // the call's setup, by the first blocks (no other work of this launch reads it)
    const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (lin < a.su.blocks) setup_work(a.su, lin);
  }
  int d, tile;
  xcd_tile(d, tile);
  TileInfo ti;
  if (!tile_info(a.sa, tile, ti)) return;  // uniform over the block
  const int t = threadIdx.x;
  for (int i = t; i < kSub * kSubStride; i += kSortThreads) s_hs[i] = 0;
  __syncthreads();
  uint32_t *s_h = s_hs + (lane_id() & (kSub - 1)) * kSubStride;
  if (a.pass == 0) {
    // every coordinate load of the thread is issued before the first count
    // (the LDS atomics would otherwise wait for each load in turn)
    const int wave = t / kWave;
    const int lane = (int)lane_id();
    const int base = ti.begin + wave * kWave * kSortItems + lane;
    int g[kSortItems][3];
    load_points(xyz, ti, base, g);  // (a tile holds at least one point)
    // Runs of equal digits are counted in registers and added once: with
    // the input in a raster order, the digit (low bits of the position
    // along the line) is often the same for a thread's items, and for every
    // lane of the wave, whose atomics on one word would serialise.
    const CodeGen cg = code_gen(a.dt, d);
    uint32_t run_digit = 0, run_count = 0;
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      if (base + j * kWave < ti.end) {
        const uint32_t digit = gen_code(cg, g[j][0], g[j][1], g[j][2]) & 255u;
        if (run_count != 0 && digit != run_digit) {
          atomicAdd(&s_h[run_digit], run_count);
          run_count = 0;
        }
        run_digit = digit;
        ++run_count;
      }
    }
    if (run_count != 0) atomicAdd(&s_h[run_digit], run_count);
  } else {
    // tile starts are multiples of 16 inside the direction's row (clouds
    // start at any position, so only the bytes of the tile are counted)
    const uint8_t *row = digits + (size_t)d * a.stride;
    const int p0 = ti.begin + 16 * t;
    if (p0 + 16 <= ti.end && (p0 & 15) == 0) {
      const uint4 q = *reinterpret_cast<const uint4 *>(row + p0);
      const uint32_t w[4] = {q.x, q.y, q.z, q.w};
      // runs of equal digits among the 16 consecutive items add once
      uint32_t rd = w[0] & 255u, rc = 0;
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const uint32_t dg = (w[j >> 2] >> (8 * (j & 3))) & 255u;
        if (dg != rd) {
          atomicAdd(&s_h[rd], rc);
          rc = 0;
        }
        rd = dg;
        ++rc;
      }
      atomicAdd(&s_h[rd], rc);
    } else {
      for (int j = 0; j < 16; ++j)
        if (p0 + j < ti.end) atomicAdd(&s_h[row[p0 + j]], 1u);
    }
  }
  __syncthreads();
  uint32_t c = 0;
#pragma unroll
  for (int k = 0; k < kSub; ++k) c += s_hs[k * kSubStride + t];
  hist[((size_t)d * a.row + tile) * 256 + t] = c;  // one 1 KB row per tile
}

// Exclusive prefix over tiles of every (direction, digit) count, and the
// total after the last tile (row ntiles).  The counts are stored tile-major,
// one row of BINS digits per tile, so every access is a contiguous row
// segment.  One block per (direction, 64 digits): lane = digit, the 16 waves
// split the tiles into 16 consecutive ranges; each wave sums its range with
// all loads of a chunk in flight, the waves' sums are scanned in LDS, and
// each wave writes its range's prefixes starting from the sums of the waves
// before it.
constexpr int kScanWaves = 16;
constexpr int kScanChunk = 16;  // tiles per wave per round trip
template <int BINS>
__global__ __launch_bounds__(kScanWaves * 64) void k_sort_scan(SortArgs a, uint32_t *__restrict__ hist) {
  __shared__ uint32_t s_sum[kScanWaves][kWave];
  constexpr int kGroups = BINS / kWave;
  const int d = blockIdx.x / kGroups;
  const int digit = (blockIdx.x % kGroups) * kWave + (int)lane_id();
  const int w = threadIdx.x / kWave;
  const int ntiles = num_tiles(a);
  const int per = (ntiles + kScanWaves - 1) / kScanWaves;
  const int t0 = w * per, t1 = min(t0 + per, ntiles);
  uint32_t *h = hist + (size_t)d * a.row * BINS + digit;  // h[tile * BINS]
  if (per <= kScanChunk) {  // (up to 256 tiles) one round trip: the counts stay in registers
    uint32_t v[kScanChunk];
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) v[j] = t0 + j < t1 ? h[(size_t)(t0 + j) * BINS] : 0u;
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) sum += v[j];
    s_sum[w][lane_id()] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
    for (int ww = 0; ww < kScanWaves; ++ww) {
      const uint32_t x = s_sum[ww][lane_id()];
      run += ww < w ? x : 0u;
      total += x;
    }
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) {
      if (t0 + j < t1) h[(size_t)(t0 + j) * BINS] = run;
      run += v[j];
    }
    if (w == kScanWaves - 1) h[(size_t)ntiles * BINS] = total;
    return;
  }
  uint32_t sum = 0;
  for (int c0 = t0; c0 < t1; c0 += kScanChunk) {
    uint32_t v[kScanChunk];
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) v[j] = c0 + j < t1 ? h[(size_t)(c0 + j) * BINS] : 0u;
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) sum += v[j];
  }
  s_sum[w][lane_id()] = sum;
  __syncthreads();
  uint32_t run = 0, total = 0;
  for (int ww = 0; ww < kScanWaves; ++ww) {
    const uint32_t x = s_sum[ww][lane_id()];
    run += ww < w ? x : 0u;
    total += x;
  }
  for (int c0 = t0; c0 < t1; c0 += kScanChunk) {
    uint32_t v[kScanChunk];
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) v[j] = c0 + j < t1 ? h[(size_t)(c0 + j) * BINS] : 0u;
#pragma unroll
    for (int j = 0; j < kScanChunk; ++j) {
      if (c0 + j < t1) h[(size_t)(c0 + j) * BINS] = run;
      run += v[j];
    }
  }
  if (w == kScanWaves - 1) h[(size_t)ntiles * BINS] = total;
}

// This pass's digit of an item (code << 32 | index).
__device__ __forceinline__ uint32_t digit_of(uint64_t item, int shift) {
  return __builtin_amdgcn_ubfe((uint32_t)(item >> 32), (uint32_t)shift, 8u);
}
// Bit b of x spread over the word: 0 or all ones.  Written out so the
// compiler keeps one sign-extending field extract instead of rebuilding the
// mask from compares.
__device__ __forceinline__ int32_t bit_mask(uint32_t x, int b) {
  int32_t m;
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(m) : "v"(x), "i"(b));
  return m;
}

// Exclusive scans of two uint32 per thread over a 256-thread block.
__device__ __forceinline__ void block_exclusive_scan2_256(uint32_t &v0, uint32_t &v1, uint32_t (*s_tmp)[4]) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x / kWave;
  uint32_t x0 = v0, x1 = v1;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y0 = __shfl_up(x0, o, kWave), y1 = __shfl_up(x1, o, kWave);
    if (lane >= (uint32_t)o) {
      x0 += y0;
      x1 += y1;
    }
  }
  if (lane == kWave - 1) {
    s_tmp[0][w] = x0;
    s_tmp[1][w] = x1;
  }
  __syncthreads();
  uint32_t b0 = 0, b1 = 0;
  for (int ww = 0; ww < w; ++ww) {
    b0 += s_tmp[0][ww];
    b1 += s_tmp[1][ww];
  }
  v0 = b0 + x0 - v0;
  v1 = b1 + x1 - v1;
}

__global__ __launch_bounds__(kSortThreads) void k_sort_downsweep(SortArgs a, const int32_t *__restrict__ xyz,
                                                                 const uint64_t *__restrict__ src,
                                                                 uint64_t *__restrict__ dst,
                                                                 const uint32_t *__restrict__ hist,
                                                                 uint8_t *__restrict__ digits,
                                                                 uint32_t *__restrict__ rank,
                                                                 fgbd_result *__restrict__ res) {
  __shared__ uint32_t s_wh[4][256];
  __shared__ uint32_t s_off[256];
  __shared__ uint32_t s_tmp[2][4];
  __shared__ uint64_t s_stage[kSortTile];

  int d, tile;
  if (a.pass == a.passes - 1)
    xcd_tile_last(d, tile);
  else
    xcd_tile(d, tile);
  TileInfo ti;
  if (!tile_info(a.sa, tile, ti)) return;  // uniform over the block
  const int t = threadIdx.x;
  const int wave = t / kWave;
  const int lane = (int)lane_id();
  const int valid = ti.end - ti.begin;

  s_wh[0][t] = 0;
  s_wh[1][t] = 0;
  s_wh[2][t] = 0;
  s_wh[3][t] = 0;
  // scanned counts of digit t: the cloud's count of t and this tile's offset
  // inside the cloud (the first cloud starts at column 0 with prefix 0)
  const uint32_t *hd = hist + (size_t)d * a.row * 256 + t;  // hd[tile * 256]: digit t of a tile row
  const uint32_t p_first = ti.first > 0 ? hd[(size_t)ti.first * 256] : 0u;
  uint32_t off_t = hd[(size_t)tile * 256] - p_first;
  uint32_t below_t = hd[(size_t)ti.next_first * 256] - p_first;  // becomes the exclusive prefix over digits

  uint64_t item[kSortItems];
  const CodeGen cg = code_gen(a.dt, d);
  const int base = ti.begin + wave * kWave * kSortItems + lane;
  int bad = 0;
  if (a.pass == 0) {
    int g[kSortItems][3];
    load_points(xyz, ti, base, g);
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      bad |= outside_grid(g[j], a.dt.bits);
      item[j] = (uint64_t)gen_code(cg, g[j][0], g[j][1], g[j][2]) << 32 | (uint32_t)(base + j * kWave);
    }
  } else {
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) item[j] = src[(size_t)d * a.stride + min(base + j * kWave, ti.end - 1)];
  }
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) item[j] = base + j * kWave < ti.end ? item[j] : ~0ull;
  // pass 0: coordinates outside the grid (flagged once, by direction 0)
  if (bad && d == 0) atomicOr(&res[ti.s].status, FGBD_ST_COORD_RANGE);
  __syncthreads();

  // Stable rank of each item among the equal digits of its wave: items are
  // visited in tile order (j major, lane minor within the wave).  The lanes
  // holding the same digit (its peers) are those that agree with it on all 8
  // ballots: with m = bit b of the digit spread over the word (0 or all
  // ones), a lane keeps ~(vote ^ m).  Each round every lane reads the wave's
  // count of its digit over the earlier rounds, and the first lane of each
  // group of peers then adds the group's size to it.  A wave's LDS
  // operations are performed in the order they are issued, so the rounds
  // need no wait between them: the reads are waited for once, after the last
  // round, and each item's rank is that count plus its peers in lower lanes.
  uint32_t rk[kSortItems], before[kSortItems];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t digit = digit_of(item[j], a.shift);
    int32_t m[8];
    uint64_t vote[8];
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      m[b] = bit_mask(digit, b);
      vote[b] = __builtin_amdgcn_ballot_w64(m[b] != 0);
    }
    uint32_t plo = ~0u, phi = ~0u;  // lanes that agree with this one in every bit
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      plo &= ~((uint32_t)vote[b] ^ (uint32_t)m[b]);
      phi &= ~((uint32_t)(vote[b] >> 32) ^ (uint32_t)m[b]);
    }
    const uint64_t peers = ((uint64_t)phi << 32) | plo;
    before[j] = count_below(peers);
    rk[j] = __hip_atomic_load(&s_wh[wave][digit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (before[j] == 0)
      __hip_atomic_fetch_add(&s_wh[wave][digit], (uint32_t)__popcll(peers), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
  }
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) rk[j] += before[j];
  __syncthreads();

  // per digit: exclusive over digits in the tile and (for the global
  // offset) over the cloud's digit totals; then each wave's start of the
  // digit in the staged tile (the tile's start of the digit plus the counts
  // of the waves before), and the global position of staged slot 0 of the
  // digit's run (its global offset minus its start in the tile, mod 2^32)
  {
    const uint32_t c0 = s_wh[0][t], c1 = s_wh[1][t], c2 = s_wh[2][t], c3 = s_wh[3][t];
    uint32_t in_tile = c0 + c1 + c2 + c3;
    block_exclusive_scan2_256(in_tile, below_t, s_tmp);
    s_wh[0][t] = in_tile;
    s_wh[1][t] = in_tile + c0;
    s_wh[2][t] = in_tile + c0 + c1;
    s_wh[3][t] = in_tile + c0 + c1 + c2;
    s_off[t] = (uint32_t)ti.seg_start + below_t + off_t - in_tile;
  }
  __syncthreads();

#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    const uint32_t digit = digit_of(item[j], a.shift);
    s_stage[s_wh[wave][digit] + rk[j]] = item[j];
  }
  __syncthreads();

  const bool last_pass = (a.pass == a.passes - 1);
  const bool wide = a.passes > kSortPasses;
  const bool rekey = wide && a.pass == kSortPasses - 1;  // the low 32 code bits are done
  uint64_t *out = dst + (size_t)d * a.stride;
  uint8_t *dig = digits + (size_t)d * a.stride;
  // Write-out in staged order: thread t takes slots t + 256 j, so each
  // store instruction of a wave covers 64 consecutive slots (runs of equal
  // digits go to consecutive global positions).  All slots' LDS reads are
  // issued before the first store (slots past the tile's items are read but
  // not stored).
  uint64_t st[kSortItems];
  uint32_t gp[kSortItems];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) st[j] = s_stage[t + j * kSortThreads];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) gp[j] = s_off[digit_of(st[j], a.shift)] + (uint32_t)(t + j * kSortThreads);
  if (last_pass) {
    // the sorted item keeps its index and carries the point's packed
    // coordinates instead of its code (the neighbour search's form); wide
    // codes keep the index only
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      if (t + j * kSortThreads < valid) {
        const uint32_t idx = (uint32_t)st[j];
        out[gp[j]] = wide ? (uint64_t)idx : ((uint64_t)decode_packed(cg, (uint32_t)(st[j] >> 32)) << 32) | idx;
        rank[(size_t)d * a.stride + idx] = gp[j];
      }
    }
  } else if (rekey) {
    // the item's key becomes the code's bits above 32
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      if (t + j * kSortThreads < valid) {
        const uint32_t idx = (uint32_t)st[j];
        const uint32_t hi =
            gen_code_hi(cg, xyz[3 * (size_t)idx + 0], xyz[3 * (size_t)idx + 1], xyz[3 * (size_t)idx + 2]);
        out[gp[j]] = ((uint64_t)hi << 32) | idx;
        dig[gp[j]] = (uint8_t)hi;  // the next pass's digit
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      if (t + j * kSortThreads < valid) {
        out[gp[j]] = st[j];
        dig[gp[j]] = (uint8_t)(st[j] >> (40 + a.shift));  // the next pass's digit
      }
    }
  }
}


// ------------------------------------------------------------ hybrid sort
// Codes of at most 32 bits (grids up to 2^10), and wider ones that leave room
// for the index in a 64-bit item (2^11 with 35-bit codes: 2^29 points; 2^13
// with 41: 2^23; see msd_index_bits), take a shorter route.  One
// pass on the kMsdBits most significant bits of each direction's code
// (upsweep, scan and downsweep as above, with 2^kMsdBits digits, the codes
// made from the coordinates) splits every cloud's points, in the order of the
// input's 64-point chunks, into buckets of equal top digit; the downsweep also records, from its counts,
// which buckets start in every window of kLocalWin of a cloud's sorted
// positions.
// k_local_sort then gives each window of a direction one block, which sorts
// the buckets that start in its window (up to the first bucket of the next
// window), by their codes less the smallest top digit's base.
// Buckets are ordered by their top digits already, so sorting a range by the
// whole code sorts each bucket and keeps the buckets in place; ties keep the
// MSD pass's order, and those of one chunk that it left out of index order
// are put right at the end.  The block writes the sorted items
// in their final form and rank, as the last LSD pass does.  A range of more
// than kLocalCap items ends in a bucket that reaches several windows, whose
// blocks sort it between them, each reading it all: fast for the planes of a
// scan (three floors of 90,000 points each beside 400,000 others on a 2^11
// grid: 305 us for the graph, 965 with a block alone on each and 538 with the
// LSD passes), slow where most of a large cloud has one top digit (a million
// points in one plane: 1.6 ms, 0.6 with the LSD passes), which a block then
// reports through a host-mapped flag so that the caller's context can choose
// the LSD passes for its next calls.
//
// In LDS a range of R items is sorted by counting: the codes, less the base,
// are split by their top 13 bits into bins (one LDS atomic per item gives its
// place in its bin, in no particular order), and each item's rank in its bin
// is the number of its bin's keys below its own, a key being the code's low
// bits and then the position in the range.  The bins are short (on the frames
// measured an item shares its bin with 5 to 12 others on average, at most
// about 230), lanes with neighbouring slots read the same keys, and nothing
// has to be matched across lanes: 20 M vector instructions per launch on the
// 1M frame against 32 M for three 8-bit LSD passes in LDS whose stable ranks
// came from 8 ballots per item and pass; 90 -> 64 us there, 410 -> 243 us on
// 8 clouds of 4.4M points, 81 -> 51 us on 421k points in 16 directions.
// Where a bin holds more than kMaxBin items, or the codes have few bits, the
// range takes stable 8-bit passes in LDS instead.
// Items stay in registers; 65 KB of LDS and 1024 threads let two blocks (all
// 32 waves) share a CU.

__device__ __forceinline__ int code_width(const DirTable &dt, int d) {
  const DirInfo di = dt.d[d];
  const uint32_t uh = (uint32_t)(di.uh < 0 ? -di.uh : di.uh);
  return 3 * dt.bits + (32 - __clz(uh)) + di.wm_extra;  // bit_length(0) = 0
}
__device__ __forceinline__ int msd_shift(const DirTable &dt, int d) {
  const int w = code_width(dt, d);
  return w > kMsdBits ? w - kMsdBits : 0;
}
// The top digit of a code (a field extract, so it stays below 2^kMsdBits
// even for the codes of coordinates outside the grid).
__device__ __forceinline__ uint32_t msd_digit(uint32_t code, int sh) {
  return __builtin_amdgcn_ubfe(code, (uint32_t)sh, (uint32_t)kMsdBits);
}

// Per-tile counts of the top digits, codes made from the coordinates (and
// the call's setup folded in, as in pass 0 of the LSD sort).
template <bool WIDE>
__global__ __launch_bounds__(kSortThreads) void k_msd_upsweep(SortArgs a, const int32_t *__restrict__ xyz,
                                                              uint32_t *__restrict__ hist) {
  constexpr int kSub = 4, kSubStride = kMsdBins + 1;
  __shared__ uint32_t s_hs[kSub * kSubStride];
  if (a.fold) {
    const int lin = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (lin < a.su.blocks) setup_work(a.su, lin);
  }
  int d, tile;
  xcd_tile(d, tile);
  TileInfo ti;
  if (!tile_info(a.sa, tile, ti)) return;  // uniform over the block
  const int t = threadIdx.x;
  for (int i = t; i < kSub * kSubStride; i += kSortThreads) s_hs[i] = 0;
  __syncthreads();
  uint32_t *s_h = s_hs + (lane_id() & (kSub - 1)) * kSubStride;
  const int wave = t / kWave;
  const int lane = (int)lane_id();
  const int base = ti.begin + wave * kWave * kSortItems + lane;
  int g[kSortItems][3];
  load_points(xyz, ti, base, g);
  const CodeGen cg = code_gen(a.dt, d);
  const int sh = msd_shift(a.dt, d);
  uint32_t run_digit = 0, run_count = 0;
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    if (base + j * kWave < ti.end) {
      uint32_t digit = 0;
      if (WIDE) {  // the digit sits at bits sh .. sh + 9 of the whole code
        const uint64_t code =
            (uint64_t)gen_code_hi(cg, g[j][0], g[j][1], g[j][2]) << 32 | gen_code(cg, g[j][0], g[j][1], g[j][2]);
        digit = (uint32_t)(code >> sh) & (kMsdBins - 1u);
      } else {
        digit = msd_digit(gen_code(cg, g[j][0], g[j][1], g[j][2]), sh);
      }
      if (run_count != 0 && digit != run_digit) {
        atomicAdd(&s_h[run_digit], run_count);
        run_count = 0;
      }
      run_digit = digit;
      ++run_count;
    }
  }
  if (run_count != 0) atomicAdd(&s_h[run_digit], run_count);
  __syncthreads();
  uint32_t *row = hist + ((size_t)d * a.row + tile) * kMsdBins;
#pragma unroll
  for (int q = 0; q < kMsdBins / kSortThreads; ++q) {
    const int c = t + q * kSortThreads;
    uint32_t v = 0;
#pragma unroll
    for (int k = 0; k < kSub; ++k) v += s_hs[k * kSubStride + c];
    row[c] = v;
  }
}

// The partition by top digit: per-wave digit counts in LDS, staging in digit
// order and runs written to their offsets.  Items keep their code
// (code << ib | index, ib = 32 unless WIDE).
// Lanes next to each other mostly hold points next to each other, so equal
// digits come in runs: the first lane of a run adds the run's length to the
// wave's count of its digit (one LDS atomic an item instead serialises on the
// same word: 52 us on 1M points in 8 directions against 29).  The partition
// is then stable between the 64-point chunks of the input, not inside one,
// where a digit may have several runs; k_local_sort orders equal codes by
// index.  Ranks from kMsdBits ballots an item, stable inside the chunk too,
// were 58 % of the vector instructions here: 44 us.
template <bool WIDE>
__global__ __launch_bounds__(kSortThreads) void k_msd_downsweep(SortArgs a, const int32_t *__restrict__ xyz,
                                                                uint64_t *__restrict__ dst,
                                                                const uint32_t *__restrict__ hist,
                                                                fgbd_result *__restrict__ res) {
  constexpr int kPer = kMsdBins / kSortThreads;  // digits per thread: kPer t .. kPer t + kPer - 1
  static_assert(kPer == 4, "one 16-byte count load per tile row and thread");
  __shared__ __align__(16) uint32_t s_wh[4][kMsdBins / 2];  // per wave, two 16-bit counts a word, then starts
  __shared__ uint64_t s_stage[kSortTile];
  __shared__ uint32_t s_off[kMsdBins];
  __shared__ uint32_t s_tmp[2][4];

  int d, tile;
  xcd_tile(d, tile);
  TileInfo ti;
  if (!tile_info(a.sa, tile, ti)) return;  // uniform over the block
  const int t = threadIdx.x;
  const int wave = t / kWave;
  const int lane = (int)lane_id();
  const int valid = ti.end - ti.begin;
  const int seg_end = a.sa.n_fixed >= 0 ? a.sa.n_fixed : a.sa.segs->start[ti.s + 1];
  for (int i = t; i < 2 * kMsdBins; i += kSortThreads) (&s_wh[0][0])[i] = 0;
  // scanned counts of the thread's digits: the cloud's count and this tile's
  // offset inside the cloud
  const uint32_t *hd = hist + (size_t)d * a.row * kMsdBins + kPer * t;
  const uint4 pf = ti.first > 0 ? *reinterpret_cast<const uint4 *>(hd + (size_t)ti.first * kMsdBins)
                                : make_uint4(0u, 0u, 0u, 0u);
  const uint4 pt = *reinterpret_cast<const uint4 *>(hd + (size_t)tile * kMsdBins);
  const uint4 pn = *reinterpret_cast<const uint4 *>(hd + (size_t)ti.next_first * kMsdBins);
  const uint32_t off_q[kPer] = {pt.x - pf.x, pt.y - pf.y, pt.z - pf.z, pt.w - pf.w};
  const uint32_t below_q[kPer] = {pn.x - pf.x, pn.y - pf.y, pn.z - pf.z, pn.w - pf.w};

  // (the index is the position: without it, a narrow item is its code)
  std::conditional_t<WIDE, uint64_t, uint32_t> held[kSortItems];
  auto top_of = [&](int j) { return (uint32_t)(WIDE ? (uint64_t)held[j] >> 32 : held[j]); };
  const CodeGen cg = code_gen(a.dt, d);
  // where the top digit sits in an item's upper word
  const int sh = msd_shift(a.dt, d) + (WIDE ? a.ib - 32 : 0);
  const int base = ti.begin + wave * kWave * kSortItems + lane;
  int bad = 0;
  {
    int g[kSortItems][3];
    load_points(xyz, ti, base, g);
#pragma unroll
    for (int j = 0; j < kSortItems; ++j) {
      bad |= outside_grid(g[j], a.dt.bits);
      const uint32_t code = gen_code(cg, g[j][0], g[j][1], g[j][2]);
      if constexpr (WIDE)
        held[j] = ((uint64_t)gen_code_hi(cg, g[j][0], g[j][1], g[j][2]) << 32 | code) << a.ib |
                  (uint32_t)(base + j * kWave);
      else
        held[j] = code;
    }
  }
  if (bad && d == 0) atomicOr(&res[ti.s].status, FGBD_ST_COORD_RANGE);
  __syncthreads();

  // rank among the wave's equal digits: the first lane of each run of equal
  // digits adds the run's length to the count, and the run's lanes take its
  // result and their place in the run
  uint32_t rk[kSortItems];  // digit << 16 | rank
  const uint64_t upto = ~0ull >> (63 - lane);  // lanes up to this one
  constexpr int kGroup = 4;                    // (atomics in flight; more spill)
#pragma unroll
  for (int g = 0; g < kSortItems; g += kGroup) {
    uint32_t head[kGroup], dg[kGroup], both[kGroup];
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int j = g + u;
      const bool in = base + j * kWave < ti.end;
      dg[u] = in ? msd_digit(top_of(j), sh) : ~0u;
      const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(~(int)dg[u], (int)dg[u], 0x138, 0xf, 0xf, false);
      const uint64_t heads = __builtin_amdgcn_ballot_w64(dg[u] != prev);  // (wave_shr:1; lane 0 is one)
      head[u] = 63u - (uint32_t)__builtin_clzll(heads & upto);
      if (in && head[u] == (uint32_t)lane) {
        const uint64_t after = heads & ~upto;  // (no run after the last one)
        const uint32_t next = after ? (uint32_t)__builtin_ctzll(after) : 64u;
        both[u] = atomicAdd(&s_wh[wave][dg[u] >> 1], (next - (uint32_t)lane) << 16 * (dg[u] & 1u));
      }
    }
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const uint32_t v = (uint32_t)__builtin_amdgcn_ds_bpermute((int)(4u * head[u]), (int)both[u]);
      rk[g + u] = dg[u] << 16 | (__builtin_amdgcn_ubfe(v, 16 * (dg[u] & 1u), 16) + ((uint32_t)lane - head[u]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();

  // per digit: exclusive over the tile's digits and over the cloud's digit
  // totals (over the thread's kPer digits, then over the threads), each
  // wave's start of the digit in the staged tile, and the global position of
  // staged slot 0 of the digit's run
  {
    uint32_t c[4][kPer], ex_in[kPer], ex_below[kPer];
    uint32_t run_in = 0, run_below = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint2 v = *reinterpret_cast<const uint2 *>(&s_wh[w][2 * t]);
      c[w][0] = v.x & 0xffffu;
      c[w][1] = v.x >> 16;
      c[w][2] = v.y & 0xffffu;
      c[w][3] = v.y >> 16;
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      ex_in[q] = run_in;
      run_in += c[0][q] + c[1][q] + c[2][q] + c[3][q];
      ex_below[q] = run_below;
      run_below += below_q[q];
    }
    block_exclusive_scan2_256(run_in, run_below, s_tmp);
    uint32_t e[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      e[q] = run_in + ex_in[q];
      s_off[kPer * t + q] = (uint32_t)ti.seg_start + run_below + ex_below[q] + off_q[q] - e[q];
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      *reinterpret_cast<uint2 *>(&s_wh[w][2 * t]) = make_uint2(e[0] | e[1] << 16, e[2] | e[3] << 16);
#pragma unroll
      for (int q = 0; q < kPer; ++q) e[q] += c[w][q];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) {
    if (base + j * kWave < ti.end)
      s_stage[reinterpret_cast<const uint16_t *>(s_wh[wave])[rk[j] >> 16] + (rk[j] & 0xffffu)] =
          WIDE ? (uint64_t)held[j] : (uint64_t)held[j] << 32 | (uint32_t)(base + j * kWave);
  }
  __syncthreads();
  uint64_t *out = dst + (size_t)d * a.stride;
  uint64_t st[kSortItems];
  uint32_t gp[kSortItems];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j) st[j] = s_stage[t + j * kSortThreads];
#pragma unroll
  for (int j = 0; j < kSortItems; ++j)
    gp[j] = s_off[msd_digit((uint32_t)(st[j] >> 32), sh)] + (uint32_t)(t + j * kSortThreads);
  // (the offsets stay inside the direction's row for counts that agree
  // with the upsweep's; the bound only keeps a broken count from writing
  // outside it)
#pragma unroll
  for (int j = 0; j < kSortItems; ++j)
    if (t + j * kSortThreads < valid && gp[j] < (uint32_t)a.stride) out[gp[j]] = st[j];
  // The cloud's first tile records the range of each of the cloud's windows,
  // the buckets that start in it: the range's first position, the digit of the
  // items there, the first digit whose bucket starts at or after the window's
  // base, and where the bucket that reaches the next window's base starts (in
  // the cloud's last window: the digit after the cloud's last).
  // A binary search over the bucket starts finds the first digit whose bucket
  // starts at or after a position; an empty bucket shares the start of the
  // next one that is not.  One store per window; an atomic minimum per bucket took 45 us instead of 26 on 64
  // clouds of 4k points, whose every tile is a first one.
  if (tile == ti.first) {  // (uniform)
    __syncthreads();       // the staged tile has been read
    uint32_t *s_start = reinterpret_cast<uint32_t *>(s_stage);
    // (the first tile's offset inside every bucket is 0)
    for (int c = t; c < kMsdBins; c += kSortThreads)
      s_start[c] = s_off[c] + reinterpret_cast<const uint16_t *>(s_wh[0])[c];
    __syncthreads();
    auto first_at = [&](uint32_t pos) {
      int l = 0, h = kMsdBins;
      while (l < h) {
        const int m = (l + h) >> 1;
        if (s_start[m] >= pos)
          h = m;
        else
          l = m + 1;
      }
      return l;
    };
    for (int w = t; w < ti.next_first - tile; w += kSortThreads) {
      const int l = first_at((uint32_t)(ti.seg_start + w * kLocalWin));
      const uint32_t lo = l < kMsdBins ? s_start[l] : (uint32_t)seg_end;
      // when bucket l is empty, the items at lo are of a later digit
      const int held = l + 1 < kMsdBins && s_start[l + 1] == lo ? first_at(lo + 1u) - 1 : l;
      const bool last = tile + w + 1 == ti.next_first;
      const int end_digit = first_at((uint32_t)(last ? seg_end : ti.seg_start + (w + 1) * kLocalWin));
      const int reach = last ? end_digit : (int)s_start[max(end_digit - 1, 0)];
      a.win[(size_t)d * a.nwin + tile + w] = make_int4((int)lo, held, l, reach);
    }
  }
}

constexpr int kLocalThreads = 1024;
constexpr int kLocalWaves = kLocalThreads / kWave;
constexpr int kLocalItems = 8;                          // per thread, in-LDS ranges
constexpr int kLocalCap = kLocalThreads * kLocalItems;  // 8192 items
constexpr int kPosBits = 13;                            // a position in an in-LDS range
constexpr int kBinBits = 13;
constexpr int kBins = 1 << kBinBits;
constexpr uint32_t kMaxBin = 512;                       // a larger bin makes its window's keys take LSD passes
static_assert(kLocalCap == 1 << kPosBits, "positions of the largest in-LDS range");
// A window's part of a large bucket: some less than a range holds, as the bins
// that start in it are taken whole.  Every part costs three reads of the
// bucket, so few are better: a million points in one plane, 2.2 ms with parts
// of a window's 4096.
constexpr int kShare = 6144;

struct LocalArgs {
  DirTable dt;
  SegArgs sa;
  int64_t stride;
  const int4 *win;     // [L][nwin]: where each window's range starts (see k_msd_downsweep)
  int32_t nwin;
  int32_t *big;        // host-mapped flag set for a range of more than kBigRange items (NULL: none)
  int32_t ib;          // index bits of the items (32 unless WIDE)
};

// Stable rank of an 8-bit digit among the wave's equal digits (the
// downsweep's ballot matching): returns the wave's count of the digit so far
// (an LDS read not yet waited for), sets `before` to the peers in lower
// lanes, and the first lane of each group of peers adds the group's size.
__device__ __forceinline__ uint32_t wave_rank8(uint32_t digit, uint32_t *cnt, uint32_t &before) {
  int32_t m[8];
  uint64_t vote[8];
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    m[b] = bit_mask(digit, b);
    vote[b] = __builtin_amdgcn_ballot_w64(m[b] != 0);
  }
  uint32_t plo = ~0u, phi = ~0u;
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    plo &= ~((uint32_t)vote[b] ^ (uint32_t)m[b]);
    phi &= ~((uint32_t)(vote[b] >> 32) ^ (uint32_t)m[b]);
  }
  const uint64_t peers = ((uint64_t)phi << 32) | plo;
  before = count_below(peers);
  const uint32_t r = __hip_atomic_load(&cnt[digit], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (before == 0)
    __hip_atomic_fetch_add(&cnt[digit], (uint32_t)__popcll(peers), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  return r;
}

// A value that every lane holds, in scalar registers (the compiler cannot tell
// of one loaded from memory that kernels write): branches on it are scalar, and
// nothing has to live through the side not taken.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int4 uniform(int4 v) {
  return make_int4(uniform(v.x), uniform(v.y), uniform(v.z), uniform(v.w));
}

__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32 | (uint32_t)uniform((int)v);
}

// Exclusive prefix of v over the threads of the block (up to 16 waves);
// every thread calls it.  s_w: 16 words.
__device__ __forceinline__ uint32_t exclusive_scan_block(uint32_t v, uint32_t *s_w) {
  const uint32_t lane = lane_id();
  const int w = threadIdx.x / kWave;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, kWave);
    if (lane >= (uint32_t)o) x += y;
  }
  if (lane == kWave - 1) s_w[w] = x;
  __syncthreads();
  uint32_t b = 0;
  for (int ww = 0; ww < w; ++ww) b += s_w[ww];
  __syncthreads();  // s_w is free again when this returns
  return b + x - v;
}

// A bucket of one top digit that several windows sort together.
struct LargeBucket {
  int start, end;   // its positions
  int parts, part;  // the windows that share it, and this one among them
};

// One block per (direction, window).  A window is kLocalWin sorted positions
// of one cloud, numbered like the radix tiles, so no window holds points of
// two clouds: with windows laid over the whole batch, every window of a batch
// of small clouds straddled some and was sorted through global memory (64
// clouds of 4k points: 144 us; 29 us with windows of their own).
// WIDE: codes above 32 bits, with a.ib index bits below them.  Keys stay 32-bit
// words, ranges of more than 32 code bits looking at whole items on ties
// (64-bit keys in LDS leave one block a CU): 700k points at b = 11, 70 us, and
// 74 with 64-bit keys.
template <bool WIDE>
__global__ __launch_bounds__(kLocalThreads, 8) void k_local_sort(LocalArgs a, const uint64_t *src, uint64_t *dst,
                                                                 uint32_t *__restrict__ rank) {
  // the bins' counts, then starts (two 16-bit values a word), then each
  // position's rank; a slot's key and its bin
  __shared__ uint32_t s_key[kLocalCap + 4];
  __shared__ uint32_t s_two[kLocalCap + 2];  // [kBins / 2 + 2] bins, then [kLocalCap] 16-bit bin numbers
  uint32_t *const s_bin = s_two;
  uint16_t *const s_of = reinterpret_cast<uint16_t *>(s_two + kBins / 2 + 2);
  __shared__ uint32_t s_w[16];
  __shared__ int s_swap;   // equal codes out of index order
  __shared__ int s_heavy;  // a bin holds more than kMaxBin items
  __shared__ unsigned long long s_min, s_max;

  // Consecutive windows of a direction go to the XCDs in turn.  Windows differ
  // in cost by direction and by part of the cloud: with one direction per XCD
  // the slowest one set the time (96 us on the 1M frame against 68 then).
  const int d = (int)blockIdx.y, win = (int)blockIdx.x;
  TileInfo ti;
  if (!tile_info(a.sa, win, ti)) return;  // uniform over the block
  const int t = threadIdx.x;
  const int wave = t / kWave;
  const int lane = (int)lane_id();
  const size_t dbase = (size_t)d * a.stride;
  const int sh = msd_shift(a.dt, d);

  // The range as the top-digit pass recorded it from its counts: it ends where
  // the cloud's next window's starts.  The digit before the next window's
  // first one that starts at or after its base is never empty.
  const int4 *wrow = a.win + (size_t)d * a.nwin;
  const int4 here = uniform(wrow[win]), next = uniform(wrow[min(win + 1, a.nwin - 1)]);
  const int before = uniform(wrow[max(win - 1, 0)].w);
  const bool last_win = win + 1 == ti.next_first;
  const int seg_end = uniform(a.sa.n_fixed >= 0 ? a.sa.n_fixed : (int)a.sa.segs->start[ti.s + 1]);
  const int hi = last_win ? seg_end : next.x;
  const uint32_t df = (uint32_t)here.y, dl = (uint32_t)(last_win ? here.w : next.z) - 1u;
  // A range past the LDS capacity ends in a bucket that reaches past the next
  // window's base; the windows whose base it reaches sort it between them
  // (below), and what comes before it is left to this one.
  const bool large = hi - here.x > kLocalCap;
  if (large && a.big && hi - here.x > kBigRange && t == 0) *a.big = 1;  // (only ever set to 1)
  const CodeGen cg = code_gen(a.dt, d);
  const uint32_t id_mask = WIDE ? (1u << a.ib) - 1u : ~0u;
  uint64_t *out = dst + dbase;

  // the range at hand: its items, first position, length, the smallest code it
  // may hold and the bits of a code less that one
  const uint64_t *items = src + dbase;
  int lo = here.x, R = (large ? here.w : hi) - here.x;
  uint64_t base = (uint64_t)df << sh;
  int range_bits = sh + (dl > df ? 32 - __clz(dl - df) : 0);
  // an item's code less the range's base, its top 32 bits where it has more
  // (WIDE: the low `drop` bits then only break ties), and its final form
  int drop = WIDE && range_bits > 32 ? range_bits - 32 : 0;
  auto rel = [&](uint64_t v) { return WIDE ? (v >> a.ib) - base : (uint64_t)((uint32_t)(v >> 32) - (uint32_t)base); };
  auto rel_top = [&](uint64_t v) {
    return WIDE ? shr64_lo(v - (base << a.ib), a.ib + drop) : (uint32_t)(v >> 32) - (uint32_t)base;
  };
  auto final_item = [&](uint64_t v) {
    if constexpr (WIDE)
      return decode_packed_wide(cg, v, a.ib);
    else
      return (uint64_t)decode_packed(cg, (uint32_t)(v >> 32)) << 32 | (uint32_t)v;
  };
  // (final forms are equal above the index where the codes are)
  auto same_code = [&](uint64_t u, uint64_t v) { return ((u ^ v) >> (WIDE ? a.ib : 32)) == 0; };
  // (of one 64-point chunk of the input too, inside which the top-digit pass
  // does not keep the order of equal digits)
  auto same_chunk = [&](uint64_t u, uint64_t v) {
    const uint32_t first = (uint32_t)ti.seg_start;
    return ((uint32_t)u & id_mask) - first >> 6 == ((uint32_t)v & id_mask) - first >> 6;
  };
  auto alike = [&](uint64_t u, uint64_t v) { return same_code(u, v) && same_chunk(u, v); };
  // The sorted range from LDS (final forms, s_two above s_key) to dst.  Points
  // of one voxel that the top-digit pass left out of index order are of one
  // chunk of the input and so lie next to each other: if there are any, each
  // item counts the smaller ones among them.
  auto store_sorted = [&] {
    auto at = [&](int s) { return (uint64_t)s_two[s] << 32 | s_key[s]; };
#pragma unroll
    for (int j = 0; j < kLocalItems; ++j) {
      if (j * kLocalThreads >= R) break;
      const int s = j * kLocalThreads + t;
      if (s < R) {
        const uint64_t v = at(s);
        out[lo + s] = v;
        if (s + 1 < R && s_two[s + 1] == s_two[s]) {  // (the upper word: rarely equal but for equal codes)
          const uint64_t nx = at(s + 1);
          if (alike(v, nx) && nx < v) s_swap = 1;
        }
      }
    }
    __syncthreads();
    if (uniform(s_swap) == 0) return;
    for (int s = t; s < R; s += kLocalThreads) {
      const uint64_t v = at(s);
      int r = s;
      for (int u = s - 1; u >= 0; --u) {
        const uint64_t o = at(u);
        if (!alike(v, o)) break;
        r -= o > v ? 1 : 0;
      }
      for (int u = s + 1; u < R; ++u) {
        const uint64_t o = at(u);
        if (!alike(v, o)) break;
        r += o < v ? 1 : 0;
      }
      if (r == s) continue;
      const uint32_t id = (uint32_t)v & id_mask;
      out[lo + r] = v;
      if (id < (uint32_t)a.stride) rank[dbase + id] = (uint32_t)(lo + r);
    }
  };
  // The range at hand by 8-bit LSD passes in LDS over the positions, whose keys
  // stay in place.  Slot (wave J + j) 64 + lane in visiting order; slots past
  // the range hold keys of all ones and so stay after every item.
  auto digit_sort = [&] {
    // (opaque: formed anew here, or what comes from it is held over the caller's loop and spills)
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    const int wave = uniform(t / kWave), lane = t % kWave;
    const int J = (R + kLocalThreads - 1) / kLocalThreads, bits = range_bits - drop;
    uint32_t(*const s_cnt)[256] = reinterpret_cast<uint32_t(*)[256]>(s_two);  // [kLocalWaves][256]
    uint16_t *const s_pos = reinterpret_cast<uint16_t *>(s_two + kLocalWaves * 256);
    const int low_passes = WIDE && drop > 0 ? (drop + 7) / 8 : 0;
    const int passes = low_passes + (bits + 7) / 8;
    const int first_slot = wave * J * kWave + lane;
    for (int s = t; s < J * kLocalThreads; s += kLocalThreads) {
      s_key[s] = s < R ? rel_top(items[lo + min(s, R - 1)]) : ~0u;
      s_pos[s] = (uint16_t)s;
    }
    __syncthreads();  // (there may be no pass: one code)
    for (int pass = 0; pass < passes; ++pass) {
      for (int i = t; i < kLocalWaves * 256; i += kLocalThreads) (&s_cnt[0][0])[i] = 0u;
      __syncthreads();
      auto digit_of_pos = [&](uint32_t pos) {
        if (pass >= low_passes) return s_key[pos] >> 8 * (pass - low_passes) & 255u;
        return (int)pos < R ? (uint32_t)(rel(items[lo + (int)pos]) >> 8 * pass) & 255u : 255u;
      };
      uint32_t pv[kLocalItems];  // rank among the wave's equal digits << 16 | position
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        pv[j] = s_pos[first_slot + j * kWave];
        uint32_t before;
        const uint32_t count = wave_rank8(digit_of_pos(pv[j]), s_cnt[wave], before);
        pv[j] |= (count + before) << 16;
        asm volatile("" : "+v"(pv[j]));  // (one register an item: its parts kept for later spill)
      }
      __syncthreads();
      uint32_t tot = 0;
      if (t < 256) {
#pragma unroll 4
        for (int w = 0; w < kLocalWaves; ++w) tot += s_cnt[w][t];
      }
      const uint32_t ex = exclusive_scan_block(tot, s_w);
      if (t < 256) {
        uint32_t run = ex;
#pragma unroll 4
        for (int w = 0; w < kLocalWaves; ++w) {
          const uint32_t c = s_cnt[w][t];
          s_cnt[w][t] = run;
          run += c;
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        const uint32_t pos = pv[j] & 0xffffu;
        s_pos[s_cnt[wave][digit_of_pos(pos)] + (pv[j] >> 16)] = (uint16_t)pos;
      }
      __syncthreads();
    }
    // Items in sorted order through LDS, as below.  (A range of a large bucket
    // stands where its result goes: every item is read before one is written.)
    uint32_t pv[kLocalItems];
#pragma unroll
    for (int j = 0; j < kLocalItems; ++j) {
      if (j >= J) break;
      pv[j] = s_pos[j * kLocalThreads + t];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kLocalItems; ++j) {
      if (j >= J) break;
      const int s = j * kLocalThreads + t;
      if (s < R) {
        const uint64_t v = items[lo + (int)pv[j]], done = final_item(v);
        const uint32_t id = (uint32_t)v & id_mask;
        s_key[s] = (uint32_t)done;
        s_two[s] = (uint32_t)(done >> 32);
        if (id < (uint32_t)a.stride) rank[dbase + id] = (uint32_t)(lo + s);
      }
    }
    __syncthreads();
    store_sorted();
  };

  bool digits = false;  // the range at hand is left to digit_sort
  if (R > 0) {          // (else no bucket starts in the window)
    const int J = (R + kLocalThreads - 1) / kLocalThreads;  // <= kLocalItems
    const int bits = range_bits - drop;
    // ---- in LDS.  Items stay with their thread (position j kLocalThreads + t
    // of the range); their codes less the range's base are counted into
    // 2^kBinBits bins by the top bits, the key of each item (the low bits,
    // then the position) goes to a slot of its bin, and the rank of a slot's
    // key among its bin's keys is counted.
    // (bits <= 32, so kPosBits + shift <= 32 and a key fits its word)
    const int shift = bits > kBinBits ? bits - kBinBits : 0;
    uint64_t item[kLocalItems];
    uint32_t place[kLocalItems];
#pragma unroll
    for (int j = 0; j < kLocalItems; ++j) {
      if (j >= J) break;  // uniform
      item[j] = items[lo + min(j * kLocalThreads + t, R - 1)];
    }
    for (int i = t; i < kBins / 2 + 2; i += kLocalThreads) s_bin[i] = 0u;
    // (few codes, so few and long bins whose counts would wait for each other:
    // one LSD pass at once; 400k points on a 2^3 grid, 65 us with bins first)
    const bool few = bits <= 8;
    if (t == 0) {
      s_heavy = few ? 1 : 0;
      s_swap = 0;
    }
    __syncthreads();
    // (codes of coordinates outside the grid can exceed the range's bits: the
    // minimum keeps their bins inside the table)
    auto bin_of = [&](uint32_t c) { return min(c >> shift, (uint32_t)kBins - 1u); };
#pragma unroll
    for (int j = 0; j < kLocalItems; ++j) {
      if (j >= J || few) break;
      if (j * kLocalThreads + t < R) {
        const uint32_t b = bin_of(rel_top(item[j])), sh16 = 16u * (b & 1u);
        place[j] = (atomicAdd(&s_bin[b >> 1], 1u << sh16) >> sh16) & 0xffffu;
      }
    }
    __syncthreads();
    {  // exclusive prefix over the bins, and the largest bin
      constexpr int kPerT = kBins / 2 / kLocalThreads;
      uint32_t w[kPerT], sum = 0, big = 0;
#pragma unroll
      for (int q = 0; q < kPerT; ++q) {
        w[q] = s_bin[t * kPerT + q];
        const uint32_t a0 = w[q] & 0xffffu, a1 = w[q] >> 16;
        big = max(big, max(a0, a1));
        sum += a0 + a1;
      }
      if (big > kMaxBin) s_heavy = 1;
      uint32_t run = exclusive_scan_block(sum, s_w);
#pragma unroll
      for (int q = 0; q < kPerT; ++q) {
        const uint32_t a0 = w[q] & 0xffffu, a1 = w[q] >> 16;
        s_bin[t * kPerT + q] = run | (run + a0) << 16;
        run += a0 + a1;
      }
      if (t == kLocalThreads - 1) s_bin[kBins / 2] = run;
    }
    __syncthreads();
    // long bins: many points in one voxel, or along one scan line
    digits = uniform(s_heavy) != 0;
    if (!digits) {
      const uint16_t *start = reinterpret_cast<const uint16_t *>(s_bin);
      const uint32_t low = (1u << shift) - 1u;
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        const int pos = j * kLocalThreads + t;
        if (pos < R) {
          const uint32_t c = rel_top(item[j]), b = bin_of(c);
          const uint32_t s = start[b] + place[j];
          s_key[s] = (c & low) << kPosBits | (uint32_t)pos;
          s_of[s] = (uint16_t)b;
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        const int s = j * kLocalThreads + t;
        if (s < R) {
          const uint32_t key = s_key[s], b = s_of[s];
          const uint32_t b0 = start[b], len = start[b + 1] - b0;
          uint32_t r = b0;
          const uint32_t *bin = s_key + b0;
          uint32_t k = 0;
          if (WIDE && drop > 0) {  // (uniform) equal keys but for the position: the whole items decide
            const uint64_t mine = items[lo + (int)(key & (kLocalCap - 1))];
            for (; k < len; ++k) {
              const uint32_t v = bin[k];
              bool less = v < key;
              if (((v ^ key) >> kPosBits) == 0 && v != key) less = items[lo + (int)(v & (kLocalCap - 1))] < mine;
              r += less ? 1u : 0u;
            }
          }
          for (; k + 8 <= len; k += 8) {
            uint32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = bin[k + u];
#pragma unroll
            for (int u = 0; u < 8; ++u) r += v[u] < key ? 1u : 0u;
          }
          for (; k < len; k += 4) {
            uint32_t v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = bin[k + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) r += (k + u < len && v[u] < key) ? 1u : 0u;
          }
          place[j] = r << kPosBits | (key & (kLocalCap - 1));
        }
      }
      __syncthreads();
      uint16_t *s_rank = reinterpret_cast<uint16_t *>(s_bin);  // (the starts have been read)
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        if (j * kLocalThreads + t < R) s_rank[place[j] & (kLocalCap - 1)] = (uint16_t)(place[j] >> kPosBits);
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        const int pos = j * kLocalThreads + t;
        if (pos < R) place[j] = s_rank[pos];
      }
      __syncthreads();
      // rank is written in the order of the range (near the input's inside a
      // bucket), the items in sorted order through LDS
#pragma unroll
      for (int j = 0; j < kLocalItems; ++j) {
        if (j >= J) break;
        const int pos = j * kLocalThreads + t;
        if (pos < R) {
          const uint64_t done = final_item(item[j]);
          const uint32_t id = (uint32_t)item[j] & id_mask;
          s_key[place[j]] = (uint32_t)done;
          s_two[place[j]] = (uint32_t)(done >> 32);
          if (id < (uint32_t)a.stride)  // (the id is a point of the range; the bound is a guard)
            rank[dbase + id] = (uint32_t)lo + place[j];
        }
      }
      __syncthreads();
      store_sorted();
    }
  }

  // ---- this window's part of a large bucket.  The windows that share it each
  // read it all: its codes, less the bucket's base, are counted into 2^kBinBits
  // bins, and a window takes the bins whose sorted positions start in its even
  // share of them.  It copies their items, in the order in which they stand,
  // to the place in dst where they will be, and sorts them there like any other
  // range.  Nothing writes the items that others read and nobody waits.  Items
  // that the bins leave too close (a bin of more than kLocalCap) are split
  // again by their own bits, and more points of one code than that are only
  // copied.
  // A bucket that starts in an earlier window and reaches this one's base, in
  // a range past the LDS capacity (`before` is its start only if it reaches it).
  bool share = win > ti.first && here.x > ti.begin && here.x - before > kLocalCap - kLocalWin;
  if (__builtin_expect(!digits && !share, 1)) return;
  const int owner = ti.first + (before - ti.seg_start) / kLocalWin;
  share = share && here.x - uniform(wrow[max(owner, 0)].x) > kLocalCap;
  LargeBucket lb;
  lb.start = before;
  lb.end = here.x;
  lb.parts = (here.x - before + kShare - 1) / kShare;  // (at most the windows it reaches: they are two or more)
  lb.part = win - owner - 1;
  share = share && lb.part < lb.parts;
  uint64_t k0 = 0, k1 = 0;   // keys of the window's items not sorted yet, k0 <= key < k1
  int left = -1, at_pos = 0; // their number (-1: not known yet), and where they begin in the bucket
  const uint64_t bucket = (uint64_t)(uint32_t)(here.z - 1) << sh;  // its smallest code
  const uint64_t key_mask = (1ull << sh) - 1ull;  // (codes of coordinates outside the grid: some place all the same)
  // an item's code (narrow: the upper word alone), and its key
  using Code = std::conditional_t<WIDE, uint64_t, uint32_t>;
  auto code_at = [&](int q) -> Code {
    const uint64_t *v = src + dbase + (size_t)(lb.start + q);
    if constexpr (WIDE)
      return *v >> a.ib;
    else
      return reinterpret_cast<const uint32_t *>(v)[1];
  };
  auto key_of = [&](Code c) { return (c - (Code)bucket) & (Code)key_mask; };
  // f(code, place in the bucket, whether there is one): the bucket's items,
  // each wave a contiguous part in order, some loads in flight (more spill)
  const int lsize = lb.end - lb.start;
  auto each_item = [&](auto f) {
    constexpr int U = WIDE ? 2 : 4;
    const int per = (lsize + kLocalThreads - 1) / kLocalThreads * kWave;
    const int q1 = min(uniform(wave) * per + per, lsize);
    for (int q = uniform(wave) * per; q < q1; q += U * kWave) {
      Code c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) c[u] = code_at(min(q + u * kWave + lane, lsize - 1));
#pragma unroll
      for (int u = 0; u < U; ++u) f(c[u], q + u * kWave + lane, q + u * kWave + lane < q1);
    }
  };
  // the starts of the bins of the keys from..to (inclusive) into s_key[0 .. kBins]; returns the keys' shift
  auto count_bins = [&](uint64_t from, uint64_t to) {
    const int width = to > from ? 64 - __clzll((long long)(to - from)) : 0;
    const int g = width > kBinBits ? width - kBinBits : 0;
    __syncthreads();
    for (int i = t; i <= kBins; i += kLocalThreads) s_key[i] = 0u;
    __syncthreads();
    each_item([&](Code c, int, bool in) {
      const Code k = key_of(c);
      const uint32_t bin = in && k >= (Code)from && k <= (Code)to ? (uint32_t)((k - (Code)from) >> g) : ~0u;
      // (runs of lanes with one bin add once: the input's order is often the keys')
      const uint32_t prev = (uint32_t)__builtin_amdgcn_update_dpp(~(int)bin, (int)bin, 0x138, 0xf, 0xf, false);
      const uint64_t heads = __builtin_amdgcn_ballot_w64(bin != prev);
      if (bin != prev && bin != ~0u) {
        const uint64_t after = heads & ~(~0ull >> (63 - lane));
        atomicAdd(&s_key[bin], (after ? (uint32_t)__builtin_ctzll(after) : 64u) - (uint32_t)lane);
      }
    });
    __syncthreads();
    constexpr int kPerT = kBins / kLocalThreads;
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < kPerT; ++q) sum += s_key[t * kPerT + q];
    uint32_t run = exclusive_scan_block(sum, s_w);
#pragma unroll
    for (int q = 0; q < kPerT; ++q) {
      const uint32_t c = s_key[t * kPerT + q];
      s_key[t * kPerT + q] = run;
      run += c;
    }
    if (t == kLocalThreads - 1) s_key[kBins] = run;
    __syncthreads();
    return g;
  };
  auto first_bin = [&](uint32_t pos) {  // the first bin that starts at or after pos
    int l = 0, h = kBins;
    while (l < h) {
      const int m = (l + h) >> 1;
      if (uniform((int)s_key[m]) >= (int)pos)
        h = m;
      else
        l = m + 1;
    }
    return l;
  };
  // f(place, sorted position) for the items of keys k0 .. kp - 1, in the order in which they stand
  auto in_order = [&](uint64_t kp, auto f) {
    auto mine = [&](Code c, bool in) {
      const Code k = key_of(c);
      return in && k >= (Code)k0 && k < (Code)kp;
    };
    int n = 0;
    each_item([&](Code c, int, bool in) { n += (int)__popcll(__builtin_amdgcn_ballot_w64(mine(c, in))); });
    __syncthreads();
    if (lane == 0) s_w[wave] = (uint32_t)n;
    __syncthreads();
    int to = at_pos;
    for (int w = 0; w < uniform(wave); ++w) to += uniform((int)s_w[w]);
    each_item([&](Code c, int q, bool in) {
      const bool m = mine(c, in);
      const uint64_t all = __builtin_amdgcn_ballot_w64(m);
      if (m) f(q, to + (int)count_below(all));
      to += (int)__popcll(all);
    });
    __syncthreads();
  };
  // an item of more than kLocalCap of one key, at sorted position `to` by the
  // order in which they stand, to its place by index: only items of its chunk,
  // which stand together, may come before it out of order
  auto store_one_key = [&](int q, int to) {
    const uint64_t v = src[dbase + (size_t)(lb.start + q)];
    const Code key = key_of(code_at(q));
    for (int u = q - 1; u >= 0; --u) {
      const uint64_t o = src[dbase + (size_t)(lb.start + u)];
      if (!same_chunk(o, v)) break;
      to -= key_of(code_at(u)) == key && o > v ? 1 : 0;
    }
    for (int u = q + 1; u < lsize; ++u) {
      const uint64_t o = src[dbase + (size_t)(lb.start + u)];
      if (!same_chunk(o, v)) break;
      to += key_of(code_at(u)) == key && o < v ? 1 : 0;
    }
    const uint32_t id = (uint32_t)v & id_mask;
    out[lb.start + to] = final_item(v);
    if (id < (uint32_t)a.stride) rank[dbase + id] = (uint32_t)(lb.start + to);
  };
  // sets the range at hand to the window's next items; false when there are none
  auto next_range = [&]() {
    if (left < 0) {  // the window's share
      const int even = (lsize + lb.parts - 1) / lb.parts, first = lb.part * even;
      uint64_t lowest = 0, highest = key_mask;
      if (WIDE && sh > 2 * kBinBits) {  // (many bits: the bins cover those in use)
        uint64_t mn = ~0ull, mx = 0ull;
        each_item([&](Code c, int, bool) {
          const uint64_t k = key_of(c);
          mn = k < mn ? k : mn;
          mx = k > mx ? k : mx;
        });
        if (t == 0) {
          s_min = ~0ull;
          s_max = 0ull;
        }
        __syncthreads();
        atomicMin(&s_min, (unsigned long long)mn);
        atomicMax(&s_max, (unsigned long long)mx);
        __syncthreads();
        lowest = uniform64(s_min);
        highest = uniform64(s_max);
      }
      left = 0;
      if (lowest == highest) {  // one code: the items stay where they are
        int q = first + t;
        asm volatile("" : "+v"(q));  // (its addresses spill when formed before the loop around this)
        for (; q < min(first + even, lsize); q += kLocalThreads) store_one_key(q, q);
        return false;
      }
      const int g = count_bins(lowest, highest);
      const int b0 = first_bin((uint32_t)first);
      const int b1 = lb.part + 1 == lb.parts ? kBins : first_bin((uint32_t)(first + even));
      at_pos = uniform((int)s_key[b0]);
      left = uniform((int)s_key[b1]) - at_pos;
      k0 = lowest + ((uint64_t)b0 << g);
      k1 = lowest + ((uint64_t)b1 << g);
    }
    uint64_t kp = k1;
    int c = left;
    while (c > kLocalCap) {
      if (kp - k0 == 1) {
        in_order(kp, store_one_key);
        at_pos += c;
        left -= c;
        k0 = kp;
        kp = k1;
        c = left;
        continue;
      }
      const int g = count_bins(k0, kp - 1);
      const int b = first_bin(kLocalCap + 1) - 1;  // the last bin that starts within a range's length
      const int s0 = uniform((int)s_key[b]);
      const uint64_t kb = k0 + ((uint64_t)b << g);
      if (s0 > 0) {
        c = s0;
        kp = kb;
      } else {  // the bins below it are empty, and it holds more than a range
        c = uniform((int)s_key[b + 1]);
        k0 = kb;
        kp = min(kp, kb + (1ull << g));
      }
    }
    if (c == 0) return false;
    in_order(kp, [&](int q, int to) { out[lb.start + to] = src[dbase + (size_t)(lb.start + q)]; });
    items = out;
    lo = lb.start + at_pos;
    R = c;
    base = bucket + k0;
    range_bits = kp - k0 > 1 ? 64 - __clzll((long long)(kp - k0 - 1)) : 0;
    drop = WIDE && range_bits > 32 ? range_bits - 32 : 0;
    at_pos += c;
    left -= c;
    k0 = kp;
    return true;
  };
  for (;;) {
    if (!digits && (!share || !next_range())) return;
    digits = false;
    if (t == 0) s_swap = 0;
    digit_sort();
    __syncthreads();  // (the LDS is the next range's)
  }
}

}  // namespace

SetupArgs setup_args(const Run &r, const int64_t *offsets, int64_t n_host, fgbd_result *res, int zero_result) {
  SetupArgs a;
  a.offsets = offsets;
  a.n_host = n_host;
  a.n_cap = r.pl.n_cap;
  a.B = r.pl.B;
  for (int g = 0; g < kNumGrids; ++g) a.grid[g] = r.pl.grid[g];
  a.zero_result = zero_result;
  a.sums_count = r.pl.B * kSweepSlots * kSweepParts;
  a.noise_count = r.pl.B * r.pl.E1 * kNoiseSlots;
  a.edge_count = r.pl.B * kEdgeSlots * kEdgeVals;
  const int most = 3 * a.sums_count > a.noise_count ? 3 * a.sums_count : a.noise_count;
  int blocks = (most + 256 * 8 - 1) / (256 * 8);
  a.blocks = blocks < 1 ? 1 : (blocks > 256 ? 256 : blocks);
  // the first sweep adds into sums buffer 1, the fused first launch into
  // buffers 2 (x_2) and 3 (x_1): buffers 1-3 start cleared (see launch_sweep)
  a.sums1 = r.b.sums + (size_t)a.sums_count;
  a.noise_acc = r.b.noise_acc;
  a.edge_acc = r.b.edge_acc;
  a.sg = r.b.segs;
  a.res = res;
  return a;
}

hipError_t launch_setup(const Run &r, const int64_t *offsets, int64_t n_host, fgbd_result *res, int zero_result) {
  const SetupArgs a = setup_args(r, offsets, n_host, res, zero_result);
  k_setup<<<a.blocks, 256, 0, r.stream>>>(a);
  return hipGetLastError();
}

hipError_t launch_sort(const Run &r, const int32_t *xyz, fgbd_result *res, Sorted *sorted) {
  SortArgs a;
  a.win = nullptr;
  a.nwin = 0;
  a.dt = r.dt;
  a.sa = r.sa;
  a.stride = r.pl.stride;
  a.row = r.pl.ntiles_cap + 1;
  a.fold = 0;
  a.su = r.setup;
  const int ntiles = r.sa.n_fixed >= 0 ? (r.sa.n_fixed + kSortTile - 1) / kSortTile : r.pl.ntiles_cap;
  const dim3 grid(ntiles > 0 ? ntiles : 1, r.dt.num_dirs);
  const int ib = msd_index_bits(r.dt, r.pl.n_cap);
  a.ib = ib;
  if (ib > 0 && !r.sort_lsd) {
    // the MSD pass, then the windows' local sorts
    const bool wide = ib < 32;
    a.nwin = (int)grid.x;  // windows are numbered like the tiles
    a.win = r.b.win;
    a.pass = 0;
    a.passes = 1;
    a.shift = 0;
    a.fold = r.fold_setup ? 1 : 0;
    if (a.fold && a.su.blocks > (int)(grid.x * grid.y)) a.su.blocks = (int)(grid.x * grid.y);
    FGBD_PRE(r.pf, kUpsweep);
    (wide ? k_msd_upsweep<true> : k_msd_upsweep<false>)<<<grid, kSortThreads, 0, r.stream>>>(a, xyz, r.b.hist);
    FGBD_POST(r.pf);
    FGBD_PRE(r.pf, kScan);
    k_sort_scan<kMsdBins><<<r.dt.num_dirs * (kMsdBins / kWave), kScanWaves * kWave, 0, r.stream>>>(a, r.b.hist);
    FGBD_POST(r.pf);
    FGBD_PRE(r.pf, kDownsweep);
    (wide ? k_msd_downsweep<true> : k_msd_downsweep<false>)<<<grid, kSortThreads, 0, r.stream>>>(a, xyz, r.b.items_a,
                                                                                                r.b.hist, res);
    FGBD_POST(r.pf);
    LocalArgs la;
    la.dt = r.dt;
    la.sa = r.sa;
    la.stride = r.pl.stride;
    la.win = r.b.win;
    la.nwin = a.nwin;
    la.big = r.sort_big;
    la.ib = ib;
    FGBD_PRE(r.pf, kLocalSort);
    (wide ? k_local_sort<true> : k_local_sort<false>)<<<dim3(a.nwin, r.dt.num_dirs), kLocalThreads, 0, r.stream>>>(
        la, r.b.items_a, r.b.items_b, r.b.rank);
    FGBD_POST(r.pf);
    *sorted = {r.b.items_b, ib};
    return hipGetLastError();
  }
  const uint64_t *src = nullptr;
  uint64_t *bufs[2] = {r.b.items_a, r.b.items_b};
  a.passes = r.dt.passes;
  for (int pass = 0; pass < a.passes; ++pass) {
    a.pass = pass;
    a.shift = 8 * (pass % kSortPasses);
    uint64_t *dst = bufs[pass & 1];
    FGBD_PRE(r.pf, kUpsweep);
    a.fold = (pass == 0 && r.fold_setup) ? 1 : 0;
    if (a.fold && a.su.blocks > (int)(grid.x * grid.y)) a.su.blocks = (int)(grid.x * grid.y);  // clears are strided
    k_sort_upsweep<<<grid, kSortThreads, 0, r.stream>>>(a, xyz, r.b.digits, r.b.hist);
    FGBD_POST(r.pf);
    FGBD_PRE(r.pf, kScan);
    k_sort_scan<256><<<r.dt.num_dirs * 4, kScanWaves * kWave, 0, r.stream>>>(a, r.b.hist);
    FGBD_POST(r.pf);
    FGBD_PRE(r.pf, kDownsweep);
    k_sort_downsweep<<<grid, kSortThreads, 0, r.stream>>>(a, xyz, src, dst, r.b.hist, r.b.digits, r.b.rank, res);
    FGBD_POST(r.pf);
    src = dst;
  }
  *sorted = {src, r.dt.passes == kSortPasses ? 32 : 0};
  return hipGetLastError();
}

}  // namespace fgbd
