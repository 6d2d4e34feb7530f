// Tile binning and depth ordering (Sec. 3.1: Gaussians sorted by camera depth,
// rendered per 16x16 tile) on gfx950.
//
// The instance order is the lexicographic order of (tile, depth bits, index).
// It is built as a least-significant-digit radix sort whose depth digits are
// hoisted in front of the duplication:
//   1. compact the visible Gaussians (index order) with their depth bits;
//   2. stable LSD radix sort of (depth bits, index) over the visible ones only;
//   3. scan the tile counts in that order and emit, for each Gaussian, one
//      instance per tile of its rectangle (row-major) - instances now appear
//      in (depth, index) order;
//   4. stable LSD radix sort of the instances by tile id (ceil(bits/8) passes);
//   5. per-tile [first, last+1) ranges.
// Step 4's stability keeps (depth, index) order inside a tile, so the result
// equals a full sort of (tile, depth, index) keys, while the passes over the
// instance array move 8 bytes per instance instead of 12.
//
// With tile culling on, step 3 lists a Gaussian only in the tiles it can
// reach (alpha >= 1/255 at some pixel).  Those form one column interval per
// tile row of its rectangle, so the culled emission works on rows: count the
// rectangle rows, compute every row's interval once, scan the interval
// lengths into instance offsets.  Fewer instances then reach the lists and
// the compositing loops, and since a row's instances are consecutive tiles of
// one tile row, steps 3 to 5 become a sort of the rows by tile row and one
// expansion that writes the finished lists and ranges (k_row_keys to
// k_row_expand).  Per view: 1M Gaussians at 1920x1280 (5 to 11M instances)
// 200 -> 106 us, 6M (20 to 70M) 640 -> 285, 200k at 960x640 (3.5M) 130 -> 78;
// eight served views of three sizes 1,935 -> 1,573 us in all.  Launches whose
// widths or rows the packed records cannot hold, and capacities too small for
// the tables, emit instances row by row (a thread per row) and sort them.
//
// Every radix pass is the classic three-kernel form: per-block digit
// histograms in LDS (atomics on LDS counters), an exclusive scan of each
// digit's row of block counts, and a scatter whose in-block ranks come from
// wave ballots (lanes with equal digits) and per-wave LDS counters, which keeps
// the sort stable.  Counts live on the device; kernels sized for a capacity
// exit early past the live count, so no host synchronisation is needed.
#include <mutex>

#include "pvg_math.hpp"

namespace pvg {

constexpr int kThreads = 256;
constexpr int kScanItems = 4;                       // items per thread in the scans / compaction
constexpr int kScanBlock = kThreads * kScanItems;   // 1024
constexpr int kRsItems = 16;                        // items per thread in a tile pass
constexpr int kRsBlock = kThreads * kRsItems;       // 4096
// Items per thread in a depth pass: 1024 keys a block, so that the visible
// Gaussians of one view (0.58M in the benchmark) fill the chip: with 4096 the
// passes had 142 blocks for 256 CUs, and their scatter ran at 0.5 TB/s.
constexpr int kDepthItems = 4;
constexpr int kDepthBlock = kThreads * kDepthItems;  // 1024
// Digits of the depth passes.  Three passes of 11 bits measured slower than
// four of 8 on the benchmark's 0.58M visible Gaussians (2048-digit block
// scans and 11 ballots per key outweigh the saved pass).
constexpr int kDepthBits = 8;
constexpr int kDepthPasses = (32 + kDepthBits - 1) / kDepthBits;

// ------------------------------------------------------------------ helpers
template <class T>
__device__ __forceinline__ T wave_incl_scan(T x, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const T y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  return x;
}

// Exclusive scan of one value per thread over a block of kN threads (lds:
// kN / 64 + 1 values).
template <class T, int kN = kThreads>
__device__ __forceinline__ T block_excl_scan(T v, T* lds, T& total) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const T x = wave_incl_scan<T>(v, lane);
  if (lane == 63) lds[wid] = x;
  __syncthreads();
  if (tid == 0) {
    T s = 0;
    for (int w = 0; w < kN / 64; ++w) {
      const T t = lds[w];
      lds[w] = s;
      s += t;
    }
    lds[kN / 64] = s;
  }
  __syncthreads();
  const T r = lds[wid] + x - v;
  total = lds[kN / 64];
  __syncthreads();
  return r;
}

__device__ __forceinline__ int64_t live_count(const uint32_t* n_dev, int64_t n_host) {
  return n_dev ? static_cast<int64_t>(*n_dev) : n_host;
}
__device__ __forceinline__ int64_t live_count64(const int64_t* n_dev, int64_t n_host) {
  return n_dev ? *n_dev : n_host;
}

// ------------------------------------------------------------------ step 1: compaction
__global__ void __launch_bounds__(kThreads) k_vis_count(const uint32_t* __restrict__ tiles, const int64_t* n_live,
                                                        int64_t n_host, unsigned long long* partials) {
  __shared__ unsigned long long lds[5];
  const int64_t n = live_count64(n_live, n_host);
  if (static_cast<int64_t>(blockIdx.x) * kScanBlock >= n) return;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * kScanItems;
  unsigned long long c = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n && tiles[base + k] > 0u) ++c;
  unsigned long long tot;
  block_excl_scan<unsigned long long>(c, lds, tot);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

// Exclusive scan of `count` block partials in place (one block of 1024).  The
// total goes to *total_out; with cap >= 0 it is checked against the capacity:
// over it, *total_out = 0 and *over_flag = 1.  sat_out (optional) receives the
// total saturated to 32 bits.
__device__ __forceinline__ void scan_partials_block(unsigned long long* partials, int64_t count,
                                                    unsigned long long* wsum, uint32_t* total_out, int64_t cap,
                                                    uint32_t* over_flag, uint32_t* sat_out) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  unsigned long long carry = 0;
  for (int64_t base = 0; base < count; base += 1024) {
    const int64_t i = base + tid;
    const unsigned long long v = i < count ? partials[i] : 0ull;
    const unsigned long long x = wave_incl_scan<unsigned long long>(v, lane);
    if (lane == 63) wsum[wid] = x;
    __syncthreads();
    if (tid == 0) {
      unsigned long long s = 0;
      for (int w = 0; w < 16; ++w) {
        const unsigned long long t = wsum[w];
        wsum[w] = s;
        s += t;
      }
      wsum[16] = s;
    }
    __syncthreads();
    if (i < count) partials[i] = carry + wsum[wid] + x - v;
    carry += wsum[16];
    __syncthreads();
  }
  if (tid == 0) {
    const bool over = cap >= 0 && carry > static_cast<unsigned long long>(cap);
    *total_out = over ? 0u : static_cast<uint32_t>(carry);
    if (over) *over_flag = 1u;
    if (sat_out) *sat_out = carry > 0xffffffffull ? 0xffffffffu : static_cast<uint32_t>(carry);
  }
}
// scan_partials_block over the blocks of `per_block` items each, unless *skip
// is set.
__global__ void __launch_bounds__(1024) k_scan_partials(unsigned long long* partials, const uint32_t* count_dev,
                                                        const int64_t* count_dev64, int64_t count_host,
                                                        int per_block, uint32_t* total_out, int64_t cap,
                                                        uint32_t* over_flag, uint32_t* sat_out,
                                                        const uint32_t* skip) {
  __shared__ unsigned long long wsum[17];
  if (skip && *skip) return;
  const int64_t items = count_dev64 ? *count_dev64 : live_count(count_dev, count_host);
  scan_partials_block(partials, (items + per_block - 1) / per_block, wsum, total_out, cap, over_flag, sat_out);
}

__global__ void __launch_bounds__(kThreads) k_vis_compact(const uint32_t* __restrict__ tiles,
                                                          const float* __restrict__ depth, const int64_t* n_live,
                                                          int64_t n_host,
                                                          const unsigned long long* __restrict__ partials,
                                                          uint32_t* keys, uint32_t* vals) {
  __shared__ unsigned long long lds[5];
  const int64_t n = live_count64(n_live, n_host);
  if (static_cast<int64_t>(blockIdx.x) * kScanBlock >= n) return;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * kScanItems;
  bool f[kScanItems];
  unsigned long long c = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    f[k] = base + k < n && tiles[base + k] > 0u;
    c += f[k] ? 1 : 0;
  }
  unsigned long long tot;
  unsigned long long pos = block_excl_scan<unsigned long long>(c, lds, tot) + partials[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (f[k]) {
      keys[pos] = __float_as_uint(depth[base + k]);
      vals[pos] = static_cast<uint32_t>(base + k);
      ++pos;
    }
  }
}

// ------------------------------------------------------------------ radix passes
// kMaxBits: the widest digit a kernel instance handles (8 for the tile
// passes, 11 for the depth passes: 32 bits in three passes); `bits` <= it.
template <int kMaxBits, int kPer>
__global__ void __launch_bounds__(kThreads) k_rs_hist(const uint32_t* __restrict__ keys, const uint32_t* n_dev,
                                                      int64_t n_host, int shift, int bits, uint32_t* hist,
                                                      int64_t cols) {
  constexpr int kR = 1 << kMaxBits;
  constexpr int kBlock = kThreads * kPer;
  __shared__ uint32_t h[kR];
  const int64_t n = live_count(n_dev, n_host);
  const int64_t nb = (n + kBlock - 1) / kBlock;
  const int radix = 1 << bits;
  const uint32_t mask = static_cast<uint32_t>(radix - 1);
  for (int64_t lb = blockIdx.x; lb < nb; lb += gridDim.x) {
    for (int d = threadIdx.x; d < radix; d += kThreads) h[d] = 0;
    __syncthreads();
    const int64_t base = lb * kBlock + threadIdx.x;
#pragma unroll 4
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = base + k * kThreads;
      if (i < n) atomicAdd(&h[(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < radix; d += kThreads) hist[d * cols + lb] = h[d];
    __syncthreads();
  }
}

// One block per digit: exclusive scan of that digit's block counts (blocks
// of `block` keys).
__global__ void __launch_bounds__(kThreads) k_rs_rowscan(uint32_t* hist, int64_t cols, const uint32_t* n_dev,
                                                         int64_t n_host, int64_t block, uint32_t* rowtot) {
  __shared__ uint32_t lds[5];
  const int64_t n = live_count(n_dev, n_host);
  const int64_t nb = (n + block - 1) / block;
  uint32_t* row = hist + blockIdx.x * cols;
  uint32_t carry = 0;
  for (int64_t base = 0; base < nb; base += kThreads * 4) {
    const int64_t i0 = base + threadIdx.x * 4;
    uint32_t v[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = i0 + k < nb ? row[i0 + k] : 0u;
      s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_excl_scan<uint32_t>(s, lds, tot) + carry;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k < nb) row[i0 + k] = run;
      run += v[k];
    }
    carry += tot;
  }
  if (threadIdx.x == 0) rowtot[blockIdx.x] = carry;
}

// Rank of the lane's digit among those its wave has passed here so far, in
// lane order: wave ballots find the lanes with equal digits and cnt[digit]
// (wave-private, in LDS) carries the count across calls.  Lanes that are not
// `valid` take no part and get 0xffffffff.
__device__ __forceinline__ uint32_t wave_rank(uint32_t dig, bool valid, int bits, uint32_t* cnt, uint64_t lt) {
  uint64_t peers = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const bool bit = (dig >> b) & 1u;
    const uint64_t bal = __ballot(bit);
    peers &= bit ? bal : ~bal;
  }
  uint32_t old = 0;
  if (valid) old = cnt[dig];
  const uint32_t rank = old + static_cast<uint32_t>(__popcll(peers & lt));
  __builtin_amdgcn_wave_barrier();
  if (valid && (peers & lt) == 0) cnt[dig] = old + static_cast<uint32_t>(__popcll(peers));
  __builtin_amdgcn_wave_barrier();
  return valid ? rank : 0xffffffffu;
}

// From the four waves' digit counts s_cnt (fewer than 2^kMaxBits digits
// used): s_off[d] becomes the block's first slot of digit d, s_cnt[w][d] wave
// w's.  tot[j] is the count of digit tid * kPerT + j.
template <int kR, int kPerT>
__device__ __forceinline__ void combine_digits(uint32_t (*s_cnt)[kR], uint32_t* s_off, int radix, uint32_t* lds,
                                               uint32_t (&tot)[kPerT]) {
  const int tid = threadIdx.x;
  uint32_t c[kPerT][kThreads / 64], sum = 0;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const int d = tid * kPerT + j;
    tot[j] = 0;
    for (int w = 0; w < kThreads / 64; ++w) {
      c[j][w] = d < radix ? s_cnt[w][d] : 0u;
      tot[j] += c[j][w];
    }
    sum += tot[j];
  }
  uint32_t all;
  uint32_t off = block_excl_scan<uint32_t>(sum, lds, all);
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const int d = tid * kPerT + j;
    if (d < radix) {
      s_off[d] = off;
      uint32_t run = off;
      for (int w = 0; w < kThreads / 64; ++w) {
        s_cnt[w][d] = run;
        run += c[j][w];
      }
    }
    off += tot[j];
  }
}

// Exclusive scan of the digits' totals: base[j] of digit tid * kPerT + j.
template <int kPerT>
__device__ __forceinline__ void digit_bases(const uint32_t* __restrict__ rowtot, int radix, uint32_t* lds,
                                            uint32_t (&base)[kPerT]) {
  uint32_t t[kPerT], sum = 0;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const int d = threadIdx.x * kPerT + j;
    t[j] = d < radix ? rowtot[d] : 0u;
    sum += t[j];
  }
  uint32_t tot;
  uint32_t run = block_excl_scan<uint32_t>(sum, lds, tot);
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    base[j] = run;
    run += t[j];
  }
}

// Scatter of one stable LSD pass.  Each wave ranks its own contiguous 64 kPer
// keys (wave_rank), the block combines the four waves per digit, stages the
// block's pairs locally sorted in LDS and writes each digit's run
// contiguously.  A thread owns kPerT consecutive digits in the block-wide
// digit scans.
template <int kMaxBits, int kPer>
__global__ void __launch_bounds__(kThreads) k_rs_scatter(const uint32_t* __restrict__ kin,
                                                         const uint32_t* __restrict__ vin, uint32_t* kout,
                                                         uint32_t* vout, const uint32_t* n_dev, int64_t n_host,
                                                         int shift, int bits, const uint32_t* __restrict__ hist,
                                                         int64_t cols, const uint32_t* __restrict__ rowtot) {
  constexpr int kR = 1 << kMaxBits;
  constexpr int kPerT = kR / kThreads > 0 ? kR / kThreads : 1;  // digits per thread in the digit scans
  constexpr int kBlock = kThreads * kPer;        // items per block
  constexpr int kWaveItems = 64 * kPer;          // contiguous items per wave
  __shared__ uint32_t s_cnt[kThreads / 64][kR];  // per-wave digit counts, then per-wave digit bases
  __shared__ uint32_t s_off[kR];                 // block-local first slot of each digit
  __shared__ uint32_t s_gbase[kR];               // global first slot of each digit for this block
  __shared__ uint32_t s_k[kBlock];
  __shared__ uint32_t s_v[kBlock];
  __shared__ uint32_t lds[5];
  const int64_t n = live_count(n_dev, n_host);
  const int64_t nb = (n + kBlock - 1) / kBlock;
  if (static_cast<int64_t>(blockIdx.x) >= nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int radix = 1 << bits;
  const uint32_t mask = static_cast<uint32_t>(radix - 1);
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t digit_base[kPerT];  // first global slot of the thread's digits
  digit_bases<kPerT>(rowtot, radix, lds, digit_base);
  for (int64_t lb = blockIdx.x; lb < nb; lb += gridDim.x) {
    for (int w = 0; w < kThreads / 64; ++w)
      for (int d = tid; d < radix; d += kThreads) s_cnt[w][d] = 0;
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
      const int d = tid * kPerT + j;
      if (d < radix) s_gbase[d] = digit_base[j] + hist[d * cols + lb];
    }
    __syncthreads();
    // phase 1: wave-local stable ranks
    const int64_t wbase = lb * kBlock + static_cast<int64_t>(wid) * kWaveItems;
    uint32_t key[kPer], val[kPer], rank[kPer];
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int64_t i = wbase + it * 64 + lane;
      const bool valid = i < n;
      key[it] = valid ? kin[i] : 0u;
      val[it] = valid ? vin[i] : 0u;
      rank[it] = wave_rank((key[it] >> shift) & mask, valid, bits, s_cnt[wid], lt);
    }
    __syncthreads();
    // phase 2: per digit, combine the waves and scan over digits
    uint32_t tot[kPerT];
    combine_digits<kR, kPerT>(s_cnt, s_off, radix, lds, tot);
    __syncthreads();
    // phase 3: stage locally sorted
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      if (rank[it] != 0xffffffffu) {
        const uint32_t dig = (key[it] >> shift) & mask;
        const uint32_t p = s_cnt[wid][dig] + rank[it];
        s_k[p] = key[it];
        s_v[p] = val[it];
      }
    }
    __syncthreads();
    // phase 4: coalesced runs out
    const int64_t live = min(static_cast<int64_t>(kBlock), n - lb * kBlock);
    for (int p = tid; p < live; p += kThreads) {
      const uint32_t k = s_k[p];
      const uint32_t dig = (k >> shift) & mask;
      const uint32_t o = s_gbase[dig] + (static_cast<uint32_t>(p) - s_off[dig]);
      kout[o] = k;
      vout[o] = s_v[p];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ step 3: tile counts and emission
__global__ void __launch_bounds__(kThreads) k_tile_count(const uint32_t* __restrict__ order,
                                                         const uint32_t* __restrict__ tiles, const uint32_t* n_dev,
                                                         int64_t n_host, unsigned long long* partials) {
  __shared__ unsigned long long lds[5];
  const int64_t n = live_count(n_dev, n_host);
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * kScanItems;
  if (static_cast<int64_t>(blockIdx.x) * kScanBlock >= n) return;
  unsigned long long c = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k)
    if (base + k < n) c += tiles[order[base + k]];
  unsigned long long tot;
  block_excl_scan<unsigned long long>(c, lds, tot);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

__device__ __forceinline__ int32_t clamp_tile_e(float v, int32_t hi) {
  const float f = floorf(v);
  if (f < 0.0f) return 0;
  if (f > static_cast<float>(hi)) return hi;
  return static_cast<int32_t>(f);
}

// First instance of each visible Gaussian in depth order: the exclusive scan
// of the tile counts (block partials already scanned).
__global__ void __launch_bounds__(kThreads) k_tile_offsets(const uint32_t* __restrict__ order,
                                                           const uint32_t* __restrict__ tiles,
                                                           const uint32_t* n_dev, int64_t n_host,
                                                           const unsigned long long* __restrict__ partials,
                                                           const uint32_t* __restrict__ counters,
                                                           uint32_t* offsets, uint32_t* first) {
  __shared__ unsigned long long lds[5];
  if (counters[2]) return;  // over capacity: offsets would not fit 32 bits, nothing is emitted
  const int64_t n = live_count(n_dev, n_host);
  if (static_cast<int64_t>(blockIdx.x) * kScanBlock >= n) return;
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanBlock + threadIdx.x * kScanItems;
  uint32_t c[kScanItems];
  unsigned long long sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    c[k] = base + k < n ? tiles[order[base + k]] : 0u;
    sum += c[k];
  }
  unsigned long long tot;
  unsigned long long r = block_excl_scan<unsigned long long>(sum, lds, tot) + partials[blockIdx.x];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) {
      offsets[base + k] = static_cast<uint32_t>(r);
      if (first) first[order[base + k]] = static_cast<uint32_t>(r);
    }
    r += c[k];
  }
}

// Last k in [0, n) with a[k] <= x, for non-decreasing a with a[0] <= x, by a
// 64-way search of the whole wave (each round shrinks the interval 64x).
__device__ __forceinline__ int64_t wave_last_le(const uint32_t* __restrict__ a, int64_t n, uint32_t x, int lane) {
  int64_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const int64_t p = lo + (((hi - lo) * (lane + 1)) >> 6);
    const bool ok = p <= lo || (p < hi && a[p] <= x);
    const int L = __popcll(__ballot(ok));  // ok holds for a prefix of the lanes
    const int64_t nlo = L > 0 ? __shfl(p, L - 1, 64) : lo;
    const int64_t nhi = __shfl(p, L, 64);
    lo = nlo > lo ? nlo : lo;
    hi = nhi;
  }
  return lo;
}

constexpr int kEmitChunk = 2048;  // instances per block iteration

// Instance emission balanced by instances: a block writes a fixed chunk of
// the instance array, finds the Gaussians that own it with a wave search over
// the offsets, stages their rectangles in LDS and fills the chunk (coalesced),
// so a few huge near-camera splats cannot serialise one block.
__global__ void __launch_bounds__(kThreads) k_emit(ViewSet vs, const uint32_t* __restrict__ order,
                                                   const float* __restrict__ xy, const int32_t* __restrict__ radius,
                                                   const uint32_t* __restrict__ offsets,
                                                   const uint32_t* __restrict__ counters, uint32_t* keys,
                                                   uint32_t* vals) {
  __shared__ uint32_t s_off[kEmitChunk];
  __shared__ uint32_t s_g[kEmitChunk];
  __shared__ uint32_t s_base[kEmitChunk];
  __shared__ uint32_t s_wg[kEmitChunk];  // rectangle width (low 16) | tile grid width (high 16)
  __shared__ int64_t s_k[2];
  if (counters[2]) return;
  const int64_t M = counters[0];
  const int64_t nvis = counters[1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t nchunks = (M + kEmitChunk - 1) / kEmitChunk;
  for (int64_t chunk = blockIdx.x; chunk < nchunks; chunk += gridDim.x) {
    const int64_t j0 = chunk * kEmitChunk;
    const int64_t j1 = min(M, j0 + kEmitChunk);
    if (wid < 2) {
      const int64_t k = wave_last_le(offsets, nvis, static_cast<uint32_t>(wid == 0 ? j0 : j1 - 1), lane);
      if (lane == 0) s_k[wid] = k;
    }
    __syncthreads();
    const int64_t k0 = s_k[0];
    const int cnt = static_cast<int>(s_k[1] - k0 + 1);  // <= kEmitChunk: each owner starts in the chunk
    for (int q = tid; q < cnt; q += kThreads) {
      const int64_t k = k0 + q;
      const uint32_t g = order[k];
      const View& v = view_at(vs, view_of_gauss(vs, g));
      const float2 m = reinterpret_cast<const float2*>(xy)[g];
      const float rr = static_cast<float>(radius[g]);
      const int32_t x0 = clamp_tile_e((m.x - rr) / 16.0f, v.GX);
      const int32_t y0 = clamp_tile_e((m.y - rr) / 16.0f, v.GY);
      const int32_t x1 = clamp_tile_e(((m.x + rr) + 15.0f) / 16.0f, v.GX);
      s_off[q] = offsets[k];
      s_g[q] = g;
      s_base[q] = static_cast<uint32_t>(v.tile_off + static_cast<int64_t>(y0) * v.GX + x0);
      s_wg[q] = static_cast<uint32_t>(x1 - x0) | (static_cast<uint32_t>(v.GX) << 16);
    }
    __syncthreads();
    for (int64_t j = j0 + tid; j < j1; j += kThreads) {
      int lo = 0, hi = cnt - 1;
      const uint32_t uj = static_cast<uint32_t>(j);
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_off[mid] <= uj) lo = mid; else hi = mid - 1;
      }
      const uint32_t q = uj - s_off[lo];
      const uint32_t wg = s_wg[lo];
      const uint32_t w = wg & 0xffffu, gx = wg >> 16;
      const uint32_t dy = q / w, dx = q - dy * w;
      keys[j] = s_base[lo] + dy * gx + dx;
      vals[j] = s_g[lo];
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ step 3 with tile culling
// Rectangle of Gaussian g (in its view) and the view.
__device__ __forceinline__ const View& rect_of(const ViewSet& vs, const float* __restrict__ xy,
                                               const int32_t* __restrict__ radius, uint32_t g, float2& m,
                                               int32_t rect[4]) {
  const View& v = view_at(vs, view_of_gauss(vs, g));
  m = reinterpret_cast<const float2*>(xy)[g];
  tile_rect(m.x, m.y, radius[g], v.GX, v.GY, rect);
  return v;
}

// The row kernels take one visible Gaussian per thread (a row loop is at
// most one image height of tiles long, and near splats sort first).
constexpr int kRowBlock = kThreads;

// Block sums of the rectangle row counts in depth order.
__global__ void __launch_bounds__(kThreads) k_row_count(ViewSet vs, const uint32_t* __restrict__ order,
                                                        const float* __restrict__ xy,
                                                        const int32_t* __restrict__ radius, const uint32_t* n_dev,
                                                        int64_t n_host, unsigned long long* partials) {
  __shared__ unsigned long long lds[5];
  const int64_t n = live_count(n_dev, n_host);
  if (static_cast<int64_t>(blockIdx.x) * kRowBlock >= n) return;
  const int64_t k = static_cast<int64_t>(blockIdx.x) * kRowBlock + threadIdx.x;
  unsigned long long c = 0;
  if (k < n) {
    float2 m;
    int32_t rect[4];
    rect_of(vs, xy, radius, order[k], m, rect);
    c = static_cast<unsigned long long>(rect[3] - rect[1]);
  }
  unsigned long long tot;
  block_excl_scan<unsigned long long>(c, lds, tot);
  if (threadIdx.x == 0) partials[blockIdx.x] = tot;
}

constexpr int kRowSort = 1024;  // rectangle rows per block of the tile-row pass

// Index of each visible Gaussian's first rectangle row (row_off[k]), for the
// adjoint row_base[g] = row_off[k] - y0 (mod 2^32), and, for the tile-row
// pass, the owner starts[b] of row kRowSort b.
__global__ void __launch_bounds__(kThreads) k_row_base(ViewSet vs, const uint32_t* __restrict__ order,
                                                       const float* __restrict__ xy,
                                                       const int32_t* __restrict__ radius, const uint32_t* n_dev,
                                                       int64_t n_host,
                                                       const unsigned long long* __restrict__ row_partials,
                                                       const uint32_t* __restrict__ counters, uint32_t* row_off,
                                                       uint32_t* row_base, uint32_t* starts, int64_t nstarts) {
  __shared__ unsigned long long lds[5];
  if (counters[2]) return;
  const int64_t n = live_count(n_dev, n_host);
  if (static_cast<int64_t>(blockIdx.x) * kRowBlock >= n) return;
  const int64_t k = static_cast<int64_t>(blockIdx.x) * kRowBlock + threadIdx.x;
  uint32_t g = 0;
  int32_t rect[4] = {0, 0, 0, 0};
  if (k < n) {
    float2 m;
    g = order[k];
    rect_of(vs, xy, radius, g, m, rect);
  }
  unsigned long long tot;
  const unsigned long long r0 =
      block_excl_scan<unsigned long long>(static_cast<unsigned long long>(rect[3] - rect[1]), lds, tot) +
      row_partials[blockIdx.x];
  if (k < n) {
    row_off[k] = static_cast<uint32_t>(r0);
    if (starts) {
      const uint32_t b = static_cast<uint32_t>((r0 + kRowSort - 1) / kRowSort);
      const uint64_t end = r0 + static_cast<uint32_t>(rect[3] - rect[1]);
      // (the bound only matters for records that changed since k_row_count)
      for (uint64_t q = b; q * kRowSort < end && static_cast<int64_t>(q) < nstarts; ++q)
        starts[q] = static_cast<uint32_t>(k);
    }
    if (row_base) row_base[g] = static_cast<uint32_t>(r0) - static_cast<uint32_t>(rect[1]);
  }
}

// Steps 1 to 2 and the row offsets for few Gaussians, in one block: the
// visible ones are compacted into LDS, sorted there by depth (over the bits
// that differ between keys, in equal digits of at most nine: three passes for
// depths within a factor of 2^16) and written as `order`; with culling their
// rows are counted, checked against the capacity and scanned as by k_row_count
// to k_row_base.  One launch of 16 us at 2,000 Gaussians (26 at 5,000) for
// twenty dependent ones of a few blocks each, some 4.5 us apart: 320x208 and
// 2,000 Gaussians 190 -> 129 us a render.  Its bound is the chain of a block's
// steps (four passes of 8 bits: 20 and 31 us), so it loses where the passes'
// own work would fill many blocks.
constexpr int kSmallOrder = 8192;
__global__ void __launch_bounds__(1024) k_order_small(ViewSet vs, Geom geom, int n, int cull, int64_t cap,
                                                      uint32_t* counters, uint32_t* order, uint32_t* num_rows,
                                                      uint32_t* row_off, uint32_t* row_base, uint32_t* starts) {
  constexpr int kWaves = 16, kPer = kSmallOrder / 1024;
  constexpr int kBits = 9, kDigits = 1 << kBits;
  __shared__ uint32_t s_key[2][kSmallOrder];
  __shared__ uint16_t s_idx[2][kSmallOrder];
  __shared__ uint32_t s_cnt[kWaves][kDigits];
  __shared__ uint32_t s_w[kPer * kWaves];
  __shared__ uint32_t lds[kWaves + 1];
  __shared__ uint32_t s_or, s_and;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  // compaction, in index order
  if (tid == 0) { s_or = 0u; s_and = 0xffffffffu; }
  uint64_t seen[kPer];
  uint32_t key[kPer];
#pragma unroll
  for (int it = 0; it < kPer; ++it) {
    const int i = 1024 * it + tid;
    const bool f = i < n && geom.tiles[i] > 0u;
    key[it] = f ? __float_as_uint(geom.depth[i]) : 0u;
    seen[it] = __ballot(f);
    if (lane == 0) s_w[kWaves * it + wid] = static_cast<uint32_t>(__popcll(seen[it]));
  }
  __syncthreads();
  if (wid == 0) {
    const uint32_t a = s_w[2 * lane], b = s_w[2 * lane + 1];
    const uint32_t x = wave_incl_scan<uint32_t>(a + b, lane);
    s_w[2 * lane] = x - a - b;
    s_w[2 * lane + 1] = x - b;
    if (lane == 63) lds[0] = x;
  }
  __syncthreads();
  const int nv = static_cast<int>(lds[0]);
  uint32_t any = 0u, all = 0xffffffffu;
#pragma unroll
  for (int it = 0; it < kPer; ++it) {
    if (!(seen[it] >> lane & 1ull)) continue;
    const uint32_t p = s_w[kWaves * it + wid] + static_cast<uint32_t>(__popcll(seen[it] & lt));
    s_key[0][p] = key[it];
    s_idx[0][p] = static_cast<uint16_t>(1024 * it + tid);
    any |= key[it];
    all &= key[it];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    any |= __shfl_xor(any, off, 64);
    all &= __shfl_xor(all, off, 64);
  }
  if (lane == 0) {
    atomicOr(&s_or, any);
    atomicAnd(&s_and, all);
  }
  __syncthreads();
  const uint32_t differ = s_or & ~s_and;  // bits that not all keys share
  const int its = ((nv + 63) / 64 + kWaves - 1) / kWaves;  // 64s per wave
  // the bits from the lowest to the highest that differ, in equal digits of at
  // most kBits
  const int low = differ ? __ffs(differ) - 1 : 0, width = differ ? 32 - __clz(differ) - low : 0;
  const int bits = width ? (width + (width + kBits - 1) / kBits - 1) / ((width + kBits - 1) / kBits) : 1;
  const uint32_t mask = (1u << bits) - 1u;
  int src = 0;
  for (int shift = low; shift < low + width; shift += bits) {
    for (int q = tid; q < kWaves * kDigits; q += 1024) (&s_cnt[0][0])[q] = 0u;
    __syncthreads();
    uint32_t rank[kPer];
    uint16_t idx[kPer];
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int i = (wid * its + it) * 64 + lane;
      rank[it] = 0xffffffffu;
      if (it < its) {
        const bool valid = i < nv;
        key[it] = valid ? s_key[src][i] : 0u;
        idx[it] = valid ? s_idx[src][i] : 0;
        rank[it] = wave_rank((key[it] >> shift) & mask, valid, bits, s_cnt[wid], lt);
      }
    }
    __syncthreads();
    uint32_t tot = 0;
    if (tid < kDigits)
      for (int w = 0; w < kWaves; ++w) tot += s_cnt[w][tid];
    uint32_t sum;
    uint32_t run = block_excl_scan<uint32_t, 1024>(tot, lds, sum);
    if (tid < kDigits) {
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_cnt[w][tid];
        s_cnt[w][tid] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      if (rank[it] == 0xffffffffu) continue;
      const uint32_t p = s_cnt[wid][(key[it] >> shift) & mask] + rank[it];
      s_key[src ^ 1][p] = key[it];
      s_idx[src ^ 1][p] = idx[it];
    }
    src ^= 1;
    __syncthreads();
  }
  for (int k = tid; k < nv; k += 1024) order[k] = s_idx[src][k];
  // rows in depth order, consecutive Gaussians to a thread
  uint32_t rows[kPer], y0[kPer], mine = 0;
  if (cull) {
    const int per = (nv + 1023) / 1024;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int k = tid * per + q;
      rows[q] = 0;
      y0[q] = 0;
      if (q < per && k < nv) {
        float2 m;
        int32_t rect[4];
        rect_of(vs, geom.xy, geom.radius, s_idx[src][k], m, rect);
        rows[q] = static_cast<uint32_t>(rect[3] - rect[1]);
        y0[q] = static_cast<uint32_t>(rect[1]);
        mine += rows[q];
      }
    }
    uint32_t total;
    uint32_t r0 = block_excl_scan<uint32_t, 1024>(mine, lds, total);
    const bool over = static_cast<int64_t>(total) > cap;
    if (tid == 0) {
      *num_rows = over ? 0u : total;
      counters[0] = 0u;
      counters[1] = static_cast<uint32_t>(nv);
      counters[2] = over ? 1u : 0u;
      counters[3] = total;
    }
    if (over) return;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int k = tid * per + q;
      if (q < per && k < nv) {
        row_off[k] = r0;
        if (row_base) row_base[s_idx[src][k]] = r0 - y0[q];
        if (starts)
          for (uint32_t b = (r0 + kRowSort - 1) / kRowSort; b * kRowSort < r0 + rows[q]; ++b) starts[b] = k;
        r0 += rows[q];
      }
    }
  } else if (tid == 0) {
    counters[0] = 0u;
    counters[1] = static_cast<uint32_t>(nv);
    counters[2] = 0u;
    counters[3] = 0u;
  }
}

// One thread per rectangle row, 256 consecutive rows per block iteration.
// The rows' owners (at most 256, consecutive in depth order) are found by a
// wave search over row_off and staged in LDS with their ellipse.  Writes
// rows[i] = (g, first reached column | count << 16, global tile id of that
// column, row index within the Gaussian) and the block's reached-tile sums.
__global__ void __launch_bounds__(kThreads) k_row_intervals(ViewSet vs, const uint32_t* __restrict__ order,
                                                            const float* __restrict__ xy,
                                                            const float* __restrict__ conic_op,
                                                            const int32_t* __restrict__ radius,
                                                            const uint32_t* __restrict__ row_off,
                                                            const uint32_t* __restrict__ num_rows,
                                                            const uint32_t* __restrict__ counters, uint4* rows,
                                                            unsigned long long* tile_partials) {
  __shared__ uint32_t s_off[kRowBlock];
  __shared__ uint32_t s_g[kRowBlock];
  __shared__ int32_t s_rect[kRowBlock][4];  // x0, x1, y0, y1
  __shared__ int32_t s_view[kRowBlock][3];  // H, GX, tile_off (32 bits)
  __shared__ ReachRows s_rr[kRowBlock];
  __shared__ int64_t s_k[2];
  __shared__ unsigned long long lds[5];
  if (counters[2]) return;
  const int64_t R = *num_rows;
  const int64_t nvis = counters[1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t nblocks = (R + kRowBlock - 1) / kRowBlock;
  for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const int64_t i0 = blk * kRowBlock;
    const int64_t i1 = min(R, i0 + kRowBlock);
    if (wid < 2) {
      const int64_t k = wave_last_le(row_off, nvis, static_cast<uint32_t>(wid == 0 ? i0 : i1 - 1), lane);
      if (lane == 0) s_k[wid] = k;
    }
    __syncthreads();
    const int64_t k0 = s_k[0];
    // <= kRowBlock as every Gaussian has a row; the bound only matters for
    // records that changed since k_row_count (a caller's race), as does the
    // row check below: such input yields wrong lists, never a write out of bounds
    const int cnt = static_cast<int>(min<int64_t>(kRowBlock, s_k[1] - k0 + 1));
    if (tid < cnt) {
      const uint32_t g = order[k0 + tid];
      float2 m;
      int32_t rect[4];
      const View& v = rect_of(vs, xy, radius, g, m, rect);
      const float4 co = reinterpret_cast<const float4*>(conic_op)[g];
      s_off[tid] = row_off[k0 + tid];
      s_g[tid] = g;
      s_rect[tid][0] = rect[0];
      s_rect[tid][1] = rect[2];
      s_rect[tid][2] = rect[1];
      s_rect[tid][3] = rect[3];
      s_view[tid][0] = v.H;
      s_view[tid][1] = v.GX;
      s_view[tid][2] = static_cast<int32_t>(v.tile_off);
      s_rr[tid] = reach_rows_init(m.x, m.y, co.x, co.y, co.z, co.w);
    }
    __syncthreads();
    const int64_t i = i0 + tid;
    uint32_t len = 0;
    if (i < i1) {
      int lo = 0, hi = cnt - 1;
      const uint32_t ui = static_cast<uint32_t>(i);
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_off[mid] <= ui) lo = mid; else hi = mid - 1;
      }
      const uint32_t r = ui - s_off[lo];
      const int ty = s_rect[lo][2] + static_cast<int>(r);
      int c0 = 0, c1 = -1;
      if (ty < s_rect[lo][3]) reach_row(s_rr[lo], ty, s_view[lo][0], s_rect[lo][0], s_rect[lo][1], c0, c1);
      len = c1 >= c0 ? static_cast<uint32_t>(c1 - c0 + 1) : 0u;
      const uint32_t tile = static_cast<uint32_t>(s_view[lo][2]) +
                            static_cast<uint32_t>(ty) * static_cast<uint32_t>(s_view[lo][1]) +
                            static_cast<uint32_t>(c0);
      rows[i] = make_uint4(s_g[lo], static_cast<uint32_t>(c0) | (len << 16), tile, r);
    }
    unsigned long long tot;
    block_excl_scan<unsigned long long>(len, lds, tot);
    if (tid == 0) tile_partials[blk] = tot;
  }
}

// One thread per row again (same blocks): instance offset of each row from
// the scanned block sums and a block scan, the adjoint's row records
// brows[i] = (offset, first column | count << 16), first[g], and the block's
// instances, which are consecutive in the output, written 256 at a time.
// Each instance's row is found 4096 instances at a time: every non-empty row
// marks its first instance in the chunk (the row holding the chunk's first
// instance marks slot 0), and a max-scan carries the marks forward (rows
// start in increasing order), so an instance finds its row with one LDS read
// instead of a binary search over the block's 256 row starts.
constexpr int kEmitRun = 4096;  // instances per chunk of the owner scan
__global__ void __launch_bounds__(kThreads) k_row_emit(const uint4* __restrict__ rows,
                                                       const uint32_t* __restrict__ num_rows,
                                                       const unsigned long long* __restrict__ tile_partials,
                                                       const uint32_t* __restrict__ counters, uint2* brows,
                                                       uint32_t* first, uint32_t* keys, uint32_t* vals) {
  constexpr int kPerT = kEmitRun / kThreads;  // 16 owner slots per thread in the scan
  __shared__ uint32_t s_start[kRowBlock];
  __shared__ uint32_t s_tile[kRowBlock];
  __shared__ uint32_t s_g[kRowBlock];
  __shared__ int s_own[kEmitRun];
  __shared__ int s_wmax[kThreads / 64];
  __shared__ unsigned long long lds[5];
  if (counters[2]) return;
  const int64_t R = *num_rows;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t nblocks = (R + kRowBlock - 1) / kRowBlock;
  for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const int64_t i = blk * kRowBlock + tid;
    uint4 rec = make_uint4(0u, 0u, 0u, 1u);
    if (i < R) rec = rows[i];
    const uint32_t len = rec.y >> 16;
    unsigned long long tot;
    const uint32_t pre = static_cast<uint32_t>(block_excl_scan<unsigned long long>(len, lds, tot));
    const uint32_t base = static_cast<uint32_t>(tile_partials[blk]);
    if (i < R) {
      if (brows) brows[i] = make_uint2(base + pre, rec.y);
      if (first && rec.w == 0u) first[rec.x] = base + pre;
    }
    s_start[tid] = pre;
    s_tile[tid] = rec.z;
    s_g[tid] = rec.x;
    const uint32_t total = static_cast<uint32_t>(tot);
    for (uint32_t c0 = 0; c0 < total; c0 += kEmitRun) {
      const uint32_t n = min(static_cast<uint32_t>(kEmitRun), total - c0);
      for (int k = tid; k < kEmitRun; k += kThreads) s_own[k] = 0;
      __syncthreads();
      if (len > 0 && pre < c0 + n && pre + len > c0)  // this row has instances in the chunk
        s_own[pre > c0 ? pre - c0 : 0] = tid;
      __syncthreads();
      // inclusive max-scan of s_own[0 .. kEmitRun): 16 slots per thread, then
      // the threads' maxima across the block
      int run = 0;
#pragma unroll
      for (int k = 0; k < kPerT; ++k) run = max(run, s_own[kPerT * tid + k]);
      int incl = run;
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl = max(incl, y);
      }
      if (lane == 63) s_wmax[wid] = incl;
      __syncthreads();
      int carry = __shfl_up(incl, 1, 64);
      if (lane == 0) carry = 0;
      for (int w = 0; w < wid; ++w) carry = max(carry, s_wmax[w]);
#pragma unroll
      for (int k = 0; k < kPerT; ++k) {
        carry = max(carry, s_own[kPerT * tid + k]);
        s_own[kPerT * tid + k] = carry;
      }
      __syncthreads();
      for (uint32_t u = tid; u < n; u += kThreads) {
        const int o = s_own[u];
        const uint32_t t = c0 + u;
        keys[base + t] = s_tile[o] + (t - s_start[o]);
        vals[base + t] = s_g[o];
      }
      __syncthreads();
    }
  }
}

// ------------------------------------------------------------------ step 4 by tile rows (culled lists)
// A rectangle row's instances are consecutive tiles of one tile row, so the
// culled lists need no sort of instances by tile id, which moved every
// instance's 8 bytes seven times: the row records (an eighth of the instances
// on large views) are sorted by tile row, which is one radix pass that also
// leaves the empty ones behind, and then every tile row's records, still in
// depth order, are expanded and dealt to their columns in one pass that
// writes the finished lists.  A record is a key (tile row << 16 | last
// reached column << 8 | first) and its Gaussian; a row with nothing reached
// has last column 255.
constexpr int kRowChunk = 256;   // sorted records per block iteration of the expansion, all of one tile row
constexpr int kMaxCols = 255;    // widest tile grid of the packed keys
constexpr int kRun = 4096;       // instances expanded at a time

__device__ __forceinline__ uint32_t key_first(uint32_t k) { return k & 255u; }
__device__ __forceinline__ uint32_t key_len(uint32_t k) {  // 255: nothing reached
  const uint32_t c1 = (k >> 8) & 255u;
  return c1 == 255u ? 0u : c1 + 1u - (k & 255u);
}

// First global tile id and number of columns of global tile row y (0 columns
// past the last live row).
__device__ __forceinline__ int2 tile_row_of(const ViewSet& vs, int y) {
  if (!vs.table) return make_int2(y * vs.one.GX, y < vs.one.GY ? vs.one.GX : 0);
  int lo = 0, hi = live_views(vs) - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (vs.table[mid].row_off <= y) lo = mid; else hi = mid - 1;
  }
  const View& v = vs.table[lo];
  const int ty = y - v.row_off;
  return make_int2(static_cast<int>(v.tile_off) + ty * v.GX, ty < v.GY ? v.GX : 0);
}

// Of 64 marks, those of lanes 0 .. lane.
__device__ __forceinline__ uint32_t marks_upto(uint32_t lo, uint32_t hi, int lane) {
  const uint32_t own = (lane < 32 ? lo >> lane : hi >> (lane - 32)) & 1u;
  return __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, own));
}

// One thread per rectangle row, kRowSort consecutive rows per block
// iteration, with the owners staged as in k_row_intervals; a bit per row
// marks where an owner starts, and a row's owner is the count of marks up to
// it.  Writes each row's
// record, the block's record counts per tile row (hist[y][block], y < nrows)
// and the sum of its reached tiles per 256 rows.
template <int kR>
__global__ void __launch_bounds__(kRowSort) k_row_keys(ViewSet vs, const uint32_t* __restrict__ order,
                                                       const float* __restrict__ xy,
                                                       const float* __restrict__ conic_op,
                                                       const int32_t* __restrict__ radius,
                                                       const uint32_t* __restrict__ row_off,
                                                       const uint32_t* __restrict__ starts,
                                                       const uint32_t* __restrict__ num_rows,
                                                       const uint32_t* __restrict__ counters, int nrows, int64_t cols,
                                                       uint32_t* keys, uint32_t* vals, uint32_t* hist,
                                                       unsigned long long* tile_partials) {
  __shared__ uint32_t s_off[kRowSort];
  __shared__ uint32_t s_g[kRowSort];
  __shared__ int2 s_x[kRowSort];   // rectangle columns [x, y)
  __shared__ int4 s_y[kRowSort];   // rectangle rows [x, y), the view's height and first global tile row
  __shared__ ReachRows s_rr[kRowSort];
  __shared__ uint32_t s_h[kR];
  __shared__ uint32_t s_w[kRowSort / 64];
  __shared__ uint32_t s_mark[kRowSort / 32];  // bit i: an owner's first row of the block is row i
  __shared__ uint32_t s_mbase[kRowSort / 64]; // owners before each 64 rows
  if (counters[2]) return;
  const int64_t R = *num_rows;
  const int64_t nvis = counters[1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t nblocks = (R + kRowSort - 1) / kRowSort;
  for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
    const int64_t i0 = blk * kRowSort;
    const int64_t i1 = min(R, i0 + kRowSort);
    for (int d = tid; d < nrows; d += kRowSort) s_h[d] = 0;
    if (tid < kRowSort / 32) s_mark[tid] = 0;
    __syncthreads();
    // the block's owners: up to the next block's first, which may own rows of
    // both.  Records that changed since k_row_count may have left any value in
    // starts and in the rectangles: the bounds here and on ty keep such input
    // to wrong lists.
    const int64_t k0 = min<int64_t>(starts[blk], nvis - 1);
    const int64_t k1 = blk + 1 < nblocks ? min<int64_t>(starts[blk + 1], nvis - 1) : nvis - 1;
    const int cnt = static_cast<int>(max<int64_t>(1, min<int64_t>(kRowSort, k1 - k0 + 1)));
    if (tid < cnt) {
      const uint32_t g = order[k0 + tid];
      float2 m;
      int32_t rect[4];
      const View& v = rect_of(vs, xy, radius, g, m, rect);
      const float4 co = reinterpret_cast<const float4*>(conic_op)[g];
      const uint32_t off = row_off[k0 + tid];
      const uint32_t at = tid == 0 ? 0u : off - static_cast<uint32_t>(i0);
      if (at < kRowSort) atomicOr(&s_mark[at >> 5], 1u << (at & 31u));
      s_off[tid] = off;
      s_g[tid] = g;
      s_x[tid] = make_int2(rect[0], rect[2]);
      s_y[tid] = make_int4(rect[1], rect[3], v.H, v.row_off);
      s_rr[tid] = reach_rows_init(m.x, m.y, co.x, co.y, co.z, co.w);
    }
    __syncthreads();
    if (wid == 0) {
      const uint32_t m = lane < kRowSort / 64 ? __popc(s_mark[2 * lane]) + __popc(s_mark[2 * lane + 1]) : 0u;
      const uint32_t x = wave_incl_scan<uint32_t>(m, lane);
      if (lane < kRowSort / 64) s_mbase[lane] = x - m;
    }
    __syncthreads();
    const int64_t i = i0 + tid;
    uint32_t len = 0;
    if (i < i1) {
      const uint32_t ui = static_cast<uint32_t>(i);
      const uint32_t lo = s_mbase[wid] + marks_upto(s_mark[2 * wid], s_mark[2 * wid + 1], lane) - 1u;
      const int4 ry = s_y[lo];
      const int ty = ry.x + static_cast<int>(ui - s_off[lo]);
      int c0 = 0, c1 = -1;
      if (ty >= ry.x && ty < ry.y) reach_row(s_rr[lo], ty, ry.z, s_x[lo].x, s_x[lo].y, c0, c1);
      len = c1 >= c0 ? static_cast<uint32_t>(c1 - c0 + 1) : 0u;
      const uint32_t y = static_cast<uint32_t>(ry.w + ty);
      keys[i] = (y << 16) | (len ? static_cast<uint32_t>(c1) << 8 : 255u << 8) | static_cast<uint32_t>(c0);
      vals[i] = s_g[lo];
      if (len) atomicAdd(&s_h[y], 1u);
    }
    const uint32_t x = wave_incl_scan<uint32_t>(len, lane);
    if (lane == 63) s_w[wid] = x;
    __syncthreads();
    if (tid < kRowSort / 256 && i0 + 256 * tid < i1)
      tile_partials[blk * (kRowSort / 256) + tid] =
          static_cast<unsigned long long>(s_w[4 * tid]) + s_w[4 * tid + 1] + s_w[4 * tid + 2] + s_w[4 * tid + 3];
    for (int d = tid; d < nrows; d += kRowSort) hist[d * cols + blk] = s_h[d];
    __syncthreads();
  }
}

// Block 0: the exclusive scan of the tile sums and the capacity check of the
// reached tiles; block 1 + y: the exclusive scan of tile row y's block counts.
__global__ void __launch_bounds__(1024) k_row_scans(unsigned long long* partials, const uint32_t* num_rows,
                                                    uint32_t* counters, int64_t cap, uint32_t* hist, int64_t cols,
                                                    uint32_t* rowtot) {
  __shared__ unsigned long long wsum[17];
  const int64_t R = *num_rows;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (blockIdx.x == 0) {
    if (counters[2]) return;
    scan_partials_block(partials, (R + 255) / 256, wsum, counters, cap, counters + 2, counters + 3);
    return;
  }
  uint32_t* row = hist + static_cast<int64_t>(blockIdx.x - 1) * cols;
  const int64_t nb = (R + kRowSort - 1) / kRowSort;
  uint32_t* w32 = reinterpret_cast<uint32_t*>(wsum);
  uint32_t carry = 0;
  for (int64_t base = 0; base < nb; base += 4096) {
    const int64_t i0 = base + tid * 4;
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      v[k] = i0 + k < nb ? row[i0 + k] : 0u;
      sum += v[k];
    }
    const uint32_t x = wave_incl_scan<uint32_t>(sum, lane);
    if (lane == 63) w32[wid] = x;
    __syncthreads();
    uint32_t run = carry + x - sum, all = 0;
    for (int w = 0; w < 16; ++w) {
      if (w < wid) run += w32[w];
      all += w32[w];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i0 + k < nb) row[i0 + k] = run;
      run += v[k];
    }
    carry += all;
    __syncthreads();
  }
  if (tid == 0) rowtot[blockIdx.x - 1] = carry;
}

// The tile-row pass: k_rs_scatter over the records' tile rows, leaving out
// the empty ones.  A wave's 256 records are also one block of the tile sums,
// so it knows every record's first instance and writes the adjoint's row
// records brows[i] = (offset, first column | count << 16) and, for a
// Gaussian's first row, first[g].
template <int kR>
__global__ void __launch_bounds__(kThreads) k_row_scatter(const uint32_t* __restrict__ kin,
                                                          const uint32_t* __restrict__ vin, uint32_t* kout,
                                                          uint32_t* vout, const uint32_t* __restrict__ num_rows,
                                                          const uint32_t* __restrict__ counters, int bits,
                                                          const uint32_t* __restrict__ hist, int64_t cols, int nrows,
                                                          const uint32_t* __restrict__ rowtot,
                                                          const unsigned long long* __restrict__ tile_partials,
                                                          uint2* brows, uint32_t* first) {
  constexpr int kPer = kRowSort / kThreads;
  constexpr int kPerT = kR / kThreads;
  __shared__ uint32_t s_cnt[kThreads / 64][kR];
  __shared__ uint32_t s_off[kR];
  __shared__ uint32_t s_gbase[kR];
  __shared__ uint32_t s_k[kRowSort];
  __shared__ uint32_t s_v[kRowSort];
  __shared__ uint32_t lds[5];
  if (counters[2]) return;
  const int64_t n = *num_rows;
  const int64_t nb = (n + kRowSort - 1) / kRowSort;
  if (static_cast<int64_t>(blockIdx.x) >= nb) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const uint64_t lt = (1ull << lane) - 1ull;
  uint32_t digit_base[kPerT];
  digit_bases<kPerT>(rowtot, nrows, lds, digit_base);
  for (int64_t lb = blockIdx.x; lb < nb; lb += gridDim.x) {
    for (int w = 0; w < kThreads / 64; ++w)
      for (int d = tid; d < nrows; d += kThreads) s_cnt[w][d] = 0;
#pragma unroll
    for (int j = 0; j < kPerT; ++j) {
      const int d = tid * kPerT + j;
      if (d < nrows) s_gbase[d] = digit_base[j] + hist[d * cols + lb];
    }
    __syncthreads();
    const int64_t wbase = lb * kRowSort + static_cast<int64_t>(wid) * 256;
    uint32_t inst = wbase < n ? static_cast<uint32_t>(tile_partials[lb * (kRowSort / 256) + wid]) : 0u;
    uint32_t key[kPer], val[kPer], rank[kPer];
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      const int64_t i = wbase + it * 64 + lane;
      const bool in = i < n;
      key[it] = in ? kin[i] : 255u << 8;
      val[it] = in ? vin[i] : 0u;
      const uint32_t len = key_len(key[it]);
      const uint32_t x = wave_incl_scan<uint32_t>(len, lane);
      const uint32_t e = inst + x - len;
      inst += __shfl(x, 63, 64);
      uint32_t before = __shfl_up(val[it], 1, 64);  // the record before belongs to the same Gaussian, or this is its first
      if (lane == 0) before = in && i > 0 ? vin[i - 1] : ~val[it];
      if (in && brows) brows[i] = make_uint2(e, key_first(key[it]) | (len << 16));
      if (in && first && before != val[it]) first[val[it]] = e;
      rank[it] = wave_rank(key[it] >> 16, len > 0, bits, s_cnt[wid], lt);
    }
    __syncthreads();
    uint32_t tot[kPerT];
    combine_digits<kR, kPerT>(s_cnt, s_off, nrows, lds, tot);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kPer; ++it) {
      if (rank[it] != 0xffffffffu) {
        const uint32_t p = s_cnt[wid][key[it] >> 16] + rank[it];
        s_k[p] = key[it];
        s_v[p] = val[it];
      }
    }
    __syncthreads();
    // the records of all digits (lds[4]: the block scan's total)
    const int live = static_cast<int>(lds[4]);
    for (int p = tid; p < live; p += kThreads) {
      const uint32_t k = s_k[p];
      const uint32_t o = s_gbase[k >> 16] + (static_cast<uint32_t>(p) - s_off[k >> 16]);
      kout[o] = k;
      vout[o] = s_v[p];
    }
    __syncthreads();
  }
}

// First sorted record and first chunk of every tile row (index nrows: the
// totals), from the rows' record counts.
template <int kR>
__device__ __forceinline__ void row_tables(const uint32_t* __restrict__ rowtot, int nrows, uint32_t* s_rec,
                                           uint32_t* s_chunk, uint32_t* lds) {
  constexpr int kPerT = kR / kThreads;
  uint32_t t[kPerT], rec = 0, chunk = 0, all_rec, all_chunk;
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const int d = threadIdx.x * kPerT + j;
    t[j] = d < nrows ? rowtot[d] : 0u;
    rec += t[j];
    chunk += (t[j] + kRowChunk - 1) / kRowChunk;
  }
  uint32_t r = block_excl_scan<uint32_t>(rec, lds, all_rec);
  uint32_t c = block_excl_scan<uint32_t>(chunk, lds, all_chunk);
#pragma unroll
  for (int j = 0; j < kPerT; ++j) {
    const int d = threadIdx.x * kPerT + j;
    if (d < nrows) { s_rec[d] = r; s_chunk[d] = c; }
    r += t[j];
    c += (t[j] + kRowChunk - 1) / kRowChunk;
  }
  if (threadIdx.x == 0) { s_rec[nrows] = all_rec; s_chunk[nrows] = all_chunk; }
  __syncthreads();
}

// Instances per column of each chunk: every record adds 1 at its first
// column and takes it away behind its last, and the prefix sum counts them.
// chunks[c] = (first record, last + 1, first tile id of its row, instances);
// *num_chunks counts them.
template <int kR>
__global__ void __launch_bounds__(kThreads) k_col_hist(ViewSet vs, const uint32_t* __restrict__ keys,
                                                       const uint32_t* __restrict__ rowtot,
                                                       const uint32_t* __restrict__ counters, int nrows, int ld,
                                                       uint32_t* chist, uint32_t* chunks, uint32_t* num_chunks) {
  __shared__ uint32_t s_rec[kR + 1], s_chunk[kR + 1];
  __shared__ uint32_t s_d[kThreads];
  __shared__ uint32_t s_sum[kThreads / 64];
  __shared__ uint32_t lds[kThreads / 64 + 1];
  if (counters[2]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  row_tables<kR>(rowtot, nrows, s_rec, s_chunk, lds);
  const uint32_t nchunks = s_chunk[nrows];
  if (blockIdx.x == 0 && tid == 0) *num_chunks = nchunks;
  for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
    int lo = 0, hi = nrows - 1;  // the tile row whose chunks include c
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_chunk[mid] <= c) lo = mid; else hi = mid - 1;
    }
    const uint32_t i0 = s_rec[lo] + (c - s_chunk[lo]) * kRowChunk;
    const uint32_t i1 = min(s_rec[lo + 1], i0 + kRowChunk);
    s_d[tid] = 0;
    __syncthreads();
    uint32_t sum = 0;
    if (i0 + tid < i1) {
      const uint32_t k = keys[i0 + tid];
      const uint32_t len = key_len(k);
      atomicAdd(&s_d[key_first(k)], 1u);
      atomicSub(&s_d[key_first(k) + len], 1u);  // at most column 255
      sum = len;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (lane == 0) s_sum[tid >> 6] = sum;
    __syncthreads();
    const uint32_t v = s_d[tid];
    sum = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
    uint32_t tot;
    const uint32_t x = block_excl_scan<uint32_t>(v, lds, tot) + v;
    if (tid < ld) chist[static_cast<int64_t>(c) * ld + tid] = x;
    if (tid == 0) {
      uint32_t* q = chunks + 4 * static_cast<int64_t>(c);
      q[0] = i0;
      q[1] = i1;
      q[2] = static_cast<uint32_t>(tile_row_of(vs, lo).x);
      q[3] = sum;
    }
  }
}

// Block y: the chunks' column counts of tile row y become each chunk's first
// output slot of each column (tile rows in order, in one the columns in order,
// in a column the chunks in order), and the row's tile ranges (empty: 0, 0)
// are written.  256 threads a column range, or 128 where the grid is that
// narrow, in as many segments of the chunks as fit.
__global__ void __launch_bounds__(1024) k_col_scan(ViewSet vs, const uint32_t* __restrict__ rowtot,
                                                   const uint32_t* __restrict__ counters, int ld, uint32_t* chist,
                                                   const uint32_t* __restrict__ chunks, uint32_t* ranges) {
  __shared__ uint32_t s_part[1024];
  __shared__ uint32_t s_start[257];
  __shared__ uint32_t s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int y = blockIdx.x;
  const int2 tr = tile_row_of(vs, y);
  if (counters[2]) {  // over capacity: every list empty
    if (tid < tr.y) ranges[2 * (tr.x + tid)] = ranges[2 * (tr.x + tid) + 1] = 0u;
    return;
  }
  auto block_sum = [&](uint32_t v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) s_w[wid] = v;
    __syncthreads();
    uint32_t all = 0;
    for (int w = 0; w < 16; ++w) all += s_w[w];
    __syncthreads();
    return all;
  };
  uint32_t v = 0;
  for (int d = tid; d < y; d += 1024) v += (rowtot[d] + kRowChunk - 1) / kRowChunk;
  const uint32_t c0 = block_sum(v);  // chunks of the rows before
  v = 0;
#pragma unroll 4
  for (uint32_t c = tid; c < c0; c += 1024) v += chunks[4 * static_cast<int64_t>(c) + 3];
  const uint32_t inst = block_sum(v);  // and their instances
  const uint32_t nch = (rowtot[y] + kRowChunk - 1) / kRowChunk;
  const int width = ld <= 128 ? 128 : 256;
  const int col = tid & (width - 1), seg = tid / width, segs = 1024 / width;
  const uint32_t q0 = static_cast<uint32_t>(static_cast<uint64_t>(nch) * seg / segs);
  const uint32_t q1 = static_cast<uint32_t>(static_cast<uint64_t>(nch) * (seg + 1) / segs);
  uint32_t* h = chist + static_cast<int64_t>(c0) * ld + col;
  uint32_t sum = 0;
  if (col < ld) {
#pragma unroll 8
    for (uint32_t q = q0; q < q1; ++q) sum += h[static_cast<int64_t>(q) * ld];
  }
  s_part[tid] = sum;
  __syncthreads();
  uint32_t run = 0, tot = 0;  // the segments before, and the column's total
  for (int k = 0; k < segs; ++k) {
    const uint32_t p = s_part[k * width + col];
    if (k < seg) run += p;
    tot += p;
  }
  // exclusive scan of the columns' totals (the first segment's threads)
  const uint32_t x = wave_incl_scan<uint32_t>(tot, lane);
  if (seg == 0 && lane == 63) s_w[wid] = x;
  __syncthreads();
  if (seg == 0) {
    uint32_t b = inst + x - tot;
    for (int w = 0; w < wid; ++w) b += s_w[w];
    s_start[col] = b;
    if (col < tr.y) {
      ranges[2 * (tr.x + col)] = tot ? b : 0u;
      ranges[2 * (tr.x + col) + 1] = tot ? b + tot : 0u;
    }
  }
  __syncthreads();
  run += s_start[col];
  if (col < ld) {
    uint32_t q = q0;
    for (; q + 8 <= q1; q += 8) {
      uint32_t t[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) t[k] = h[static_cast<int64_t>(q + k) * ld];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        h[static_cast<int64_t>(q + k) * ld] = run;
        run += t[k];
      }
    }
    for (; q < q1; ++q) {
      const uint32_t t = h[static_cast<int64_t>(q) * ld];
      h[static_cast<int64_t>(q) * ld] = run;
      run += t;
    }
  }
}

// The expansion: a chunk's records become instances kRun at a time.  A bit
// per instance marks where a record starts, so an instance's record is the
// count of marks up to it.  Every instance then sets its record's bit in its
// column's mask (256 records: eight words), which makes its rank in the
// column the number of bits below; ranked, the instances are staged sorted in
// LDS and written in runs at the chunk's first slots of its columns.
//
// Bound: the instances' 8 bytes out, 320 MB in 106 us on a 6M view; on a 1M
// view (60 MB in 40 us) the latency of a chunk's eight steps, as 1,400 chunks
// are one round of the chip: 512 threads 40 us, 256 44, 1,024 67.  Ranks by
// wave_rank, a ballot per bit of the column: 75 us against 49 (256 threads).
// Chunks of 128 records: 51 against 49, on the 6M view 145 against 120.
constexpr int kExpand = 512;  // threads of the expansion
__global__ void __launch_bounds__(kExpand) k_row_expand(const uint32_t* __restrict__ keys_in,
                                                        const uint32_t* __restrict__ vals_in,
                                                        const uint32_t* __restrict__ chist,
                                                        const uint32_t* __restrict__ chunks,
                                                        const uint32_t* __restrict__ num_chunks,
                                                        const uint32_t* __restrict__ counters, int ld, uint32_t* keys,
                                                        uint32_t* vals) {
  constexpr int kPer = kRun / kExpand;
  constexpr int kWords = kRowChunk / 32;
  constexpr int kCols = kMaxCols + 1;
  __shared__ uint32_t s_mask[kWords][kCols];  // per column: the records with an instance there
  __shared__ uint16_t s_slot[kWords][kCols];  // staging slot of a column's first instance of each word
  __shared__ uint32_t s_to[kCols];            // output slot minus staging slot of each column
  __shared__ uint2 s_own[kRowChunk];          // Gaussian; first column minus first instance in the chunk
  __shared__ uint32_t s_mark[kRun / 32];      // bit i: a record starts at instance i of the run
  __shared__ uint32_t s_mbase[kRun / 64];     // records started before each 64 instances, in the chunk
  __shared__ uint8_t s_t[kRun];
  __shared__ uint32_t s_v[kRun];
  __shared__ uint32_t lds[kExpand / 64 + 1];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (counters[2]) return;
  const uint32_t nchunks = *num_chunks;
  for (uint32_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
    const uint32_t* desc = chunks + 4 * static_cast<int64_t>(c);
    const uint32_t i = desc[0] + tid, tile0 = desc[2], total = desc[3];
    uint32_t key = 255u << 8, g = 0;
    if (tid < kRowChunk && i < desc[1]) {
      key = keys_in[i];
      g = vals_in[i];
    }
    // the thread's column: its next output slot
    uint32_t out = tid < ld ? chist[static_cast<int64_t>(c) * ld + tid] : 0u;
    const uint32_t len = key_len(key);
    uint32_t all;
    const uint32_t pre = block_excl_scan<uint32_t, kExpand>(len, lds, all);
    if (tid < kRowChunk) s_own[tid] = make_uint2(g, key_first(key) - pre);
    uint32_t started = 0;  // records that start before the run
    for (uint32_t r0 = 0; r0 < total; r0 += kRun) {
      const uint32_t n = min(static_cast<uint32_t>(kRun), total - r0);
      if (tid < kRun / 32) s_mark[tid] = 0;
      for (int q = tid; q < kWords * kCols; q += kExpand) (&s_mask[0][0])[q] = 0;
      __syncthreads();
      if (len > 0 && pre >= r0 && pre < r0 + n) atomicOr(&s_mark[(pre - r0) >> 5], 1u << ((pre - r0) & 31u));
      __syncthreads();
      if (wid == 0) {
        const uint32_t m = static_cast<uint32_t>(__popc(s_mark[2 * lane]) + __popc(s_mark[2 * lane + 1]));
        const uint32_t x = wave_incl_scan<uint32_t>(m, lane);
        s_mbase[lane] = started + x - m;
        if (lane == 63) lds[0] = started + x;
      }
      __syncthreads();
      started = lds[0];
      // whole 64s per wave, as even as they go
      const uint32_t per = ((n + 63) / 64 + kExpand / 64 - 1) / (kExpand / 64);
      uint32_t at[kPer], val[kPer];  // record in the chunk << 8 | column; Gaussian
#pragma unroll
      for (int it = 0; it < kPer; ++it) {
        const uint32_t grp = wid * per + it;
        const uint32_t q = grp * 64 + lane;
        at[it] = 0;
        val[it] = 0;
        if (static_cast<uint32_t>(it) < per && q < n) {
          const uint32_t rec = s_mbase[grp] + marks_upto(s_mark[2 * grp], s_mark[2 * grp + 1], lane) - 1u;
          const uint2 o = s_own[rec];
          const uint32_t x = o.y + r0 + q;
          atomicOr(&s_mask[rec >> 5][x], 1u << (rec & 31u));
          at[it] = rec << 8 | x;
          val[it] = o.x;
        }
      }
      __syncthreads();
      {
        uint32_t m[kWords], cnt = 0;
        if (tid < kCols) {
#pragma unroll
          for (int w = 0; w < kWords; ++w) {
            m[w] = __popc(s_mask[w][tid]);
            cnt += m[w];
          }
        }
        uint32_t slot = block_excl_scan<uint32_t, kExpand>(cnt, lds, all);
        if (tid < kCols) {
          s_to[tid] = out - slot;
          out += cnt;
#pragma unroll
          for (int w = 0; w < kWords; ++w) {
            s_slot[w][tid] = static_cast<uint16_t>(slot);
            slot += m[w];
          }
        }
      }
      __syncthreads();
#pragma unroll
      for (int it = 0; it < kPer; ++it) {
        const uint32_t q = (wid * per + it) * 64 + lane;
        if (static_cast<uint32_t>(it) < per && q < n) {
          const uint32_t x = at[it] & 255u, rec = at[it] >> 8;
          const uint32_t below = s_mask[rec >> 5][x] & ((1u << (rec & 31u)) - 1u);
          const uint32_t p = s_slot[rec >> 5][x] + static_cast<uint32_t>(__popc(below));
          s_t[p] = static_cast<uint8_t>(x);
          s_v[p] = val[it];
        }
      }
      __syncthreads();
      for (uint32_t p = tid; p < n; p += kExpand) {
        const uint32_t t = s_t[p];
        const uint32_t o = s_to[t] + p;
        keys[o] = tile0 + t;
        vals[o] = s_v[p];
      }
      __syncthreads();
    }
    __syncthreads();
  }
}

// Four keys a thread (one 16-byte read, plus the keys either side): the
// tile of each is a range's first entry where the key before differs, its
// last where the key after does.
__global__ void k_ranges(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ counters,
                         uint32_t* ranges, int64_t ntiles) {
  const int64_t n = counters[0];
  const int64_t n4 = (n + 3) / 4;
  const bool vec = (reinterpret_cast<uintptr_t>(keys) & 15u) == 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n4;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t j0 = 4 * i;
    uint32_t k[6];  // keys j0 - 1 .. j0 + 4 (the outer two only where they exist)
    if (vec && j0 + 4 <= n) {
      const uint4 q = reinterpret_cast<const uint4*>(keys)[i];
      k[1] = q.x; k[2] = q.y; k[3] = q.z; k[4] = q.w;
    } else {
      for (int c = 0; c < 4; ++c) k[1 + c] = j0 + c < n ? keys[j0 + c] : 0u;
    }
    k[0] = j0 > 0 ? keys[j0 - 1] : 0u;
    k[5] = j0 + 4 < n ? keys[j0 + 4] : 0u;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int64_t j = j0 + c;
      const uint32_t t = k[1 + c];
      if (j >= n || static_cast<int64_t>(t) >= ntiles) continue;  // only records changed under a running sort
      if (j == 0 || k[c] != t) ranges[2 * static_cast<int64_t>(t)] = static_cast<uint32_t>(j);
      if (j == n - 1 || k[2 + c] != t) ranges[2 * static_cast<int64_t>(t) + 1] = static_cast<uint32_t>(j + 1);
    }
  }
}

// ------------------------------------------------------------------ host pipeline
static int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
static size_t align256(size_t x) { return (x + 255) & ~static_cast<size_t>(255); }

BinPlan plan_bins(int64_t n, int64_t tiles, int64_t capacity) {
  BinPlan p{};
  p.n = n;
  p.tiles = tiles;
  p.capacity = capacity;
  int bits = 0;
  while ((int64_t{1} << bits) < tiles) ++bits;
  p.tile_bits = bits;
  p.tile_passes = static_cast<int>(cdiv(bits, 8));
  p.hist_cols = std::max<int64_t>(1, cdiv(capacity, kRsBlock));
  p.hist_cols_depth = std::max<int64_t>(1, cdiv(n, kDepthBlock));
  size_t off = 0;
  p.off_vis_keys = off; off = align256(off + sizeof(uint32_t) * 2 * std::max<int64_t>(n, 1));
  p.off_vis_vals = off; off = align256(off + sizeof(uint32_t) * 2 * std::max<int64_t>(n, 1));
  p.off_offsets = off;  off = align256(off + sizeof(uint32_t) * std::max<int64_t>(n, 1));
  const int64_t nparts = std::max<int64_t>(1, cdiv(n, kThreads));  // blocks of the row kernels (the most)
  p.off_partials = off; off = align256(off + sizeof(unsigned long long) * (nparts + 1));
  p.off_hist = off;
  off = align256(off + sizeof(uint32_t) * std::max<int64_t>((int64_t{1} << kDepthBits) * p.hist_cols_depth,
                                                            256 * p.hist_cols));
  p.off_rowtot = off;   off = align256(off + sizeof(uint32_t) * (1 << kDepthBits));
  p.off_partials2 = off;
  off = align256(off + sizeof(unsigned long long) * (std::max<int64_t>(1, cdiv(capacity, kThreads)) + 1));
  p.off_rows = off;     off = align256(off + sizeof(uint4) * std::max<int64_t>(capacity, 1));
  p.off_num_rows = off; off = align256(off + sizeof(uint32_t) * 4);
  p.total = off;
  return p;
}

// One stable LSD pass of `bits` bits at `shift` from (kin, vin) to (kout, vout).
constexpr int64_t kMaxGrid = 8192;  // physical blocks of a grid-stride pass

template <int kMaxBits, int kPer>
static hipError_t radix_pass(const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout,
                             const uint32_t* n_dev, int64_t n_grid, int shift, int bits, uint32_t* hist,
                             int64_t cols, uint32_t* rowtot, hipStream_t s) {
  if (bits < 1 || bits > kMaxBits) return hipErrorInvalidValue;
  constexpr int64_t kBlock = int64_t{kThreads} * kPer;
  const unsigned nb = static_cast<unsigned>(std::min(kMaxGrid, std::max<int64_t>(1, cdiv(n_grid, kBlock))));
  auto hist_kernel = k_rs_hist<kMaxBits, kPer>;
  auto scatter_kernel = k_rs_scatter<kMaxBits, kPer>;
  hipLaunchKernelGGL(hist_kernel, dim3(nb), dim3(kThreads), 0, s, kin, n_dev, n_grid, shift, bits, hist, cols);
  hipLaunchKernelGGL(k_rs_rowscan, dim3(1u << bits), dim3(kThreads), 0, s, hist, cols, n_dev, n_grid, kBlock,
                     rowtot);
  hipLaunchKernelGGL(scatter_kernel, dim3(nb), dim3(kThreads), 0, s, kin, vin, kout, vout, n_dev, n_grid,
                     shift, bits, hist, cols, rowtot);
  return hipGetLastError();
}

// Device arrays of the tile-row path: the records before their sort lie in the
// unused halves of keys and vals, everything else in the rows scratch.
struct RowSort {
  int nrows, ld, row_bits;
  int64_t cols;  // blocks of the tile-row pass at full capacity
  uint32_t *rkeys, *rvals, *skeys, *svals, *hist, *chist, *rowtot, *starts, *chunks, *num_chunks;
};

// Whether sorting row records beats sorting instances.  It moves every record
// twice and every instance once; the instance sort moves instances once per 8
// bits of the tile id and once more, so where rows are short (few columns) or
// the tile ids take one pass, only launches small enough for the shorter chain
// of kernels to count gain.  Lists of a driving path of 200k - 500k - 1M - 5M
// Gaussians, us, by instances against by row records:
//   16 x 16 tiles (one pass) 136 - 134, 178 - 180, 256 - 266, 1,012 - 1,117
//   4 x 64 (one pass)        137 - 138, 180 - 194, 266 - 299, 1,086 - 1,326
//   20 x 15                  158 - 132, 199 - 174, 278 - 268, 1,057 - 1,092
//   32 x 32                  (300k) 172 - 151, 289 - 276, 1,153 - 1,151
//   6 x 1,024                164 - 156, 204 - 203, 265 - 289, 997 - 1,047
//   8 x 512                  162 - 145, 200 - 178, 288 - 261, 1,037 - 978
//   60 x 40                  (300k) 183 - 158, 330 - 288, 1,358 - 1,195
// and 1M at 120 x 80 480 - 342, at 128 x 1,024 1,313 - 590.
static bool rows_pay(const ViewSet& vs) {
  const int64_t n = vs.total_gauss;
  if (n <= 1 << 17) return true;
  if (vs.total_tiles <= 256) return false;
  if (vs.total_rows > 256 && vs.max_cols < 8) return n <= 1 << 19;
  return vs.total_tiles > 512 || n <= 3 << 19;
}

// The tile-row path takes every culled launch whose view widths fit the packed
// keys, whose tile rows fit one digit (10 bits), whose tables fit the rows
// scratch, which is sized for the other path (from a capacity of some 100
// instances a tile row of 120 columns on they do), and which gains by it.
static bool plan_rows(const ViewSet& vs, const pvg_bins* bins, uint32_t* scratch, RowSort& r) {
  const int64_t cap = bins->capacity;
  if (!bins->tile_cull || vs.total_rows < 1 || vs.total_rows > 1024 || vs.max_cols > kMaxCols) return false;
  if (!rows_pay(vs)) return false;
  r.nrows = static_cast<int>(vs.total_rows);
  r.ld = vs.max_cols;
  r.cols = cdiv(cap, kRowSort);
  const int64_t hist = r.nrows * r.cols, chunks = cdiv(cap, kRowChunk) + r.nrows;
  if (hist + chunks * (r.ld + 4) + r.nrows + r.cols + 1 > 2 * cap) return false;
  r.row_bits = 0;
  while ((1 << r.row_bits) < r.nrows) ++r.row_bits;
  r.rkeys = bins->keys + cap;
  r.rvals = bins->vals + cap;
  r.skeys = scratch;
  r.svals = r.skeys + cap;
  r.hist = r.svals + cap;
  r.chist = r.hist + hist;
  r.chunks = r.chist + chunks * r.ld;
  r.rowtot = r.chunks + 4 * chunks;
  r.starts = r.rowtot + r.nrows;
  r.num_chunks = r.starts + r.cols;
  return true;
}

constexpr int64_t kRowGrid = 2048;  // physical blocks of the tile-row kernels (two to four rounds of the chip)

template <int kR>
static void launch_row_keys(const ViewSet& vs, const RowSort& r, const uint32_t* order, const Geom& geom,
                            const uint32_t* row_off, const uint32_t* num_rows, pvg_bins* bins,
                            unsigned long long* partials, hipStream_t s) {
  // two blocks a CU, all that its LDS holds; 2,048 blocks, most of them empty: 26 us for 23
  const unsigned nb = static_cast<unsigned>(std::min<int64_t>(512, std::max<int64_t>(1, r.cols)));
  hipLaunchKernelGGL(k_row_keys<kR>, dim3(nb), dim3(kRowSort), 0, s, vs, order, geom.xy, geom.conic_op, geom.radius,
                     row_off, r.starts, num_rows, bins->counters, r.nrows, r.cols, r.rkeys, r.rvals, r.hist, partials);
  hipLaunchKernelGGL(k_row_scans, dim3(static_cast<unsigned>(1 + r.nrows)), dim3(1024), 0, s, partials, num_rows,
                     bins->counters, bins->capacity, r.hist, r.cols, r.rowtot);
}

// max_rows bounds the rectangle rows (the capacity, or the counted rows).
template <int kR>
static void launch_row_lists(const ViewSet& vs, const RowSort& r, int64_t max_rows, const uint32_t* num_rows,
                             pvg_bins* bins, const unsigned long long* partials, hipStream_t s) {
  const unsigned nb = static_cast<unsigned>(std::min(kRowGrid, std::max<int64_t>(1, cdiv(max_rows, kRowSort))));
  hipLaunchKernelGGL(k_row_scatter<kR>, dim3(nb), dim3(kThreads), 0, s, r.rkeys, r.rvals, r.skeys, r.svals, num_rows,
                     bins->counters, r.row_bits, r.hist, r.cols, r.nrows, r.rowtot, partials,
                     reinterpret_cast<uint2*>(bins->rows), bins->first);
  const unsigned nc = static_cast<unsigned>(std::min(2 * kRowGrid, cdiv(max_rows, kRowChunk) + r.nrows));
  hipLaunchKernelGGL(k_col_hist<kR>, dim3(nc), dim3(kThreads), 0, s, vs, r.skeys, r.rowtot, bins->counters, r.nrows,
                     r.ld, r.chist, r.chunks, r.num_chunks);
  hipLaunchKernelGGL(k_col_scan, dim3(static_cast<unsigned>(r.nrows)), dim3(1024), 0, s, vs, r.rowtot, bins->counters,
                     r.ld, r.chist, r.chunks, bins->ranges);
  hipLaunchKernelGGL(k_row_expand, dim3(nc), dim3(kExpand), 0, s, r.skeys, r.svals, r.chist, r.chunks, r.num_chunks,
                     bins->counters, r.ld, bins->keys, bins->vals);
}

int run_bin_sort(const ViewSet& vs, const Geom& geom, pvg_bins* bins, void* tmp, const BinPlan& plan,
                 int sync_count, hipStream_t s) {
  char* base = static_cast<char*>(tmp);
  uint32_t* vkeys = reinterpret_cast<uint32_t*>(base + plan.off_vis_keys);
  uint32_t* vvals = reinterpret_cast<uint32_t*>(base + plan.off_vis_vals);
  unsigned long long* partials = reinterpret_cast<unsigned long long*>(base + plan.off_partials);
  uint32_t* hist = reinterpret_cast<uint32_t*>(base + plan.off_hist);
  uint32_t* rowtot = reinterpret_cast<uint32_t*>(base + plan.off_rowtot);
  uint32_t* offsets = reinterpret_cast<uint32_t*>(base + plan.off_offsets);
  uint32_t* counters = bins->counters;
  const int64_t n = plan.n;
  const int64_t cap = plan.capacity;
  const int64_t nvis_stride = std::max<int64_t>(n, 1);

  const bool cull = bins->tile_cull != 0;
  unsigned long long* partials2 = reinterpret_cast<unsigned long long*>(base + plan.off_partials2);
  uint4* rows = reinterpret_cast<uint4*>(base + plan.off_rows);
  uint32_t* num_rows = reinterpret_cast<uint32_t*>(base + plan.off_num_rows);
  RowSort rs{};
  const bool by_rows = plan_rows(vs, bins, reinterpret_cast<uint32_t*>(rows), rs);
  // as many as one block's LDS holds: there the launches are the cost (a render at
  // 320x208 of 1,000 Gaussians 182 -> 125 us, of 8,192 194 -> 149)
  const bool small = n > 0 && n <= kSmallOrder && !vs.table;
  if (small) {
    StageScope sc(PVG_STAGE_DEPTH_SORT, s);
    hipLaunchKernelGGL(k_order_small, dim3(1), dim3(1024), 0, s, vs, geom, static_cast<int>(n), cull ? 1 : 0, cap,
                       counters, vvals, num_rows, offsets, bins->row_base, by_rows ? rs.starts : nullptr);
    PVG_HIP(hipGetLastError());
  } else {
    PVG_HIP(launch_fill_u32(counters, 0u, 4, s));
  }
  if (n > 0 && !small) {
    StageScope sc(PVG_STAGE_COMPACT, s);
    const unsigned nb = static_cast<unsigned>(cdiv(n, kScanBlock));
    hipLaunchKernelGGL(k_vis_count, dim3(nb), dim3(kThreads), 0, s, geom.tiles, vs.live, n, partials);
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, partials, static_cast<const uint32_t*>(nullptr),
                       vs.live, n, kScanBlock, counters + 1, int64_t{-1}, static_cast<uint32_t*>(nullptr),
                       static_cast<uint32_t*>(nullptr), static_cast<const uint32_t*>(nullptr));
    // into buffer 1 when the depth passes are odd in number, so they end in buffer 0
    const int64_t start = (kDepthPasses & 1) * nvis_stride;
    hipLaunchKernelGGL(k_vis_compact, dim3(nb), dim3(kThreads), 0, s, geom.tiles, geom.depth, vs.live, n, partials,
                       vkeys + start, vvals + start);
    PVG_HIP(hipGetLastError());
  }
  // depth sort of the visible Gaussians: kDepthPasses LSD passes, ending in buffer 0
  if (n > 0 && !small) {
    StageScope sc(PVG_STAGE_DEPTH_SORT, s);
    const auto depth_pass = radix_pass<kDepthBits, kDepthItems>;
    for (int pass = 0; pass < kDepthPasses; ++pass) {
      const int src = ((kDepthPasses & 1) + pass) & 1, dst = src ^ 1;
      const int shift = kDepthBits * pass;
      PVG_HIP(depth_pass(vkeys + src * nvis_stride, vvals + src * nvis_stride, vkeys + dst * nvis_stride,
                                     vvals + dst * nvis_stride, counters + 1, n, shift,
                                     std::min(kDepthBits, 32 - shift), hist, plan.hist_cols_depth, rowtot, s));
    }
  }
  const uint32_t* order = vvals;  // buffer 0 after the depth passes
  const unsigned nbv_max = static_cast<unsigned>(std::max<int64_t>(1, cdiv(n, kScanBlock)));
  // instance counts in depth order and the capacity check: rectangle tiles, or
  // (culled) rectangle rows, their reached intervals and the reached tiles
  if (n > 0) {
    StageScope sc(PVG_STAGE_SCAN_EMIT, s);
    if (!cull) {
      hipLaunchKernelGGL(k_tile_count, dim3(nbv_max), dim3(kThreads), 0, s, order, geom.tiles, counters + 1, n,
                         partials);
      hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, partials, counters + 1,
                         static_cast<const int64_t*>(nullptr), n, kScanBlock, counters, cap, counters + 2,
                         counters + 3, static_cast<const uint32_t*>(nullptr));
    } else {
      const unsigned nrb = static_cast<unsigned>(std::min(kMaxGrid, std::max<int64_t>(1, cdiv(cap, kRowBlock))));
      if (!small) {
        PVG_HIP(launch_fill_u32(num_rows, 0u, 1, s));
        const unsigned nbr = static_cast<unsigned>(cdiv(n, kRowBlock));
        hipLaunchKernelGGL(k_row_count, dim3(nbr), dim3(kThreads), 0, s, vs, order, geom.xy, geom.radius,
                           counters + 1, n, partials);
        hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, partials, counters + 1,
                           static_cast<const int64_t*>(nullptr), n, kRowBlock, num_rows, cap, counters + 2,
                           counters + 3, static_cast<const uint32_t*>(nullptr));
        hipLaunchKernelGGL(k_row_base, dim3(nbr), dim3(kThreads), 0, s, vs, order, geom.xy, geom.radius, counters + 1,
                           n, partials, counters, offsets, bins->row_base, by_rows ? rs.starts : nullptr, rs.cols);
      }
      if (by_rows) {
        (rs.nrows <= 256 ? launch_row_keys<256> : launch_row_keys<1024>)(vs, rs, order, geom, offsets, num_rows, bins,
                                                                         partials2, s);
      } else {
        hipLaunchKernelGGL(k_row_intervals, dim3(nrb), dim3(kThreads), 0, s, vs, order, geom.xy, geom.conic_op,
                           geom.radius, offsets, num_rows, counters, rows, partials2);
        hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(1024), 0, s, partials2, num_rows,
                           static_cast<const int64_t*>(nullptr), int64_t{0}, kRowBlock, counters, cap, counters + 2,
                           counters + 3, counters + 2);
      }
    }
    PVG_HIP(hipGetLastError());
  }
  int64_t m_grid = cap;
  int64_t vis_grid = n;
  int64_t row_grid = cap;
  if (sync_count) {
    uint32_t host_counts[4], host_rows = 0;
    PVG_HIP(hipMemcpyAsync(host_counts, counters, sizeof(host_counts), hipMemcpyDeviceToHost, s));
    if (cull && n > 0) PVG_HIP(hipMemcpyAsync(&host_rows, num_rows, sizeof(host_rows), hipMemcpyDeviceToHost, s));
    PVG_HIP(hipStreamSynchronize(s));
    bins->num_instances = host_counts[3] == 0xffffffffu ? int64_t{0xffffffff} : int64_t{host_counts[3]};
    bins->num_visible = host_counts[1];
    if (host_counts[2]) {
      set_error("instance capacity %lld is smaller than the %lld %s of this render", static_cast<long long>(cap),
                static_cast<long long>(bins->num_instances),
                cull && host_rows == 0 ? "rectangle rows" : "instances");
      return PVG_ERR_CAPACITY;
    }
    m_grid = host_counts[0];
    vis_grid = host_counts[1];
    row_grid = host_rows;
  }
  if (by_rows && n > 0 && vis_grid > 0 && row_grid > 0) {
    StageScope sc(PVG_STAGE_TILE_SORT, s);
    (rs.nrows <= 256 ? launch_row_lists<256> : launch_row_lists<1024>)(vs, rs, row_grid, num_rows, bins, partials2, s);
    PVG_HIP(hipGetLastError());
    return PVG_OK;
  }
  const int passes = plan.tile_passes;
  const int start = passes & 1;  // so that the last pass lands in buffer 0
  // culled lists: the row pass also writes the adjoint's row records and
  // first[], so it runs whenever there are rows, even with nothing listed
  if (n > 0 && vis_grid > 0 && (cull ? row_grid > 0 : m_grid > 0)) {
    StageScope sc(PVG_STAGE_SCAN_EMIT, s);
    const unsigned nbv = static_cast<unsigned>(cdiv(vis_grid, kScanBlock));
    if (!cull) {
      hipLaunchKernelGGL(k_tile_offsets, dim3(nbv), dim3(kThreads), 0, s, order, geom.tiles, counters + 1, n,
                         partials, counters, offsets, bins->first);
      const unsigned nbe = static_cast<unsigned>(std::min(kMaxGrid, cdiv(m_grid, kEmitChunk)));
      hipLaunchKernelGGL(k_emit, dim3(nbe), dim3(kThreads), 0, s, vs, order, geom.xy, geom.radius, offsets,
                         counters, bins->keys + start * cap, bins->vals + start * cap);
    } else {
      const unsigned nre = static_cast<unsigned>(std::min(kMaxGrid, std::max<int64_t>(1, cdiv(row_grid, kRowBlock))));
      hipLaunchKernelGGL(k_row_emit, dim3(nre), dim3(kThreads), 0, s, rows, num_rows, partials2, counters,
                         reinterpret_cast<uint2*>(bins->rows), bins->first, bins->keys + start * cap,
                         bins->vals + start * cap);
    }
    PVG_HIP(hipGetLastError());
  }
  if (passes > 0 && m_grid > 0) {
    StageScope sc(PVG_STAGE_TILE_SORT, s);
    const auto tile_pass = radix_pass<8, kRsItems>;
    const int per = (plan.tile_bits + passes - 1) / passes;
    for (int pass = 0; pass < passes; ++pass) {
      const int src = (start + pass) & 1, dst = src ^ 1;
      const int shift = per * pass;
      const int bits = std::min(per, plan.tile_bits - shift);
      PVG_HIP(tile_pass(bins->keys + src * cap, bins->vals + src * cap, bins->keys + dst * cap,
                            bins->vals + dst * cap, counters, m_grid, shift, bits, hist, plan.hist_cols, rowtot, s));
    }
  }
  {
    StageScope sc(PVG_STAGE_RANGES, s);
    PVG_HIP(launch_fill_u32(bins->ranges, 0u, 2 * plan.tiles, s));
    if (m_grid > 0) {
      hipLaunchKernelGGL(k_ranges, dim3(static_cast<unsigned>(std::min(kMaxGrid * 4, cdiv(m_grid, 1024)))),
                         dim3(256), 0, s, bins->keys, counters, bins->ranges, static_cast<int64_t>(plan.tiles));
      PVG_HIP(hipGetLastError());
    }
  }
  return PVG_OK;
}

// ------------------------------------------------- library-held bin_sort scratch
// The scratch of pvg_bin_sort_noalloc, for callers that cannot allocate device
// memory.  Each device the library runs on holds its own copy until the
// process ends.  In host code `scratch` names a host-side stand-in, never a
// device address: host code uses only the address hipGetSymbolAddress returns,
// looked up once per device with that device current.
static __device__ __align__(256) unsigned char scratch[PVG_NOALLOC_SCRATCH_BYTES];

hipError_t noalloc_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    addr[dev] = p;
  }
  *out = addr[dev];
  return hipSuccess;
}

}  // namespace pvg
