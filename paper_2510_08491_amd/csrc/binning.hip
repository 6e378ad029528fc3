// Tile binning and depth sorting (the tiling / sorting stages the paper's
// App. A lists beside preprocessing; the blending of Eq. 4 needs the
// primitives of every pixel in depth order).
//
//   depth  : stable LSD radix sort of the (view, primitive) pairs by their
//            float32 depth bits (ties keep the index order); it also puts
//            the pairs' tile counts into that order
//   scan   : exclusive prefix sum of the tile counts in that order
//   emit   : one (key, value) instance per covered tile, primitives in depth
//            order, key = (global tile id << 31) | float32 depth bits,
//            value = primitive id
//   sort   : stable LSD radix sort of the instances by the tile bits of the
//            key only: the input is already in depth order and every pass
//            is stable, so the result is ordered by the whole key (and by
//            primitive index for equal depths), as a sort over all bits
//            would order it, with 1-3 passes over the instances instead of
//            5-6 (8-bit digits, 3 kernels per pass: digit histogram per
//            block, prefix per digit over the blocks, stable scatter).  With
//            bin_order 2 the pairs stay in primitive order and the sort
//            covers depth and tile bits.
//   ranges : [start, end) of every global tile in the sorted array
//
// At the sizes of one view every kernel here is a few microseconds, most of
// it launch and drain, so the launches are counted: with few pairs those of a
// view are ordered, counted and scanned by one workgroup in LDS, a pass takes three
// kernels at any size, a scan one or two, and what a neighbour can do on the
// way (first keys, last gather, clears, checks) has no launch of its own.
//
// Sizes only known on the device (the instance count) are read from device
// memory; launches are sized by the workspace capacity, so the sequence can
// be captured in a graph.  Writes past the capacity are dropped and flagged.
#include <algorithm>

#include "snp_internal.h"

namespace snp {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int64_t kScanChunk = (int64_t)kScanThreads * kScanItems;  // 4096
constexpr int64_t kScanBlocksMax = 8192;  // blocks whose totals each block can sum for itself

constexpr int kSortThreads = 256;
constexpr int kRadix = 256;

// Keys per block of a radix pass: 4096 (16 rounds of the block), or 1024 (4
// rounds) for up to 2^18 keys, where 4096 would leave most CUs idle: depth
// sort of 100k pairs, 25 or 98 blocks: a scatter takes 12.0 or 5.9 us, a
// histogram 6.2 or 4.5 us.
int sort_rounds(int64_t n) { return n <= ((int64_t)1 << 18) ? 4 : 16; }
static int64_t sort_blocks(int64_t n, int rounds) {
  const int64_t chunk = (int64_t)kSortThreads * rounds;
  return (n + chunk - 1) / chunk;
}

__global__ void fill_u32_kernel(uint32_t* p, int64_t n, uint32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) p[i] = v;
}

hipError_t fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  int64_t blocks = (n + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// exclusive scan: uint32 values -> uint32 offsets (wrapping), uint64 total
// ---------------------------------------------------------------------------
// Exclusive prefix of x over the NT threads of the block and its total.  Ends
// with a barrier (s_warp may be reused).
template <int NT, typename T>
__device__ __forceinline__ T block_exclusive_scan(T x, T* total, T* s_warp) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T inc = x;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const T y = __shfl_up(inc, o);
    if (lane >= o) inc += y;
  }
  if (lane == 63) s_warp[w] = inc;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    if (k < w) base += s_warp[k];
    tot += s_warp[k];
  }
  __syncthreads();
  *total = tot;
  return base + inc - x;
}

// (the row of the grid picks the array)
struct ScanArrays {
  const uint32_t* in[2];
  uint32_t* out[2];
};

__global__ void __launch_bounds__(kScanThreads) scan_totals_kernel(ScanArrays a, int64_t n, uint64_t* totals) {
  __shared__ uint64_t s_warp[kScanThreads / 64];
  const uint32_t* __restrict__ in = a.in[blockIdx.y];
  totals += (int64_t)blockIdx.y * gridDim.x;
  const int64_t base = (int64_t)blockIdx.x * kScanChunk;
  uint64_t sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k * kScanThreads + threadIdx.x;
    sum += i < n ? in[i] : 0u;
  }
  uint64_t total;
  block_exclusive_scan<kScanThreads>(sum, &total, s_warp);
  if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

// One block's chunk, after the totals of the blocks before it: summed here
// (prefixed = 0), or already in totals as exclusive prefixes.
__global__ void __launch_bounds__(kScanThreads) scan_chunk_kernel(ScanArrays a, int64_t n, const uint64_t* totals,
                                                                  int prefixed, uint64_t* total_out) {
  __shared__ uint64_t s_warp[kScanThreads / 64];
  const uint32_t* __restrict__ in = a.in[blockIdx.y];
  uint32_t* __restrict__ out = a.out[blockIdx.y];
  totals += (int64_t)blockIdx.y * gridDim.x;
  uint64_t before = 0;
  if (prefixed) {
    before = totals[blockIdx.x];
  } else if (blockIdx.x > 0) {
    uint64_t part = 0;
    for (unsigned b = threadIdx.x; b < blockIdx.x; b += kScanThreads) part += totals[b];
    block_exclusive_scan<kScanThreads>(part, &before, s_warp);
  }
  const int64_t base = (int64_t)blockIdx.x * kScanChunk + (int64_t)threadIdx.x * kScanItems;
  uint32_t v[kScanItems];
  uint64_t sum = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    v[k] = i < n ? in[i] : 0u;
    sum += v[k];
  }
  uint64_t total;
  uint64_t run = before + block_exclusive_scan<kScanThreads>(sum, &total, s_warp);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + k;
    if (i < n) out[i] = (uint32_t)run;
    run += v[k];
  }
  if (total_out && blockIdx.y == 0 && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *total_out = before + total;
}

// totals -> exclusive prefixes in place, one workgroup (more blocks than
// kScanBlocksMax: 2^25 values and up)
__global__ void __launch_bounds__(1024) scan_prefix_kernel(uint64_t* totals, int64_t n) {
  __shared__ uint64_t s_warp[16];
  totals += (int64_t)blockIdx.y * n;
  uint64_t carry = 0;
  for (int64_t i0 = 0; i0 < n; i0 += 1024) {
    const int64_t i = i0 + threadIdx.x;
    uint64_t total;
    const uint64_t x = i < n ? totals[i] : 0;
    const uint64_t e = block_exclusive_scan<1024>(x, &total, s_warp);
    if (i < n) totals[i] = carry + e;
    carry += total;
  }
}

// Scratch needed by scan_exclusive_u32 for n elements of one or two arrays (bytes).
size_t scan_scratch_bytes(int64_t n, int arrays) {
  const int64_t nb = (n + kScanChunk - 1) / kScanChunk;
  return ((size_t)nb * arrays * 8 + 255) / 256 * 256 + 256;
}

// Exclusive scan of n uint32 values into out (wrapping) and the exact total
// into *total_out (uint64, device) if non-null; with in2, of a second array
// into out2 in the same launches.
hipError_t scan_exclusive_u32(const uint32_t* in, uint32_t* out, int64_t n, void* scratch, uint64_t* total_out,
                              hipStream_t st, const uint32_t* in2, uint32_t* out2) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = (n + kScanChunk - 1) / kScanChunk;
  uint64_t* totals = reinterpret_cast<uint64_t*>(scratch);
  const ScanArrays a = {{in, in2}, {out, out2}};
  const unsigned rows = in2 ? 2 : 1;
  const bool prefixed = nb > kScanBlocksMax;
  if (nb > 1) hipLaunchKernelGGL(scan_totals_kernel, dim3((unsigned)nb, rows), dim3(kScanThreads), 0, st, a, n, totals);
  if (prefixed) hipLaunchKernelGGL(scan_prefix_kernel, dim3(1, rows), dim3(1024), 0, st, totals, nb);
  hipLaunchKernelGGL(scan_chunk_kernel, dim3((unsigned)nb, rows), dim3(kScanThreads), 0, st, a, n, totals,
                     prefixed ? 1 : 0, total_out);
  return hipGetLastError();
}

// lanes of the wave (among those valid) that hold the same 8-bit digit
__device__ __forceinline__ unsigned long long same_digit(uint32_t d, bool valid) {
  const unsigned long long v = __ballot(valid);
  uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const unsigned long long bal = __ballot((d >> b) & 1u);
    const uint32_t m = (uint32_t)((int32_t)(d << (31 - b)) >> 31);  // all ones where the bit is set
    lo &= ~((uint32_t)bal ^ m);
    hi &= ~((uint32_t)(bal >> 32) ^ m);
  }
  return ((unsigned long long)hi << 32) | lo;
}

// ---------------------------------------------------------------------------
// order of the pairs of views of up to kOrderMax primitives, a workgroup per view
// ---------------------------------------------------------------------------
// Depth bits of the pairs -> their order (view by view, ascending depth,
// stable: the sort by tiles that follows needs no more), the tile counts in
// that order, the counts' exclusive scan and its total.  LSD radix of 8-bit
// passes over depth - least depth, three of them unless the depths span more
// than a factor of four or so: every wave owns up to 16 x 64 consecutive
// keys, a key's rank among its wave's equal digits comes from ballots, a scan
// over (digit, wave) gives the digits' places, and the keys change places
// through LDS.  A view's first place is the sum of the counts of the views
// before it, which its workgroup adds up itself.  Bound by its own chain of
// barriers and rounds (a CU per view).  3 x 3001 pairs: twenty launches of
// passes over all pairs 0.16 ms, one workgroup for all views and four passes
// 46 us, this 22; 2 x 7919 pairs 79 -> 39 us; 256 pairs 14 us.  A second
// row of workgroups, beside the first, scans the counts in primitive order.
constexpr int kOrderThreads = 1024;
constexpr int kOrderWaves = kOrderThreads / 64;
constexpr int kOrderItems = 16;
constexpr int kOrderMax = kOrderThreads * kOrderItems;  // 16384

__global__ void __launch_bounds__(kOrderThreads) order_small_kernel(const uint32_t* __restrict__ depth_bits,
                                                                    const uint32_t* __restrict__ counts, int n,
                                                                    uint32_t* __restrict__ order,
                                                                    uint32_t* __restrict__ counts_sorted,
                                                                    uint32_t* __restrict__ offsets,
                                                                    uint32_t* __restrict__ plain,
                                                                    unsigned long long* total_out) {
  const int64_t v0 = (int64_t)blockIdx.x * n;  // the view's first pair
  __shared__ uint32_t s_key[kOrderMax];
  __shared__ uint16_t s_idx[kOrderMax];
  __shared__ uint16_t s_cnt[kOrderWaves][kRadix];  // count, then first place, of each (wave, digit)
  __shared__ uint64_t s_warp[kOrderWaves];
  __shared__ uint32_t s_min, s_max;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // rounds of 64 keys per wave: the waves share the keys evenly
  const int rounds = (n + kOrderThreads - 1) / kOrderThreads;
  if (blockIdx.y == 1) {  // the scan in primitive order: `rounds` consecutive counts per thread, read twice
    const int end = min((t + 1) * rounds, n);
    uint64_t sum = 0, before = 0, total;
    for (int64_t i = t; i < v0; i += kOrderThreads) before += counts[i];
    for (int i = t * rounds; i < end; ++i) sum += counts[v0 + i];
    block_exclusive_scan<kOrderThreads>(before, &total, s_warp);
    uint64_t run = total;
    run += block_exclusive_scan<kOrderThreads>(sum, &total, s_warp);
    for (int i = t * rounds; i < end; ++i) {
      plain[v0 + i] = (uint32_t)run;
      run += counts[v0 + i];
    }
    return;
  }
  const int first = w * rounds * 64 + lane;
  const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  uint32_t key[kOrderItems];
  uint16_t idx[kOrderItems];
#pragma unroll
  for (int r = 0; r < kOrderItems; ++r) {
    const int i = first + 64 * r;
    key[r] = r < rounds && i < n ? depth_bits[v0 + i] : 0u;
    idx[r] = (uint16_t)i;
  }
  // depths relative to the least (culled pairs, depth 0, stay first)
  if (t == 0) {
    s_min = ~0u;
    s_max = 0u;
  }
  __syncthreads();
  uint32_t lo = ~0u, hi = 0u;
#pragma unroll
  for (int r = 0; r < kOrderItems; ++r) {
    lo = min(lo, key[r] - 1u);  // 0 wraps to the largest
    hi = max(hi, key[r]);
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o));
  }
  if (lane == 0) {
    atomicMin(&s_min, lo);
    atomicMax(&s_max, hi);
  }
  __syncthreads();
  const uint32_t least = s_min, most = s_max;  // (least depth - 1: the differences start at 1)
#pragma unroll
  for (int r = 0; r < kOrderItems; ++r) key[r] = key[r] ? key[r] - least : 0u;
  const int bits = most ? 32 - __builtin_clz(most - least) : 0;
  for (int shift = 0; shift < bits; shift += 8) {
    for (int i = t; i < kRadix * kOrderWaves / 2; i += kOrderThreads) reinterpret_cast<uint32_t*>(s_cnt)[i] = 0u;
    __syncthreads();
    uint16_t rank[kOrderItems];
#pragma unroll
    for (int r = 0; r < kOrderItems; ++r) {
      if (r >= rounds) break;
      const bool valid = first + 64 * r < n;
      const uint32_t d = (key[r] >> shift) & 0xFF;
      const unsigned long long peers = same_digit(d, valid);
      // the wave's own counter: read by all its equal digits, then advanced by the first
      const uint32_t seen = s_cnt[w][d];
      rank[r] = (uint16_t)(seen + __popcll(peers & below));
      __builtin_amdgcn_wave_barrier();
      if (valid && (peers & below) == 0) s_cnt[w][d] = (uint16_t)(seen + __popcll(peers));
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // exclusive scan over (digit, wave): four waves of a digit per thread
    static_assert(kRadix * kOrderWaves == 4 * kOrderThreads, "four counters per thread");
    uint16_t* mine = &s_cnt[4 * (t & 3)][t >> 2];
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c[k] = mine[k * kRadix];
      sum += c[k];
    }
    uint32_t total;
    uint32_t run = block_exclusive_scan<kOrderThreads>(sum, &total, reinterpret_cast<uint32_t*>(s_warp));
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      mine[k * kRadix] = (uint16_t)run;
      run += c[k];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kOrderItems; ++r) {
      if (r >= rounds || first + 64 * r >= n) continue;
      const uint32_t pos = (uint32_t)s_cnt[w][(key[r] >> shift) & 0xFF] + rank[r];
      s_key[pos] = key[r];
      s_idx[pos] = idx[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kOrderItems; ++r) {
      const int i = first + 64 * r;
      if (r < rounds && i < n) {
        key[r] = s_key[i];
        idx[r] = s_idx[i];
      }
    }
    __syncthreads();
  }
  // tile counts in order (through LDS, for the scan over consecutive entries)
#pragma unroll
  for (int r = 0; r < kOrderItems; ++r) {
    const int i = first + 64 * r;
    if (r < rounds && i < n) {
      const uint32_t cnt = counts[v0 + idx[r]];
      order[v0 + i] = (uint32_t)v0 + idx[r];
      counts_sorted[v0 + i] = cnt;
      s_key[i] = cnt;
    }
  }
  uint64_t sum = 0, before = 0;
  for (int64_t i = t; i < v0; i += kOrderThreads) sum += counts[i];
  if (v0) block_exclusive_scan<kOrderThreads>(sum, &before, s_warp);
  __syncthreads();
  sum = 0;
  for (int k = 0; k < rounds; ++k) {
    const int i = t * rounds + k;
    sum += i < n ? s_key[i] : 0u;
  }
  uint64_t total;
  uint64_t run = before + block_exclusive_scan<kOrderThreads>(sum, &total, s_warp);
  for (int k = 0; k < rounds; ++k) {
    const int i = t * rounds + k;
    if (i < n) {
      offsets[v0 + i] = (uint32_t)run;
      run += s_key[i];
    }
  }
  if (t == 0 && blockIdx.x == gridDim.x - 1) *total_out = before + total;
}

// A workgroup holds a CU, and reads the counts of all views before its own, so
// with many views the passes over all pairs win.  Binning and sorting, a
// workgroup per view / passes: 64 views of 1023 primitives 52 / 86 us, 256 of
// 255 63 / 88, 512 of 127 86 / 90, 512 of 15 69 / 85, 1024 of 63 133 / 95,
// 1024 of 15 111 / 93, 4096 of 15 389 / 94.
constexpr int kOrderViews = 512;

bool order_small(int64_t P, int32_t V) { return P <= kOrderMax && V <= kOrderViews; }

hipError_t launch_order_small(const uint32_t* depth_bits, const uint32_t* counts, int64_t P, int32_t V, uint32_t* order,
                              uint32_t* counts_sorted, uint32_t* offsets, uint32_t* plain,
                              unsigned long long* total_out, hipStream_t st) {
  hipLaunchKernelGGL(order_small_kernel, dim3((unsigned)V, 2), dim3(kOrderThreads), 0, st, depth_bits, counts, (int)P,
                     order, counts_sorted, offsets, plain, total_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// emit instances
// ---------------------------------------------------------------------------

// Instances of the pairs j (in depth order, or primitive order when order is
// null) at offsets[j] on.  A workgroup takes 64 consecutive pairs, whose
// instances form one contiguous output range, and its four waves write that
// range 256 instances at a time (thread t writes position base + t), so the
// writes are coalesced: each thread finds its pair by a binary search over
// the pairs' offsets in LDS and its tile from the pair's tile rectangle.
// Latency bound: a pair with many tiles holds its workgroup, so few pairs
// share one (100k Gaussians, 2.07e6 instances: one wave per 64 pairs 41 us,
// this 13 us).
constexpr int kEmitPairs = 64;

__global__ void __launch_bounds__(256) emit_kernel(EmitArgs a) {
  if (pair_block() == 0 && threadIdx.x == 0) {
    if (a.counters[CNT_INSTANCES] > (unsigned long long)a.capacity) a.counters[CNT_OVERFLOW] = 1ull;
    a.counters[CNT_DEPTH_SORT] = (unsigned long long)a.depth_sorted;
  }
  __shared__ uint32_t s_off[kEmitPairs + 1];  // first instance of each pair, relative to the block's base; then the end
  __shared__ int32_t s_tx0[kEmitPairs], s_nx[kEmitPairs], s_tile0[kEmitPairs], s_ntx[kEmitPairs];
  __shared__ uint32_t s_p[kEmitPairs], s_d[kEmitPairs];
  const int64_t n = a.P * a.V;
  const int64_t j0 = pair_block() * kEmitPairs;
  if (j0 >= n) return;
  const int last = (int)min((int64_t)(kEmitPairs - 1), n - 1 - j0);
  // uint32 arithmetic: the differences stay exact if the scan wrapped
  const uint32_t base = a.offsets[j0];
  if ((int)threadIdx.x <= last) {
    const int l = threadIdx.x;
    const int64_t j = j0 + l;
    const int64_t i = a.order ? (int64_t)a.order[j] : j;
    const int v = (int)(i / a.P);
    const CamDev& cam = a.cams[v];
    const int4 rc = reinterpret_cast<const int4*>(a.rects)[i];
    const int tx0 = rc.x / cam.tile_w, tx1 = rc.y / cam.tile_w;
    s_tx0[l] = tx0;
    s_nx[l] = tx1 - tx0 + 1;
    s_tile0[l] = cam.tile_base + (rc.z / cam.tile_h) * cam.ntx;
    s_ntx[l] = cam.ntx;
    s_p[l] = (uint32_t)(i - (int64_t)v * a.P);
    s_d[l] = a.depth_bits[i];
    const uint32_t off = a.offsets[j] - base;
    s_off[l] = off;
    if (l == last) s_off[kEmitPairs] = off + a.tile_counts[i];
  }
  __syncthreads();
  const uint32_t total = s_off[kEmitPairs];
  for (uint32_t o = threadIdx.x; o < total; o += 256) {
    // the last pair k with s_off[k] <= o (pairs without instances share
    // their offset with the next one and are skipped by taking the last)
    int lo = 0, hi = last;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (s_off[mid] <= o) lo = mid; else hi = mid - 1;
    }
    const uint32_t k = o - s_off[lo], nx = (uint32_t)s_nx[lo];
    const uint32_t row = k / nx;
    const int64_t pos = (int64_t)base + (int64_t)o;
    if (pos < a.capacity) {
      const unsigned long long tile =
          (unsigned long long)(s_tile0[lo] + (int)row * s_ntx[lo] + s_tx0[lo] + (int)(k - row * nx));
      a.keys[pos] = (tile << 31) | (unsigned long long)s_d[lo];
      a.values[pos] = s_p[lo];
    }
  }
}

hipError_t launch_emit(const EmitArgs& a, hipStream_t st) {
  const int64_t n = a.P * a.V;
  hipLaunchKernelGGL(emit_kernel, pair_grid((n + kEmitPairs - 1) / kEmitPairs), dim3(256), 0, st, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// stable LSD radix sort
// ---------------------------------------------------------------------------
// number of elements to sort: *count, at most the capacity of the buffers
__device__ __forceinline__ int64_t sort_count(const unsigned long long* count, int64_t capacity) {
  const unsigned long long n = *count;
  return n > (unsigned long long)capacity ? capacity : (int64_t)n;
}

// Digit counts of each block's chunk, hist[digit][block].  clear / n_clear:
// words to zero on the way.
template <typename K, int R>
__global__ void __launch_bounds__(kSortThreads) radix_hist_kernel(const K* __restrict__ keys,
                                                                  const unsigned long long* count,
                                                                  int64_t capacity, int shift,
                                                                  uint32_t* __restrict__ hist, int64_t nblocks,
                                                                  uint32_t* __restrict__ clear, int64_t n_clear) {
  __shared__ uint32_t s_h[kRadix];
  s_h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t n = count ? sort_count(count, capacity) : capacity;
  const int64_t base = (int64_t)blockIdx.x * (kSortThreads * R);
  for (int r = 0; r < R; ++r) {
    const int64_t i = base + (int64_t)r * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&s_h[(keys[i] >> shift) & 0xFF], 1u);
  }
  for (int64_t i = (int64_t)blockIdx.x * kSortThreads + threadIdx.x; i < n_clear; i += nblocks * kSortThreads)
    clear[i] = 0u;
  __syncthreads();
  hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = s_h[threadIdx.x];
}

// Per digit (one block each): exclusive prefix of its counts over the blocks,
// and its total.
__global__ void __launch_bounds__(kScanThreads) radix_prefix_kernel(const uint32_t* __restrict__ hist,
                                                                    uint32_t* __restrict__ offs, int64_t nblocks,
                                                                    uint32_t* __restrict__ totals) {
  __shared__ uint32_t s_warp[kScanThreads / 64];
  const uint32_t* row = hist + (int64_t)blockIdx.x * nblocks;
  uint32_t* out = offs + (int64_t)blockIdx.x * nblocks;
  uint32_t carry = 0;
  if (nblocks <= kScanThreads) {
    const uint32_t x = threadIdx.x < nblocks ? row[threadIdx.x] : 0u;
    const uint32_t e = block_exclusive_scan<kScanThreads>(x, &carry, s_warp);
    if (threadIdx.x < nblocks) out[threadIdx.x] = e;
  } else {
    for (int64_t b0 = 0; b0 < nblocks; b0 += kScanChunk) {
      const int64_t base = b0 + (int64_t)threadIdx.x * kScanItems;
      uint32_t v[kScanItems], sum = 0, total;
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) {
        v[k] = base + k < nblocks ? row[base + k] : 0u;
        sum += v[k];
      }
      uint32_t run = carry + block_exclusive_scan<kScanThreads>(sum, &total, s_warp);
#pragma unroll
      for (int k = 0; k < kScanItems; ++k) {
        if (base + k < nblocks) out[base + k] = run;
        run += v[k];
      }
      carry += total;
    }
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Stable scatter of one block's chunk.  The chunk's keys are first placed
// in LDS in digit order (the block's own digit counts from the histogram
// give each digit's local start; ballot ranks keep the input order within a
// digit), then written out from LDS in that order, so consecutive threads
// write consecutive addresses of a digit's output run (runs of about
// chunk / 256 keys) instead of one scattered key each.  vin null: the values
// are the positions.  gather: the last pass over the pairs -- instead of the
// keys, gout receives gather[value].
template <typename K, int R>
__global__ void __launch_bounds__(kSortThreads) radix_scatter_kernel(
    const K* __restrict__ kin, const uint32_t* __restrict__ vin, K* __restrict__ kout, uint32_t* __restrict__ vout,
    const unsigned long long* count, int64_t capacity, int shift, const uint32_t* __restrict__ offs,
    const uint32_t* __restrict__ hist, const uint32_t* __restrict__ totals, int64_t nblocks,
    const uint32_t* __restrict__ gather, uint32_t* __restrict__ gout) {
  constexpr int NW = kSortThreads / 64;
  constexpr int CHUNK = kSortThreads * R;
  __shared__ K s_key[CHUNK];
  __shared__ uint32_t s_val[CHUNK];
  __shared__ uint32_t s_lstart[kRadix];     // first local position of each digit
  __shared__ uint32_t s_run[kRadix];        // running local position of each digit
  __shared__ uint32_t s_goff[kRadix];       // global start of each digit for this block
  __shared__ uint32_t s_wcnt[NW][kRadix];   // per-wave digit counts in the current round
  __shared__ uint32_t s_wsum[NW];
  const int64_t n = count ? sort_count(count, capacity) : capacity;
  const int64_t base = (int64_t)blockIdx.x * CHUNK;
  if (base >= n) return;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // all of this thread's keys and values first, so their loads are in flight together
  K rkey[R];
  uint32_t rval[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = base + (int64_t)r * kSortThreads + t;
    rkey[r] = i < n ? kin[i] : (K)0;
    rval[r] = i < n ? (vin ? vin[i] : (uint32_t)i) : 0u;
  }
  // local digit starts: exclusive scan of this block's digit counts; global
  // ones: the digits' totals scanned, plus this digit's prefix over the blocks
  uint32_t all;
  const uint32_t local = block_exclusive_scan<kSortThreads>(hist[(int64_t)t * nblocks + blockIdx.x], &all, s_wsum);
  const uint32_t digit = block_exclusive_scan<kSortThreads>(totals[t], &all, s_wsum);
  s_goff[t] = digit + offs[(int64_t)t * nblocks + blockIdx.x];
  s_lstart[t] = local;
  s_run[t] = local;
  const unsigned long long lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t rbase = base + (int64_t)r * kSortThreads;
    if (rbase >= n) break;  // uniform over the block
#pragma unroll
    for (int k = 0; k < NW; ++k) s_wcnt[k][t] = 0;
    __syncthreads();
    const int64_t i = rbase + t;
    const bool valid = i < n;
    const K key = rkey[r];
    const uint32_t val = rval[r];
    const uint32_t d = valid ? (uint32_t)((key >> shift) & 0xFF) : 0u;
    // lanes of this wave holding the same digit
    const unsigned long long peers = same_digit(d, valid);
    const uint32_t rank_w = (uint32_t)__popcll(peers & lt_mask);
    if (valid && rank_w == 0) s_wcnt[w][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    // per digit: prefix over the waves, advance the running local position
    {
      uint32_t run = s_run[t];
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        const uint32_t cw = s_wcnt[k][t];
        s_wcnt[k][t] = run;
        run += cw;
      }
      s_run[t] = run;
    }
    __syncthreads();
    if (valid) {
      const uint32_t lpos = s_wcnt[w][d] + rank_w;
      s_key[lpos] = key;
      s_val[lpos] = val;
    }
    __syncthreads();
  }
  // write the chunk out in digit order
  const int64_t nloc = n - base < CHUNK ? n - base : CHUNK;
  for (int q = t; q < nloc; q += kSortThreads) {
    const K key = s_key[q];
    const uint32_t d = (uint32_t)((key >> shift) & 0xFF);
    const uint32_t pos = s_goff[d] + ((uint32_t)q - s_lstart[d]);
    const uint32_t val = s_val[q];
    vout[pos] = val;
    if (gather)
      gout[pos] = gather[val];
    else
      kout[pos] = key;
  }
}

size_t sort_scratch_bytes(int64_t n, int rounds) {
  const int64_t nh = sort_blocks(n, rounds) * kRadix;
  return ((size_t)nh * 4 + 255) / 256 * 256 * 2 + kRadix * 4;
}

struct SortScratch {
  uint32_t *hist, *offs, *totals;
  int64_t nblocks;
  int rounds;
  SortScratch(int64_t n, int r, void* scratch) : nblocks(sort_blocks(n, r)), rounds(r) {
    const size_t row = ((size_t)nblocks * kRadix * 4 + 255) / 256 * 256;
    char* sp = reinterpret_cast<char*>(scratch);
    hist = reinterpret_cast<uint32_t*>(sp);
    offs = reinterpret_cast<uint32_t*>(sp + row);
    totals = reinterpret_cast<uint32_t*>(sp + 2 * row);
  }
};

template <typename K, int R>
static void radix_pass(const K* ki, const uint32_t* vi, K* ko, uint32_t* vo, int64_t capacity,
                       const unsigned long long* count, int shift, const SortScratch& sc, uint32_t* clear,
                       int64_t n_clear, const uint32_t* gather, uint32_t* gout, hipStream_t st) {
  const dim3 grid((unsigned)sc.nblocks), block(kSortThreads);
  hipLaunchKernelGGL((radix_hist_kernel<K, R>), grid, block, 0, st, ki, count, capacity, shift, sc.hist, sc.nblocks,
                     clear, n_clear);
  hipLaunchKernelGGL(radix_prefix_kernel, dim3(kRadix), dim3(kScanThreads), 0, st, sc.hist, sc.offs, sc.nblocks,
                     sc.totals);
  hipLaunchKernelGGL((radix_scatter_kernel<K, R>), grid, block, 0, st, ki, vi, ko, vo, count, capacity, shift, sc.offs,
                     sc.hist, sc.totals, sc.nblocks, gather, gout);
}

template <typename K>
static void radix_pass(const K* ki, const uint32_t* vi, K* ko, uint32_t* vo, int64_t capacity,
                       const unsigned long long* count, int shift, const SortScratch& sc, uint32_t* clear,
                       int64_t n_clear, const uint32_t* gather, uint32_t* gout, hipStream_t st) {
  if (sc.rounds == 4)
    radix_pass<K, 4>(ki, vi, ko, vo, capacity, count, shift, sc, clear, n_clear, gather, gout, st);
  else
    radix_pass<K, 16>(ki, vi, ko, vo, capacity, count, shift, sc, clear, n_clear, gather, gout, st);
}

// Sorts the first min(*count, capacity) keys/values by bits [lo_bit, lo_bit +
// key_bits), stably, and zeroes n_clear words at `clear` on the way.  Buffers
// ping-pong between (k0,v0) and (k1,v1); the input is in (k0,v0) and the
// result ends in (k0,v0) if the number of passes is even, else in (k1,v1).
hipError_t radix_sort(unsigned long long* k0, uint32_t* v0, unsigned long long* k1, uint32_t* v1, int64_t capacity,
                      const unsigned long long* count, int lo_bit, int key_bits, int rounds, void* scratch,
                      uint32_t* clear, int64_t n_clear, hipStream_t st) {
  if (capacity <= 0) return hipSuccess;
  const SortScratch sc(capacity, rounds, scratch);
  const int passes = (key_bits + 7) / 8;
  unsigned long long *ki = k0, *ko = k1;
  uint32_t *vi = v0, *vo = v1;
  for (int ps = 0; ps < passes; ++ps) {
    radix_pass<unsigned long long>(ki, vi, ko, vo, capacity, count, lo_bit + 8 * ps, sc, clear,
                                   ps == 0 ? n_clear : 0, nullptr, nullptr, st);
    std::swap(ki, ko);
    std::swap(vi, vo);
  }
  return hipGetLastError();
}

// Order of n pairs by their depth bits (stable): pair indices in `order`,
// counts[order] in `counts_sorted`.  ka, kb, va: scratch of n words each.
hipError_t order_pairs(const uint32_t* depth_bits, const uint32_t* counts, int64_t n, uint32_t* ka, uint32_t* kb,
                       uint32_t* va, uint32_t* order, uint32_t* counts_sorted, int rounds, void* scratch,
                       hipStream_t st) {
  const SortScratch sc(n, rounds, scratch);
  radix_pass<uint32_t>(depth_bits, nullptr, ka, va, n, nullptr, 0, sc, nullptr, 0, nullptr, nullptr, st);
  radix_pass<uint32_t>(ka, va, kb, order, n, nullptr, 8, sc, nullptr, 0, nullptr, nullptr, st);
  radix_pass<uint32_t>(kb, order, ka, va, n, nullptr, 16, sc, nullptr, 0, nullptr, nullptr, st);
  radix_pass<uint32_t>(ka, va, nullptr, order, n, nullptr, 24, sc, nullptr, 0, counts, counts_sorted, st);
  return hipGetLastError();
}

int radix_passes(int key_bits) { return (key_bits + 7) / 8; }

// ---------------------------------------------------------------------------
// tile ranges
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) ranges_kernel(const unsigned long long* __restrict__ keys,
                                                     const unsigned long long* counters, int64_t capacity,
                                                     uint32_t* __restrict__ ranges) {
  const int64_t n = sort_count(counters + CNT_INSTANCES, capacity);
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    const unsigned long long tile = keys[i] >> 31;
    if (i == 0 || (keys[i - 1] >> 31) != tile) ranges[2 * tile] = (uint32_t)i;
    if (i == n - 1 || (keys[i + 1] >> 31) != tile) ranges[2 * tile + 1] = (uint32_t)(i + 1);
  }
}

// The order in which the rasterizers take the tiles: most instances first, in
// steps of 64 instances (tiles of a step in any order -- the order only
// balances the load).  A counting sort over 1024 steps, by one workgroup up to
// kTileOrderOne tiles, else spread over blocks that share global counters (four
// launches).  The whole sort with one primitive, one workgroup / spread: 2500
// tiles 20.2 / 21.9 us, 4096 23.1 / 22.0, 5700 30.6 / 27.5, 8160 34.9 / 27.3,
// 32400 76 / 30; with 50000 primitives 51.9 / 55.7, 54.2 / 56.2, 58.6 / 58.1,
// 64.5 / 60.2, 108 / 69.
constexpr int kOrderSteps = 1024;
constexpr int64_t kTileOrderOne = 5120;

__device__ __forceinline__ int tile_step(const uint32_t* ranges, int64_t t) {
  const uint2 r = reinterpret_cast<const uint2*>(ranges)[t];
  const uint32_t s = (r.y - r.x + 63) >> 6;  // empty tiles alone in the last step
  return kOrderSteps - 1 - (int)(s < kOrderSteps - 1 ? s : kOrderSteps - 1);
}

__global__ void __launch_bounds__(1024) tile_order_kernel(const uint32_t* __restrict__ ranges, int64_t n,
                                                          uint32_t* __restrict__ order) {
  __shared__ uint32_t s_place[kOrderSteps];
  __shared__ uint32_t s_warp[16];
  const int t = threadIdx.x;
  s_place[t] = 0;
  __syncthreads();
  for (int64_t i = t; i < n; i += 1024) atomicAdd(&s_place[tile_step(ranges, i)], 1u);
  __syncthreads();
  uint32_t total;
  const uint32_t c = s_place[t];
  const uint32_t e = block_exclusive_scan<1024>(c, &total, s_warp);
  s_place[t] = e;
  __syncthreads();
  for (int64_t i = t; i < n; i += 1024) order[atomicAdd(&s_place[tile_step(ranges, i)], 1u)] = (uint32_t)i;
}

// many tiles: counts, their scan and the placing as three kernels over all CUs
__global__ void __launch_bounds__(256) tile_step_counts_kernel(const uint32_t* __restrict__ ranges, int64_t n,
                                                               uint32_t* __restrict__ counts) {
  __shared__ uint32_t s_c[kOrderSteps];
  for (int i = threadIdx.x; i < kOrderSteps; i += 256) s_c[i] = 0;
  __syncthreads();
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    atomicAdd(&s_c[tile_step(ranges, i)], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kOrderSteps; i += 256)
    if (s_c[i]) atomicAdd(&counts[i], s_c[i]);
}

__global__ void __launch_bounds__(1024) tile_step_scan_kernel(uint32_t* counts) {
  __shared__ uint32_t s_warp[16];
  uint32_t total;
  const uint32_t e = block_exclusive_scan<1024>(counts[threadIdx.x], &total, s_warp);
  counts[threadIdx.x] = e;
}

// Each block places `chunk` consecutive tiles: it counts them by step, takes
// its share of every step's places with one addition, and deals them out in
// LDS.  (With an addition per tile, tiles of one step waited for each other:
// 36864 empty tiles 0.3 ms, this 10 us.)
__global__ void __launch_bounds__(256) tile_place_kernel(const uint32_t* __restrict__ ranges, int64_t n, int64_t chunk,
                                                         uint32_t* __restrict__ places, uint32_t* __restrict__ order) {
  __shared__ uint32_t s_place[kOrderSteps];
  for (int i = threadIdx.x; i < kOrderSteps; i += 256) s_place[i] = 0;
  __syncthreads();
  const int64_t i0 = (int64_t)blockIdx.x * chunk + threadIdx.x, i1 = min((int64_t)(blockIdx.x + 1) * chunk, n);
  for (int64_t i = i0; i < i1; i += 256) atomicAdd(&s_place[tile_step(ranges, i)], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kOrderSteps; i += 256)
    if (s_place[i]) s_place[i] = atomicAdd(&places[i], s_place[i]);
  __syncthreads();
  for (int64_t i = i0; i < i1; i += 256) order[atomicAdd(&s_place[tile_step(ranges, i)], 1u)] = (uint32_t)i;
}

size_t tile_order_scratch_bytes(int64_t n_tiles) { return n_tiles > kTileOrderOne ? kOrderSteps * sizeof(uint32_t) : 0; }

hipError_t launch_tile_order(const uint32_t* ranges, int64_t n_tiles, uint32_t* order, uint32_t* scratch,
                             hipStream_t st) {
  if (n_tiles <= 0) return hipSuccess;
  if (n_tiles <= kTileOrderOne) {
    hipLaunchKernelGGL(tile_order_kernel, dim3(1), dim3(1024), 0, st, ranges, n_tiles, order);
    return hipGetLastError();
  }
  hipError_t e = fill_u32(scratch, kOrderSteps, 0u, st);
  if (e != hipSuccess) return e;
  int64_t blocks = (n_tiles + 255) / 256;
  if (blocks > 512) blocks = 512;
  hipLaunchKernelGGL(tile_step_counts_kernel, dim3((unsigned)blocks), dim3(256), 0, st, ranges, n_tiles, scratch);
  hipLaunchKernelGGL(tile_step_scan_kernel, dim3(1), dim3(1024), 0, st, scratch);
  hipLaunchKernelGGL(tile_place_kernel, dim3((unsigned)blocks), dim3(256), 0, st, ranges, n_tiles,
                     (n_tiles + blocks - 1) / blocks, scratch, order);
  return hipGetLastError();
}

// ranges are cleared by the sort before (tiles without instances keep [0, 0))
hipError_t launch_ranges(const unsigned long long* keys, const unsigned long long* counters, int64_t capacity,
                         uint32_t* ranges, hipStream_t st) {
  int64_t blocks = (capacity + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(ranges_kernel, dim3((unsigned)blocks), dim3(256), 0, st, keys, counters, capacity, ranges);
  return hipGetLastError();
}

}  // namespace snp
