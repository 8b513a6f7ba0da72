// Index binding, gather and scatter for gfx950 (section 3.2.2 of the paper: index arrays are
// checked and negative indices converted; boolean masks are counted and converted to explicit
// indices; bound to strides both become relative offsets into the data buffer, after which the
// indexed elements are copied out of, or into, the tensor).
//
//   ocn_index_offsets  one lane per index: wrap, range check, multiply by the stride; invalid
//                      indices are counted (one integer atomic per wavefront that saw any)
//   ocn_mask_offsets   stream compaction in the mask's row-major order, one to three launches and no
//                      waiting between workgroups: per-workgroup counts, an exclusive scan of
//                      the counts by one workgroup (through LDS, coalesced both ways), then every workgroup writes the offsets of
//                      its selected elements behind its prefix (smaller masks: behind the sum of the counts,
//                      or of the mask itself, before it) (staged in LDS so that the
//                      stores are coalesced).  Lanes own 16 consecutive mask bytes (one 128-bit
//                      load when the mask is contiguous), four in smaller masks.
//   ocn_gather/scatter one lane per copied item (an element, or 16 bytes where the rows' fastest
//                      dimension is contiguous and aligned), rows of `inner` elements per offset
//                      (gapless rows in 16-byte pieces of any alignment: row_pieces_kernel);
//                      short rows share a workgroup, long ones take several.  Offsets outside the stated range are skipped, never followed.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <type_traits>

#include "../../include/ocn.h"
#include "dtypes.hpp"
#include "dev_types.hpp"
#include "planner.hpp"

namespace ocn {
namespace {

constexpr int kMaskPerLane = 16;                       // mask elements per lane
constexpr int kMaskChunk = kBlock * kMaskPerLane;      // per workgroup
constexpr int kScanBlock = 1024;

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv &f) { return (__umulhi(n, f.m) + n) >> f.s; }

// ---------------------------------------------------------------------------------------
// index arrays
// ---------------------------------------------------------------------------------------

struct IndexArgs {
  const char *idx;
  char *off;
  int32_t ndim;
  int64_t size[kMaxDims], si[kMaxDims], so[kMaxDims];  // row-major: last dim fastest
  int64_t n, dim_size, stride;
  unsigned long long *invalid;
};

__global__ void fill_u64_kernel(unsigned long long *p, unsigned long long v) { *p = v; }

__global__ __launch_bounds__(kBlock) void index_offsets_kernel(const IndexArgs p) {
  // the grid is capped (a launch cannot have 2^32 lanes): longer index arrays loop; every lane
  // of a wavefront makes the same number of trips, so that the vote below stays whole
  const int64_t step = (int64_t)gridDim.x * kBlock;
  for (int64_t e0 = (int64_t)blockIdx.x * kBlock; e0 < p.n; e0 += step) {
  const int64_t e = e0 + threadIdx.x;
  bool bad = false;
  if (e < p.n) {
    int64_t rem = e, oi = 0, oo = 0;
#pragma unroll
    for (int d = kMaxDims - 1; d >= 0; --d) {
      if (d < p.ndim) {
        const int64_t q = rem / p.size[d];
        const int64_t i = rem - q * p.size[d];
        rem = q;
        oi += i * p.si[d];
        oo += i * p.so[d];
      }
    }
    int64_t i = *reinterpret_cast<const int64_t *>(p.idx + oi);
    if (i < 0) i += p.dim_size;
    bad = i < 0 || i >= p.dim_size;
    *reinterpret_cast<int64_t *>(p.off + oo) = bad ? 0 : i * p.stride;
  }
  const unsigned long long votes = __ballot(bad);
  if (votes != 0 && (threadIdx.x & (kWave - 1)) == 0) atomicAdd(p.invalid, (unsigned long long)__popcll(votes));
  }
}

// Both tensors contiguous (and 16-byte aligned): two indices per lane, one 16-byte load and one
// 16-byte store each, streamed when the arrays are too large to stay cached; no index
// decomposition (the kernel above divides 64-bit numbers once per dim and element: 2^26
// indices 264 us).
__global__ __launch_bounds__(kBlock) void index_offsets_flat_kernel(const IndexArgs p, int nt) {
  using L2 = long long __attribute__((ext_vector_type(2)));
  const int64_t npair = (p.n + 1) / 2;
  const int64_t step = (int64_t)gridDim.x * kBlock;
  for (int64_t e0 = (int64_t)blockIdx.x * kBlock; e0 < npair; e0 += step) {
    const int64_t e = e0 + threadIdx.x;
    int nbad = 0;
    if (e < npair) {
      const bool both = 2 * e + 1 < p.n;
      L2 v;
      if (both) {
        if (nt) { asm volatile(""); v = __builtin_nontemporal_load(reinterpret_cast<const L2 *>(p.idx) + e); asm volatile(""); }
        else v = reinterpret_cast<const L2 *>(p.idx)[e];
      } else {
        v.x = reinterpret_cast<const long long *>(p.idx)[2 * e];
        v.y = 0;
      }
      long long i0 = v.x < 0 ? v.x + p.dim_size : v.x, i1 = v.y < 0 ? v.y + p.dim_size : v.y;
      const bool bad0 = i0 < 0 || i0 >= p.dim_size, bad1 = both && (i1 < 0 || i1 >= p.dim_size);
      nbad = (bad0 ? 1 : 0) + (bad1 ? 1 : 0);
      L2 r;
      r.x = bad0 ? 0 : i0 * p.stride;
      r.y = bad1 ? 0 : i1 * p.stride;
      if (both) {
        if (nt) { asm volatile(""); __builtin_nontemporal_store(r, reinterpret_cast<L2 *>(p.off) + e); asm volatile(""); }
        else reinterpret_cast<L2 *>(p.off)[e] = r;
      } else {
        reinterpret_cast<long long *>(p.off)[2 * e] = r.x;
      }
    }
    // every lane of a wavefront makes the same number of trips, so the shuffles stay whole
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) nbad += __shfl_xor(nbad, d, kWave);
    if (nbad != 0 && (threadIdx.x & (kWave - 1)) == 0) atomicAdd(p.invalid, (unsigned long long)nbad);
  }
}

// Few indices, both tensors contiguous: one workgroup of 1024 lanes binds them all and writes the
// number of invalid ones itself, where several would add to a counter that another launch has to
// clear first (launch and gap of that one: 2.5 us of a call's host time, 1.3 us on the device).
constexpr int64_t kIndexOneBlock = 4096, kIndexCounted = 16384;
__global__ __launch_bounds__(1024) void index_offsets_small_kernel(const IndexArgs p) {
  constexpr int U = 4;
  __shared__ int32_t waves[1024 / kWave];
  int32_t nbad = 0;
  for (int64_t e0 = threadIdx.x; e0 < p.n; e0 += 1024 * U) {
    int64_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e0 + u * 1024 < p.n) v[u] = reinterpret_cast<const int64_t *>(p.idx)[e0 + u * 1024];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (e0 + u * 1024 < p.n) {
        const int64_t i = v[u] < 0 ? v[u] + p.dim_size : v[u];
        const bool bad = i < 0 || i >= p.dim_size;
        reinterpret_cast<int64_t *>(p.off)[e0 + u * 1024] = bad ? 0 : i * p.stride;
        nbad += bad ? 1 : 0;
      }
    }
  }
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) nbad += __shfl_xor(nbad, d, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) waves[threadIdx.x / kWave] = nbad;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t all = 0;
    for (int w = 0; w < 1024 / kWave; ++w) all += waves[w];
    *p.invalid = (unsigned long long)all;
  }
}

// Some more of them, also aligned for pairs and the tensors apart: the first workgroup reads all indices and
// writes the number of invalid ones, the others bind a pair per lane and count nothing, so that no launch clears a
// counter and no workgroup waits for another.  What one workgroup reads and writes in turn bounds the kernel above:
// 10000 indices with a gather 7.0 -> 5.4 us, 16000 8.7 -> 6.2, 5000 5.2 -> 4.9, 2000 the same.  The one that counts
// is the last to end beyond that: at 20000 clearing a counter is as fast (6.9 us and 6.7), at 65536 faster (11.1, 7.3).
__global__ __launch_bounds__(1024) void index_offsets_counted_kernel(const IndexArgs p) {
  using L2 = long long __attribute__((ext_vector_type(2)));
  constexpr uint32_t U = 8;
  __shared__ uint32_t waves[1024 / kWave];
  const uint32_t n = (uint32_t)p.n, pairs = n / 2, tid = threadIdx.x;
  const L2 *idx = reinterpret_cast<const L2 *>(p.idx);
  const long long *one = reinterpret_cast<const long long *>(p.idx) + (n - 1);   // of an odd number the last
  auto invalid = [&](long long i) { return (i < 0 ? i + p.dim_size < 0 : i >= p.dim_size) ? 1u : 0u; };
  auto bound = [&](long long i) { return invalid(i) ? 0ll : (i < 0 ? i + p.dim_size : i) * p.stride; };
  if (blockIdx.x != 0) {
    const uint32_t e = (blockIdx.x - 1) * 1024 + tid;
    if (e < pairs) {
      const L2 v = idx[e];
      L2 r;
      r.x = bound(v.x);
      r.y = bound(v.y);
      reinterpret_cast<L2 *>(p.off)[e] = r;
    } else if (e == pairs && (n & 1)) {
      reinterpret_cast<long long *>(p.off)[n - 1] = bound(*one);
    }
    return;
  }
  uint32_t bad = tid == 0 && (n & 1) ? invalid(*one) : 0;
  for (uint32_t e0 = tid; e0 < pairs; e0 += 1024 * U) {
    L2 v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) v[u] = idx[e0 + u * 1024 < pairs ? e0 + u * 1024 : e0];   // (all on their way at once)
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (e0 + u * 1024 < pairs) bad += invalid(v[u].x) + invalid(v[u].y);
  }
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) bad += __shfl_xor(bad, d, kWave);
  if ((tid & (kWave - 1)) == 0) waves[tid / kWave] = bad;
  __syncthreads();
  if (tid == 0) {
    uint32_t all = 0;
    for (int w = 0; w < 1024 / kWave; ++w) all += waves[w];
    *p.invalid = all;
  }
}

// ---------------------------------------------------------------------------------------
// boolean masks
// ---------------------------------------------------------------------------------------

struct MaskArgs {
  const char *mask;
  int32_t ndim;                       // canonical dims, row-major: last fastest
  FastDiv div[kMaxDims];
  int64_t sm[kMaxDims], st[kMaxDims]; // mask / target byte strides
  uint32_t n;                         // mask elements (< 2^31)
  int32_t contig;                     // the mask is one contiguous, 16-byte aligned run
  uint32_t *block_counts;             // [nblocks]; after the scan: exclusive prefixes
  uint32_t nblocks;
  int64_t *offsets;
  int64_t capacity;
  int64_t *count;
  int32_t nt_store;                   // large result: streaming stores
};

__device__ __forceinline__ void mask_decode(const MaskArgs &p, uint32_t e, int64_t &om, int64_t &ot) {
  om = 0;
  ot = 0;
#pragma unroll
  for (int d = kMaxDims - 1; d >= 0; --d) {
    if (d < p.ndim) {
      const uint32_t q = d == 0 ? 0u : fdiv(e, p.div[d]);
      const uint32_t i = e - q * p.div[d].d;
      e = q;
      om += (int64_t)i * p.sm[d];
      ot += (int64_t)i * p.st[d];
    }
  }
}

// bit k set: element e0 + k is selected
__device__ __forceinline__ uint32_t mask_flags(const MaskArgs &p, uint32_t e0) {
  uint32_t flags = 0;
  if (e0 >= p.n) return 0;
  if (p.contig && e0 + kMaskPerLane <= p.n) {
    const uint4 v = *reinterpret_cast<const uint4 *>(p.mask + e0);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int k = 0; k < kMaskPerLane; ++k)
      if ((w[k >> 2] >> (8 * (k & 3))) & 0xffu) flags |= 1u << k;
    return flags;
  }
#pragma unroll 4
  for (int k = 0; k < kMaskPerLane; ++k) {
    const uint32_t e = e0 + (uint32_t)k;
    if (e < p.n) {
      int64_t om, ot;
      mask_decode(p, e, om, ot);
      if (*reinterpret_cast<const uint8_t *>(p.mask + om) != 0) flags |= 1u << k;
    }
  }
  return flags;
}

// exclusive prefix of `v` over the workgroup's lanes; total in `sum` (all lanes)
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *lds, uint32_t &sum) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t inc = v;
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const uint32_t up = (uint32_t)__shfl_up((int)inc, d, kWave);
    if (lane >= d) inc += up;
  }
  if (lane == kWave - 1) lds[wave] = inc;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) {
    if (w < wave) before += lds[w];
    total += lds[w];
  }
  sum = total;
  return before + inc - v;
}

// bytes that are not zero: bit 7 of each byte of ((w & 0x7f..) + 0x7f..) | w
__device__ __forceinline__ uint32_t nonzero_bytes(const uint4 &v) {
  auto word = [](uint32_t w) { return (uint32_t)__popc((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) & 0x80808080u); };
  return word(v.x) + word(v.y) + word(v.z) + word(v.w);
}

__global__ __launch_bounds__(kBlock) void mask_count_kernel(const MaskArgs p) {
  __shared__ uint32_t lds[kBlock / kWave];
  const uint32_t e0 = (blockIdx.x * kBlock + threadIdx.x) * kMaskPerLane;
  const uint32_t c = (uint32_t)__popc(mask_flags(p, e0));
  uint32_t sum;
  (void)block_exclusive_scan(c, lds, sum);
  if (threadIdx.x == 0) p.block_counts[blockIdx.x] = sum;
}

// The same counts for a contiguous mask: a wavefront per chunk of kMaskChunk bytes, every lane with four
// 16-byte loads in flight (the loads of a wavefront cover 1 KiB each).  TOTALS: a workgroup per
// kMaskGroup chunks, and its total as well; else four chunks per workgroup, which fill the chip earlier
// (64 chunks 3.4 us, 4.3 in groups).  (One load per lane and a workgroup per chunk read a 64 MB mask at
// 3 TB/s; four chunks per wavefront 30 MB in 7.5 us, 6.7 so.)
constexpr int kMaskGroup = 16;
template <bool TOTALS> __global__ __launch_bounds__((TOTALS ? kMaskGroup : kBlock / kWave) * kWave) void mask_count_contig_kernel(const MaskArgs p) {
  __shared__ uint32_t lds[kMaskGroup];
  const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t chunk = blockIdx.x * (uint32_t)(TOTALS ? kMaskGroup : kBlock / kWave) + wave;
  uint32_t c = 0;
  if (chunk < p.nblocks) {            // (the same for all lanes of a wavefront)
    const uint32_t base = chunk * (uint32_t)kMaskChunk;
    constexpr int kPieces = kMaskChunk / (kWave * 16);
    uint4 v[kPieces];
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      const uint32_t e = base + (uint32_t)k * (kWave * 16) + lane * 16u;
      v[k] = make_uint4(0u, 0u, 0u, 0u);
      if (e + 16u <= p.n) {
        v[k] = *reinterpret_cast<const uint4 *>(p.mask + e);
      } else if (e < p.n) {               // the ragged end of the mask, byte by byte
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        for (uint32_t i = 0; e + i < p.n; ++i)
          w[i >> 2] |= (uint32_t) * reinterpret_cast<const uint8_t *>(p.mask + e + i) << (8 * (i & 3));
        v[k] = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
#pragma unroll
    for (int k = 0; k < kPieces; ++k) c += nonzero_bytes(v[k]);
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) c += (uint32_t)__shfl_xor((int)c, d, kWave);
    if (lane == 0) p.block_counts[chunk] = c;
  }
  if constexpr (TOTALS) {
    if (lane == 0) lds[wave] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t total = 0;
#pragma unroll
      for (int w = 0; w < kMaskGroup; ++w) total += lds[w];
      p.block_counts[p.nblocks + blockIdx.x] = total;
    }
  }
}

// one workgroup: block_counts[i] := sum of block_counts[0 .. i), *count := total.  Rounds of
// 1024 x 16 counts: read coalesced into LDS, each lane adds up 16 consecutive ones, the lane
// sums are scanned with wavefront shuffles, and the prefixes go back through LDS so that the
// stores are coalesced too.  Counts are at most kMaskChunk and a round's total stays below
// 2^26; a mask has fewer than 2^31 elements, so every prefix fits 32 bits.
__global__ __launch_bounds__(kScanBlock) void mask_scan_kernel(const MaskArgs p) {
  constexpr int kPer = 16, kRound = kScanBlock * kPer, kWaves = kScanBlock / kWave;
  __shared__ uint32_t tile[kRound + kRound / kPer];   // one pad word per lane segment: no bank conflicts
  __shared__ uint32_t wave_sum[kWaves];
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
  int64_t carry = 0;
  for (int64_t base = 0; base < (int64_t)p.nblocks; base += kRound) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = base + k * kScanBlock + t;
      const int j = k * kScanBlock + t;
      tile[j + j / kPer] = i < (int64_t)p.nblocks ? p.block_counts[i] : 0u;
    }
    __syncthreads();
    uint32_t own[kPer], s = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      own[k] = tile[t * (kPer + 1) + k];
      s += own[k];
    }
    uint32_t inc = s;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const uint32_t up = (uint32_t)__shfl_up((int)inc, d, kWave);
      if (lane >= d) inc += up;
    }
    if (lane == kWave - 1) wave_sum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += wave_sum[w];
      total += wave_sum[w];
    }
    uint32_t run = before + inc - s;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      tile[t * (kPer + 1) + k] = run;
      run += own[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int64_t i = base + k * kScanBlock + t;
      const int j = k * kScanBlock + t;
      if (i < (int64_t)p.nblocks) p.block_counts[i] = (uint32_t)carry + tile[j + j / kPer];
    }
    carry += (int64_t)total;
    __syncthreads();   // the next round overwrites tile and wave_sum
  }
  if (t == 0) *p.count = carry;
}

// A workgroup of a write kernel needs the number of elements that are selected before its chunk:
//   kBeforeCount  adds up the mask itself up to there: no other launch at all (contiguous masks of at
//                 most kMaskDirect elements: the last workgroup reads 96 KiB in three trips of eight
//                 loads, against the 2.5 us and more that each further launch costs; with the chunk counts
//                 of another launch 40000 elements take 8.3 us instead of 7.3, 98304 8.6 instead of 9.0);
//   kBeforeGroups adds up the totals of the groups of chunks before its own and the counts inside it
//                 (contiguous masks of up to kMaskSumGroups groups, 67 million elements: 4 KiB read
//                 per workgroup at most, which hide behind the others' stores);
//   kBeforeSum    adds up the chunk counts (up to kMaskSumChunks chunks, 8.4 million elements);
//   kBeforeScan   reads its prefix, for which a launch of one workgroup scans the counts (6.0 us for the
//                 7325 chunks of 30 million elements).
enum { kBeforeCount = 0, kBeforeSum = 1, kBeforeScan = 2, kBeforeGroups = 3 };
constexpr uint32_t kMaskDirect = 98304, kMaskQuarters = 1 << 20, kMaskSumChunks = 2048, kMaskSumGroups = 1024;

// FLAT: a contiguous mask and offsets that advance by one stride.  Bound by instructions as much as by the
// 120 MB of offsets of 30 million elements with half of them selected: two offsets per lane and store, whole
// lines, no index decomposition (35.1 -> 30.4 us in a trace of threshold, count and this, 5 TB/s).
// (BEFORE: one of the above.  Told at run time, the ways that a launch does not take cost every small launch
// 0.3 to 0.8 us, masks with gaps 5 %.)
template <bool FLAT, int BEFORE> __global__ __launch_bounds__(kBlock) void mask_write_kernel(const MaskArgs p) {
  __shared__ uint32_t lds[kBlock / kWave], lds_before[kBlock / kWave];
  // the positions (inside this workgroup's chunk) of its selected elements, in order: 8 KiB,
  // where the offsets themselves would take 32 KiB and leave room for five workgroups per CU
  __shared__ uint16_t staged[kMaskChunk];
  static_assert(kMaskChunk <= 65536, "positions inside a chunk are staged as 16-bit values");
  const uint32_t chunk = blockIdx.x, chunk0 = chunk * (uint32_t)kMaskChunk;
  const uint32_t flags = mask_flags(p, chunk0 + threadIdx.x * kMaskPerLane);
  if constexpr (BEFORE != kBeforeScan) {
    uint32_t c = 0;
    if constexpr (BEFORE == kBeforeGroups) {
      const uint32_t g = chunk / kMaskGroup;
      if (threadIdx.x < chunk % kMaskGroup) c = p.block_counts[g * kMaskGroup + threadIdx.x];
#pragma unroll 4
      for (uint32_t i = threadIdx.x; i < g; i += kBlock) c += p.block_counts[p.nblocks + i];
    } else {
#pragma unroll 4
      for (uint32_t i = threadIdx.x; i < chunk; i += kBlock) c += p.block_counts[i];
    }
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) c += (uint32_t)__shfl_xor((int)c, d, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0) lds_before[threadIdx.x / kWave] = c;   // read behind the next barrier
  }
  uint32_t sum;
  uint32_t slot = block_exclusive_scan((uint32_t)__popc(flags), lds, sum);
  uint32_t f = flags;
  while (f) {
    const int k = __ffs((int)f) - 1;
    f &= f - 1;
    staged[slot++] = (uint16_t)(threadIdx.x * kMaskPerLane + (uint32_t)k);
  }
  __syncthreads();
  int64_t base = 0;
  if constexpr (BEFORE == kBeforeScan) {
    base = p.block_counts[chunk];
  } else {
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) base += lds_before[w];
    if (chunk + 1 == p.nblocks && threadIdx.x == 0) *p.count = base + sum;
  }
  // coalesced stores behind this workgroup's prefix; a position becomes its offset on the way out
  if constexpr (FLAT) {
    using Two = long long __attribute__((ext_vector_type(2)));
    const int64_t stride = p.ndim > 0 ? p.st[0] : 0, origin = (int64_t)chunk0 * stride;
    const int64_t room = p.capacity - base;          // offsets that may be stored
    const uint32_t end = room < 0 ? 0u : room < (int64_t)sum ? (uint32_t)room : sum;
    int64_t *out = p.offsets + base;
    // up to the first line, pairs in whole lines from there (a streaming store of part of a line is slow),
    // the one behind the last pair
    const uint32_t to_line = (uint32_t)((128u - ((uintptr_t)out & 127u)) & 127u) / 8u, head = to_line < end ? to_line : end;
    if (threadIdx.x < head) out[threadIdx.x] = origin + (int64_t)staged[threadIdx.x] * stride;
    if (threadIdx.x == kBlock - 1 && ((end - head) & 1u)) out[end - 1] = origin + (int64_t)staged[end - 1] * stride;
    for (uint32_t i = head + threadIdx.x * 2u; i + 1u < end; i += kBlock * 2u) {
      const Two t = {(long long)(origin + (int64_t)staged[i] * stride), (long long)(origin + (int64_t)staged[i + 1] * stride)};
      if (p.nt_store) {  // (the empty asm keeps the compiler from merging the two stores and dropping the hint)
        asm volatile("");
        __builtin_nontemporal_store(t, reinterpret_cast<Two *>(out + i));
        asm volatile("");
      } else {
        *reinterpret_cast<Two *>(out + i) = t;
      }
    }
  } else {
    for (uint32_t i = threadIdx.x; i < sum; i += kBlock)
      if (base + i < p.capacity) {
        int64_t om, ot;
        mask_decode(p, chunk0 + (uint32_t)staged[i], om, ot);
        if (p.nt_store) {
          asm volatile("");
          __builtin_nontemporal_store(ot, p.offsets + base + i);
          asm volatile("");
        } else {
          p.offsets[base + i] = ot;
        }
      }
  }
}

// Contiguous masks of at most kMaskQuarters elements: a workgroup per quarter of a chunk, a lane per four elements
// instead of sixteen, the quarters before its own counted from the mask.  Bound by the latency of one workgroup,
// most of it the sixteen turns of the loop that stages a lane's positions and the stores behind it; four times the
// workgroups of a quarter of that work, which still run all at once: with the threshold and the count before it 1000
// elements 7.2 -> 5.1 us, 98304 10.2 -> 9.0, 10^6 12.6 -> 11.7; 2 * 10^6 the same, 4 * 10^6 19.7 -> 21.1.
template <int BEFORE> __global__ __launch_bounds__(kBlock) void mask_write_quarters_kernel(const MaskArgs p) {
  constexpr uint32_t kQuarter = kMaskChunk / 4;
  static_assert(kQuarter == kBlock * 4, "four mask bytes per lane");
  __shared__ uint32_t lds[kBlock / kWave], lds_before[kBlock / kWave];
  __shared__ uint16_t staged[kQuarter];
  const uint32_t tid = threadIdx.x, chunk = blockIdx.x / 4, chunk0 = chunk * (uint32_t)kMaskChunk, q0 = blockIdx.x * kQuarter;
  const uint32_t e0 = q0 + tid * 4u;
  uint32_t own = 0;
  if (e0 + 4u <= p.n) own = *reinterpret_cast<const uint32_t *>(p.mask + e0);
  else
    for (uint32_t i = 0; e0 + i < p.n; ++i) own |= (uint32_t) * reinterpret_cast<const uint8_t *>(p.mask + e0 + i) << (8 * i);
  uint32_t c = 0;                       // (the quarters before a workgroup's own are whole)
  if (chunk0 + tid * 16u < q0) c = nonzero_bytes(*reinterpret_cast<const uint4 *>(p.mask + chunk0 + tid * 16u));
  if constexpr (BEFORE == kBeforeCount) {
    // eight loads in flight, past the end the first one again
    constexpr uint32_t kAhead = 8;
    for (uint32_t j = 0; j < chunk; j += kAhead) {
      uint4 v[kAhead];
#pragma unroll
      for (uint32_t k = 0; k < kAhead; ++k)
        v[k] = *reinterpret_cast<const uint4 *>(p.mask + (j + k < chunk ? j + k : 0u) * (uint32_t)kMaskChunk + tid * 16u);
#pragma unroll
      for (uint32_t k = 0; k < kAhead; ++k) c += j + k < chunk ? nonzero_bytes(v[k]) : 0u;
    }
  } else {
#pragma unroll 4
    for (uint32_t i = tid; i < chunk; i += kBlock) c += p.block_counts[i];
  }
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) c += (uint32_t)__shfl_xor((int)c, d, kWave);
  if ((tid & (kWave - 1)) == 0) lds_before[tid / kWave] = c;   // read behind the next barrier
  const uint32_t set = (((own & 0x7f7f7f7fu) + 0x7f7f7f7fu) | own) & 0x80808080u;
  uint32_t sum;
  uint32_t slot = block_exclusive_scan((uint32_t)__popc(set), lds, sum);
#pragma unroll
  for (uint32_t k = 0; k < 4; ++k)
    if ((set >> (8 * k + 7)) & 1u) staged[slot++] = (uint16_t)(tid * 4u + k);
  __syncthreads();
  int64_t base = 0;
#pragma unroll
  for (int w = 0; w < kBlock / kWave; ++w) base += lds_before[w];
  if (blockIdx.x + 1 == gridDim.x && tid == 0) *p.count = base + sum;
  const int64_t stride = p.ndim > 0 ? p.st[0] : 0, origin = (int64_t)q0 * stride;
  const int64_t room = p.capacity - base;          // offsets that may be stored
  const uint32_t end = room < 0 ? 0u : room < (int64_t)sum ? (uint32_t)room : sum;
  for (uint32_t i = tid; i < end; i += kBlock) p.offsets[base + i] = origin + (int64_t)staged[i] * stride;
}

// ---------------------------------------------------------------------------------------
// gather / scatter
// ---------------------------------------------------------------------------------------

struct GatherArgs {
  const char *src;                    // gather: the indexed tensor; scatter: the rows
  char *dst;
  const int64_t *offsets;
  int64_t n, lo, hi;
  int32_t ndim;                       // canonical inner dims, last fastest
  FastDiv div[kMaxDims];
  int64_t ss[kMaxDims], sd[kMaxDims]; // inner byte strides on the source / destination side
  int64_t row_stride;                 // bytes between rows on the side that is not indexed
  uint32_t inner;                     // elements per row
  uint32_t vec;                       // elements a lane copies at once (1, or 16 bytes' worth)
  uint32_t items;                     // lane items per row: inner / vec
  int32_t items_log2;                 // >= 0: rows of at most 256 items, padded to 1 << items_log2 lanes,
                                      // 256 >> items_log2 rows per workgroup; -1: workgroups per row below
  FastDiv chunks_div;                 // workgroups per row
  int32_t nt_rows;                    // gather of single elements: stream the (large) result past the caches
  int32_t swap_sc;                    // the two sides are stored in different byte orders: bytes of one scalar (0: same order)
};

// reverses every scalar of `sc` bytes in a piece that is moved between byte orders
template <class P> __device__ __forceinline__ void reorder(P &v, int sc) {
  if (sc == 0) return;
  if constexpr (sizeof(P) >= 2) { if (sc == 2) reverse_scalars<2>(v); }
  if constexpr (sizeof(P) >= 4) { if (sc == 4) reverse_scalars<4>(v); }
  if constexpr (sizeof(P) >= 8) { if (sc == 8) reverse_scalars<8>(v); }
}

template <int ES> struct Bytes { unsigned char b[ES]; };
template <> struct alignas(2) Bytes<2> { unsigned char b[2]; };
template <> struct alignas(4) Bytes<4> { unsigned char b[4]; };
template <> struct alignas(8) Bytes<8> { unsigned char b[8]; };
template <> struct alignas(16) Bytes<16> { unsigned char b[16]; };

// SCATTER = false: dst[j, i] = src[offsets[j] + i];  true: dst[offsets[j] + i] = src[j, i]
// A lane copies one item: an element, or 16 bytes of the rows' fastest dim when that dim is
// contiguous and aligned on both sides (an offset that is not a multiple of 16 falls back to
// element copies for its row).  Short rows share a workgroup.
template <int ES, bool SCATTER> __global__ __launch_bounds__(kBlock) void gather_kernel(const GatherArgs p) {
  constexpr int V = 16 / ES;
  int64_t j;
  uint32_t item;
  if (p.items_log2 >= 0) {
    j = (int64_t)blockIdx.x * (kBlock >> p.items_log2) + (threadIdx.x >> p.items_log2);
    item = threadIdx.x & ((1u << p.items_log2) - 1u);
    if (j >= p.n) return;
  } else {
    const uint32_t row = fdiv(blockIdx.x, p.chunks_div);
    j = row;
    item = (blockIdx.x - row * p.chunks_div.d) * kBlock + threadIdx.x;
  }
  if (item >= p.items) return;
  const int64_t off = p.offsets[j];
  if (off < p.lo || off > p.hi) return;
  int64_t os = 0, od = 0;
  uint32_t rem = item * p.vec;
#pragma unroll
  for (int d = kMaxDims - 1; d >= 0; --d) {
    if (d < p.ndim) {
      const uint32_t q = d == 0 ? 0u : fdiv(rem, p.div[d]);
      const uint32_t k = rem - q * p.div[d].d;
      rem = q;
      os += (int64_t)k * p.ss[d];
      od += (int64_t)k * p.sd[d];
    }
  }
  if (SCATTER) { os += j * p.row_stride; od += off; }
  else { os += off; od += j * p.row_stride; }
  if (V > 1 && p.vec > 1) {
    if ((off & 15) == 0) {
      Bytes<16> v = *reinterpret_cast<const Bytes<16> *>(p.src + os);
      reorder(v, p.swap_sc);
      *reinterpret_cast<Bytes<16> *>(p.dst + od) = v;
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) {
        Bytes<ES> v = *reinterpret_cast<const Bytes<ES> *>(p.src + os + e * ES);
        reorder(v, p.swap_sc);
        *reinterpret_cast<Bytes<ES> *>(p.dst + od + e * ES) = v;
      }
    }
  } else {
    Bytes<ES> v = *reinterpret_cast<const Bytes<ES> *>(p.src + os);
    reorder(v, p.swap_sc);
    *reinterpret_cast<Bytes<ES> *>(p.dst + od) = v;
  }
}

// Single elements per offset, the rows side contiguous (a[mask], a[index array] on a flat list):
// a lane takes four consecutive offsets (two 16-byte loads), moves the four elements, and
// handles the rows side as one piece of 4 * ES bytes - four times the bytes in flight per lane
// of the kernel above, whose lanes each wait on one offset and then on one element.  An
// offset outside [lo, hi] still skips its element alone.
template <int ES, bool SCATTER> __global__ __launch_bounds__(kBlock) void gather_scalar4_kernel(const GatherArgs p) {
  using E = Bytes<ES>;
  struct alignas(4 * ES) E4 { E e[4]; };
  using L2 = long long __attribute__((ext_vector_type(2)));
  const int64_t j0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
  if (j0 >= p.n) return;
  char *dst = p.dst;
  const char *src = p.src;
  if (j0 + 4 <= p.n) {
    const L2 o01 = *reinterpret_cast<const L2 *>(p.offsets + j0), o23 = *reinterpret_cast<const L2 *>(p.offsets + j0 + 2);
    const int64_t off[4] = {o01.x, o01.y, o23.x, o23.y};
    bool ok[4], all = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      ok[i] = off[i] >= p.lo && off[i] <= p.hi;
      all = all && ok[i];
    }
    if (SCATTER) {
      E4 v = *reinterpret_cast<const E4 *>(src + j0 * ES);
      reorder(v, p.swap_sc);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (ok[i]) *reinterpret_cast<E *>(dst + off[i]) = v.e[i];
    } else {
      E4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (ok[i]) v.e[i] = *reinterpret_cast<const E *>(src + off[i]);
      reorder(v, p.swap_sc);
      if (all) {
        if (ES == 4 && p.nt_rows) {   // (16 bytes per lane: a wavefront's store covers whole lines)
          using Q = uint32_t __attribute__((ext_vector_type(4)));
          Q q;
          __builtin_memcpy(&q, &v, 16);
          asm volatile("");
          __builtin_nontemporal_store(q, reinterpret_cast<Q *>(dst + j0 * ES));
          asm volatile("");
        } else {
          *reinterpret_cast<E4 *>(dst + j0 * ES) = v;
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (ok[i]) *reinterpret_cast<E *>(dst + (j0 + i) * ES) = v.e[i];
      }
    }
  } else {
    for (int64_t j = j0; j < p.n; ++j) {
      const int64_t off = p.offsets[j];
      if (off < p.lo || off > p.hi) continue;
      E v = SCATTER ? *reinterpret_cast<const E *>(src + j * ES) : *reinterpret_cast<const E *>(src + off);
      reorder(v, p.swap_sc);
      if (SCATTER) *reinterpret_cast<E *>(dst + off) = v;
      else *reinterpret_cast<E *>(dst + j * ES) = v;
    }
  }
}

// Rows that are one contiguous run on both sides, of any length and alignment, in pieces of P
// bytes: 16, or the largest power of two that fits into a shorter row.  The last piece of a row
// ends with the row and may overlap the one before it (the same bytes are written twice).  Lanes
// are numbered through all pieces of all rows, so none idles for padding, and take U pieces each,
// a workgroup apart, so that a lane has several of the dependent loads (offset, then row) in
// flight.  65536 rows of 1200 bytes gathered: 44.4 us with 75 pieces of a row in 128 lanes and one
// piece per lane, 27 us here.
struct RowPieceArgs {
  const char *src;
  char *dst;
  const int64_t *offsets;
  int64_t lo, hi, row_stride;
  uint32_t total;                     // pieces: rows x items (below 2^31)
  uint32_t bytes;                     // of a row
  FastDiv items_div;                  // pieces per row
  int32_t nt_rows, swap_sc;           // as GatherArgs
};
template <int P, bool SCATTER, int U> __global__ __launch_bounds__(kBlock) void row_pieces_kernel(const RowPieceArgs p) {
  using QU = uint32_t __attribute__((ext_vector_type(4), aligned(1)));
  struct __attribute__((packed, aligned(1))) Any { unsigned char b[P]; };
  const uint32_t t0 = blockIdx.x * (uint32_t)(kBlock * U) + threadIdx.x;
  int64_t off[U], at[U];
  Bytes<P> v[U];
  bool ok[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t t = t0 + (uint32_t)(u * kBlock);
    ok[u] = t < p.total;
    const uint32_t row = fdiv(ok[u] ? t : 0u, p.items_div);
    const uint32_t b = ((ok[u] ? t : 0u) - row * p.items_div.d) * (uint32_t)P;
    at[u] = b + (uint32_t)P <= p.bytes ? b : p.bytes - (uint32_t)P;
    off[u] = p.offsets[row];
    ok[u] = ok[u] && off[u] >= p.lo && off[u] <= p.hi;
    off[u] += at[u];
    at[u] += (int64_t)row * p.row_stride;
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (ok[u]) {
      const char *src = p.src + (SCATTER ? at[u] : off[u]);
      if constexpr (P == 16) {
        const QU q = *reinterpret_cast<const QU *>(src);
        __builtin_memcpy(&v[u], &q, 16);
      } else {
        const Any a = *reinterpret_cast<const Any *>(src);
        __builtin_memcpy(&v[u], &a, P);
      }
    }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (ok[u]) {
      reorder(v[u], p.swap_sc);
      char *dst = p.dst + (SCATTER ? off[u] : at[u]);
      if constexpr (P == 16) {
        QU q;
        __builtin_memcpy(&q, &v[u], 16);
        if (!SCATTER && p.nt_rows) {
          asm volatile("");
          __builtin_nontemporal_store(q, reinterpret_cast<QU *>(dst));
          asm volatile("");
        } else {
          *reinterpret_cast<QU *>(dst) = q;
        }
      } else {
        Any a;
        __builtin_memcpy(&a, &v[u], P);
        *reinterpret_cast<Any *>(dst) = a;
      }
    }
}

int done(hipError_t e) {
  if (e == hipSuccess) return OCN_OK;
  record_hip_error((int)e);
  return OCN_ERR_LAUNCH;
}

// the indexing kernels take tensors in native byte order only (one-byte scalars have no order)
bool other_byte_order(const ocn_tensor *t) {
  return t && t->byteswapped && t->dtype >= 0 && t->dtype < DT_COUNT && dt_size(dt_real_of(t->dtype)) > 1;
}

bool bad_tensor(const ocn_tensor *t) {
  if (!t || t->ndim < 0 || t->ndim > kMaxDims || t->dtype < 0 || t->dtype >= DT_COUNT) return true;
  for (int d = 0; d < t->ndim; ++d)
    if (t->size[d] < 0) return true;
  return false;
}
int64_t numel_of(const ocn_tensor *t) {
  int64_t n = 1;
  for (int d = 0; d < t->ndim; ++d) n *= t->size[d];
  return n;
}

int plan_mask(const ocn_tensor *mask, const int64_t *target_strides, MaskArgs *m) {
  if (bad_tensor(mask)) return mask ? OCN_ERR_SHAPE : OCN_ERR_NULLPTR;
  if (mask->dtype != DT_BOOL) return OCN_ERR_DTYPE;
  if (mask->ndim > 0 && !target_strides) return OCN_ERR_NULLPTR;
  const int64_t n = numel_of(mask);
  if (n >= ((int64_t)1 << 31)) return OCN_ERR_SHAPE;
  std::memset(m, 0, sizeof *m);
  m->n = (uint32_t)n;
  m->mask = (const char *)mask->base + mask->offset;
  // canonical dims in the mask's own (row-major) order: drop size 1, merge neighbours that both
  // the mask and the target walk as one longer dim
  int nd = 0;
  int64_t size[kMaxDims];
  for (int d = 0; d < mask->ndim; ++d) {
    if (mask->size[d] == 1) continue;
    const int64_t sz = mask->size[d], sm = mask->stride[d], st = target_strides[d];
    if (nd > 0 && m->sm[nd - 1] == sm * sz && m->st[nd - 1] == st * sz) {
      size[nd - 1] *= sz;
      m->sm[nd - 1] = sm;
      m->st[nd - 1] = st;
    } else {
      size[nd] = sz; m->sm[nd] = sm; m->st[nd] = st;
      ++nd;
    }
  }
  m->ndim = nd;
  for (int d = 0; d < nd; ++d) m->div[d] = make_fastdiv((uint32_t)size[d]);
  m->contig = (nd == 0 || (nd == 1 && m->sm[0] == 1)) && ((uintptr_t)m->mask % 16 == 0);
  m->nblocks = (uint32_t)((n + kMaskChunk - 1) / kMaskChunk);
  return OCN_OK;
}

}  // namespace
}  // namespace ocn

using namespace ocn;

extern "C" {

int ocn_index_offsets(const ocn_tensor *index, int64_t dim_size, int64_t stride_bytes, const ocn_tensor *offsets,
                      void *invalid_count, void *stream) {
  if (bad_tensor(index) || bad_tensor(offsets)) return (!index || !offsets) ? OCN_ERR_NULLPTR : OCN_ERR_SHAPE;
  if (other_byte_order(index) || other_byte_order(offsets)) return OCN_ERR_BYTEORDER;
  if (!invalid_count) return OCN_ERR_NULLPTR;
  if (index->dtype != DT_I64 || offsets->dtype != DT_I64) return OCN_ERR_DTYPE;
  if (index->ndim != offsets->ndim || dim_size < 0) return OCN_ERR_SHAPE;
  if (index->device != offsets->device) return OCN_ERR_DEVICE;
  IndexArgs a;
  std::memset(&a, 0, sizeof a);
  a.n = 1;
  for (int d = 0; d < index->ndim; ++d) {
    if (index->size[d] != offsets->size[d]) return OCN_ERR_SHAPE;
    a.size[d] = index->size[d];
    a.si[d] = index->stride[d];
    a.so[d] = offsets->stride[d];
    a.n *= index->size[d];
  }
  if (((intptr_t)index->base + index->offset) % 8 || ((intptr_t)offsets->base + offsets->offset) % 8) return OCN_ERR_ALIGN;
  for (int d = 0; d < index->ndim; ++d)
    if (index->size[d] > 1 && (a.si[d] % 8 || a.so[d] % 8)) return OCN_ERR_ALIGN;
  a.ndim = index->ndim;
  a.idx = (const char *)index->base + index->offset;
  a.off = (char *)offsets->base + offsets->offset;
  a.dim_size = dim_size;
  a.stride = stride_bytes;
  a.invalid = (unsigned long long *)invalid_count;
  // every check comes before the first launch: on error nothing has been enqueued or written
  const int64_t grid = std::min<int64_t>((a.n + kBlock - 1) / kBlock, max_launch_blocks());   // the kernel loops beyond that
  if (a.n > 0 && (!index->base || !offsets->base)) return OCN_ERR_NULLPTR;
  hipStream_t s = (hipStream_t)stream;
  // both tensors contiguous in row-major order: one workgroup for few indices, else, if they are
  // 16-byte aligned too, the flat kernel
  bool contiguous = true;
  int64_t expect = 8;
  for (int d = index->ndim - 1; d >= 0 && contiguous; --d) {
    if (a.size[d] != 1 && (a.si[d] != expect || a.so[d] != expect)) contiguous = false;
    expect *= a.size[d];
  }
  const bool flat = contiguous && ((uintptr_t)a.idx % 16) == 0 && ((uintptr_t)a.off % 16) == 0;
  const int64_t cgrid = 1 + ((a.n + 1) / 2 + 1023) / 1024;
  const bool apart = a.idx + a.n * 8 <= a.off || a.off + a.n * 8 <= a.idx;    // (offsets may replace the indices)
  if (flat && apart && a.n > kIndexOneBlock && a.n <= kIndexCounted && cgrid <= max_launch_blocks()) {
    hipLaunchKernelGGL(index_offsets_counted_kernel, dim3((unsigned)cgrid), dim3(1024), 0, s, a);
    return done(hipGetLastError());
  }
  if (contiguous && a.n > 0 && a.n <= kIndexCounted) {
    hipLaunchKernelGGL(index_offsets_small_kernel, dim3(1), dim3(1024), 0, s, a);
    return done(hipGetLastError());
  }
  hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, a.invalid, 0ull);
  if (a.n > 0 && flat) {
    const int64_t npair = (a.n + 1) / 2;
    const int64_t fgrid = std::min<int64_t>((npair + kBlock - 1) / kBlock, max_launch_blocks());
    hipLaunchKernelGGL(index_offsets_flat_kernel, dim3((unsigned)fgrid), dim3(kBlock), 0, s, a, a.n * 8 >= ((int64_t)32 << 20) ? 1 : 0);
  } else if (a.n > 0) {
    hipLaunchKernelGGL(index_offsets_kernel, dim3((unsigned)grid), dim3(kBlock), 0, s, a);
  }
  return done(hipGetLastError());
}

size_t ocn_mask_offsets_workspace_bytes(const ocn_tensor *mask) {
  if (bad_tensor(mask)) return 0;
  const int64_t n = numel_of(mask);
  return (size_t)((n + kMaskChunk - 1) / kMaskChunk + 1) * sizeof(int64_t);
}

int ocn_mask_offsets(const ocn_tensor *mask, const int64_t *target_strides, void *offsets, int64_t capacity,
                     void *count, void *workspace, size_t workspace_bytes, void *stream) {
  MaskArgs m;
  const int rc = plan_mask(mask, target_strides, &m);
  if (rc != OCN_OK) return rc;
  if (!count || capacity < 0 || (capacity > 0 && !offsets)) return OCN_ERR_NULLPTR;
  if (((uintptr_t)offsets % 8) || ((uintptr_t)count % 8)) return OCN_ERR_ALIGN;
  hipStream_t s = (hipStream_t)stream;
  if (m.n == 0) {
    hipLaunchKernelGGL(fill_u64_kernel, dim3(1), dim3(1), 0, s, (unsigned long long *)count, 0ull);
    return done(hipGetLastError());
  }
  if (!mask->base) return OCN_ERR_NULLPTR;
  if (!workspace || workspace_bytes < ocn_mask_offsets_workspace_bytes(mask)) return OCN_ERR_WORKSPACE;
  if ((uintptr_t)workspace % 8) return OCN_ERR_ALIGN;
  m.block_counts = (uint32_t *)workspace;
  m.offsets = (int64_t *)offsets;
  m.capacity = capacity;
  m.count = (int64_t *)count;
  m.nt_store = std::min<int64_t>(capacity, m.n) * 8 >= ((int64_t)32 << 20);  // too large to stay cached
  const uint32_t groups = (m.nblocks + kMaskGroup - 1) / kMaskGroup;
  const int before = m.contig && m.n <= kMaskDirect ? kBeforeCount : m.nblocks <= kMaskSumChunks ? kBeforeSum
                     : m.contig && groups <= kMaskSumGroups ? kBeforeGroups : kBeforeScan;
  if (before != kBeforeCount) {
    if (before == kBeforeGroups) hipLaunchKernelGGL(mask_count_contig_kernel<true>, dim3(groups), dim3(kMaskGroup * kWave), 0, s, m);
    else if (m.contig)
      hipLaunchKernelGGL(mask_count_contig_kernel<false>, dim3((m.nblocks + kBlock / kWave - 1) / (kBlock / kWave)), dim3(kBlock), 0, s, m);
    else hipLaunchKernelGGL(mask_count_kernel, dim3(m.nblocks), dim3(kBlock), 0, s, m);
  }
  if (before == kBeforeScan) hipLaunchKernelGGL(mask_scan_kernel, dim3(1), dim3(kScanBlock), 0, s, m);
  const bool quarters = m.contig && m.n <= kMaskQuarters;
  auto write = [&](auto before) {
    constexpr int BEFORE = decltype(before)::value;
    if constexpr (BEFORE == kBeforeCount || BEFORE == kBeforeSum) {
      if (BEFORE == kBeforeCount || quarters) {
        const dim3 grid((m.n + kMaskChunk / 4 - 1) / (kMaskChunk / 4));
        hipLaunchKernelGGL(mask_write_quarters_kernel<BEFORE>, grid, dim3(kBlock), 0, s, m);
        return;
      }
    }
    if constexpr (BEFORE != kBeforeCount) {
      if (m.contig && m.ndim <= 1) hipLaunchKernelGGL((mask_write_kernel<true, BEFORE>), dim3(m.nblocks), dim3(kBlock), 0, s, m);
      else hipLaunchKernelGGL((mask_write_kernel<false, BEFORE>), dim3(m.nblocks), dim3(kBlock), 0, s, m);
    }
  };
  switch (before) {
    case kBeforeCount: write(std::integral_constant<int, kBeforeCount>{}); break;
    case kBeforeGroups: write(std::integral_constant<int, kBeforeGroups>{}); break;
    case kBeforeSum: write(std::integral_constant<int, kBeforeSum>{}); break;
    default: write(std::integral_constant<int, kBeforeScan>{}); break;
  }
  return done(hipGetLastError());
}

// shared by gather and scatter: `rows` has shape [n, inner...], `inner` describes one indexed
// sub-tensor of the tensor the offsets point into
static int run_gather(bool scatter, const ocn_tensor *inner, const void *offsets, int64_t n, int64_t lo, int64_t hi,
                      const ocn_tensor *rows, void *stream) {
  if (bad_tensor(inner) || bad_tensor(rows)) return (!inner || !rows) ? OCN_ERR_NULLPTR : OCN_ERR_SHAPE;
  if (inner->dtype != rows->dtype) return OCN_ERR_DTYPE;
  // a copy of elements between two tensors of the same byte order needs no reversal; between
  // different orders every scalar is reversed on the way (section 3.1.3)
  const bool reorder_scalars = other_byte_order(inner) != other_byte_order(rows);
  if (inner->device != rows->device) return OCN_ERR_DEVICE;
  if (n < 0 || rows->ndim != inner->ndim + 1 || rows->size[0] != n) return OCN_ERR_SHAPE;
  for (int d = 0; d < inner->ndim; ++d)
    if (rows->size[d + 1] != inner->size[d]) return OCN_ERR_SHAPE;
  const int es = dt_size(inner->dtype);
  const int sc = dt_size(dt_real_of(inner->dtype));
  GatherArgs g;
  std::memset(&g, 0, sizeof g);
  const int64_t inner_elems = numel_of(inner);
  if (n == 0 || inner_elems == 0) return OCN_OK;
  if (!offsets || !inner->base || !rows->base) return OCN_ERR_NULLPTR;
  if ((uintptr_t)offsets % 8) return OCN_ERR_ALIGN;
  if (((intptr_t)inner->base + inner->offset) % sc || ((intptr_t)rows->base + rows->offset) % sc || rows->stride[0] % sc)
    return OCN_ERR_ALIGN;
  if (inner_elems >= ((int64_t)1 << 31)) return OCN_ERR_SHAPE;
  // canonical inner dims: drop size 1, order by the stride on the rows side (slowest first), merge
  struct D { int64_t size, si, sr; } d[kMaxDims];
  int nd = 0;
  for (int k = 0; k < inner->ndim; ++k) {
    if (inner->size[k] == 1) continue;
    if (inner->stride[k] % sc || rows->stride[k + 1] % sc) return OCN_ERR_ALIGN;
    d[nd++] = D{inner->size[k], inner->stride[k], rows->stride[k + 1]};
  }
  auto mag = [](int64_t v) { return v < 0 ? -v : v; };
  for (int a = 1; a < nd; ++a)
    for (int b = a; b > 0 && mag(d[b].sr) > mag(d[b - 1].sr); --b) std::swap(d[b], d[b - 1]);
  int m = 0;
  for (int k = 0; k < nd; ++k) {
    if (m > 0 && d[m - 1].si == d[k].si * d[k].size && d[m - 1].sr == d[k].sr * d[k].size) {
      d[m - 1].size *= d[k].size; d[m - 1].si = d[k].si; d[m - 1].sr = d[k].sr;
    } else {
      d[m++] = d[k];
    }
  }
  g.ndim = m;
  for (int k = 0; k < m; ++k) {
    g.div[k] = make_fastdiv((uint32_t)d[k].size);
    g.ss[k] = scatter ? d[k].sr : d[k].si;
    g.sd[k] = scatter ? d[k].si : d[k].sr;
  }
  g.src = scatter ? (const char *)rows->base + rows->offset : (const char *)inner->base + inner->offset;
  g.dst = scatter ? (char *)inner->base + inner->offset : (char *)rows->base + rows->offset;
  g.offsets = (const int64_t *)offsets;
  g.n = n;
  g.lo = lo;
  g.hi = hi;
  g.row_stride = rows->stride[0];
  g.swap_sc = reorder_scalars ? sc : 0;
  g.inner = (uint32_t)inner_elems;
  // 16-byte items along the rows' fastest dim when it is contiguous and everything else keeps
  // such items aligned (the offsets themselves are checked row by row in the kernel)
  const int vfull = 16 / es;
  g.vec = 1;
  if (vfull > 1 && m > 0 && d[m - 1].si == es && d[m - 1].sr == es && d[m - 1].size % vfull == 0 &&
      ((intptr_t)inner->base + inner->offset) % 16 == 0 && ((intptr_t)rows->base + rows->offset) % 16 == 0 &&
      rows->stride[0] % 16 == 0) {
    bool ok = true;
    for (int k = 0; k + 1 < m; ++k) ok = ok && d[k].si % 16 == 0 && d[k].sr % 16 == 0;
    if (ok) g.vec = (uint32_t)vfull;
  }
  g.items = (uint32_t)(inner_elems / g.vec);
  int64_t grid;
  if (g.items <= (uint32_t)kBlock) {   // short rows share a workgroup
    g.items_log2 = 0;
    while ((1u << g.items_log2) < g.items) ++g.items_log2;
    const int64_t rows_per_block = kBlock >> g.items_log2;
    grid = (n + rows_per_block - 1) / rows_per_block;
    g.chunks_div = make_fastdiv(1);
  } else {
    g.items_log2 = -1;
    const int64_t chunks = ((int64_t)g.items + kBlock - 1) / kBlock;
    g.chunks_div = make_fastdiv((uint32_t)chunks);
    grid = n * chunks;
  }
  const int64_t max_blocks = max_launch_blocks();
  hipStream_t s = (hipStream_t)stream;
  // single elements, the rows side contiguous and aligned for pieces of four: four offsets per lane
  if (inner_elems == 1 && es <= 8 && rows->stride[0] == es && (uintptr_t)offsets % 16 == 0 &&
      ((intptr_t)rows->base + rows->offset) % (4 * es) == 0) {
    const int64_t per_launch = max_blocks * kBlock * 4;   // a multiple of four offsets: later launches stay aligned
    for (int64_t j0 = 0; j0 < n; j0 += per_launch) {
      GatherArgs q = g;
      q.nt_rows = !scatter && n * es >= ((int64_t)32 << 20);
      q.n = std::min<int64_t>(per_launch, n - j0);
      q.offsets = g.offsets + j0;
      if (scatter) q.src = g.src + j0 * es;
      else q.dst = g.dst + j0 * es;
      const int64_t launch_grid = (q.n + 4 * kBlock - 1) / (4 * kBlock);
#define OCN_LAUNCH4(ES)                                                                                                  \
  if (scatter) hipLaunchKernelGGL((gather_scalar4_kernel<ES, true>), dim3((unsigned)launch_grid), dim3(kBlock), 0, s, q); \
  else hipLaunchKernelGGL((gather_scalar4_kernel<ES, false>), dim3((unsigned)launch_grid), dim3(kBlock), 0, s, q);
      switch (es) {
        case 1: OCN_LAUNCH4(1) break;
        case 2: OCN_LAUNCH4(2) break;
        case 4: OCN_LAUNCH4(4) break;
        default: OCN_LAUNCH4(8) break;
      }
#undef OCN_LAUNCH4
    }
    return done(hipGetLastError());
  }
  // rows that are one contiguous run on both sides
  if (inner_elems == 1 || (m == 1 && d[0].si == es && d[0].sr == es && inner_elems * es < ((int64_t)1 << 31))) {
    const int64_t bytes = inner_elems * es;
    int piece = 16;
    while (piece > bytes) piece /= 2;
    const int64_t items = (bytes + piece - 1) / piece;
    const bool many = n * items >= kNumCUs * kBlock * 4;       // enough for four pieces per lane
    const int64_t per_block = (int64_t)kBlock * (many ? 4 : 1);
    const int64_t rows_max = std::min<int64_t>((((int64_t)1 << 31) - 8 * kBlock) / items, max_blocks * per_block / items);
    if (rows_max >= 1) {
      RowPieceArgs r;
      r.lo = lo;
      r.hi = hi;
      r.row_stride = g.row_stride;
      r.bytes = (uint32_t)bytes;
      r.items_div = make_fastdiv((uint32_t)items);
      r.nt_rows = !scatter && n * bytes >= ((int64_t)32 << 20);
      r.swap_sc = g.swap_sc;
      for (int64_t j0 = 0; j0 < n; j0 += rows_max) {
        const int64_t rows_now = std::min<int64_t>(rows_max, n - j0);
        r.src = g.src + (scatter ? j0 * g.row_stride : 0);
        r.dst = g.dst + (scatter ? 0 : j0 * g.row_stride);
        r.offsets = g.offsets + j0;
        r.total = (uint32_t)(rows_now * items);
        const unsigned launch_grid = (unsigned)(((int64_t)r.total + per_block - 1) / per_block);
#define OCN_LAUNCH_ROWS(P, S, U) hipLaunchKernelGGL((row_pieces_kernel<P, S, U>), dim3(launch_grid), dim3(kBlock), 0, s, r)
#define OCN_LAUNCH_PIECE(P)                                                        \
  case P:                                                                          \
    if (scatter) { if (many) OCN_LAUNCH_ROWS(P, true, 4); else OCN_LAUNCH_ROWS(P, true, 1); }     \
    else { if (many) OCN_LAUNCH_ROWS(P, false, 4); else OCN_LAUNCH_ROWS(P, false, 1); }           \
    break;
        switch (piece) {
          OCN_LAUNCH_PIECE(1) OCN_LAUNCH_PIECE(2) OCN_LAUNCH_PIECE(4) OCN_LAUNCH_PIECE(8) OCN_LAUNCH_PIECE(16)
          default: break;
        }
#undef OCN_LAUNCH_PIECE
#undef OCN_LAUNCH_ROWS
      }
      return done(hipGetLastError());
    }
  }
  // A launch may not exceed 2^32 lanes: longer lists of offsets go out in several launches,
  // each over a contiguous run of rows (the kernels are independent of one another).
  const int64_t blocks_per_row_num = g.items_log2 >= 0 ? 1 : (int64_t)g.chunks_div.d;      // blocks per row ...
  const int64_t rows_per_block = g.items_log2 >= 0 ? (kBlock >> g.items_log2) : 1;          // ... or rows per block
  if (blocks_per_row_num > max_blocks) return OCN_ERR_SHAPE;   // a single row of 2^40 items: not a gather any more
  const int64_t rows_per_launch = g.items_log2 >= 0 ? max_blocks * rows_per_block : max_blocks / blocks_per_row_num;
  (void)grid;
  const GatherArgs all = g;
  for (int64_t j0 = 0; j0 < n; j0 += rows_per_launch) {
    g = all;
    g.n = std::min<int64_t>(rows_per_launch, n - j0);
    g.offsets = all.offsets + j0;
    if (scatter) g.src = all.src + j0 * all.row_stride;
    else g.dst = all.dst + j0 * all.row_stride;
    const int64_t launch_grid = g.items_log2 >= 0 ? (g.n + rows_per_block - 1) / rows_per_block : g.n * blocks_per_row_num;
#define OCN_LAUNCH(ES)                                                                                               \
  if (scatter) hipLaunchKernelGGL((gather_kernel<ES, true>), dim3((unsigned)launch_grid), dim3(kBlock), 0, s, g);   \
  else hipLaunchKernelGGL((gather_kernel<ES, false>), dim3((unsigned)launch_grid), dim3(kBlock), 0, s, g);
    switch (es) {
      case 1: OCN_LAUNCH(1) break;
      case 2: OCN_LAUNCH(2) break;
      case 4: OCN_LAUNCH(4) break;
      case 8: OCN_LAUNCH(8) break;
      default: OCN_LAUNCH(16) break;
    }
  }
#undef OCN_LAUNCH
  return done(hipGetLastError());
}

int ocn_gather(const ocn_tensor *a_inner, const void *offsets, int64_t n, int64_t lo, int64_t hi,
               const ocn_tensor *out, void *stream) {
  return run_gather(false, a_inner, offsets, n, lo, hi, out, stream);
}

int ocn_scatter(const ocn_tensor *src, const void *offsets, int64_t n, int64_t lo, int64_t hi,
                const ocn_tensor *out_inner, void *stream) {
  return run_gather(true, out_inner, offsets, n, lo, hi, src, stream);
}

}  // extern "C"
