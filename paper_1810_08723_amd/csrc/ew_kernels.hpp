// Elementwise kernels of the tensor engine for gfx950 (wave64, 256-lane workgroups).
//
// These kernels cover every canonical plan the host planner can produce:
//   ew_rows_kernel    every operand is contiguous (or broadcast) along the innermost canonical
//                     dimension: 128-bit lane accesses, several vectors in flight per lane.
//   ew_tiled_kernel   operands disagree on their fastest axis: a power-of-two tile spanning
//                     those axes is staged through LDS so that every operand is read and
//                     written along its own fastest axis.  Without staging it is the plain
//                     strided kernel for specialised dtypes.
//   ew_tiled_fast_kernel, ew_tiled_any_kernel  the same tiles for the plans that are whole, aligned
//                     vectors throughout, and for clipped tiles and any alignment.
//   ew_interp_kernel  any dtype combination, conversions chosen by runtime switches.
// The operations follow sections 3.2 and 3.2.1 of the paper (elementwise arithmetic with
// implicit type casting fused into the kernel: no intermediate tensors).
#pragma once

#include "dev_types.hpp"
#include "planner.hpp"
#include "sigs.hpp"

namespace ocn {

// ---------------------------------------------------------------------------------------
// kernel arguments (plain data, passed by value)
// ---------------------------------------------------------------------------------------

// Arguments of the kernel for rows of any length and alignment.
struct RowsArgs {
  char *out;
  const char *a, *b;
  int64_t numel;
  int64_t nvec;      // vectors in total
  uint32_t flags;    // kRows* bits; operands in the other byte order in bits 8..10
  uint32_t block;    // lanes per workgroup
  uint32_t shift;    // flat form: elements by which the first vector starts before the output
  uint32_t inner;    // flat form: elements per row (row form: 0, no vector crosses into the next row)
  uint32_t last;     // row form: elements of a row's last vector
  FastDiv rdiv;      // flat form: elements per row; row form: vectors per row
  int32_t nouter;
  int64_t so[kMaxDims - 1], sa[kMaxDims - 1], sb[kMaxDims - 1];  // outer strides, fastest outer first
  FastDiv odiv[kMaxDims - 1];                                    // outer sizes, same order
};
enum : uint32_t {
  kRowsFlat = 1,        // the output is one contiguous run: vectors are aligned pieces of it and may cross rows
  kRowsALinear = 2, kRowsBLinear = 4,   // flat form: that input is contiguous along with the output
  kRowsABcast = 8, kRowsBBcast = 16,    // that input is broadcast along the rows
  kRowsNtA = 32, kRowsNtB = 64,         // read that input with streaming (non-temporal) loads
  kRowsNtStore = 128,                   // stream the output past the caches
  kRowsSwapShift = 8
};

// Launches of at most this many tiles fetch all their arguments first (warm_arguments); in larger
// ones the extra scalar loads of every wavefront cost more than the few first misses.
constexpr int64_t kWarmTiles = 2048;

constexpr int kMaxTilePasses = 16;  // a tile holds at most 4096 elements = 16 passes of 256 lanes

// One enumeration order of a tile's elements (fastest dim of some operand first).
struct TileOrder {
  int8_t nord;                     // tiled dims
  int8_t vecw;                     // log2 of the vector length along the first enumerated dim
  int8_t width[kMaxDims];          // log2 tile extent of the k-th enumerated dim
  int8_t dim[kMaxDims];            // which canonical dim that is
  int8_t lds_shift[kMaxDims];      // bit position of that dim in the LDS slot number
  int32_t niter;                   // passes of 256 lanes that cover the tile
  int64_t stride[3][kMaxDims];     // byte stride of that dim for out / a / b
  int64_t hi_off[3][kMaxTilePasses];  // byte offsets contributed by the pass number
  uint32_t hi_slot[kMaxTilePasses];   // LDS slot contributed by the pass number
};

// slot -> physical LDS element: slot ^ (((slot >> src) & mask) << dst)
struct TileSwizzle {
  uint32_t src, mask, dst;
};

struct TiledArgs {
  char *out;
  const char *a, *b;
  int32_t ndim, tile_bits;
  uint32_t total_tiles;
  int64_t size[kMaxDims];
  int64_t so[kMaxDims], sa[kMaxDims], sb[kMaxDims];
  int32_t tl[kMaxDims];
  FastDiv ntdiv[kMaxDims];
  int32_t stage_a, stage_b;
  int32_t nt_store;                // stream the output past the caches
  int32_t swap;                    // operands stored in the other byte order: bit 0 a, bit 1 b, bit 2 out
  uint32_t lds_off_b;              // byte offset of b's staging area in dynamic LDS
  TileSwizzle swz[2];              // for a, b
  TileOrder ord[3];                // enumeration orders: out's, a's, b's
};

// Arguments of the unclipped, all-vector form of the tiled kernel.  Everything that does not
// depend on the lane is tabulated by the host, and all offsets inside a tile are unsigned
// 32-bit, so that an access costs one scalar add (tile base + pass offset) and no vector
// address arithmetic.  LDS addresses are XORs of three host- or once-computed terms: the
// swizzle is linear over GF(2) and the lane, pass and element-in-vector parts of a slot number
// occupy disjoint bits, so swizzle(lane + pass + element) is the XOR of their swizzles.
constexpr int kFastLaneDims = 8;
struct FastOrder {
  int32_t nlane;                            // dims reached by the 8 lane bits
  int32_t niter;                            // passes of 256 lanes
  uint32_t shift[kFastLaneDims];            // bit field of the lane number holding dim k's index
  uint32_t mask[kFastLaneDims];
  uint32_t up[kFastLaneDims];               // left shift of the extracted index (vector length for k = 0)
  uint32_t slot_shift[kFastLaneDims];       // bit position of dim k in the LDS slot number
  uint32_t stride[3][kFastLaneDims];        // byte strides for out / a / b
  uint32_t hi_off[3][kMaxTilePasses];       // byte offsets contributed by the pass number
};
struct FastTiledArgs {
  char *out;
  const char *a, *b;
  int32_t warm;                             // few workgroups: touch all argument lines first
  int32_t ntd;                              // entries of the tile-number decomposition, fastest first
  int32_t stage_a, stage_b;
  int32_t nt_store;                         // stream the output past the caches
  int32_t swap;                             // operands stored in the other byte order: bit 0 a, bit 1 b, bit 2 out
  int32_t pair_log2;                        // groups of 1 << pair_log2 consecutive tiles share input lines
  int32_t nt_a, nt_b;                       // read that input with streaming loads (its runs inside a tile are whole lines)
  uint32_t lds_base[2];                     // byte offset of a's / b's staging area
  FastDiv ntdiv[kMaxDims + 1];              // (one more than dims: a dim's tile index may be split in two)
  int64_t step[3][kMaxDims + 1];            // bytes from one tile to the next along that dim
  TileSwizzle swz[2];
  uint32_t es_log2[2];
  uint32_t vc_log2;                         // log2 of the compute vector length
  FastOrder ord[3];
  uint32_t st_hi[2][kMaxTilePasses];        // staging writes: swizzled byte address from the pass number
  uint32_t st_el[2][16];                    // ... from the element number inside a vector
  uint32_t rd_hi[2][kMaxTilePasses];        // compute-phase reads: from the pass number
  uint32_t rd_ch[2][16];                    // ... from the 16-byte chunk inside a vector
};

// Arguments of the tiled kernel for clipped tiles and operands that are aligned to their elements
// only: the tables of the form above, plus what it takes to tell which elements of a clipped tile
// exist.  A tile's limits, and the coordinates contributed by a pass number, are packed as 16 bits
// per tiled dim, in the enumeration order of the operand they are compared for.
constexpr int kAnyDims = 4;                 // most tiled dims
constexpr int kAnyMaxBlock = 1024;
struct AnyOrder {
  int32_t niter;                            // passes of the workgroup's lanes
  int32_t vecw;                             // log2 of the vector length along the first dim
  uint32_t nvec;                            // vectors of the tile
  uint32_t shift[kAnyDims], mask[kAnyDims], up[kAnyDims];  // lane number -> coordinate, as FastOrder
  uint32_t slot_shift[kAnyDims];
  uint32_t stride[3][kAnyDims];             // byte strides for out / a / b
  uint32_t lim_shift[kAnyDims];             // where that dim's limit sits in the packed limits
  uint32_t hi_off[3][kMaxTilePasses];       // byte offsets contributed by the pass number
  uint64_t hi_c[kMaxTilePasses];            // packed coordinates contributed by the pass number
};
struct AnyTiledArgs {
  char *out;
  const char *a, *b;
  int32_t warm;                             // few workgroups: touch all argument lines first
  uint32_t block;                           // lanes per workgroup: 256, 512 or 1024
  int32_t nord;                             // tiled dims
  int32_t ntd;                              // entries of the tile-number decomposition, fastest first
  int32_t stage_a, stage_b;
  int32_t nt_store, swap;                   // as FastTiledArgs
  uint32_t sa0, sb0;                        // byte strides of the inputs along the output's fastest dim
  uint32_t stage_stride[2];                 // byte stride of a staged input along its own fastest dim
  const char *end[2];                       // ends of the inputs: one past the highest byte
  uint32_t lds_base[2], es_log2[2];
  uint64_t inner;                           // the limits of a tile that is not the last along any dim
  uint64_t whole;                           // the limits of an unclipped tile: its extents
  FastDiv ntdiv[kMaxDims];
  int64_t step[3][kMaxDims];                // bytes from one tile to the next along that dim
  uint32_t dim_shift[kMaxDims];             // where the dim's limit sits in the packed limits (64: not a tiled dim)
  uint32_t last[kMaxDims];                  // the limit of the dim's last tile
  TileSwizzle swz[2];
  AnyOrder ord[3];
  uint32_t st_hi[2][kMaxTilePasses];        // LDS byte addresses, as FastTiledArgs
  uint32_t st_el[2][16];
  uint32_t rd_hi[2][kMaxTilePasses];
  uint32_t rd_el[2][16];                    // compute-phase reads: from the element number inside a vector
};

struct InterpArgs {
  char *out;
  const char *a, *b;
  int32_t ndim, nin, op, T, dt_a, dt_b, dt_o;
  int64_t size[kMaxDims], so[kMaxDims], sa[kMaxDims], sb[kMaxDims];
  int64_t numel;
  int32_t idx32;              // fewer than 2^31 elements: 32-bit multiply-shift index arithmetic
  int32_t swap;               // operands stored in the other byte order: bit 0 a, bit 1 b, bit 2 out
  int32_t vec;                // 4: a lane takes four consecutive elements of the innermost dim (sizes, strides and
                              // numel then count groups of four); 1: one element
  int32_t nt_store;           // stream the output past the caches
  int32_t back[3];            // vec == 4: bytes (out / a / b) by which a row's last group is moved back to end with the row
  int32_t inner_a, inner_b;   // vec == 4: the input is contiguous along the innermost dim (else broadcast there)
  FastDiv div[kMaxDims];
};

#if defined(__HIPCC__)

#define OCN_HDF __host__ __device__ __forceinline__

OCN_HDF uint32_t fastdiv(uint32_t n, const FastDiv &f) {
  return (uint32_t)((((uint64_t)n * f.m) >> 32) + n) >> f.s;
}

// four stored bools: any byte but zero is true, written as 1
OCN_HDF uint32_t bool_bytes(uint32_t w) { return ((((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w) >> 7) & 0x01010101u; }

// ---------------------------------------------------------------------------------------
// raw vector access
// ---------------------------------------------------------------------------------------

template <class S, int V> struct alignas(sizeof(S) * V >= 16 ? 16 : sizeof(S) * V) Pack {
  S v[V];
};

#define OCN_KEEP_BRANCH() asm volatile("")
// `nt`: a streaming (non-temporal) load, for inputs too large to be found in a cache again
// (the hint is only ever set for a single piece of at most 16 bytes per lane).  The empty asm
// statements keep the two branches apart; merged, the hint would be dropped.
template <class S, int V> OCN_DEV void load_pack(const char *p, Pack<S, V> &dst, bool nt = false) {
  constexpr int B = sizeof(S) * V;
  if constexpr (B >= 16) {
    using Q = uint32_t __attribute__((ext_vector_type(4)));
    if (B == 16 && nt) {
      OCN_KEEP_BRANCH();
      reinterpret_cast<Q *>(&dst)[0] = __builtin_nontemporal_load(reinterpret_cast<const Q *>(p));
      OCN_KEEP_BRANCH();
    } else {
#pragma unroll
      for (int i = 0; i < B / 16; ++i) {
        reinterpret_cast<Q *>(&dst)[i] = reinterpret_cast<const Q *>(p)[i];
      }
    }
  } else if constexpr (B == 8) {
    using D = uint32_t __attribute__((ext_vector_type(2)));
    if (nt) {
      OCN_KEEP_BRANCH();
      *reinterpret_cast<D *>(&dst) = __builtin_nontemporal_load(reinterpret_cast<const D *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<D *>(&dst) = *reinterpret_cast<const D *>(p);
    }
  } else if constexpr (B == 4) {
    if (nt) {
      OCN_KEEP_BRANCH();
      *reinterpret_cast<uint32_t *>(&dst) = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<uint32_t *>(&dst) = *reinterpret_cast<const uint32_t *>(p);
    }
  } else if constexpr (B == 2) {
    *reinterpret_cast<uint16_t *>(&dst) = *reinterpret_cast<const uint16_t *>(p);
  } else {
    *reinterpret_cast<uint8_t *>(&dst) = *reinterpret_cast<const uint8_t *>(p);
  }
}

// `nt`: a streaming (non-temporal) store.  Outputs too large to stay in the Infinity Cache are
// written this way: an ordinary store leaves the lines dirty in that cache, and the next
// kernel then pays for writing them back while it reads (measured: up to a third of its time).
// (The empty asm statements fence the streaming branch: without them the compiler merges the
// two stores of an if/else into one and drops the hint.)
template <class S, int V> OCN_DEV void store_pack(char *p, const Pack<S, V> &src, bool nt = false) {
  constexpr int B = sizeof(S) * V;
  if constexpr (B >= 16) {
    using Q = uint32_t __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int i = 0; i < B / 16; ++i) {
      if (nt) {
        OCN_KEEP_BRANCH();
        __builtin_nontemporal_store(reinterpret_cast<const Q *>(&src)[i], reinterpret_cast<Q *>(p) + i);
        OCN_KEEP_BRANCH();
      } else {
        reinterpret_cast<Q *>(p)[i] = reinterpret_cast<const Q *>(&src)[i];
      }
    }
  } else if constexpr (B == 8) {
    using D = uint32_t __attribute__((ext_vector_type(2)));
    if (nt) {
      OCN_KEEP_BRANCH();
      __builtin_nontemporal_store(*reinterpret_cast<const D *>(&src), reinterpret_cast<D *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<D *>(p) = *reinterpret_cast<const D *>(&src);
    }
  } else if constexpr (B == 4) {
    if (nt) {
      OCN_KEEP_BRANCH();
      __builtin_nontemporal_store(*reinterpret_cast<const uint32_t *>(&src), reinterpret_cast<uint32_t *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<uint32_t *>(p) = *reinterpret_cast<const uint32_t *>(&src);
    }
  } else if constexpr (B == 2) {
    *reinterpret_cast<uint16_t *>(p) = *reinterpret_cast<const uint16_t *>(&src);
  } else {
    *reinterpret_cast<uint8_t *>(p) = *reinterpret_cast<const uint8_t *>(&src);
  }
}

// The same accesses for addresses that are only multiples of the scalar size.  gfx950 loads and
// stores up to 16 bytes per lane at any such address; a wavefront's access then touches one
// cache line more than an aligned one (a flat copy with the inputs off by one element: 61.8
// against 60.2 us for 48 M floats).  Copied through packed types, so that the compiler knows.
template <class S, int V, int AL> OCN_DEV void load_pack_any(const char *p, Pack<S, V> &dst, bool nt = false) {
  using X = Unaligned<AL>;
  constexpr int B = sizeof(S) * V;
  if constexpr (B >= 16) {
    typename X::W4 w[B / 16];
    if (B == 16 && nt) {
      OCN_KEEP_BRANCH();
      w[0] = __builtin_nontemporal_load(reinterpret_cast<const typename X::W4 *>(p));
      OCN_KEEP_BRANCH();
    } else {
#pragma unroll
      for (int i = 0; i < B / 16; ++i) w[i] = reinterpret_cast<const typename X::W4 *>(p)[i];
    }
    __builtin_memcpy(&dst, w, B);
  } else if constexpr (B == 8) {
    const typename X::W2 w = *reinterpret_cast<const typename X::W2 *>(p);
    __builtin_memcpy(&dst, &w, B);
  } else if constexpr (B == 4) {
    const uint32_t w = *reinterpret_cast<const typename X::W1 *>(p);
    __builtin_memcpy(&dst, &w, B);
  } else if constexpr (B == 2) {
    const uint16_t w = *reinterpret_cast<const typename X::H1 *>(p);
    __builtin_memcpy(&dst, &w, B);
  } else {
    __builtin_memcpy(&dst, p, B);
  }
}
template <class S, int V, int AL> OCN_DEV void store_pack_any(char *p, const Pack<S, V> &src, bool nt = false) {
  using X = Unaligned<AL>;
  constexpr int B = sizeof(S) * V;
  if constexpr (B >= 16) {
    typename X::W4 w[B / 16];
    __builtin_memcpy(w, &src, B);
#pragma unroll
    for (int i = 0; i < B / 16; ++i) {
      if (nt) {
        OCN_KEEP_BRANCH();
        __builtin_nontemporal_store(w[i], reinterpret_cast<typename X::W4 *>(p) + i);
        OCN_KEEP_BRANCH();
      } else {
        reinterpret_cast<typename X::W4 *>(p)[i] = w[i];
      }
    }
  } else if constexpr (B == 8) {
    typename X::W2 w;
    __builtin_memcpy(&w, &src, B);
    if (nt) {
      OCN_KEEP_BRANCH();
      __builtin_nontemporal_store(w, reinterpret_cast<typename X::W2 *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<typename X::W2 *>(p) = w;
    }
  } else if constexpr (B == 4) {
    uint32_t w;
    __builtin_memcpy(&w, &src, B);
    if (nt) {
      OCN_KEEP_BRANCH();
      __builtin_nontemporal_store(w, reinterpret_cast<typename X::W1 *>(p));
      OCN_KEEP_BRANCH();
    } else {
      *reinterpret_cast<typename X::W1 *>(p) = w;
    }
  } else if constexpr (B == 2) {
    uint16_t w;
    __builtin_memcpy(&w, &src, B);
    *reinterpret_cast<typename X::H1 *>(p) = w;
  } else {
    __builtin_memcpy(p, &src, B);
  }
}

// ---------------------------------------------------------------------------------------
// one element: load-convert, operate, convert-store
// ---------------------------------------------------------------------------------------

template <int OP, int SA, int SB, int SO, int NIN> struct Sig {
  // compute type: inputs of a specialised comparison have equal types, so T is that type
  static constexpr int T = NIN == 2 ? (is_logical(OP) ? (int)DT_BOOL : is_compare(OP) ? SA : SO)
                                    : unary_compute_dtype(OP, SA, SO);
  using SAt = storage_t<SA>;
  using SBt = storage_t<SB>;
  using SOt = storage_t<SO>;
  static constexpr int ES_MIN = imin(imin((int)sizeof(SAt), (int)sizeof(SOt)), NIN == 2 ? (int)sizeof(SBt) : 16);
  static constexpr int ES_MAX = imax(imax((int)sizeof(SAt), (int)sizeof(SOt)), NIN == 2 ? (int)sizeof(SBt) : 1);
  static constexpr bool NIN2 = NIN == 2;
  static constexpr int SA_DT = SA, SB_DT = SB, SO_DT = SO;
  static constexpr int V = rows_vec((int)sizeof(SOt), ES_MAX);
  static constexpr int U = rows_unroll(V, ES_MAX);
  static constexpr int VR = rows_stream_vec((int)sizeof(SOt), ES_MIN, ES_MAX);  // the rows kernel's vector
  static constexpr int UR = rows_stream_unroll(VR, ES_MIN);

  // operands stored in the other byte order: un-reverse inputs after the load, reverse the
  // result before the store (sw: bit 0 a, bit 1 b, bit 2 out; uniform over the launch)
  template <class PA, class PB> OCN_DEV static void order_inputs(int sw, PA &a, PB &b) {
    if (sw & 1) reverse_scalars<scalar_bytes(SA)>(a);
    if constexpr (NIN == 2) {
      if (sw & 2) reverse_scalars<scalar_bytes(SB)>(b);
    }
  }
  template <class PO> OCN_DEV static void order_output(int sw, PO &r) {
    if (sw & 4) reverse_scalars<scalar_bytes(SO)>(r);
  }

  OCN_DEV static SOt eval(SAt a, SBt b) {
    reg_t<T> ra = convert<T>(from_storage<SA>(a));
    if constexpr (NIN == 2) {
      reg_t<T> rb = convert<T>(from_storage<SB>(b));
      auto r = apply_binary<OP, T>(ra, rb);
      return to_storage<SO>(convert<SO>(r));
    } else {
      auto r = apply_unary<OP, T>(ra);
      return to_storage<SO>(convert<SO>(r));
    }
  }
};

// ---------------------------------------------------------------------------------------
// rows kernel
// ---------------------------------------------------------------------------------------

// The common shapes - at most one outer dim, rows of whole vectors, fewer than 2^31 vectors -
// get a kernel of their own.  With one vector per lane a wavefront lives for one memory round
// trip, so what it executes before its first load is time during which it has nothing in
// flight: this kernel reads 72 bytes of arguments with two scalar loads (the general kernel's
// 340 bytes of strides and divisors arrive in eight loads that are all waited for), needs one
// division per vector and no per-element conditions, and issues every load of a lane before it
// waits for any (2^26 floats negated: 84.4 us in the general kernel's body for these shapes,
// a plain copy of the same size written for the purpose 80.7 us).
struct RowsSlimArgs {
  char *out;
  const char *a, *b;
  int64_t so, sa, sb;   // byte strides of the outer dim (zero and unused without one)
  uint32_t nvec;        // vectors in total
  FastDiv vpr_div;      // vectors per row
  uint32_t flags;       // kSlim* bits; operands in the other byte order in bits 8..10; from bit 16: elements behind
                        // the last whole vector (without an outer dim only)
};
enum : uint32_t { kSlimABcast = 1, kSlimBBcast = 2, kSlimNtA = 4, kSlimNtB = 8, kSlimNtStore = 16, kSlimSwapShift = 8, kSlimTailShift = 16 };
#ifndef OCN_SLIM_BLOCK
#define OCN_SLIM_BLOCK 64
#endif
constexpr int kSlimBlock = OCN_SLIM_BLOCK;

template <class G> __global__ __launch_bounds__(kSlimBlock) void ew_rows_slim_kernel(const RowsSlimArgs q) {
  constexpr int V = G::VR, U = G::UR;
  RowsSlimArgs p = q;
  OCN_ARGS_NOW("s"(p.out), "s"(p.a), "s"(p.b), "s"(p.so), "s"(p.sa), "s"(p.sb), "s"(p.nvec), "s"(p.vpr_div.d),
               "s"(p.vpr_div.m), "s"(p.vpr_div.s), "s"(p.flags));
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr bool BIN = G::NIN2;
  const uint32_t g0 = blockIdx.x * (uint32_t)(kSlimBlock * U) + threadIdx.x;
  const uint32_t flags = p.flags;
  Pack<SAt, V> va[U];
  Pack<SBt, V> vb[U];
  int64_t oo[U];
  // every load of the lane is issued before anything waits for one
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t g = g0 + (uint32_t)u * kSlimBlock;
    oo[u] = 0;
    if (g < p.nvec) {
      const uint32_t row = fastdiv(g, p.vpr_div);
      const int64_t e0 = (int64_t)(g - row * p.vpr_div.d) * V;
      oo[u] = (int64_t)row * p.so + e0 * (int64_t)sizeof(SOt);
      const char *pa = p.a + (int64_t)row * p.sa;
      // (an operand broadcast along the row: its one element lands in the vector's first slot
      // and is spread out after the loads; a register of its own would have to be cleared on
      // the other path, which the compiler does behind a wait for the loads issued so far)
      if (flags & kSlimABcast) va[u].v[0] = *reinterpret_cast<const SAt *>(pa);
      else load_pack<SAt, V>(pa + e0 * (int64_t)sizeof(SAt), va[u], (flags & kSlimNtA) != 0);
      if constexpr (BIN) {
        const char *pb = p.b + (int64_t)row * p.sb;
        if (flags & kSlimBBcast) vb[u].v[0] = *reinterpret_cast<const SBt *>(pb);
        else load_pack<SBt, V>(pb + e0 * (int64_t)sizeof(SBt), vb[u], (flags & kSlimNtB) != 0);
      }
    }
  }
  const int swap = (int)(flags >> kSlimSwapShift) & 7;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (g0 + (uint32_t)u * kSlimBlock < p.nvec) {
      if (flags & kSlimABcast) {
#pragma unroll
        for (int i = 1; i < V; ++i) va[u].v[i] = va[u].v[0];
      }
      if constexpr (BIN) {
        if (flags & kSlimBBcast) {
#pragma unroll
          for (int i = 1; i < V; ++i) vb[u].v[i] = vb[u].v[0];
        }
      }
      Pack<SOt, V> r;
      if (swap) G::order_inputs(swap, va[u], vb[u]);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(va[u].v[i], vb[u].v[i]);
        else r.v[i] = G::eval(va[u].v[i], SBt{});
      }
      if (swap) G::order_output(swap, r);
      store_pack<SOt, V>(p.out + oo[u], r, (flags & kSlimNtStore) != 0);
    }
  }
  // The elements behind the last whole vector of a one-dimensional tensor, by the lane that the next
  // vector would be (a > b over 30 000 001 floats: 28.6 us in the kernel for rows of any length, which
  // holds four vectors per lane here, 25.5 with the tail in this one).
  if constexpr (U > 1) {
    const uint32_t tail = flags >> kSlimTailShift;
    if (tail == 0) return;          // (a scalar branch: nothing else is left to do for all other launches)
    OCN_KEEP_BRANCH();
    const uint32_t ahead = p.nvec - g0;
    if (ahead % kSlimBlock == 0 && ahead / kSlimBlock < (uint32_t)U) {
      const int64_t e0 = (int64_t)p.nvec * V;
      for (uint32_t i = 0; i < tail; ++i) {
        Pack<SAt, 1> x;
        Pack<SBt, 1> y;
        Pack<SOt, 1> r;
        x.v[0] = reinterpret_cast<const SAt *>(p.a)[flags & kSlimABcast ? 0 : e0 + i];
        if constexpr (BIN) y.v[0] = reinterpret_cast<const SBt *>(p.b)[flags & kSlimBBcast ? 0 : e0 + i];
        if (swap) G::order_inputs(swap, x, y);
        if constexpr (BIN) r.v[0] = G::eval(x.v[0], y.v[0]);
        else r.v[0] = G::eval(x.v[0], SBt{});
        if (swap) G::order_output(swap, r);
        reinterpret_cast<SOt *>(p.out)[e0 + i] = r.v[0];
      }
    }
  }
}

// Rows of any length and alignment, any number of outer dims.  Bound by HBM like the kernel
// above; what it has to avoid is element-sized accesses where rows do not start on vector
// boundaries (an odd row length).  Two forms:
//   flat  The output is one contiguous run, which is cut into aligned vectors regardless of where
//         rows end, so that stores are whole lines.  An input that runs along with it is read
//         in the same aligned vectors; any other input (broadcast along some dim, rows in
//         another order) is read at its own, possibly unaligned, address, and element by
//         element by the few lanes whose vector crosses from one row into the next.
//   rows  Vectors start where rows start; a row's last, partial vector goes element by element.
// int32 [8000, 6001] times a float row of 6001: 126 us as single elements, 61.4 us here (6.25 TB/s;
// starting vectors where rows start took 67 us).  64-lane workgroups as above.
// byte offsets of a row in the three operands
template <class P> OCN_HDF void rows_outer(const P &p, uint32_t row, int64_t (&off)[3]) {
  off[0] = off[1] = off[2] = 0;
  const int nouter = p.nouter;
  for (int k = 0; k < nouter; ++k) {
    const uint32_t d = p.odiv[k].d;
    const uint32_t q = k + 1 < nouter ? fastdiv(row, FastDiv{d, p.odiv[k].m, p.odiv[k].s}) : 0u;
    const int64_t i = (int64_t)(row - q * d);
    row = q;
    off[0] += i * p.so[k];
    off[1] += i * p.sa[k];
    off[2] += i * p.sb[k];
  }
}

// where vector number g lies (es_*: element sizes)
struct RowsPlace {
  int64_t first;    // flat form: its first element (may lie before the output)
  int64_t off[3];   // byte offsets of its row in out / a / b (row form: of its first element)
  uint32_t row, col; // (row form: col counts from the vector's first element; a row may be longer than 2^32)
  int lo, hi;       // the elements of the vector that exist: lo .. hi - 1
  bool inrow;       // all of them lie in one row
};
template <int V, class P> OCN_HDF RowsPlace rows_place(const P &p, int64_t g, int es_o, int es_a, int es_b) {
  RowsPlace r;
  r.first = 0;
  r.row = r.col = 0;
  r.lo = 0;
  r.inrow = true;
  r.off[0] = r.off[1] = r.off[2] = 0;
  const uint32_t flags = p.flags;
  const FastDiv rdiv{p.rdiv.d, p.rdiv.m, p.rdiv.s};
  if (flags & kRowsFlat) {
    const int64_t numel = p.numel;
    r.first = g * V - (int64_t)p.shift;
    r.lo = r.first < 0 ? (int)-r.first : 0;
    r.hi = numel - r.first < V ? (int)(numel - r.first) : V;
    if (p.nouter) {
      const uint32_t e = (uint32_t)(r.first + r.lo);
      r.row = fastdiv(e, rdiv);
      r.col = e - r.row * rdiv.d;
      r.inrow = r.col + (uint32_t)(r.hi - r.lo) <= p.inner;
      rows_outer(p, r.row, r.off);
    }
  } else {
    r.row = fastdiv((uint32_t)g, rdiv);
    const uint32_t c = (uint32_t)g - r.row * rdiv.d;
    r.hi = c + 1 == rdiv.d ? (int)p.last : V;
    rows_outer(p, r.row, r.off);
    const int64_t e0 = (int64_t)c * V;
    r.off[0] += e0 * es_o;
    if (!(flags & kRowsABcast)) r.off[1] += e0 * es_a;
    if (!(flags & kRowsBBcast)) r.off[2] += e0 * es_b;
  }
  return r;
}
// byte offset of element i of vector r in operand x (0 out, 1 a, 2 b; es its element size, lin:
// it runs along with a contiguous output, bc: it is broadcast along the rows); r.row, r.col and
// r.off are those of element i
template <class R> OCN_HDF int64_t rows_offset(const R &r, int x, int i, int es, bool lin, bool bc) {
  return lin ? (r.first + i) * es : r.off[x] + (bc ? 0 : (int64_t)r.col * es);
}
// on to the next element (past the last row nothing is read)
template <class P> OCN_HDF void rows_next(const P &p, RowsPlace &r) {
  if (++r.col == p.inner && p.nouter) {
    r.col = 0;
    rows_outer(p, ++r.row, r.off);
  }
}

template <class G> __global__ __launch_bounds__(kBlock) void ew_rows_kernel(const RowsArgs by_value) {
  constexpr int V = G::VR, U = G::UR;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr int ALA = scalar_bytes(G::SA_DT), ALB = scalar_bytes(G::SB_DT), ALO = scalar_bytes(G::SO_DT);
  constexpr int ESA = (int)sizeof(SAt), ESB = (int)sizeof(SBt), ESO = (int)sizeof(SOt);
  constexpr bool BIN = G::NIN2;
  (void)by_value;  // read through the kernarg segment: the outer dims are indexed at run time
  using KArgs = const __attribute__((address_space(4))) RowsArgs;
  KArgs &p = *(KArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  OCN_ARGS_NOW("s"(p.out), "s"(p.a), "s"(p.b), "s"(p.numel), "s"(p.nvec), "s"(p.flags), "s"(p.block), "s"(p.shift),
               "s"(p.inner), "s"(p.last), "s"(p.rdiv.d), "s"(p.rdiv.m), "s"(p.rdiv.s), "s"(p.nouter));
  const uint32_t flags = p.flags, block = p.block;
  const bool flat = (flags & kRowsFlat) != 0;
  const bool alin = (flags & kRowsALinear) != 0, blin = (flags & kRowsBLinear) != 0;
  const bool abc = (flags & kRowsABcast) != 0, bbc = (flags & kRowsBBcast) != 0;

  const int64_t g0 = (int64_t)blockIdx.x * (int64_t)(block * U) + threadIdx.x;
  Pack<SAt, V> va[U];
  Pack<SBt, V> vb[U];
  char *po[U];
  int lo[U], hi[U];
  bool inrow[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t g = g0 + (int64_t)u * block;
    lo[u] = hi[u] = 0;
    inrow[u] = true;
    if (g < p.nvec) {
      RowsPlace r = rows_place<V>(p, g, ESO, ESA, ESB);
      lo[u] = r.lo;
      hi[u] = r.hi;
      inrow[u] = r.inrow;
      po[u] = p.out + rows_offset(r, 0, 0, ESO, flat, false);
      const bool whole = r.hi - r.lo == V;
      const bool va_ok = whole && (alin || r.inrow), vb_ok = !BIN || (whole && (blin || r.inrow));
      if (va_ok) {
        const char *pa = p.a + rows_offset(r, 1, 0, ESA, alin, abc);
        if (abc && !alin) va[u].v[0] = *reinterpret_cast<const SAt *>(pa);
        else load_pack_any<SAt, V, ALA>(pa, va[u], (flags & kRowsNtA) != 0);
      }
      if constexpr (BIN) {
        if (vb_ok) {
          const char *pb = p.b + rows_offset(r, 2, 0, ESB, blin, bbc);
          if (bbc && !blin) vb[u].v[0] = *reinterpret_cast<const SBt *>(pb);
          else load_pack_any<SBt, V, ALB>(pb, vb[u], (flags & kRowsNtB) != 0);
        }
      }
      // element by element: a vector that is not whole, or an input whose rows it crosses
      if (!va_ok || !vb_ok) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          if (i >= r.lo && i < r.hi) {
            if (!va_ok) va[u].v[i] = *reinterpret_cast<const SAt *>(p.a + rows_offset(r, 1, i, ESA, alin, abc));
            if constexpr (BIN) {
              if (!vb_ok) vb[u].v[i] = *reinterpret_cast<const SBt *>(p.b + rows_offset(r, 2, i, ESB, blin, bbc));
            }
            rows_next(p, r);
          }
        }
      }
    }
  }
  const int swap = (int)(flags >> kRowsSwapShift);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int n = hi[u] - lo[u];
    if (n > 0) {
      if (n == V && inrow[u]) {   // an input broadcast along the row: its one element, spread out
        if (abc && !alin) {
#pragma unroll
          for (int i = 1; i < V; ++i) va[u].v[i] = va[u].v[0];
        }
        if constexpr (BIN) {
          if (bbc && !blin) {
#pragma unroll
            for (int i = 1; i < V; ++i) vb[u].v[i] = vb[u].v[0];
          }
        }
      }
      Pack<SOt, V> r;
      if (swap) G::order_inputs(swap, va[u], vb[u]);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(va[u].v[i], vb[u].v[i]);
        else r.v[i] = G::eval(va[u].v[i], SBt{});
      }
      if (swap) G::order_output(swap, r);
      if (n == V) {
        store_pack_any<SOt, V, ALO>(po[u], r, (flags & kRowsNtStore) != 0);
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (i >= lo[u] && i < hi[u]) reinterpret_cast<SOt *>(po[u])[i] = r.v[i];
      }
    }
  }
}

// ---------------------------------------------------------------------------------------
// tiled kernel
// ---------------------------------------------------------------------------------------
//
// A workgroup owns one tile: a box of power-of-two extents over the canonical dims that are
// the fastest axis of the output or of an input.  The tile's elements are enumerated in up to
// three orders (the output's and each staged input's own fastest-axis-first order).  Because
// every extent is a power of two, an enumeration index e = lane + 256 * pass splits into a
// lane part (computed once per lane) and a pass part (the same for every lane and every
// workgroup, tabulated by the host), so the inner loops only add two offsets.
//
// Staged inputs are copied global -> LDS along their own fastest axis (128-bit loads when
// the layout allows), stored at slot = position in the OUTPUT's enumeration order, and read
// back along the output's fastest axis.  Slots are XOR-swizzled so that neither the
// column-wise writes nor the row-wise reads pile onto one LDS bank.

struct LanePos {
  int64_t off[3];   // byte offsets for out / a / b
  uint32_t slot;    // LDS slot (element position in the output's enumeration order)
};

// lane part of the position of vector number e (bits below 8 only) in enumeration order o
template <class O> OCN_HDF LanePos lane_pos(const O &o, uint32_t e) {
  LanePos r;
  r.off[0] = r.off[1] = r.off[2] = 0;
  r.slot = 0;
  uint32_t shift = 0;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    if (k < o.nord) {
      const uint32_t vw = k == 0 ? (uint32_t)o.vecw : 0u;
      const uint32_t w = (uint32_t)o.width[k] - vw;
      const uint32_t c = ((e >> shift) & ((1u << w) - 1u)) << vw;
      shift += w;
#pragma unroll
      for (int x = 0; x < 3; ++x) r.off[x] += (int64_t)c * o.stride[x][k];
      r.slot += c << o.lds_shift[k];
    }
  }
  return r;
}

// How many elements of vector number e lie inside a clipped tile (0 .. 1 << vecw).
template <class O> OCN_HDF int vec_inside(const O &o, uint32_t e, const uint32_t *lim_dim) {
  int n = 1 << o.vecw;
  uint32_t shift = 0;
#pragma unroll
  for (int k = 0; k < kMaxDims; ++k) {
    if (k < o.nord) {
      const uint32_t vw = k == 0 ? (uint32_t)o.vecw : 0u;
      const uint32_t w = (uint32_t)o.width[k] - vw;
      const uint32_t c = ((e >> shift) & ((1u << w) - 1u)) << vw;
      shift += w;
      uint32_t lim = 1;
#pragma unroll
      for (int dd = 0; dd < kMaxDims; ++dd)
        if (dd == o.dim[k]) lim = lim_dim[dd];
      if (k == 0) {
        const int left = (int)lim - (int)c;
        n = left < n ? left : n;
      } else if (c >= lim) {
        n = 0;
      }
    }
  }
  return n < 0 ? 0 : n;
}

OCN_HDF uint32_t swizzle(uint32_t slot, uint32_t src, uint32_t mask, uint32_t dst) {
  return slot ^ (((slot >> src) & mask) << dst);
}
OCN_HDF uint32_t swizzle(uint32_t slot, const TileSwizzle &z) { return swizzle(slot, z.src, z.mask, z.dst); }

extern __shared__ uint4 ocn_lds_raw[];

// The kernel reads its argument struct through the constant address space (the kernarg
// segment itself): indexing the per-pass tables with a runtime pass number then becomes a
// scalar load instead of forcing a private copy of the whole struct.
using KTiledArgs = const __attribute__((address_space(4))) TiledArgs;
using KTileOrder = const __attribute__((address_space(4))) TileOrder;

// global -> LDS copy of one staged input, enumerated in that input's own order
// FULL: the tile is not clipped and every lane has a whole vector in every pass, so the loop
// body carries no per-lane conditions at all.
template <class S, int V, int WHICH, bool FULL>
OCN_DEV void stage_operand(KTiledArgs &p, const char *base, S *lds,
                           const uint32_t *lim_dim, uint32_t nvec) {
  constexpr int J = V > 1 ? 2 : 4;  // vectors in flight per lane
  KTileOrder &o = p.ord[WHICH];
  const uint32_t zsrc = p.swz[WHICH - 1].src, zmask = p.swz[WHICH - 1].mask, zdst = p.swz[WHICH - 1].dst;
  const uint32_t tid = threadIdx.x;
  const LanePos lo = lane_pos(o, tid);
  const uint32_t step = 1u << o.lds_shift[0];  // slot distance between a vector's elements
  const int niter = o.niter;
  for (int j0 = 0; j0 < niter; j0 += J) {
    Pack<S, V> v[J];
    uint32_t slot[J];
    int nv[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int jj = j0 + j;
      nv[j] = 0;
      if (jj < niter) {
        const uint32_t e = tid + (uint32_t)jj * kBlock;
        int n = V;
        if constexpr (!FULL) {
          n = e < nvec ? V : 0;
          if (n) n = vec_inside(o, e, lim_dim);
        }
        nv[j] = n;
        slot[j] = lo.slot + o.hi_slot[jj];
        const char *src = base + lo.off[WHICH] + o.hi_off[WHICH][jj];
        if (FULL || n == V) {
          load_pack<S, V>(src, v[j]);
        } else {
#pragma unroll
          for (int i = 0; i < V; ++i)
            if (i < n) v[j].v[i] = reinterpret_cast<const S *>(src)[i];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (j0 + j >= niter) break;  // uniform: the last batch of passes may be short
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (FULL || i < nv[j]) lds[swizzle(slot[j] + (uint32_t)i * step, zsrc, zmask, zdst)] = v[j].v[i];
    }
  }
}

// read V consecutive slots of a staged operand (consecutive along the output's fastest axis)
template <class S, int V>
OCN_DEV void read_staged(const S *lds, uint32_t slot0, uint32_t zsrc, uint32_t zmask, uint32_t zdst, Pack<S, V> &dst) {
  constexpr int EPC = (16 / (int)sizeof(S)) < V ? (16 / (int)sizeof(S)) : V;  // elements per LDS access
  using Chunk = Pack<S, EPC>;
#pragma unroll
  for (int c = 0; c < V / EPC; ++c)
    *reinterpret_cast<Chunk *>(&dst.v[c * EPC]) =
        *reinterpret_cast<const Chunk *>(&lds[swizzle(slot0 + c * EPC, zsrc, zmask, zdst)]);
}

// V elements of a non-staged input along the output's fastest axis (byte stride s0 there)
template <class S, int V> OCN_DEV void read_direct(const char *src, int64_t s0, int n, Pack<S, V> &dst) {
  if (s0 == (int64_t)sizeof(S) && n == V) {
    load_pack<S, V>(src, dst);
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i < n) dst.v[i] = *reinterpret_cast<const S *>(src + (int64_t)i * s0);
  }
}

template <class G, int V, bool FULL>
OCN_DEV void tiled_compute(KTiledArgs &p, char *out, const char *pa, const char *pb,
                           const typename G::SAt *lds_a, const typename G::SBt *lds_b,
                           const uint32_t *lim_dim, uint32_t nvec) {
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr bool BIN = G::NIN2;
  constexpr int J = V > 1 ? 2 : 4;
  KTileOrder &o = p.ord[0];
  const uint32_t tid = threadIdx.x;
  const LanePos lo = lane_pos(o, tid);
  const int64_t sa0 = o.stride[1][0], sb0 = o.stride[2][0];
  const bool stage_a = p.stage_a, stage_b = p.stage_b;
  const uint32_t asrc = p.swz[0].src, amask = p.swz[0].mask, adst = p.swz[0].dst;
  const uint32_t bsrc = p.swz[1].src, bmask = p.swz[1].mask, bdst = p.swz[1].dst;
  const int niter = o.niter;
  for (int j0 = 0; j0 < niter; j0 += J) {
    Pack<SAt, V> av[J];
    Pack<SBt, V> bv[J];
    int64_t offo[J];
    int nv[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int jj = j0 + j;
      nv[j] = 0;
      if (jj < niter) {
        const uint32_t e = tid + (uint32_t)jj * kBlock;
        int n = V;
        if constexpr (!FULL) {
          n = e < nvec ? V : 0;
          if (n) n = vec_inside(o, e, lim_dim);
        }
        nv[j] = n;
        offo[j] = lo.off[0] + o.hi_off[0][jj];
        if (FULL || n) {
          const uint32_t slot0 = e * V;  // the output's order is the slot order
          if (stage_a) read_staged<SAt, V>(lds_a, slot0, asrc, amask, adst, av[j]);
          else read_direct<SAt, V>(pa + lo.off[1] + o.hi_off[1][jj], sa0, n, av[j]);
          if constexpr (BIN) {
            if (stage_b) read_staged<SBt, V>(lds_b, slot0, bsrc, bmask, bdst, bv[j]);
            else read_direct<SBt, V>(pb + lo.off[2] + o.hi_off[2][jj], sb0, n, bv[j]);
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if (j0 + j >= niter) break;  // uniform: the last batch of passes may be short
      const int n = nv[j];
      if (!FULL && n == 0) continue;
      Pack<SOt, V> r;
      if (p.swap) G::order_inputs(p.swap, av[j], bv[j]);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(av[j].v[i], bv[j].v[i]);
        else r.v[i] = G::eval(av[j].v[i], SBt{});
      }
      if (p.swap) G::order_output(p.swap, r);
      char *po = out + offo[j];
      if (FULL || n == V) {
        store_pack<SOt, V>(po, r, p.nt_store != 0);
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (i < n) reinterpret_cast<SOt *>(po)[i] = r.v[i];
      }
    }
  }
}

template <class S, int V, int WHICH>
OCN_DEV void stage_dispatch(KTiledArgs &p, const char *base, S *lds, bool full, const uint32_t *lim_dim,
                            uint32_t nvec) {
  if (full && nvec >= (uint32_t)kBlock) stage_operand<S, V, WHICH, true>(p, base, lds, lim_dim, nvec);
  else stage_operand<S, V, WHICH, false>(p, base, lds, lim_dim, nvec);
}

// One tile per loop trip; workgroup b takes tiles b, b + gridDim.x, ...
template <class G> __global__ __launch_bounds__(kBlock) void ew_tiled_kernel(const TiledArgs by_value) {
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  constexpr bool BIN = G::NIN2;
  constexpr int VA = 16 / (int)sizeof(SAt) > 1 ? 16 / (int)sizeof(SAt) : 1;
  constexpr int VB = 16 / (int)sizeof(SBt) > 1 ? 16 / (int)sizeof(SBt) : 1;
  constexpr int VC = G::V;
  (void)by_value;  // read through the kernarg segment instead (it is the only argument)
  KTiledArgs &p = *(KTiledArgs *)__builtin_amdgcn_kernarg_segment_ptr();

  const uint32_t tile_elems = 1u << p.tile_bits;
  SAt *lds_a = reinterpret_cast<SAt *>(ocn_lds_raw);
  SBt *lds_b = reinterpret_cast<SBt *>(reinterpret_cast<char *>(ocn_lds_raw) + p.lds_off_b);
  const bool stage_a = p.stage_a, stage_b = BIN && p.stage_b;
  const bool staged = stage_a || stage_b;
  const uint32_t total_tiles = p.total_tiles;
  const int ndim = p.ndim;

  for (uint32_t tile = blockIdx.x; tile < total_tiles; tile += gridDim.x) {
    // tile origin and clipped extents (uniform over the workgroup)
    uint32_t t = tile;
    int64_t base_o = 0, base_a = 0, base_b = 0;
    uint32_t lim_dim[kMaxDims];
    bool full = true;
#pragma unroll
    for (int d = kMaxDims - 1; d >= 0; --d) {
      lim_dim[d] = 1;
      if (d < ndim) {
        const uint32_t dv = p.ntdiv[d].d, dm = p.ntdiv[d].m, ds = p.ntdiv[d].s;
        const uint32_t q = (d == 0) ? 0u : (uint32_t)((((uint64_t)t * dm) >> 32) + t) >> ds;
        const uint32_t tc = t - q * dv;
        t = q;
        const int64_t i0 = (int64_t)tc << p.tl[d];
        const int64_t ext = (int64_t)1 << p.tl[d];
        const int64_t rem = p.size[d] - i0;
        lim_dim[d] = (uint32_t)(rem < ext ? rem : ext);
        full = full && rem >= ext;
        base_o += i0 * p.so[d];
        base_a += i0 * p.sa[d];
        if constexpr (BIN) base_b += i0 * p.sb[d];
      }
    }

    if (stage_a) {
      if (p.ord[1].vecw) stage_dispatch<SAt, VA, 1>(p, p.a + base_a, lds_a, full, lim_dim, tile_elems >> p.ord[1].vecw);
      else stage_dispatch<SAt, 1, 1>(p, p.a + base_a, lds_a, full, lim_dim, tile_elems);
    }
    if constexpr (BIN) {
      if (stage_b) {
        if (p.ord[2].vecw) stage_dispatch<SBt, VB, 2>(p, p.b + base_b, lds_b, full, lim_dim, tile_elems >> p.ord[2].vecw);
        else stage_dispatch<SBt, 1, 2>(p, p.b + base_b, lds_b, full, lim_dim, tile_elems);
      }
    }
    if (staged) __syncthreads();

    char *out = p.out + base_o;
    const char *pa = p.a + base_a;
    const char *pb = BIN ? p.b + base_b : nullptr;
    if (p.ord[0].vecw) {
      const uint32_t nvec = tile_elems >> p.ord[0].vecw;
      if (full && nvec >= (uint32_t)kBlock) tiled_compute<G, VC, true>(p, out, pa, pb, lds_a, lds_b, lim_dim, nvec);
      else tiled_compute<G, VC, false>(p, out, pa, pb, lds_a, lds_b, lim_dim, nvec);
    } else {
      if (full && tile_elems >= (uint32_t)kBlock) tiled_compute<G, 1, true>(p, out, pa, pb, lds_a, lds_b, lim_dim, tile_elems);
      else tiled_compute<G, 1, false>(p, out, pa, pb, lds_a, lds_b, lim_dim, tile_elems);
    }
    if (staged && tile + gridDim.x < total_tiles) __syncthreads();  // LDS is reused by the next tile
  }
}

// ---------------------------------------------------------------------------------------
// tiled kernel, unclipped all-vector form
// ---------------------------------------------------------------------------------------
//
// Same tiles, enumeration orders, LDS layout and swizzle as ew_tiled_kernel, for the plans the
// host proves simple: no tile is clipped, every order moves whole 16-byte vectors, inputs
// that are not staged are contiguous along the output's fastest axis, and all strides inside
// a tile are non-negative and small enough for 32-bit offsets.

using KFastArgs = const __attribute__((address_space(4))) FastTiledArgs;
using KFastOrder = const __attribute__((address_space(4))) FastOrder;

#ifndef OCN_FAST_J
#define OCN_FAST_J 2
#endif

// lane part of byte offsets (operands selected by WANT: bit 0 out, 1 a, 2 b) and of the slot
template <int WANT, class O> OCN_HDF void fast_lane(const O &o, uint32_t tid, uint32_t (&off)[3], uint32_t &slot) {
  off[0] = off[1] = off[2] = 0;
  slot = 0;
  const int n = o.nlane;
  for (int k = 0; k < n; ++k) {
    const uint32_t c = ((tid >> o.shift[k]) & o.mask[k]) << o.up[k];
    if constexpr ((WANT & 1) != 0) off[0] += c * o.stride[0][k];
    if constexpr ((WANT & 2) != 0) off[1] += c * o.stride[1][k];
    if constexpr ((WANT & 4) != 0) off[2] += c * o.stride[2][k];
    slot += c << o.slot_shift[k];
  }
}

template <class G> __global__ __launch_bounds__(kBlock) void ew_tiled_fast_kernel(const FastTiledArgs by_value) {
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr bool BIN = G::NIN2;
  constexpr int VA = 16 / (int)sizeof(SAt) > 1 ? 16 / (int)sizeof(SAt) : 1;
  constexpr int VB = 16 / (int)sizeof(SBt) > 1 ? 16 / (int)sizeof(SBt) : 1;
  constexpr int VC = G::V;
  constexpr int J = OCN_FAST_J;  // vectors in flight per lane and operand
  (void)by_value;  // read through the kernarg segment instead (it is the only argument)
  KFastArgs &p = *(KFastArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  char *lds = reinterpret_cast<char *>(ocn_lds_raw);
  if (p.warm) warm_arguments<FastTiledArgs>();

  // tile origin (uniform over the workgroup).  Workgroups go to the eight XCDs in turn, each
  // with an L2 of its own: tiles that share input lines (consecutive tile numbers, in groups
  // of 2 or 4) are given to workgroups b, b + 8, ... which the same XCD starts one after the
  // other, so that the line is fetched from memory once.
  uint32_t t = blockIdx.x;
  if (p.pair_log2) {
    const uint32_t lg = (uint32_t)p.pair_log2, r = t & 7u, h = (t >> 3) & ((1u << lg) - 1u), q = t >> (3 + lg);
    t = (q << (3 + lg)) | (r << lg) | h;
  }
  int64_t bo = 0, ba = 0, bb = 0;
  const int ntd = p.ntd;
  for (int j = 0; j < ntd; ++j) {
    const uint32_t dv = p.ntdiv[j].d, dm = p.ntdiv[j].m, ds = p.ntdiv[j].s;
    const uint32_t q = (uint32_t)((((uint64_t)t * dm) >> 32) + t) >> ds;
    const uint32_t tc = t - q * dv;
    t = q;
    bo += (int64_t)tc * p.step[0][j];
    ba += (int64_t)tc * p.step[1][j];
    if constexpr (BIN) bb += (int64_t)tc * p.step[2][j];
  }
  char *out = p.out + bo;
  const char *pa = p.a + ba;
  const char *pb = BIN ? p.b + bb : nullptr;

  const uint32_t tid = threadIdx.x;
  const bool stage_a = p.stage_a, stage_b = BIN && p.stage_b;

  if (stage_a || stage_b) {
    uint32_t offa[3] = {0, 0, 0}, offb[3] = {0, 0, 0}, slot;
    uint32_t la = 0, lb = 0;  // lane part of the swizzled LDS byte address
    int na = 0, nb = 0;
    if (stage_a) {
      fast_lane<2>(p.ord[1], tid, offa, slot);
      la = (swizzle(slot, p.swz[0].src, p.swz[0].mask, p.swz[0].dst) << p.es_log2[0]) | p.lds_base[0];
      na = p.ord[1].niter;
    }
    if constexpr (BIN) {
      if (stage_b) {
        fast_lane<4>(p.ord[2], tid, offb, slot);
        lb = (swizzle(slot, p.swz[1].src, p.swz[1].mask, p.swz[1].dst) << p.es_log2[1]) | p.lds_base[1];
        nb = p.ord[2].niter;
      }
    }
    const int nmax = na > nb ? na : nb;
    for (int j0 = 0; j0 < nmax; j0 += J) {
      Pack<SAt, VA> va[J];
      Pack<SBt, VB> vb[J];
#pragma unroll
      for (int j = 0; j < J; ++j)
        if (j0 + j < na) load_pack<SAt, VA>(pa + p.ord[1].hi_off[1][j0 + j] + offa[1], va[j], p.nt_a != 0);
      if constexpr (BIN) {
#pragma unroll
        for (int j = 0; j < J; ++j)
          if (j0 + j < nb) load_pack<SBt, VB>(pb + p.ord[2].hi_off[2][j0 + j] + offb[2], vb[j], p.nt_b != 0);
      }
#pragma unroll
      for (int j = 0; j < J; ++j) {
        if (j0 + j < na) {
          const uint32_t h = p.st_hi[0][j0 + j];
#pragma unroll
          for (int i = 0; i < VA; ++i) *reinterpret_cast<SAt *>(lds + (la ^ (h ^ p.st_el[0][i]))) = va[j].v[i];
        }
      }
      if constexpr (BIN) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
          if (j0 + j < nb) {
            const uint32_t h = p.st_hi[1][j0 + j];
#pragma unroll
            for (int i = 0; i < VB; ++i) *reinterpret_cast<SBt *>(lds + (lb ^ (h ^ p.st_el[1][i]))) = vb[j].v[i];
          }
        }
      }
    }
    __syncthreads();
  }

  // compute phase, in the output's order
  uint32_t off[3], slot_unused;
  fast_lane<BIN ? 7 : 3>(p.ord[0], tid, off, slot_unused);
  (void)slot_unused;
  const uint32_t lane_slot = tid << p.vc_log2;
  uint32_t ra = 0, rb = 0;
  if (stage_a) ra = (swizzle(lane_slot, p.swz[0].src, p.swz[0].mask, p.swz[0].dst) << p.es_log2[0]) | p.lds_base[0];
  if (stage_b) rb = (swizzle(lane_slot, p.swz[1].src, p.swz[1].mask, p.swz[1].dst) << p.es_log2[1]) | p.lds_base[1];
  constexpr int EPA = (16 / (int)sizeof(SAt)) < VC ? (16 / (int)sizeof(SAt)) : VC;  // elements per LDS access
  constexpr int EPB = (16 / (int)sizeof(SBt)) < VC ? (16 / (int)sizeof(SBt)) : VC;
  const int no = p.ord[0].niter;
  for (int j0 = 0; j0 < no; j0 += J) {
    Pack<SAt, VC> av[J];
    Pack<SBt, VC> bv[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int jj = j0 + j;
      if (jj < no) {
        if (stage_a) {
          const uint32_t h = p.rd_hi[0][jj];
#pragma unroll
          for (int c = 0; c < VC / EPA; ++c)
            *reinterpret_cast<Pack<SAt, EPA> *>(&av[j].v[c * EPA]) =
                *reinterpret_cast<const Pack<SAt, EPA> *>(lds + (ra ^ (h ^ p.rd_ch[0][c])));
        } else {
          load_pack<SAt, VC>(pa + p.ord[0].hi_off[1][jj] + off[1], av[j], p.nt_a != 0);
        }
        if constexpr (BIN) {
          if (stage_b) {
            const uint32_t h = p.rd_hi[1][jj];
#pragma unroll
            for (int c = 0; c < VC / EPB; ++c)
              *reinterpret_cast<Pack<SBt, EPB> *>(&bv[j].v[c * EPB]) =
                  *reinterpret_cast<const Pack<SBt, EPB> *>(lds + (rb ^ (h ^ p.rd_ch[1][c])));
          } else {
            load_pack<SBt, VC>(pb + p.ord[0].hi_off[2][jj] + off[2], bv[j], p.nt_b != 0);
          }
        }
      }
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
      const int jj = j0 + j;
      if (jj >= no) break;  // uniform: the last batch of passes may be short
      Pack<SOt, VC> r;
      if (p.swap) G::order_inputs(p.swap, av[j], bv[j]);
#pragma unroll
      for (int i = 0; i < VC; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(av[j].v[i], bv[j].v[i]);
        else r.v[i] = G::eval(av[j].v[i], SBt{});
      }
      if (p.swap) G::order_output(p.swap, r);
      store_pack<SOt, VC>(out + p.ord[0].hi_off[0][jj] + off[0], r, p.nt_store != 0);
    }
  }
}

// ---------------------------------------------------------------------------------------
// tiled kernel, any size and alignment
// ---------------------------------------------------------------------------------------
//
// The all-vector form above for tiles that are clipped by the end of the tensor and operands
// whose rows start anywhere: unaligned 16-byte accesses, and per vector a comparison of its
// coordinates with the tile's limits, which costs a scalar subtraction and a vector compare per
// tiled dim where the tile is clipped and nothing where it is not.  Inputs that are not
// staged may be contiguous, broadcast or strided along the output's fastest dim.

using KAnyArgs = const __attribute__((address_space(4))) AnyTiledArgs;
using KAnyOrder = const __attribute__((address_space(4))) AnyOrder;

// lane part of a vector's position: coordinates, byte offsets, LDS slot
struct AnyLane {
  uint32_t c[kAnyDims];
  uint32_t off[3];
  uint32_t slot;
};
template <class O> OCN_HDF AnyLane any_lane(const O &o, int nord, uint32_t tid) {
  AnyLane r;
  r.off[0] = r.off[1] = r.off[2] = r.slot = 0;
#pragma unroll
  for (int k = 0; k < kAnyDims; ++k) {
    r.c[k] = 0;
    if (k < nord) {
      r.c[k] = ((tid >> o.shift[k]) & o.mask[k]) << o.up[k];
#pragma unroll
      for (int x = 0; x < 3; ++x) r.off[x] += r.c[k] * o.stride[x][k];
      r.slot += r.c[k] << o.slot_shift[k];
    }
  }
  return r;
}
// how many elements of the lane's vector in this pass lie inside a tile with these limits
template <class O> OCN_HDF int any_inside(const O &o, int nord, const AnyLane &l, uint64_t lim, uint64_t hi_c, int v) {
  int n = v;
#pragma unroll
  for (int k = 0; k < kAnyDims; ++k) {
    if (k < nord) {
      const int left = (int)((uint32_t)(lim >> o.lim_shift[k]) & 0xffffu) - (int)((uint32_t)(hi_c >> (16 * k)) & 0xffffu) -
                       (int)l.c[k];
      if (k == 0) n = left < n ? left : n;
      else if (left <= 0) n = 0;
    }
  }
  return n < 0 ? 0 : n;
}
// tile number -> offsets of its origin and its limits (packed in the output's order)
template <class P> OCN_HDF uint64_t any_tile(const P &p, uint32_t t, int64_t (&base)[3]) {
  uint64_t lim = p.inner;
  base[0] = base[1] = base[2] = 0;
  const int ntd = p.ntd;
  for (int j = 0; j < ntd; ++j) {
    const uint32_t dv = p.ntdiv[j].d;
    const uint32_t q = j + 1 < ntd ? fastdiv(t, FastDiv{dv, p.ntdiv[j].m, p.ntdiv[j].s}) : 0u;
    const uint32_t tc = t - q * dv;
    t = q;
    for (int x = 0; x < 3; ++x) base[x] += (int64_t)tc * p.step[x][j];
    const uint32_t sh = p.dim_shift[j];
    if (sh < 64 && tc + 1 == dv) lim = (lim & ~((uint64_t)0xffffu << sh)) | ((uint64_t)p.last[j] << sh);
  }
  return lim;
}

// Where a lane loads the whole vector at `src` from: at src, or - a vector at the end of a clipped
// tile, of which only the first elements exist - so many whole elements before it that it ends
// with the operand's last byte or before (views of complex elements may have rows an odd number
// of scalars apart); `back` is the distance in elements.  The elements in between belong to the
// operand's storage and are dropped.  (Loading just the elements that exist takes a branch with
// loads on both sides, and the compiler waits for one side before it issues the other.)
OCN_HDF const char *any_address(const char *src, const char *last, int es_log2, int &back) {
  back = src > last ? (int)((src - last + (((int64_t)1 << es_log2) - 1)) >> es_log2) : 0;
  return src - ((int64_t)back << es_log2);
}
// element i of the vector is element i + back of what was loaded
template <class S, int V> OCN_DEV void any_shift(Pack<S, V> &v, int back) {
  while (back > 0) {
#pragma unroll
    for (int i = 0; i + 1 < V; ++i) v.v[i] = v.v[i + 1];
    --back;
  }
}
// n of V elements from global memory, s0 bytes apart
template <class S, int V, int AL> OCN_DEV void any_load(const char *src, const char *last, uint32_t s0, int n, Pack<S, V> &v, int &back) {
  back = 0;
  if (n > 0) {
    if (s0 == (uint32_t)sizeof(S)) {
      constexpr int L = sizeof(S) == 16 ? 4 : sizeof(S) == 8 ? 3 : sizeof(S) == 4 ? 2 : sizeof(S) == 2 ? 1 : 0;
      load_pack_any<S, V, AL>(any_address(src, last, L, back), v);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)   // (past the last element that exists: that one again)
        v.v[i] = *reinterpret_cast<const S *>(src + (uint32_t)(i < n ? i : n - 1) * s0);
    }
  }
}
// one vector of a staged input into LDS
template <class S, int V> OCN_DEV void any_park(char *lds, uint32_t addr, const Pack<S, V> &v, int n, KTable *el) {
#pragma unroll
  for (int i = 0; i < V; ++i)
    if (i < n) *reinterpret_cast<S *>(lds + (addr ^ el[i])) = v.v[i];
}
template <class S, int V> OCN_DEV void any_staged(const char *lds, uint32_t addr, KTable *el, Pack<S, V> &v) {
  constexpr int EP = (16 / (int)sizeof(S)) < V ? (16 / (int)sizeof(S)) : V;  // elements per LDS access
#pragma unroll
  for (int c = 0; c < V; c += EP)
    *reinterpret_cast<Pack<S, EP> *>(&v.v[c]) = *reinterpret_cast<const Pack<S, EP> *>(lds + (addr ^ el[c]));
}

// One vector per lane, operand and pass, and enough lanes (256 to 1024, the planner's choice) that
// a tile takes one or two passes: two or four vectors per lane held over the same loop needed 92
// to 151 vector registers instead of 58 and ran 10 to 25 % slower.  float 6000 x 5000 plus a
// transpose: 86.7 us in the general form, 74.8 here; 500 x 381 x 250: 243 -> 133; complex products
// of five-dimensional views [15, 31, 63, 61, 7]: 163 -> 98, [12, 6, 11, 3, 19]: 16.2 -> 7.7.
template <class G> __global__ __launch_bounds__(kAnyMaxBlock) void ew_tiled_any_kernel(const AnyTiledArgs by_value) {
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr bool BIN = G::NIN2;
  constexpr int VA = 16 / (int)sizeof(SAt) > 1 ? 16 / (int)sizeof(SAt) : 1;
  constexpr int VB = 16 / (int)sizeof(SBt) > 1 ? 16 / (int)sizeof(SBt) : 1;
  constexpr int V = G::V;
  constexpr int ALA = scalar_bytes(G::SA_DT), ALB = scalar_bytes(G::SB_DT), ALO = scalar_bytes(G::SO_DT);
  (void)by_value;  // read through the kernarg segment instead (it is the only argument)
  KAnyArgs &p = *(KAnyArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  char *lds = reinterpret_cast<char *>(ocn_lds_raw);
  if (p.warm) warm_arguments<AnyTiledArgs>();
  const uint32_t tid = threadIdx.x, block = p.block;
  const int nord = p.nord;
  const bool stage_a = p.stage_a, stage_b = BIN && p.stage_b;
  int64_t base[3];
  const uint64_t lim = any_tile(p, blockIdx.x, base);
  const bool full = lim == p.whole;
  char *out = p.out + base[0];
  const char *pa = p.a + base[1];
  const char *pb = BIN ? p.b + base[2] : nullptr;

  // How many elements of the lane's vector in this pass exist.  (A pass never reaches niter; the
  // comparison is there for what the compiler makes of the loads around it: without it the
  // complex products of [15, 31, 63, 61, 7] took 106 us instead of 97.)
  auto inside = [&](KAnyOrder &o, const AnyLane &l, int pass, int v) -> int {
    if (pass >= o.niter || tid + (uint32_t)pass * block >= o.nvec) return 0;
    return full ? v : any_inside(o, nord, l, lim, o.hi_c[pass], v);
  };

  // inputs read in place: the first pass is on its way while the staged ones are fetched
  KAnyOrder &oo = p.ord[0];
  const AnyLane lo = any_lane(oo, nord, tid);
  Pack<SAt, V> av;
  Pack<SBt, V> bv;
  int n, back_a, back_b;
  auto fetch = [&](int j) {
    n = inside(oo, lo, j, V);
    if (!stage_a)
      any_load<SAt, V, ALA>(pa + oo.hi_off[1][j] + lo.off[1], p.end[0] - V * (int)sizeof(SAt), p.sa0, n, av, back_a);
    if constexpr (BIN) {
      if (!stage_b)
        any_load<SBt, V, ALB>(pb + oo.hi_off[2][j] + lo.off[2], p.end[1] - V * (int)sizeof(SBt), p.sb0, n, bv, back_b);
    }
  };
  fetch(0);

  if (stage_a || stage_b) {
    AnyLane la, lb;
    uint32_t wa = 0, wb = 0;  // lane part of the swizzled LDS byte address
    int na = 0, nb = 0;
    if (stage_a) {
      la = any_lane(p.ord[1], nord, tid);
      wa = (swizzle(la.slot, p.swz[0].src, p.swz[0].mask, p.swz[0].dst) << p.es_log2[0]) | p.lds_base[0];
      na = p.ord[1].niter;
    }
    if (stage_b) {
      lb = any_lane(p.ord[2], nord, tid);
      wb = (swizzle(lb.slot, p.swz[1].src, p.swz[1].mask, p.swz[1].dst) << p.es_log2[1]) | p.lds_base[1];
      nb = p.ord[2].niter;
    }
    const int nmax = na > nb ? na : nb;
    for (int j = 0; j < nmax; ++j) {
      Pack<SAt, VA> va;
      Pack<SBt, VB> vb;
      int ca = 0, cb = 0, da, db;
      // (both loads are issued before either vector is parked)
      if (j < na) {
        ca = inside(p.ord[1], la, j, VA);
        any_load<SAt, VA, ALA>(pa + p.ord[1].hi_off[1][j] + la.off[1], p.end[0] - VA * (int)sizeof(SAt), p.stage_stride[0], ca, va, da);
      }
      if constexpr (BIN) {
        if (j < nb) {
          cb = inside(p.ord[2], lb, j, VB);
          any_load<SBt, VB, ALB>(pb + p.ord[2].hi_off[2][j] + lb.off[2], p.end[1] - VB * (int)sizeof(SBt), p.stage_stride[1], cb, vb, db);
        }
      }
      if (j < na) {
        if (!full) any_shift<SAt, VA>(va, da);
        any_park<SAt, VA>(lds, wa ^ p.st_hi[0][j], va, ca, p.st_el[0]);
      }
      if constexpr (BIN) {
        if (j < nb) {
          if (!full) any_shift<SBt, VB>(vb, db);
          any_park<SBt, VB>(lds, wb ^ p.st_hi[1][j], vb, cb, p.st_el[1]);
        }
      }
    }
    __syncthreads();
  }

  // compute phase, in the output's order
  const uint32_t slot = tid * (uint32_t)V;
  uint32_t ra = 0, rb = 0;
  if (stage_a) ra = (swizzle(slot, p.swz[0].src, p.swz[0].mask, p.swz[0].dst) << p.es_log2[0]) | p.lds_base[0];
  if (stage_b) rb = (swizzle(slot, p.swz[1].src, p.swz[1].mask, p.swz[1].dst) << p.es_log2[1]) | p.lds_base[1];
  const int niter = oo.niter;
  for (int j = 0;;) {
    if (n > 0) {
      if (stage_a) any_staged<SAt, V>(lds, ra ^ p.rd_hi[0][j], p.rd_el[0], av);
      else if (!full) any_shift<SAt, V>(av, back_a);
      if constexpr (BIN) {
        if (stage_b) any_staged<SBt, V>(lds, rb ^ p.rd_hi[1][j], p.rd_el[1], bv);
        else if (!full) any_shift<SBt, V>(bv, back_b);
      }
    }
    if (n > 0) {
      Pack<SOt, V> r;
      if (p.swap) G::order_inputs(p.swap, av, bv);
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(av.v[i], bv.v[i]);
        else r.v[i] = G::eval(av.v[i], SBt{});
      }
      if (p.swap) G::order_output(p.swap, r);
      char *po = out + oo.hi_off[0][j] + lo.off[0];
      if (n == V) {
        store_pack_any<SOt, V, ALO>(po, r, p.nt_store != 0);
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (i < n) reinterpret_cast<SOt *>(po)[i] = r.v[i];
      }
    }
    if (++j >= niter) break;  // uniform
    fetch(j);
  }
}

#endif  // __HIPCC__

}  // namespace ocn
