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

// Arguments of the kernel for boxes of any extents (ew_box_kernel).  A box is walked three times, by
// the output and by each staged input, in the operand's own order: runs of contiguous elements (one
// dim, or several the box covers whole), cut into vectors, and rows of runs along the other dims.
// Dividends are below 2^16, so a division is the high half of a product with ceil(2^32 / d); zero in
// its place leaves the quotient zero.  Everything is read whether a box has that many dims or not
// (what is missing is neutral): a test per dim is a scalar load and a wait of its own.  The largest
// coordinates a clipped box has are packed as 16 bits per dim.
constexpr uint32_t kBoxSlack = 64;          // offsets into an input start here: they stay positive for vectors moved back
constexpr int kBoxRows = 3;                 // most dims of a box (four) besides the first of a run
constexpr int kBoxRunDims = 3;              // most dims of the output's run
constexpr int kBoxGrid = 4;                 // box coordinates that are split off without a test
enum { kBoxStaged, kBoxInPlace };
struct BoxInput {
  uint32_t nvec, vpr, vpr_m;                // vectors of a whole box and of a run
  uint32_t pitch, base;                     // LDS bytes from run to run, and where the first one lies
  uint32_t epv;                             // elements of a vector
  uint32_t ext[2], ext_m[2];                // rows: extents of the first two dims
  uint32_t stride[kBoxRows];
  uint32_t unit;                            // a run's elements are unit times the extent of its last dim
  // one pass of the workgroup's lanes further on: digits of that many vectors (vector in the run, then
  // rows), bytes, and what a carry out of each digit adds
  uint32_t add[3], add_c2, add_off, add_lds, wrap_off[3], wrap_lds;
  uint32_t wrap[3];                         // radix of each digit
  uint32_t lim_run, lim[kBoxRows];          // where the limits sit
  uint32_t niter;                           // passes of the workgroup's lanes
  int32_t how;                              // staged, or read in place
  uint32_t reach;                           // bytes from a box's origin to the end of its last vector
};
struct BoxOutput {
  uint32_t nvec, vpr, vpr_m;
  uint32_t ext[2], ext_m[2];                // rows: extents of the first two dims
  uint32_t step, stride[kBoxRows];          // of the output: bytes from vector to vector, and per coordinate
  uint32_t start[2];                        // of the inputs: where the first element lies, in LDS or in place
  uint32_t run[2], pos[2][kBoxRows];        // ... bytes from element to element of a run's first dim, and per coordinate
  uint32_t add[3], add_c2, add_off, add_pos[2];   // one pass further on, as BoxInput
  uint32_t wrap[3], wrap_off[3], wrap_pos[2][3];
  uint32_t unit, lim_run, lim[kBoxRows];
  uint32_t run_ext[kBoxRunDims - 1], run_m[kBoxRunDims - 1];
  uint32_t run_pos[2][kBoxRunDims - 1];     // what a carry from one run dim into the next adds
  uint32_t niter;
  int32_t nrun;
};
struct BoxArgs {
  char *out;
  const char *a, *b;
  const char *end[2];                       // ends of the inputs: one past the highest byte
  uint64_t inner;                           // the limits of a box that is not the last along any dim
  int32_t warm, ntd;
  FastDiv ntdiv[kMaxDims];                  // box number -> box coordinates, fastest first
  int64_t step[3][kMaxDims];
  uint64_t cut[kMaxDims];                   // what the dim's last box takes off the limits
  int32_t nt_store, swap;
  uint32_t block;
  uint32_t group, regular;                  // boxes in a row that one XCD takes; boxes numbered that way
  FastDiv group_div;                        // eight such groups
  BoxInput in[2];
  BoxOutput o;
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
  static constexpr int EW = OP, SA_DT = SA, SB_DT = SB, SO_DT = SO;
  static constexpr int V = rows_vec((int)sizeof(SOt), ES_MAX);
  static constexpr int U = rows_unroll(V, ES_MAX);
  static constexpr int VR = rows_stream_vec((int)sizeof(SOt), ES_MIN, ES_MAX);  // the rows kernel's vector
  static constexpr int UR = rows_stream_unroll(VR, ES_MIN);
  static constexpr int VB = box_vec_len((int)sizeof(SOt), ES_MAX);  // the box kernel's vector

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
      // (scalar branches: computed for every vector and selected away, the reversals are a tenth of what a function of
      // complex floats executes; with the reciprocal of sinh_cosh_any sines of 2^24 of them 54.9 -> 52.7 us, hyperbolic
      // tangents 60.8 -> 56.9; logarithms, by the branches alone, 71.3 -> 67.2)
      if (swap) {
        OCN_KEEP_BRANCH();
        G::order_inputs(swap, va[u], vb[u]);
        OCN_KEEP_BRANCH();
      }
#pragma unroll
      for (int i = 0; i < V; ++i) {
        if constexpr (BIN) r.v[i] = G::eval(va[u].v[i], vb[u].v[i]);
        else r.v[i] = G::eval(va[u].v[i], SBt{});
      }
      if (swap) {
        OCN_KEEP_BRANCH();
        G::order_output(swap, r);
        OCN_KEEP_BRANCH();
      }
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

// V elements from element s on (0 <= s < V) of the 2 V that lie in a and b one after the other
template <class S, int V> OCN_DEV Pack<S, V> two_pieces(const Pack<S, V> &a, const Pack<S, V> &b, uint32_t s) {
  Pack<S, V> r;
  constexpr int B = (int)sizeof(S) * V;
  if constexpr (V == 1) {
    r = a;
  } else if constexpr (B % 4 != 0) {
    S c[2 * V];
#pragma unroll
    for (int i = 0; i < V; ++i) c[i] = a.v[i], c[V + i] = b.v[i];
#pragma unroll
    for (int step = 1; step < V; step *= 2)
#pragma unroll
      for (int i = 0; i + step < 2 * V; ++i) c[i] = s & step ? c[i + step] : c[i];
#pragma unroll
    for (int i = 0; i < V; ++i) r.v[i] = c[i];
  } else {
    constexpr int W = B / 4;
    uint32_t w[2 * W + 1];
    __builtin_memcpy(w, &a, B);
    __builtin_memcpy(w + W, &b, B);
    w[2 * W] = 0;
    const uint32_t bytes = s * (uint32_t)sizeof(S), words = bytes / 4;
#pragma unroll
    for (int step = W / 2 > 0 ? W / 2 : 1; step >= 1; step /= 2) {
      if (step < W) {
#pragma unroll
        for (int i = 0; i + step < 2 * W; ++i) w[i] = words & step ? w[i + step] : w[i];
      }
    }
    if constexpr (sizeof(S) < 4) {
#pragma unroll
      for (int i = 0; i < W; ++i) w[i] = __builtin_amdgcn_alignbyte(w[i + 1], w[i], bytes & 3);
    }
    __builtin_memcpy(&r, w, B);
  }
  return r;
}

// PIECES: vectors that go on into the next row in two whole pieces, not element by element.  The code for them costs every
// other vector registers and time (two inputs of bytes 85 registers, 49 without, and three wavefronts of eight from every SIMD;
// flat calls of any length 1 to 4 %, negated halves 4, sines of floats 2), so that it is a kernel of its own, chosen by
// rows_in_pieces.
template <class G, bool PIECES> __global__ __launch_bounds__(kBlock) void ew_rows_kernel(const RowsArgs by_value) {
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
      if (!va_ok || !vb_ok) {
        if (PIECES && whole && p.inner >= (uint32_t)V) {
          // An input whose vector goes on into the next row: the last V elements of the one row and the first
          // V of the other, whole vectors both.  (Element by element, in a lane or two of every wavefront, products
          // of halves [78078, 666] with a row took 58 us, 36 so, [1268292, 41] 81, 45; of doubles [292682, 41] 39, 34.
          // Not with several vectors per lane, where each would be waited for before the next is asked for: halves
          // times floats [548387, 62] 48 us, 72 so.)
          const uint32_t from = r.col - (p.inner - (uint32_t)V);
          const int here = V - (int)from;
          RowsPlace next = r;
          next.col = 0;
          rows_outer(p, r.row + 1, next.off);
          r.col = p.inner - (uint32_t)V;
          Pack<SAt, V> na;
          Pack<SBt, V> nb;
          if (!va_ok) {
            if (abc) {
              va[u].v[0] = *reinterpret_cast<const SAt *>(p.a + r.off[1]);
              na.v[0] = *reinterpret_cast<const SAt *>(p.a + next.off[1]);
            } else {
              load_pack_any<SAt, V, ALA>(p.a + rows_offset(r, 1, 0, ESA, false, false), va[u]);
              load_pack_any<SAt, V, ALA>(p.a + next.off[1], na);
            }
          }
          if constexpr (BIN) {
            if (!vb_ok) {
              if (bbc) {
                vb[u].v[0] = *reinterpret_cast<const SBt *>(p.b + r.off[2]);
                nb.v[0] = *reinterpret_cast<const SBt *>(p.b + next.off[2]);
              } else {
                load_pack_any<SBt, V, ALB>(p.b + rows_offset(r, 2, 0, ESB, false, false), vb[u]);
                load_pack_any<SBt, V, ALB>(p.b + next.off[2], nb);
              }
            }
          }
          if (!va_ok) {
            if (abc) {
#pragma unroll
              for (int i = V - 1; i >= 0; --i) va[u].v[i] = i < here ? va[u].v[0] : na.v[0];
            } else {
              va[u] = two_pieces(va[u], na, from);
            }
          }
          if constexpr (BIN) {
            if (!vb_ok) {
              if (bbc) {
#pragma unroll
                for (int i = V - 1; i >= 0; --i) vb[u].v[i] = i < here ? vb[u].v[0] : nb.v[0];
              } else {
                vb[u] = two_pieces(vb[u], nb, from);
              }
            }
          }
        } else {   // element by element: a vector that is not whole, or rows shorter than one
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

// ---------------------------------------------------------------------------------------
// boxes of any extents
// ---------------------------------------------------------------------------------------
//
// The tiles above have power-of-two extents: axes of 5, 17 or 71 leave up to half of the lanes
// without work per axis, and only an operand's fastest axis is lengthened, however short its runs
// stay.  Here extents are whole numbers (an axis is cut into equal parts, or not at all), runs go on
// along every axis the box covers whole, and lane numbers are split by multiplication.  A
// staged input lies in LDS in its own order, run after run, as its 16-byte pieces arrive; the
// compute phase picks its elements one by one.

using KBoxArgs = const __attribute__((address_space(4))) BoxArgs;
using KBoxOutput = const __attribute__((address_space(4))) BoxOutput;
using KBoxInput = const __attribute__((address_space(4))) BoxInput;

OCN_HDF uint32_t box_mulhi(uint32_t n, uint32_t m) { return (uint32_t)(((uint64_t)n * m) >> 32); }
OCN_HDF uint32_t box_limit(uint64_t lims, uint32_t shift) { return (uint32_t)(lims >> shift) & 0xffffu; }

// Workgroup number -> box number.  Workgroups go to the eight XCDs in turn, each with an L2 of its own:
// every XCD takes `group` boxes in a row, so that lines which neighbouring boxes share are fetched once.
template <class P> OCN_HDF uint32_t box_number(const P &p, uint32_t b) {
  if (b >= p.regular) return b;
  const uint32_t w = fastdiv(b, FastDiv{p.group_div.d, p.group_div.m, p.group_div.s}), r = b - w * p.group_div.d;
  return w * p.group_div.d + r % kXcds * p.group + r / kXcds;
}
// box number -> offsets of its origin and its limits
template <class P> OCN_HDF uint64_t box_origin(const P &p, uint32_t t, int64_t (&base)[3]) {
  uint64_t lims = p.inner;
  base[0] = base[1] = base[2] = 0;
  auto split = [&](int j) {
    const uint32_t dv = p.ntdiv[j].d;
    const uint32_t q = fastdiv(t, FastDiv{dv, p.ntdiv[j].m, p.ntdiv[j].s});
    const uint32_t tc = t - q * dv;
    t = q;
    for (int x = 0; x < 3; ++x) base[x] += (int64_t)tc * p.step[x][j];
    lims -= tc + 1 == dv ? p.cut[j] : 0;
  };
#pragma unroll
  for (int j = 0; j < kBoxGrid; ++j) split(j);
  const int ntd = p.ntd;
  for (int j = kBoxGrid; j < ntd; ++j) split(j);
  return lims;
}

// Where a lane is on its way through a staged input: vector number, digits, bytes from the box's
// origin, LDS address.
struct BoxLane {
  uint32_t t, iv, c[kBoxRows], off, lds;
};
template <class I> OCN_HDF BoxLane box_lane(const I &x, uint32_t t) {
  BoxLane r;
  const uint32_t row = x.vpr == 1 ? t : box_mulhi(t, x.vpr_m);
  r.t = t;
  r.iv = t - row * x.vpr;
  const uint32_t q0 = box_mulhi(row, x.ext_m[0]), q1 = box_mulhi(q0, x.ext_m[1]);
  r.c[0] = row - q0 * x.ext[0];
  r.c[1] = q0 - q1 * x.ext[1];
  r.c[2] = q1;
  r.off = kBoxSlack + r.iv * 16u + r.c[0] * x.stride[0] + r.c[1] * x.stride[1] + r.c[2] * x.stride[2];
  r.lds = x.base + row * x.pitch + r.iv * 16u;
  return r;
}
// one pass of the workgroup's lanes further on (all ones or zero instead of a branch per carry)
template <class I> OCN_HDF void box_advance(const I &x, uint32_t block, BoxLane &r) {
  r.t += block;
  r.iv += x.add[0];
  const uint32_t w0 = r.iv >= x.wrap[0] ? ~0u : 0u;
  r.iv -= w0 & x.wrap[0];
  r.c[0] += x.add[1] - w0;
  const uint32_t w1 = r.c[0] >= x.wrap[1] ? ~0u : 0u;
  r.c[0] -= w1 & x.wrap[1];
  r.c[1] += x.add[2] - w1;
  const uint32_t w2 = r.c[1] >= x.wrap[2] ? ~0u : 0u;
  r.c[1] -= w2 & x.wrap[2];
  r.c[2] += x.add_c2 - w2;
  r.off += x.add_off + (w0 & x.wrap_off[0]) + (w1 & x.wrap_off[1]) + (w2 & x.wrap_off[2]);
  r.lds += x.add_lds + (w0 & x.wrap_lds);
}
// does any of the lane's vector exist in a box with these limits
template <class I> OCN_HDF bool box_exists(const I &x, uint64_t lims, const BoxLane &r) {
  const uint32_t in_run = r.iv * x.epv < x.unit * (box_limit(lims, x.lim_run) + 1), in0 = r.c[0] <= box_limit(lims, x.lim[0]),
                 in1 = r.c[1] <= box_limit(lims, x.lim[1]), in2 = r.c[2] <= box_limit(lims, x.lim[2]);
  return (in_run & in0 & in1 & in2) != 0;
}

// The same for the output: where its vector, and the inputs' elements for it, lie.
struct BoxVec {
  uint32_t t, iv, c[kBoxRows], off, pos[2];
};
template <class O> OCN_HDF BoxVec box_vec(const O &o, uint32_t t) {
  BoxVec r;
  const uint32_t row = o.vpr == 1 ? t : box_mulhi(t, o.vpr_m);
  r.t = t;
  r.iv = t - row * o.vpr;
  const uint32_t q0 = box_mulhi(row, o.ext_m[0]), q1 = box_mulhi(q0, o.ext_m[1]);
  r.c[0] = row - q0 * o.ext[0];
  r.c[1] = q0 - q1 * o.ext[1];
  r.c[2] = q1;
  r.off = r.iv * o.step + r.c[0] * o.stride[0] + r.c[1] * o.stride[1] + r.c[2] * o.stride[2];
#pragma unroll
  for (int y = 0; y < 2; ++y) r.pos[y] = o.start[y] + r.iv * o.run[y] + r.c[0] * o.pos[y][0] + r.c[1] * o.pos[y][1] + r.c[2] * o.pos[y][2];
  return r;
}
template <class O> OCN_HDF void box_advance_out(const O &o, uint32_t block, BoxVec &r) {
  r.t += block;
  r.iv += o.add[0];
  const uint32_t w0 = r.iv >= o.wrap[0] ? ~0u : 0u;
  r.iv -= w0 & o.wrap[0];
  r.c[0] += o.add[1] - w0;
  const uint32_t w1 = r.c[0] >= o.wrap[1] ? ~0u : 0u;
  r.c[0] -= w1 & o.wrap[1];
  r.c[1] += o.add[2] - w1;
  const uint32_t w2 = r.c[1] >= o.wrap[2] ? ~0u : 0u;
  r.c[1] -= w2 & o.wrap[2];
  r.c[2] += o.add_c2 - w2;
  r.off += o.add_off + (w0 & o.wrap_off[0]) + (w1 & o.wrap_off[1]) + (w2 & o.wrap_off[2]);
#pragma unroll
  for (int y = 0; y < 2; ++y)
    r.pos[y] += o.add_pos[y] + (w0 & o.wrap_pos[y][0]) + (w1 & o.wrap_pos[y][1]) + (w2 & o.wrap_pos[y][2]);
}
// how many elements of the vector exist
template <int V, class O> OCN_HDF int box_count(const O &o, uint64_t lims, bool clipped, const BoxVec &r) {
  const int left = (int)(o.unit * (box_limit(lims, o.lim_run) + 1)) - (int)(r.iv * (uint32_t)V);
  int n = left < V ? left : V;
  if (clipped) {
    const uint32_t out0 = r.c[0] > box_limit(lims, o.lim[0]), out1 = r.c[1] > box_limit(lims, o.lim[1]), out2 = r.c[2] > box_limit(lims, o.lim[2]);
    n = (out0 | out1 | out2) != 0 ? 0 : n;
  }
  return r.t < o.nvec ? n : 0;
}
// Runs along two or three dims: the vector's coordinates in the run, and what they add to its place.
// (run[y] is bytes per vector here and in box_vec; a carry takes back what the elements of a whole
// dim were counted for.)
struct BoxRun {
  uint32_t c[kBoxRunDims - 1];
};
template <int V, class O> OCN_HDF BoxRun box_run(const O &o, const BoxVec &r, uint32_t (&pos)[2]) {
  const uint32_t e0 = r.iv * (uint32_t)V, d1 = box_mulhi(e0, o.run_m[0]), d2 = box_mulhi(d1, o.run_m[1]);
#pragma unroll
  for (int y = 0; y < 2; ++y) pos[y] = r.pos[y] + d1 * o.run_pos[y][0] + d2 * o.run_pos[y][1];
  return BoxRun{{e0 - d1 * o.run_ext[0], d1 - d2 * o.run_ext[1]}};
}
// the next element of such a run
template <int V, class O> OCN_HDF void box_next(const O &o, BoxRun &r, uint32_t (&pos)[2]) {
  const uint32_t w0 = ++r.c[0] == o.run_ext[0] ? ~0u : 0u;
  r.c[0] &= ~w0;
  r.c[1] -= w0;
  const uint32_t w1 = r.c[1] == o.run_ext[1] ? ~0u : 0u;
  r.c[1] &= ~w1;
#pragma unroll
  for (int y = 0; y < 2; ++y) pos[y] += o.run[y] / V + (w0 & o.run_pos[y][0]) + (w1 & o.run_pos[y][1]);
}

// A vector that would run past its operand's end is loaded from so many whole elements before it
// (see any_address); room: bytes from the box's origin to the last place a vector may start at.
OCN_HDF uint32_t box_back(uint32_t off, int32_t room, int es_log2) {
  const int32_t over = (int32_t)(off - kBoxSlack) - room;
  return over > 0 ? (uint32_t)(over + ((1 << es_log2) - 1)) >> es_log2 : 0u;
}
OCN_HDF int32_t box_room(const char *end, const char *origin, int bytes) {
  const int64_t room = end - origin - bytes;
  return room > INT32_MAX ? INT32_MAX : (int32_t)room;
}

// the fields of a staged input that box_lane and box_advance read, all fetched at once
OCN_DEV void box_input(KBoxInput &k, BoxInput &x) {
  x.nvec = k.nvec; x.vpr = k.vpr; x.vpr_m = k.vpr_m; x.pitch = k.pitch; x.base = k.base;
  x.add_c2 = k.add_c2; x.add_off = k.add_off; x.add_lds = k.add_lds; x.wrap_lds = k.wrap_lds;
#pragma unroll
  for (int i = 0; i < 2; ++i) { x.ext[i] = k.ext[i]; x.ext_m[i] = k.ext_m[i]; }
#pragma unroll
  for (int i = 0; i < 3; ++i) { x.stride[i] = k.stride[i]; x.add[i] = k.add[i]; x.wrap[i] = k.wrap[i]; x.wrap_off[i] = k.wrap_off[i]; }
  OCN_ARGS_NOW("s"(x.nvec), "s"(x.vpr), "s"(x.vpr_m), "s"(x.pitch), "s"(x.base), "s"(x.ext[0]), "s"(x.ext[1]),
               "s"(x.ext_m[0]), "s"(x.ext_m[1]), "s"(x.stride[0]), "s"(x.stride[1]), "s"(x.stride[2]), "s"(x.add[0]), "s"(x.add[1]), "s"(x.add[2]),
               "s"(x.add_c2), "s"(x.add_off), "s"(x.add_lds), "s"(x.wrap_lds), "s"(x.wrap[0]), "s"(x.wrap[1]), "s"(x.wrap[2]), "s"(x.wrap_off[0]),
               "s"(x.wrap_off[1]), "s"(x.wrap_off[2]));
}

OCN_DEV void box_output(KBoxOutput &k, BoxOutput &x) {
  x.nvec = k.nvec; x.vpr = k.vpr; x.vpr_m = k.vpr_m; x.step = k.step; x.add_c2 = k.add_c2; x.add_off = k.add_off; x.unit = k.unit; x.lim_run = k.lim_run;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    x.ext[i] = k.ext[i]; x.ext_m[i] = k.ext_m[i]; x.start[i] = k.start[i]; x.run[i] = k.run[i]; x.add_pos[i] = k.add_pos[i];
    x.run_ext[i] = k.run_ext[i]; x.run_m[i] = k.run_m[i];
    for (int y = 0; y < 2; ++y) x.run_pos[y][i] = k.run_pos[y][i];
  }
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    x.stride[i] = k.stride[i]; x.add[i] = k.add[i]; x.wrap[i] = k.wrap[i]; x.wrap_off[i] = k.wrap_off[i]; x.lim[i] = k.lim[i];
    for (int y = 0; y < 2; ++y) { x.pos[y][i] = k.pos[y][i]; x.wrap_pos[y][i] = k.wrap_pos[y][i]; }
  }
  OCN_ARGS_NOW("s"(x.nvec), "s"(x.vpr), "s"(x.vpr_m), "s"(x.step), "s"(x.ext[0]), "s"(x.ext[1]), "s"(x.ext_m[0]), "s"(x.ext_m[1]), "s"(x.stride[0]),
               "s"(x.stride[1]), "s"(x.stride[2]), "s"(x.start[0]), "s"(x.start[1]), "s"(x.run[0]), "s"(x.run[1]), "s"(x.pos[0][0]), "s"(x.pos[0][1]),
               "s"(x.pos[0][2]), "s"(x.pos[1][0]), "s"(x.pos[1][1]), "s"(x.pos[1][2]), "s"(x.unit), "s"(x.lim_run));
}

// Vectors of a staged input, and passes of inputs read in place, that a lane has in flight.  With two and
// two, kernels of two inputs take 53 to 86 registers (5 to 7 wavefronts per SIMD; floats 65), 134 of one-byte
// types (3); those of one input 38 to 68, unless an elementary function takes more.  Four of either take 87 to
// 97 of floats, and fewer wavefronts lose more than the loads win (6000 x 5000 plus a transpose 69 us with
// two and two, 76 with four passes, 72 with one).
// The private segment of 68 or 132 bytes that kernels of two inputs reserve holds scalar registers that the
// compiler then keeps in lanes of a vector register: no instruction accesses it.
constexpr int kBoxLoads = 2, kBoxAhead = 2;
// STA, STB: the input is staged in LDS (else read in place).
template <class G, bool STA, bool STB>
OCN_DEV void box_body(KBoxArgs &p, char *lds, uint64_t lims, char *out, const char *pa, const char *pb) {
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  using SOt = typename G::SOt;
  constexpr bool BIN = G::NIN2;
  constexpr int VA = 16 / (int)sizeof(SAt), VB = 16 / (int)sizeof(SBt);
  constexpr int V = G::VB;
  constexpr int ALA = scalar_bytes(G::SA_DT), ALB = scalar_bytes(G::SB_DT), ALO = scalar_bytes(G::SO_DT);
  constexpr int LA = sizeof(SAt) == 16 ? 4 : sizeof(SAt) == 8 ? 3 : sizeof(SAt) == 4 ? 2 : sizeof(SAt) == 2 ? 1 : 0;
  constexpr int LB = sizeof(SBt) == 16 ? 4 : sizeof(SBt) == 8 ? 3 : sizeof(SBt) == 4 ? 2 : sizeof(SBt) == 2 ? 1 : 0;
  constexpr int U = kBoxLoads;
  const uint32_t tid = threadIdx.x, block = p.block;
  const bool clipped = lims != p.inner;
  // (does a vector of the box reach past the operand's end?  Only those of its last boxes do.)
  const bool end_a = p.end[0] - pa < (int64_t)p.in[0].reach, end_b = BIN && p.end[1] - pb < (int64_t)p.in[1].reach;
  const char *qa = pa - kBoxSlack, *qb = BIN ? pb - kBoxSlack : nullptr;

  // Inputs read in place: the first pass is on its way while the others are fetched.  (Every lane
  // loads, one without a vector from the box's origin: a load under a condition of its own makes the
  // compiler wait for those before it.)
  BoxOutput o;
  box_output(p.o, o);
  // PU passes of the inputs read in place are on their way at a time
  constexpr int PU = !STA || (BIN && !STB) ? kBoxAhead : 1;
  const uint32_t niter = p.o.niter;
  BoxVec walker = box_vec(o, tid), vs[PU];
  int ns[PU];
  Pack<SAt, V> as[PU];
  Pack<SBt, V> bs[PU];
  uint32_t back_a[PU], back_b[PU];
  const bool one_a = !STA && o.run[0] == 0, one_b = BIN && !STB && o.run[1] == 0;
  auto fetch = [&](uint32_t j) {
#pragma unroll
    for (int u = 0; u < PU; ++u) {
      if (j + u < niter) {
        const BoxVec v = vs[u] = walker;
        box_advance_out(o, block, walker);
        const int n = ns[u] = box_count<V>(o, lims, clipped, v);
        back_a[u] = back_b[u] = 0;
        if constexpr (!STA) {
          uint32_t off = n > 0 ? v.pos[0] : kBoxSlack;
          if (one_a) {
            as[u].v[0] = *reinterpret_cast<const SAt *>(qa + off);
          } else {
            if (end_a) {
              back_a[u] = box_back(off, box_room(p.end[0], pa, V * (int)sizeof(SAt)), LA);
              off -= back_a[u] << LA;
            }
            load_pack_any<SAt, V, ALA>(qa + off, as[u]);
          }
        }
        if constexpr (BIN && !STB) {
          uint32_t off = n > 0 ? v.pos[1] : kBoxSlack;
          if (one_b) {
            bs[u].v[0] = *reinterpret_cast<const SBt *>(qb + off);
          } else {
            if (end_b) {
              back_b[u] = box_back(off, box_room(p.end[1], pb, V * (int)sizeof(SBt)), LB);
              off -= back_b[u] << LB;
            }
            load_pack_any<SBt, V, ALB>(qb + off, bs[u]);
          }
        }
      }
    }
  };
  fetch(0);

  if constexpr (STA || (BIN && STB)) {
    // Staged inputs: all loads of U passes are issued before any vector is parked.
    {
      BoxInput xa, xb;
      uint32_t na = 0, nb = 0;
      BoxLane la{}, lb{};
      if constexpr (STA) {
        box_input(p.in[0], xa);
        na = p.in[0].niter;
        la = box_lane(xa, tid);
      }
      if constexpr (BIN && STB) {
        box_input(p.in[1], xb);
        nb = p.in[1].niter;
        lb = box_lane(xb, tid);
      }
      const uint32_t nmax = na > nb ? na : nb;
      for (uint32_t j = 0; j < nmax; j += U) {
        Pack<SAt, VA> va[U];
        Pack<SBt, VB> vb[U];
        uint32_t wa[U], wb[U], da[U], db[U];   // LDS addresses (all ones: no such vector)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          wa[u] = wb[u] = ~0u;
          da[u] = db[u] = 0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if constexpr (STA) {
            if (j + u < na) {
              bool is = la.t < xa.nvec;
              if (clipped) is = is & box_exists(p.in[0], lims, la);
              wa[u] = is ? la.lds : ~0u;
              uint32_t off = is ? la.off : kBoxSlack;
              if (end_a) {
                da[u] = box_back(off, box_room(p.end[0], pa, 16), LA);
                off -= da[u] << LA;
              }
              load_pack_any<SAt, VA, ALA>(qa + off, va[u]);
              box_advance(xa, block, la);
            }
          }
          if constexpr (BIN && STB) {
            if (j + u < nb) {
              bool is = lb.t < xb.nvec;
              if (clipped) is = is & box_exists(p.in[1], lims, lb);
              wb[u] = is ? lb.lds : ~0u;
              uint32_t off = is ? lb.off : kBoxSlack;
              if (end_b) {
                db[u] = box_back(off, box_room(p.end[1], pb, 16), LB);
                off -= db[u] << LB;
              }
              load_pack_any<SBt, VB, ALB>(qb + off, vb[u]);
              box_advance(xb, block, lb);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if constexpr (STA) {
            if (j + u < na) {
              if (end_a) any_shift<SAt, VA>(va[u], (int)da[u]);
              if (wa[u] != ~0u) *reinterpret_cast<Pack<SAt, VA> *>(lds + wa[u]) = va[u];
            }
          }
          if constexpr (BIN && STB) {
            if (j + u < nb) {
              if (end_b) any_shift<SBt, VB>(vb[u], (int)db[u]);
              if (wb[u] != ~0u) *reinterpret_cast<Pack<SBt, VB> *>(lds + wb[u]) = vb[u];
            }
          }
        }
        // (vmcnt(0): parked under conditions, the loads count as outstanding in the next trip, and each
        // load there would wait for the one before it)
        __builtin_amdgcn_s_waitcnt(0x0f70);
      }
    }
    __syncthreads();
  }

  // compute phase, in the output's order
  const int swap = p.swap;
  const bool nt = p.nt_store != 0;
  auto compute = [&](auto runs, int u) {
    constexpr bool RUNS = decltype(runs)::value;   // runs go along several dims
    const BoxVec &v = vs[u];
    const int n = ns[u];
    Pack<SAt, V> av = as[u];
    Pack<SBt, V> bv = bs[u];
    if constexpr (!STA) {
      if (end_a) any_shift<SAt, V>(av, (int)back_a[u]);
      if (one_a) {
#pragma unroll
        for (int i = 1; i < V; ++i) av.v[i] = av.v[0];
      }
    }
    if constexpr (BIN && !STB) {
      if (end_b) any_shift<SBt, V>(bv, (int)back_b[u]);
      if (one_b) {
#pragma unroll
        for (int i = 1; i < V; ++i) bv.v[i] = bv.v[0];
      }
    }
    if (n <= 0) return;
    uint32_t pos[2] = {v.pos[0], v.pos[1]};
    BoxRun run;
    if constexpr (RUNS) run = box_run<V>(o, v, pos);
#pragma unroll
    for (int i = 0; i < V; ++i) {   // (elements that do not exist are read from where the last one lies)
      if constexpr (STA) av.v[i] = *reinterpret_cast<const SAt *>(lds + pos[0]);
      if constexpr (BIN && STB) bv.v[i] = *reinterpret_cast<const SBt *>(lds + pos[1]);
      if (i + 1 < V) {
        uint32_t next[2] = {pos[0], pos[1]};
        if constexpr (RUNS) {
          box_next<V>(o, run, next);
        } else {
          next[0] += o.run[0] / V;
          next[1] += o.run[1] / V;
        }
        pos[0] = i + 1 < n ? next[0] : pos[0];
        pos[1] = i + 1 < n ? next[1] : pos[1];
      }
    }
    Pack<SOt, V> r;
    if (swap) G::order_inputs(swap, av, bv);
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if constexpr (BIN) r.v[i] = G::eval(av.v[i], bv.v[i]);
      else r.v[i] = G::eval(av.v[i], SBt{});
    }
    if (swap) G::order_output(swap, r);
    char *po = out + v.off;
    if (n == V) {
      store_pack_any<SOt, V, ALO>(po, r, nt);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < n) reinterpret_cast<SOt *>(po)[i] = r.v[i];
    }
  };
  auto passes = [&](auto runs) {
    for (uint32_t j = 0;;) {
#pragma unroll
      for (int u = 0; u < PU; ++u)
        if (j + u < niter) compute(runs, u);
      if ((j += PU) >= niter) break;  // uniform
      fetch(j);
    }
  };
  if (p.o.nrun > 1) passes(std::true_type{});
  else passes(std::false_type{});
}

template <class G> __global__ __launch_bounds__(kBlock) void ew_box_kernel(const BoxArgs by_value) {
  constexpr bool BIN = G::NIN2;
  (void)by_value;  // read through the kernarg segment instead (it is the only argument)
  KBoxArgs &p = *(KBoxArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  char *lds = reinterpret_cast<char *>(ocn_lds_raw);
  if (p.warm) warm_arguments<BoxArgs>();
  int64_t base[3];
  const uint64_t lims = box_origin(p, box_number(p, blockIdx.x), base);
  char *out = p.out + base[0];
  const char *pa = p.a + base[1];
  const char *pb = BIN ? p.b + base[2] : nullptr;
  const bool in_a = p.in[0].how == kBoxInPlace;
  if constexpr (BIN) {
    if (p.in[1].how == kBoxInPlace) box_body<G, true, false>(p, lds, lims, out, pa, pb);
    else if (in_a) box_body<G, false, true>(p, lds, lims, out, pa, pb);
    else box_body<G, true, true>(p, lds, lims, out, pa, pb);
  } else {
    box_body<G, true, true>(p, lds, lims, out, pa, pb);
  }
}

#endif  // __HIPCC__

}  // namespace ocn
