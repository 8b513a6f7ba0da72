// Reduction kernels of the tensor engine for gfx950 (section 3.2 of the paper: tensor
// reductions along one or more axes).
//
//   red_rows_kernel     lanes share an output: a power-of-two group of 1 to 64 lanes (short
//                       rows: a wavefront then covers several outputs) or a whole workgroup
//                       (long rows) streams one output's addends, with 128-bit loads when the
//                       reduced axis is the input's fastest; lanes fold privately, then a
//                       shuffle tree and an LDS step combine them.  Long reductions with few outputs are split over
//                       several workgroups; each writes a partial result to the workspace and a
//                       second launch folds the partials (two-pass grid reduction).
//   red_rows_short_kernel  the same for rows of at most one vector per lane, without loops
//   red_cols_kernel     a kept axis is the input's fastest: lanes own adjacent output columns
//                       (with few columns a wavefront covers several rows at a time), the
//                       wavefronts of a workgroup take interleaved rows and are combined
//                       through LDS; row ranges can be split the same way.
//   red_cols_bits_kernel  the same for any and all of bytes, sixteen columns of a lane in four registers
//   red_generic_kernel  any layout and 64-bit extents: one output per lane, sequential fold.
// No floating-point atomics anywhere: the grouping of addends is fixed by the launch
// geometry, so results are reproducible bit for bit.
#pragma once

#include <type_traits>

#include "dev_types.hpp"
#include "planner.hpp"

namespace ocn {

struct RedArgs {
  const char *a;
  char *out;                        // final output (used when split == 1)
  char *partial;                    // workspace (used when split > 1)
  int32_t warm;                     // few workgroups: touch all argument lines first
  int32_t nkept, nred, out_dtype, vec, group;
  int64_t ksa[kMaxDims], kso[kMaxDims];    // kept dims: input / output byte strides, fastest first
  FastDiv kdiv[kMaxDims];                  // kept sizes, same order
  int64_t rsa[kMaxDims];                   // reduced dims: input byte strides, fastest first
  FastDiv rdiv[kMaxDims];                  // reduced sizes, same order
  int64_t ksize[kMaxDims], rsize[kMaxDims];// the same sizes in 64 bits (generic kernel)
  int64_t nout, nredtot;
  int64_t n0;                              // length of the fastest reduced dim (rows)
  FastDiv vpr_div;                         // rows: vectors per innermost run
  int64_t nvec;                            // rows: vectors per output
  int64_t split, chunk;
  int64_t nc;                              // cols: number of columns (fastest kept dim)
  FastDiv colblocks_div;                   // cols: column blocks per row of outputs
  // second input of a fused elementwise+reduce kernel (unused by the plain kernels)
  const char *b;
  int64_t ksb[kMaxDims], rsb[kMaxDims];    // its byte strides, same order as ksa / rsa
  int32_t a_bcast, b_bcast;                // broadcast along the vectorised dim
  int32_t cpw;                             // cols: lanes per row of columns (power of two <= 64; any number with cpw_m)
  uint32_t cpw_m;                          // cols: lanes numbered through whole rows: ceil(2^32 / cpw); else zero
  int32_t nt_load;                         // vector loads carry the streaming (non-temporal) hint
  int32_t swap_a, swap_o;                  // the input / the output is stored in the other byte order
};

// arguments of the kernel that folds [split][output] partial results
struct RedFoldArgs {
  const char *partial;
  char *out;
  int64_t kso;             // byte stride of the (one) kept dim in the output
  uint32_t nout, split;
  int32_t out_dtype, swap_o;
};

// arguments of the lean rows kernel: one reduced dim read in whole 16-byte vectors, at most one
// kept dim, everything below 2^31
struct RedLeanArgs {
  const char *a;
  const char *b;           // second input of a fused elementwise+reduce call
  char *out, *partial;
  int64_t ksa, kso;        // byte strides of the kept dim in the input and the output
  int64_t ksb;             // ... in the second input
  uint32_t nout, split;    // outputs; partial results per output
  uint32_t nvec, chunk;    // whole vectors per output; vectors per split
  int32_t out_dtype, group, nt_load;
  int32_t swap_a, swap_o;  // the input / the output is stored in the other byte order
  uint32_t tail;           // elements of an output behind its last whole vector
};

#if defined(__HIPCC__)

OCN_DEV uint32_t rfastdiv(uint32_t n, const FastDiv &f) { return (__umulhi(n, f.m) + n) >> f.s; }

// The general kernels read their arguments where they lie, in the constant address space, and loop
// over the dims there are.  Passed by value and unrolled over eight dims, the arguments of all of
// them were fetched ahead into scalar registers and spilled (160 to 200 of them).
using KRedArgs = const __attribute__((address_space(4))) RedArgs;
OCN_DEV FastDiv args_div(const __attribute__((address_space(4))) FastDiv &f) { return FastDiv{f.d, f.m, f.s}; }

// ---------------------------------------------------------------------------------------
// accumulators
// ---------------------------------------------------------------------------------------

constexpr int red_acc_dtype(int op, int dt) {
  const int k = dt_kind(dt);
  if (op == R_SUM || op == R_PROD) {
    if (k == K_BOOL || k == K_SINT) return DT_I64;
    if (k == K_UINT) return DT_U64;
    if (dt == DT_F16) return DT_F32;
    if (dt == DT_F32 || dt == DT_F64) return DT_F64;
    return dt == DT_C16 ? DT_C32 : DT_C64;
  }
  if (op == R_MIN || op == R_MAX) return dt;
  return DT_BOOL;
}
constexpr bool red_supported(int op, int dt) {
  return op == R_SUM || op == R_ANY || op == R_ALL || dt_kind(dt) != K_CPLX;
}

template <int S, int OP> struct Reducer {
  static constexpr int ACC = red_acc_dtype(OP, S);
  using A = reg_t<ACC>;     // accumulator register type
  using P = storage_t<ACC>; // how a partial result is stored

  OCN_DEV static A identity() {
    constexpr int k = dt_kind(ACC);
    if constexpr (OP == R_SUM) {
      if constexpr (k == K_CPLX) return A{0, 0};
      else return (A)0;
    } else if constexpr (OP == R_PROD) {
      return (A)1;
    } else if constexpr (OP == R_ANY) {
      return false;
    } else if constexpr (OP == R_ALL) {
      return true;
    } else {  // min / max start from the far end of the type's range
      constexpr bool mx = OP == R_MAX;
      if constexpr (k == K_BOOL) return !mx;
      else if constexpr (ACC == DT_F16) return hreg{mx ? -__builtin_inff() : __builtin_inff()};
      else if constexpr (ACC == DT_F32) return mx ? -__builtin_inff() : __builtin_inff();
      else if constexpr (ACC == DT_F64) return mx ? -__builtin_inf() : __builtin_inf();
      else return mx ? std::numeric_limits<A>::min() : std::numeric_limits<A>::max();
    }
  }

  OCN_DEV static A lift(reg_t<S> x) {
    if constexpr (OP == R_SUM || OP == R_PROD) return convert<ACC>(x);  // exact widening
    else if constexpr (OP == R_MIN || OP == R_MAX) return x;
    else return convert<DT_BOOL>(x);
  }

  OCN_DEV static A combine(A x, A y) {
    constexpr int k = dt_kind(ACC);
    if constexpr (OP == R_SUM) {
      if constexpr (k == K_CPLX) return A{x.re + y.re, x.im + y.im};
      else if constexpr (k == K_SINT) return (A)((uint64_t)x + (uint64_t)y);
      else return x + y;
    } else if constexpr (OP == R_PROD) {
      if constexpr (k == K_SINT) return (A)((uint64_t)x * (uint64_t)y);
      else return x * y;
    } else if constexpr (OP == R_ANY) {
      return x || y;
    } else if constexpr (OP == R_ALL) {
      return x && y;
    } else {
      constexpr bool mx = OP == R_MAX;
      if constexpr (k == K_BOOL) return mx ? (x || y) : (x && y);
      else if constexpr (ACC == DT_F16) return hreg{mx ? nan_max(x.v, y.v) : nan_min(x.v, y.v)};
      else if constexpr (k == K_REAL) return mx ? nan_max(x, y) : nan_min(x, y);
      else return mx ? (x > y ? x : y) : (x < y ? x : y);
    }
  }
};

// ---------------------------------------------------------------------------------------
// cross-lane movement of an accumulator of any size (32-bit pieces through the shuffle unit)
// ---------------------------------------------------------------------------------------

template <class A> OCN_DEV A shfl_down_any(A v, int delta) {
  constexpr int W = (sizeof(A) + 3) / 4;
  union { A a; uint32_t w[W]; } u, r;
#pragma unroll
  for (int i = 0; i < W; ++i) u.w[i] = 0;
  u.a = v;
#pragma unroll
  for (int i = 0; i < W; ++i) r.w[i] = (uint32_t)__shfl_down((int)u.w[i], delta, kWave);
  return r.a;
}

// after this, lane 0 of the wavefront holds the fold of all 64 lanes
template <class R> OCN_DEV typename R::A wave_fold(typename R::A v) {
#pragma unroll
  for (int d = kWave / 2; d >= 1; d >>= 1) v = R::combine(v, shfl_down_any(v, d));
  return v;
}

// lane i receives lane i + N of its row of 16 lanes (data-parallel primitive "row shift left";
// lanes past the end of the row read zero)
template <int N, class A> OCN_DEV A row_down_any(A v) {
  constexpr int W = (sizeof(A) + 3) / 4;
  union { A a; uint32_t w[W]; } u, r;
#pragma unroll
  for (int i = 0; i < W; ++i) u.w[i] = 0;
  u.a = v;
#pragma unroll
  for (int i = 0; i < W; ++i) r.w[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)u.w[i], 0x100 + N, 0xf, 0xf, true);
  return r.a;
}

// the same over aligned groups of `width` lanes (a power of two, the same for the whole
// wavefront): the first lane of every group ends up with its group's fold.  Steps that stay
// inside a row of 16 lanes use the row shift, which costs one instruction per 32-bit word.
template <class R> OCN_DEV typename R::A group_fold(typename R::A v, int width) {
  if (width > 32) v = R::combine(v, shfl_down_any(v, 32));
  if (width > 16) v = R::combine(v, shfl_down_any(v, 16));
  if (width > 8) v = R::combine(v, row_down_any<8>(v));
  if (width > 4) v = R::combine(v, row_down_any<4>(v));
  if (width > 2) v = R::combine(v, row_down_any<2>(v));
  if (width > 1) v = R::combine(v, row_down_any<1>(v));
  return v;
}

// convert an accumulator to the runtime output dtype and store it (once per output)
template <class A> __device__ __noinline__ void store_result(char *p, int dt, A r, bool swapped = false) {
  switch (dt) {
#define OCN_CASE(D)                                      \
  case D: {                                              \
    storage_t<D> s = to_storage<D>(convert<D>(r));       \
    if (swapped) reverse_scalars<scalar_bytes(D)>(s);    \
    *reinterpret_cast<storage_t<D> *>(p) = s;            \
  } break;
    OCN_CASE(DT_BOOL) OCN_CASE(DT_I8) OCN_CASE(DT_I16) OCN_CASE(DT_I32) OCN_CASE(DT_I64)
    OCN_CASE(DT_U8) OCN_CASE(DT_U16) OCN_CASE(DT_U32) OCN_CASE(DT_U64)
    OCN_CASE(DT_F16) OCN_CASE(DT_F32) OCN_CASE(DT_F64)
    OCN_CASE(DT_C16) OCN_CASE(DT_C32) OCN_CASE(DT_C64)
#undef OCN_CASE
    default: break;
  }
}

// byte offsets of output number `o` (linear over the kept dims) in the input and the output
OCN_DEV void kept_offsets(KRedArgs &p, uint32_t o, int64_t &off_a, int64_t &off_o) {
  off_a = 0;
  off_o = 0;
  const int nkept = p.nkept;
  for (int k = 0; k < nkept; ++k) {
    const uint32_t q = (k == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[k]));
    const uint32_t i = o - q * p.kdiv[k].d;
    o = q;
    off_a += (int64_t)i * p.ksa[k];
    off_o += (int64_t)i * p.kso[k];
  }
}

// input byte offset of reduced index q over the reduced dims from `first` upward
OCN_DEV int64_t reduced_offset(KRedArgs &p, uint32_t q, int first) {
  int64_t off = 0;
  const int nred = p.nred;
  for (int k = first; k < nred; ++k) {
    const uint32_t qq = (k == nred - 1) ? 0u : rfastdiv(q, args_div(p.rdiv[k]));
    const uint32_t i = q - qq * p.rdiv[k].d;
    q = qq;
    off += (int64_t)i * p.rsa[k];
  }
  return off;
}

// ---------------------------------------------------------------------------------------
// rows
// ---------------------------------------------------------------------------------------

// Any and all (of bools also their maximum and minimum) over one-byte elements, four to a register: what is
// not zero is or-ed as it is, what is zero is found through the carry into a byte's highest bit.
template <int S, int OP> struct BitFold {
  static constexpr bool kAny = OP == R_ANY || OP == R_MAX;
  static constexpr uint32_t kStart = kAny ? 0u : 0x80808080u;
  static constexpr uint32_t kNeutral = kAny ? 0u : 0x01010101u;   // elements that change nothing
  OCN_DEV static uint32_t add(uint32_t acc, uint32_t w) {
    if constexpr (kAny) return acc | w;
    else return acc & (((w & 0x7f7f7f7fu) + 0x7f7f7f7fu) | w);
  }
  OCN_DEV static uint32_t combine(uint32_t x, uint32_t y) { return kAny ? x | y : x & y; }
  OCN_DEV static bool result(uint32_t acc, int byte) { return kAny ? ((acc >> (8 * byte)) & 0xffu) != 0 : ((acc >> (8 * byte + 7)) & 1u) != 0; }
  OCN_DEV static bool whole(uint32_t acc) { return kAny ? acc != 0 : (acc & 0x80808080u) == 0x80808080u; }
};

// A lane's running fold over whole vectors of V consecutive elements.  The generic form
// folds element by element; two specialisations use packed instructions:
//   * sums of 8-bit integers add four bytes per instruction (dot product with ones) into a
//     32-bit register that is flushed into the 64-bit total long before it can overflow;
//   * min/max of half-precision values compares order-preserving 16-bit integer keys two at
//     a time and tracks NaNs on the side, which keeps the NaN-propagating, +0-above--0
//     semantics exact without any floating-point comparison.
template <int S, int OP, int V, class Enable = void> struct VecFold {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  struct alignas(sizeof(St) * V >= 16 ? 16 : sizeof(St) * V) Pk { St v[V]; };
  A acc;
  OCN_DEV void init() { acc = R::identity(); }
  OCN_DEV void add_full(const Pk &pk) {
#pragma unroll
    for (int i = 0; i < V; ++i) acc = R::combine(acc, R::lift(from_storage<S>(pk.v[i])));
  }
  OCN_DEV void add_partial(const Pk &pk, int n) {
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i < n) acc = R::combine(acc, R::lift(from_storage<S>(pk.v[i])));
  }
  // elements first .. V - 1
  OCN_DEV void add_from(const Pk &pk, int first) {
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i >= first) acc = R::combine(acc, R::lift(from_storage<S>(pk.v[i])));
  }
  OCN_DEV A result() { return acc; }
};

// sum of int8 / uint8, sixteen per vector
template <int S, int V>
struct VecFold<S, R_SUM, V, std::enable_if_t<(S == DT_I8 || S == DT_U8) && V == 16>> {
  using R = Reducer<S, R_SUM>;
  using A = typename R::A;  // int64_t or uint64_t
  using St = storage_t<S>;
  struct alignas(16) Pk { St v[V]; };
  A total;
  int32_t part;      // at most 2^11 per add_full in magnitude
  uint32_t pending;  // add_full calls since the last flush
  OCN_DEV void init() { total = 0; part = 0; pending = 0; }
  OCN_DEV void flush() {
    if constexpr (S == DT_I8) total += (A)part;
    else total += (A)(uint32_t)part;
    part = 0;
    pending = 0;
  }
  OCN_DEV void add_full(const Pk &pk) {
    const int32_t *w = reinterpret_cast<const int32_t *>(&pk);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if constexpr (S == DT_I8) part = __builtin_amdgcn_sdot4(w[k], 0x01010101, part, false);
      else part = (int32_t)__builtin_amdgcn_udot4((uint32_t)w[k], 0x01010101u, (uint32_t)part, false);
    }
    if (++pending == (1u << 19)) flush();  // 2^19 * 2^11 < 2^31 (uint8: 2^19 * 4080 < 2^32)
  }
  OCN_DEV void add_partial(const Pk &pk, int n) {
#pragma unroll
    for (int i = 0; i < V; ++i)
      if (i < n) total += (A)pk.v[i];
  }
  OCN_DEV void add_from(const Pk &pk, int first) {   // (the bytes before the first cleared: zeros add nothing)
    Pk q;
    const uint32_t *w = reinterpret_cast<const uint32_t *>(&pk);
    uint32_t *m = reinterpret_cast<uint32_t *>(&q);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int c = first - 4 * k;
      m[k] = c >= 4 ? 0u : w[k] & (c > 0 ? ~0u << (8 * c) : ~0u);
    }
    add_full(q);
  }
  OCN_DEV A result() { flush(); return total; }
};

// min / max of half precision, eight per vector: the packed IEEE 754-2019 maximum / minimum of
// gfx950 (NaN-propagating, +0 above -0) folds two elements per instruction
template <int OP, int V>
struct VecFold<DT_F16, OP, V, std::enable_if_t<(OP == R_MIN || OP == R_MAX) && V == 8>> {
  using R = Reducer<DT_F16, OP>;
  using A = typename R::A;  // hreg
  using St = storage_t<DT_F16>;
  struct alignas(16) Pk { St v[V]; };
  using h2 = _Float16 __attribute__((ext_vector_type(2)));
  static constexpr bool MX = OP == R_MAX;
  h2 best;
  OCN_DEV void init() {
    const _Float16 start = MX ? (_Float16)-__builtin_inff() : (_Float16)__builtin_inff();
    best = h2{start, start};
  }
  OCN_DEV void add_word(uint32_t w) {
    const h2 x = __builtin_bit_cast(h2, w);
    best = MX ? __builtin_elementwise_maximum(best, x) : __builtin_elementwise_minimum(best, x);
  }
  OCN_DEV void add_full(const Pk &pk) {
    const uint32_t *w = reinterpret_cast<const uint32_t *>(&pk);
#pragma unroll
    for (int k = 0; k < 4; ++k) add_word(w[k]);
  }
  OCN_DEV void add_partial(const Pk &pk, int n) {
    // pad the missing slots by repeating the first element (n >= 1 here).  The bits are taken
    // element by element from the values that were stored (no access through another type: the
    // elements were written as halves, and only the first n of them).
    uint32_t h[V];
#pragma unroll
    for (int i = 0; i < V; ++i) h[i] = __builtin_bit_cast(uint16_t, pk.v[i < n ? i : 0]);
#pragma unroll
    for (int k = 0; k < 4; ++k) add_word(h[2 * k] | (h[2 * k + 1] << 16));
  }
  OCN_DEV void add_from(const Pk &pk, int) { add_full(pk); }   // (an element seen twice changes nothing)
  OCN_DEV A result() {
    const _Float16 r = MX ? __builtin_elementwise_maximum(best.x, best.y) : __builtin_elementwise_minimum(best.x, best.y);
    return hreg{(float)r};
  }
};

// NT: the load carries the streaming (non-temporal) hint.  An input far larger than the caches
// is read once and never again; read this way a wavefront's whole-line requests stream about
// 7 % faster from HBM (fp32 row sums over 256 MiB: 43.9 -> 40.4 us).  Only for 16-byte pieces
// that neighbouring lanes read side by side: with partial lines the hint costs time.
// A pack whose tensor is stored in the other byte order is put right as soon as it is loaded.
template <int S, class Pk> OCN_DEV void order_pack(bool swapped, Pk &pk) {
  if constexpr (scalar_bytes(S) > 1) {
    if (swapped) reverse_scalars<scalar_bytes(S)>(pk);
  }
}
template <int S> OCN_DEV storage_t<S> load_one(bool swapped, const char *src) {
  storage_t<S> v = *reinterpret_cast<const storage_t<S> *>(src);
  order_pack<S>(swapped, v);
  return v;
}

// (four-byte elements are scalars except for complex halves)
template <class St> constexpr int vec_scalar() { return std::is_same<St, chalf_s>::value ? 2 : 4; }
// at any address that is a multiple of the scalar size (of four bytes for wider scalars)
template <class St, int V, bool NT = false, class Pk> OCN_DEV void load_vec(const char *src, Pk &pk) {
  if constexpr (sizeof(St) * V >= 16) {
    using Q = typename Unaligned<(sizeof(St) < 4 ? (int)alignof(St) < 2 ? 1 : 2 : sizeof(St) == 4 ? (int)vec_scalar<St>() : 4)>::W4;
    Q w[sizeof(St) * V / 16];
#pragma unroll
    for (int i = 0; i < (int)(sizeof(St) * V / 16); ++i) {
      if constexpr (NT) w[i] = __builtin_nontemporal_load(reinterpret_cast<const Q *>(src) + i);
      else w[i] = reinterpret_cast<const Q *>(src)[i];
    }
    __builtin_memcpy(&pk, w, sizeof(St) * V);
  } else {
#pragma unroll
    for (int i = 0; i < V; ++i) pk.v[i] = reinterpret_cast<const St *>(src)[i];
  }
}

// Fold vectors t0 .. t1-1 of one output's addends, `lanes` lanes cooperating.  The bulk runs
// in a loop without any per-lane condition (every lane loads U whole vectors per trip); the
// ragged remainder - the last few vectors, and the partial vector at the end of a run whose
// length is not a multiple of V - goes through a checked loop.
template <int S, int OP, int V, bool SINGLE, bool NT>
OCN_DEV typename Reducer<S, OP>::A rows_accumulate_impl(KRedArgs &p, const char *base, int64_t t0,
                                                        int64_t t1, int lane, int lanes) {
  using R = Reducer<S, OP>;
  using St = storage_t<S>;
  using F = VecFold<S, OP, V>;
  using Pk = typename F::Pk;
  constexpr int U = 4;  // independent folds and loads in flight per lane
  auto address = [&](int64_t tt, int64_t &e0) -> const char * {
    int64_t off = 0, iv = tt;
    if constexpr (!SINGLE) {
      const uint32_t q = rfastdiv((uint32_t)tt, args_div(p.vpr_div));
      iv = (uint32_t)tt - q * p.vpr_div.d;
      off = reduced_offset(p, q, 1);
    }
    e0 = iv * V;
    // single elements may be strided along the innermost reduced dim, vectors are contiguous
    return base + off + e0 * (V == 1 ? p.rsa[0] : (int64_t)sizeof(St));
  };
  if (t1 - t0 <= lanes) {  // short rows: at most one vector per lane, no loops
    F one;
    one.init();
    const int64_t tt = t0 + lane;
    if (tt < t1) {
      Pk pk;
      int64_t e0;
      const char *src = address(tt, e0);
      const int64_t left = p.n0 - e0;
      if (left >= V) {
        load_vec<St, V, NT>(src, pk);
        order_pack<S>(p.swap_a != 0, pk); one.add_full(pk);
      } else {
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (i < (int)left) pk.v[i] = reinterpret_cast<const St *>(src)[i];
        order_pack<S>(p.swap_a != 0, pk); one.add_partial(pk, (int)left);
      }
    }
    return one.result();
  }
  F fold[U];
#pragma unroll
  for (int u = 0; u < U; ++u) fold[u].init();
  // vectors below t_full are known to be whole
  int64_t t_full = t0;
  if constexpr (SINGLE) {
    t_full = p.n0 / V;
    if (t_full > t1) t_full = t1;
  } else if (p.n0 % V == 0) {
    t_full = t1;
  }
  int64_t t = t0;
  // (The loops stay as they are written: with single elements the compiler would make four trips
  // one, sixteen loads each waited for by itself, and over 64 registers for all of the kernel.
  // any over 16.8 M int16 [65536, 7, 3, 40], two reduced dims: 328 us and 154 spilled registers
  // vectorised, 63 as written; maxima of every other int8 of 16.8 M: 33 and 17.5.)
#pragma clang loop vectorize(disable) interleave(disable)
  for (; t + (int64_t)lanes * U <= t_full; t += (int64_t)lanes * U) {
    Pk pk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int64_t e0;
      load_vec<St, V, NT>(address(t + (int64_t)u * lanes + lane, e0), pk[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      order_pack<S>(p.swap_a != 0, pk[u]);
      fold[u].add_full(pk[u]);
    }
  }
#pragma clang loop vectorize(disable) interleave(disable)
  for (; t + lanes <= t_full; t += lanes) {  // whole vectors, one per lane and trip
    Pk pk;
    int64_t e0;
    load_vec<St, V, NT>(address(t + lane, e0), pk);
    order_pack<S>(p.swap_a != 0, pk); fold[0].add_full(pk);
  }
  if constexpr (!SINGLE && V > 1) {
    // Rows that end inside a vector, several reduced dims: a row's last vector is read so that it ends
    // with the row, and the elements that the one before it had are left out (maxima and the like may
    // see them twice).  Every load is a whole vector, and a lane has four in flight; one by one in
    // the loop below int8 [1234, 91] rows 92 apart took 28 us, 8.7 here with more splits.
    constexpr bool TWICE = OP == R_MIN || OP == R_MAX || OP == R_ANY || OP == R_ALL;
    if (p.n0 >= V) {
#pragma clang loop vectorize(disable) interleave(disable)
      for (; t + (int64_t)lanes * U <= t1; t += (int64_t)lanes * U) {
        Pk pk[U];
        int cut[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          int64_t e0;
          const char *src = address(t + (int64_t)u * lanes + lane, e0);
          const int64_t left = p.n0 - e0;
          cut[u] = left < V ? V - (int)left : 0;
          load_vec<St, V, NT>(src - cut[u] * (int)sizeof(St), pk[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          order_pack<S>(p.swap_a != 0, pk[u]);
          if (TWICE || cut[u] == 0) fold[u].add_full(pk[u]);
          else fold[u].add_from(pk[u], cut[u]);
        }
      }
    }
  }
#pragma clang loop vectorize(disable) interleave(disable)
  for (int64_t tt = t + lane; tt < t1; tt += lanes) {
    Pk pk;
    int64_t e0;
    const char *src = address(tt, e0);
    const int64_t left = p.n0 - e0;
    if (left >= V) {
      load_vec<St, V, NT>(src, pk);
      order_pack<S>(p.swap_a != 0, pk); fold[0].add_full(pk);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < (int)left) pk.v[i] = reinterpret_cast<const St *>(src)[i];
      order_pack<S>(p.swap_a != 0, pk); fold[0].add_partial(pk, (int)left);
    }
  }
  typename R::A acc = fold[0].result();
#pragma unroll
  for (int u = 1; u < U; ++u) acc = R::combine(acc, fold[u].result());
  return acc;
}

// Fold vectors t0 .. t1-1 of one output's addends, `lanes` lanes cooperating.  The bulk runs
// in a loop without any per-lane condition (every lane loads U whole vectors per trip); the
// ragged remainder - the last few vectors, and the partial vector at the end of a run whose
// length is not a multiple of V - goes through a checked loop.  A single reduced dimension
// (the common case) needs no index decomposition at all.
template <int S, int OP, int V>
OCN_DEV typename Reducer<S, OP>::A rows_accumulate(KRedArgs &p, const char *base, int64_t t0, int64_t t1,
                                                   int lane, int lanes) {
  if (p.nred == 1) {
    if (V > 1 && p.nt_load) return rows_accumulate_impl<S, OP, V, true, (V > 1)>(p, base, t0, t1, lane, lanes);
    return rows_accumulate_impl<S, OP, V, true, false>(p, base, t0, t1, lane, lanes);
  }
  return rows_accumulate_impl<S, OP, V, false, false>(p, base, t0, t1, lane, lanes);
}

// Eight wavefronts per SIMD (at most 64 vector registers): 16384 one-wavefront rows then fill
// the chip in exactly two rounds instead of two and two thirds.
#ifndef OCN_ROWS_OCC
#define OCN_ROWS_OCC __attribute__((amdgpu_waves_per_eu(8, 8)))
#endif
template <int S, int OP> __global__ __launch_bounds__(kBlock) OCN_ROWS_OCC void red_rows_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using R = Reducer<S, OP>;
  using A = typename R::A;
  constexpr int VF = 16 / (int)sizeof(storage_t<S>) > 0 ? 16 / (int)sizeof(storage_t<S>) : 1;
  __shared__ A lds[kBlock / kWave];

  const int tid = threadIdx.x;
  const int lane_in_wave = tid & (kWave - 1);
  const int wave = tid / kWave;
  // p.group lanes share one output: a whole workgroup, or a power of two up to a wavefront
  const bool per_block = p.group == kBlock;
  const int width = per_block ? kWave : p.group;
  const int64_t gidx = per_block ? (int64_t)blockIdx.x : ((int64_t)blockIdx.x * kBlock + tid) >> (__ffs(width) - 1);
  const int64_t ngroups = p.nout * p.split;
  const bool active = gidx < ngroups;
  const int lane = per_block ? tid : (lane_in_wave & (width - 1));
  A acc = R::identity();
  int64_t o = 0, s = 0, off_o = 0;
  if (active) {
    int64_t t0 = 0, t1 = p.nvec;
    o = gidx;
    if (p.split != 1) {
      o = gidx / p.split;
      s = gidx - o * p.split;
      t0 = s * p.chunk;
      t1 = t0 + p.chunk;
      if (t1 > p.nvec) t1 = p.nvec;
    }
    int64_t off_a;
    kept_offsets(p, (uint32_t)o, off_a, off_o);
    const int lanes = per_block ? kBlock : width;
    if (p.vec > 1) acc = rows_accumulate<S, OP, VF>(p, p.a + off_a, t0, t1, lane, lanes);
    else acc = rows_accumulate<S, OP, 1>(p, p.a + off_a, t0, t1, lane, lanes);
  }
  acc = group_fold<R>(acc, width);   // every lane takes part, whether its group has work or not
  if (per_block) {  // combine the four wavefronts of the workgroup
    if (lane_in_wave == 0) lds[wave] = acc;
    __syncthreads();
    if (tid == 0) {
#pragma unroll
      for (int w = 1; w < kBlock / kWave; ++w) acc = R::combine(acc, lds[w]);
    }
  }
  if (active && lane == 0) {
    if (p.split == 1) {
      store_result<A>(p.out + off_o, p.out_dtype, acc, p.swap_o != 0);
    } else {
      reinterpret_cast<typename R::P *>(p.partial)[o * p.split + s] = to_storage<R::ACC>(acc);
    }
  }
}

// The common row reduction - one reduced dim, contiguous and read in whole 16-byte vectors, at
// most one kept dim, a wavefront or a workgroup per output (or per split of it) - without the
// index decomposition and the 64-bit bookkeeping of the general kernel.  A wavefront lives for
// only a few loop trips on rows of some KiB, so what it executes before its first load and
// after its last one is time during which it has nothing in flight (half-precision maxima
// over rows of 8 KiB: 24.6 us in the general kernel).  Same fold order as the general kernel.
// (SW, the input's byte order, is a template parameter like NT: decided per vector inside the
// loop, the reversal is computed for every vector and selected away - a quarter of the loop's
// instructions for half-precision maxima)
template <int S, int OP, bool NT, bool SW>
OCN_DEV typename Reducer<S, OP>::A lean_fold(const char *base, uint32_t t0, uint32_t t1, uint32_t lane, uint32_t lanes) {
  constexpr bool sw = SW;
  using R = Reducer<S, OP>;
  using St = storage_t<S>;
  constexpr int V = 16 / (int)sizeof(St);
  using F = VecFold<S, OP, V>;
  using Pk = typename F::Pk;
  constexpr int U = 4;
  F fold[U];
#pragma unroll
  for (int u = 0; u < U; ++u) fold[u].init();
  uint32_t t = t0 + lane;
  for (; t + (U - 1) * lanes < t1; t += U * lanes) {
    Pk pk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) load_vec<St, V, NT>(base + (uint64_t)(t + u * lanes) * 16u, pk[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      order_pack<S>(sw, pk[u]);
      fold[u].add_full(pk[u]);
    }
  }
  // two vectors at a time while they last: a row of two or three vectors per lane takes one
  // round trip less
  for (; t + lanes < t1; t += 2 * lanes) {
    Pk pk[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) load_vec<St, V, NT>(base + (uint64_t)(t + u * lanes) * 16u, pk[u]);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      order_pack<S>(sw, pk[u]);
      fold[u].add_full(pk[u]);
    }
  }
  for (; t < t1; t += lanes) {
    Pk pk;
    load_vec<St, V, NT>(base + (uint64_t)t * 16u, pk);
    order_pack<S>(sw, pk); fold[0].add_full(pk);
  }
  typename R::A acc = fold[0].result();
#pragma unroll
  for (int u = 1; u < U; ++u) acc = R::combine(acc, fold[u].result());
  return acc;
}

// Wavefronts that share an output: one, four, or sixteen where a single output is short enough that
// one workgroup takes it whole (no second launch).
constexpr int kLeanWaves = 16;
// (TAIL: outputs have elements behind their last whole vector.  A kernel of its own, so that whole
// vectors do not pay for the test: int8 full sum of 2^28 41.5 us, 41.8 with it.)
template <int S, int OP, bool TAIL> __global__ __launch_bounds__(kLeanWaves * kWave) OCN_ROWS_OCC void red_rows_lean_kernel(const RedLeanArgs q) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  if constexpr (sizeof(storage_t<S>) < 16) {
    RedLeanArgs p = q;
    OCN_ARGS_NOW("s"(p.a), "s"(p.out), "s"(p.partial), "s"(p.ksa), "s"(p.kso), "s"(p.nout), "s"(p.split), "s"(p.nvec),
                 "s"(p.chunk), "s"(p.out_dtype), "s"(p.group), "s"(p.nt_load), "s"(p.swap_a), "s"(p.swap_o));
    __shared__ A lds[kLeanWaves];
    const uint32_t tid = threadIdx.x, lane_in_wave = tid & (kWave - 1), wave = tid / kWave;
    const bool per_block = p.group > kWave;
    const uint32_t gidx = per_block ? blockIdx.x : blockIdx.x * (kBlock / kWave) + wave;
    const bool active = gidx < p.nout * p.split;
    const uint32_t lane = per_block ? tid : lane_in_wave;
    uint32_t o = gidx, sp = 0, t0 = 0, t1 = p.nvec;
    A acc = R::identity();
    // (the row's address is formed before the branch, for every wavefront: inside it, the
    // compiler fetches the pointer with a scalar load of its own, one more round trip
    // before the wavefront's first load)
    if (p.split != 1) {
      o = gidx / p.split;
      sp = gidx - o * p.split;
      t0 = sp * p.chunk;
      t1 = t0 + p.chunk < p.nvec ? t0 + p.chunk : p.nvec;
    }
    const char *base = p.a + (int64_t)o * p.ksa;
    if (active) {
      const uint32_t lanes = (uint32_t)p.group;
      if (p.swap_a) {
        if (p.nt_load) acc = lean_fold<S, OP, true, true>(base, t0, t1, lane, lanes);
        else acc = lean_fold<S, OP, false, true>(base, t0, t1, lane, lanes);
      } else {
        if (p.nt_load) acc = lean_fold<S, OP, true, false>(base, t0, t1, lane, lanes);
        else acc = lean_fold<S, OP, false, false>(base, t0, t1, lane, lanes);
      }
      // the elements behind the last whole vector: one lane of the last split
      if constexpr (TAIL) {
        if (lane == 0 && sp + 1 == p.split) {
          const char *src = base + (uint64_t)p.nvec * 16u;
#pragma clang loop vectorize(disable) interleave(disable)
          for (uint32_t i = 0; i < p.tail; ++i)
            acc = R::combine(acc, R::lift(from_storage<S>(load_one<S>(p.swap_a != 0, src + i * (uint32_t)sizeof(storage_t<S>)))));
        }
      }
    }
    acc = group_fold<R>(acc, kWave);
    if (per_block) {
      if (lane_in_wave == 0) lds[wave] = acc;
      __syncthreads();
      if (tid == 0) {
#pragma unroll
        for (int w = 1; w < kBlock / kWave; ++w) acc = R::combine(acc, lds[w]);
        for (int w = kBlock / kWave; w < p.group / kWave; ++w) acc = R::combine(acc, lds[w]);
      }
    }
    if (active && lane == 0) {
      if (p.split == 1) store_result<A>(p.out + (int64_t)o * p.kso, p.out_dtype, acc, p.swap_o != 0);
      else reinterpret_cast<typename R::P *>(p.partial)[(uint64_t)o * p.split + sp] = to_storage<R::ACC>(acc);
    }
  }
}

// Rows of at most one vector per lane of their group, a single reduced dim, no split: the
// same groups, loads and fold order as red_rows_kernel without its loops and its 64-bit
// bookkeeping (short rows are bound by instruction issue, not by memory).
template <int S, int OP, int V, bool NT>
OCN_DEV typename Reducer<S, OP>::A short_row_fold(KRedArgs &p, const char *base, uint32_t lane) {
  using St = storage_t<S>;
  using F = VecFold<S, OP, V>;
  using Pk = typename F::Pk;
  F one;
  one.init();
  if (lane < (uint32_t)p.nvec) {
    Pk pk;
    const uint32_t e0 = lane * V;
    const char *src = base + (int64_t)e0 * (V == 1 ? p.rsa[0] : (int64_t)sizeof(St));
    const uint32_t left = (uint32_t)p.n0 - e0;
    if (left >= (uint32_t)V) {
      load_vec<St, V, NT>(src, pk);
      order_pack<S>(p.swap_a != 0, pk); one.add_full(pk);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < (int)left) pk.v[i] = reinterpret_cast<const St *>(src)[i];
      order_pack<S>(p.swap_a != 0, pk); one.add_partial(pk, (int)left);
    }
  }
  return one.result();
}

template <int S, int OP> __global__ __launch_bounds__(kBlock) void red_rows_short_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using R = Reducer<S, OP>;
  using A = typename R::A;
  constexpr int VF = 16 / (int)sizeof(storage_t<S>) > 0 ? 16 / (int)sizeof(storage_t<S>) : 1;
  const uint32_t width = (uint32_t)p.group;
  const uint32_t gl = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t o = gl >> (__ffs(p.group) - 1), lane = gl & (width - 1);
  const bool active = o < (uint32_t)p.nout;
  A acc = R::identity();
  int64_t off_o = 0;
  if (active) {
    int64_t off_a;
    kept_offsets(p, o, off_a, off_o);
    if (p.vec > 1) {
      if (p.nt_load) acc = short_row_fold<S, OP, VF, (VF > 1)>(p, p.a + off_a, lane);
      else acc = short_row_fold<S, OP, VF, false>(p, p.a + off_a, lane);
    } else {
      acc = short_row_fold<S, OP, 1, false>(p, p.a + off_a, lane);
    }
  }
  acc = group_fold<R>(acc, (int)width);
  if (active && lane == 0) store_result<A>(p.out + off_o, p.out_dtype, acc, p.swap_o != 0);
}

// The second launch of a split column reduction: partial results [split][output].  The launch is a chain
// of latencies (arguments, partial results, store), so it gets few arguments and no index arithmetic (fp32
// column sums of [16384, 4096], 16 x 4096 partial results: 7.1 us in the column kernel), and four or
// sixteen wavefronts share the splits of 64 outputs, a part each in order with up to eight loads in flight, and
// combine through LDS in that order: one wavefront folding 64 splits of 1000 outputs by itself took
// eight round trips (4.6 us, 2.8 here).
constexpr int kFoldWaves = 16;   // at most
template <int S, int OP> __global__ __launch_bounds__(kFoldWaves * kWave) void red_fold_kernel(const RedFoldArgs p) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  __shared__ A lds[kFoldWaves - 1][kWave];
  const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const uint32_t o = blockIdx.x * kWave + lane;
  const uint32_t waves = blockDim.x / kWave, per = (p.split + waves - 1) / waves;
  uint32_t s = wave * per;
  const uint32_t end = s + per < p.split ? s + per : p.split;
  A acc = R::identity();
  if (o < p.nout) {
    const St *src = reinterpret_cast<const St *>(p.partial) + o;
    constexpr uint32_t U = 8;
    for (; s + U <= end; s += U) {
      St v[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) v[u] = src[(uint64_t)(s + u) * p.nout];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) acc = R::combine(acc, R::lift(from_storage<S>(v[u])));
    }
    St v[U];   // what is left, fewer than U: all on their way together
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (s + u < end) v[u] = src[(uint64_t)(s + u) * p.nout];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (s + u < end) acc = R::combine(acc, R::lift(from_storage<S>(v[u])));
  }
  if (wave > 0) lds[wave - 1][lane] = acc;
  __syncthreads();
  if (wave == 0 && o < p.nout) {
#pragma unroll
    for (int w = 0; w < 3; ++w) acc = R::combine(acc, lds[w][lane]);
    for (uint32_t w = 3; w + 1 < waves; ++w) acc = R::combine(acc, lds[w][lane]);
    store_result<A>(p.out + (int64_t)o * p.kso, p.out_dtype, acc, p.swap_o != 0);
  }
}

// ---------------------------------------------------------------------------------------
// cols
// ---------------------------------------------------------------------------------------

constexpr int kColsMaxWaves = 16;  // the cols kernel runs with 4 or 16 wavefronts per workgroup
// columns of a lane's vector that the wavefronts of a workgroup combine through LDS at a time
// (32 KiB for sixteen wavefronts; the launcher sizes the dynamic LDS accordingly)
template <class A> OCN_HD constexpr int cols_lds_columns() { return sizeof(A) <= 8 ? 4 : 2; }
template <class A> OCN_HD constexpr size_t cols_lds_bytes(int block, int vec) {
  return (size_t)(block / kWave) * kWave * sizeof(A) * (size_t)(cols_lds_columns<A>() < vec ? cols_lds_columns<A>() : vec);
}
// any and all of bytes: a lane's whole vector (16 KiB for sixteen wavefronts)
template <int S, int OP> OCN_HD constexpr bool cols_bits() {
  return dt_size(S) == 1 && (OP == R_ANY || OP == R_ALL || (S == DT_BOOL && (OP == R_MIN || OP == R_MAX)));
}

// What a lane of the column kernels takes: V columns (of elements of ES bytes) and rows r, r + rpw, ... below r1.
struct ColsPlace {
  int lane, wave, waves;            // waves: of the workgroup
  uint32_t split, other;            // which split of the rows, which of the other kept dims' outputs
  int lr, rpw;                      // its row among those that a wavefront takes at a time, and their number
  int ncol, skip;                   // its columns; how many of the first are its neighbour's
  int64_t col0, off_a, off_o;       // the first one, and the byte offsets of it in the input and the output
  int64_t r, r1, per_wave;          // per_wave: rows of a wavefront
};
template <int ES, int V> OCN_DEV ColsPlace cols_place(KRedArgs &p) {
  ColsPlace k;
  const int tid = threadIdx.x;
  k.lane = tid & (kWave - 1);
  k.wave = tid / kWave;
  k.waves = (int)blockDim.x / kWave;

  // block -> (split, other kept dims, column block)
  uint32_t b = blockIdx.x;
  const uint32_t per_split = (uint32_t)(p.colblocks_div.d * (uint32_t)(p.nout / p.nc));
  k.split = b / per_split;
  b -= k.split * per_split;
  k.other = rfastdiv(b, args_div(p.colblocks_div));
  const uint32_t cb = b - k.other * p.colblocks_div.d;
  // p.cpw lanes (a power of two) cover one row of columns; with fewer than 64 of them a
  // wavefront takes 64 / cpw rows at a time
  const int cpw_log2 = __ffs(p.cpw) - 1;
  const int lc = k.lane & (p.cpw - 1);
  k.lr = k.lane >> cpw_log2;
  k.rpw = kWave >> cpw_log2;
  k.col0 = ((int64_t)cb * p.cpw + lc) * V;
  const int64_t left = p.nc - k.col0;
  k.ncol = left >= V ? V : (left > 0 ? (int)left : 0);
  // The lane with the last few columns takes a whole vector that ends with the last column: the
  // first `skip` of its columns are its neighbour's and are dropped at the end.
  k.skip = 0;
  if (k.ncol > 0 && k.ncol < V && p.nc >= V) {
    k.skip = V - k.ncol;
    k.col0 -= k.skip;
    k.ncol = V;
  }

  // offsets of the other kept dims (kept dim 0 is the column dim)
  k.off_a = k.col0 * (int64_t)ES;
  k.off_o = k.col0 * p.kso[0];
  {
    uint32_t o = k.other;
    const int nkept = p.nkept;
    for (int d = 1; d < nkept; ++d) {
      const uint32_t q = (d == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[d]));
      const uint32_t i = o - q * p.kdiv[d].d;
      o = q;
      k.off_a += (int64_t)i * p.ksa[d];
      k.off_o += (int64_t)i * p.kso[d];
    }
  }

  const int64_t r0 = (int64_t)k.split * p.chunk;
  k.r1 = r0 + p.chunk;
  if (k.r1 > p.nredtot) k.r1 = p.nredtot;
  // Each wavefront takes one contiguous run of the workgroup's rows (rpw rows at a time).
  // Dealing the rows out in turn instead - wavefront w taking rows w, w + waves, ... - measured
  // 10 % slower (fp32 column sums of [16384, 4096]: 46.2 against 41.5 us).
  k.per_wave = (((k.r1 - r0) + k.waves - 1) / k.waves + k.rpw - 1) / k.rpw * k.rpw;
  const int64_t w0 = r0 + (int64_t)k.wave * k.per_wave;   // this wavefront's rows: w0 .. r1 - 1
  if (w0 + k.per_wave < k.r1) k.r1 = w0 + k.per_wave;
  k.r = w0 + k.lr;
  return k;
}
// SINGLE: one reduced dim, so that row r lies r strides further on (no index decomposition)
template <bool SINGLE> OCN_DEV int64_t cols_row_offset(KRedArgs &p, int64_t r) {
  if constexpr (SINGLE) return r * p.rsa[0];
  else return reduced_offset(p, (uint32_t)r, 0);
}

template <int S, int OP, int V, bool NT, bool SINGLE>
OCN_DEV void cols_body(KRedArgs &p, typename Reducer<S, OP>::A *lds) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  auto row_offset = [&](int64_t r) { return cols_row_offset<SINGLE>(p, r); };
  const ColsPlace k0 = cols_place<(int)sizeof(St), V>(p);
  const int lane = k0.lane, wave = k0.wave, NW = k0.waves, lr = k0.lr, RPW = k0.rpw, ncol = k0.ncol, skip = k0.skip;
  const uint32_t s = k0.split, other = k0.other;
  const int64_t col0 = k0.col0, off_a = k0.off_a, off_o = k0.off_o, r1 = k0.r1, per_wave = k0.per_wave;
  int64_t r = k0.r;
  A acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = R::identity();
  constexpr int U = 4;  // rows in flight per wavefront
  struct alignas(sizeof(St) * V >= 16 ? 16 : sizeof(St) * V) Pk { St v[V]; };
  const int RS = RPW;                // rows between two rows of the same lane
  // Sums of 8-bit integers: the sixteen columns of a vector are added two at a time, as 16-bit
  // halves of 32-bit words (signed bytes biased by 128 to make them unsigned), and spilled into
  // the 64-bit accumulators every 256 rows, before a half can overflow (256 * 255 < 2^16).
  constexpr bool PACKED8 = (S == DT_I8 || S == DT_U8) && OP == R_SUM && V == 16;
  bool packed_done = false;
  if constexpr (PACKED8) {
    // Up to 256 rows per wavefront: its lanes meet in those halves, and so do the wavefronts, each word
    // widened by the wavefront that adds it up (sixteen 64-bit sums a lane took a hundred shuffles
    // and four rounds through LDS: sums over [3840, 72] 16.7 -> 10.7 us, [1000, 500] 14.4 -> 7.5).
    if (per_wave <= 256 && p.nc >= V) {
      uint32_t sums[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // bytes 0 and 2 of each word, then 1 and 3
      auto add_row = [&](const Pk &pk) {
        uint32_t w[4];
        __builtin_memcpy(w, &pk, 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t x = S == DT_I8 ? w[k] ^ 0x80808080u : w[k];
          sums[k] += x & 0x00ff00ffu;
          sums[4 + k] += (x >> 8) & 0x00ff00ffu;
        }
      };
      if (ncol == V) {
        for (; r + (int64_t)(2 * U - 1) * RS < r1; r += RS * 2 * U) {
          Pk pk[2 * U];
#pragma unroll
          for (int u = 0; u < 2 * U; ++u) load_vec<St, V, NT>(p.a + off_a + row_offset(r + (int64_t)u * RS), pk[u]);
#pragma unroll
          for (int u = 0; u < 2 * U; ++u) add_row(pk[u]);
        }
        if (r < r1) {   // the last rows, all on their way together
          Pk pk[2 * U - 1];
#pragma unroll
          for (int u = 0; u < 2 * U - 1; ++u) load_vec<St, V, NT>(p.a + off_a + row_offset(r + (int64_t)u * RS < r1 ? r + (int64_t)u * RS : r), pk[u]);
#pragma unroll
          for (int u = 0; u < 2 * U - 1; ++u)
            if (r + (int64_t)u * RS < r1) add_row(pk[u]);
        }
      }
      uint32_t *words = reinterpret_cast<uint32_t *>(lds);   // [word][wavefront][lane]
      const uint64_t bias = S == DT_I8 ? (uint64_t)128 * (uint64_t)(((int64_t)s * p.chunk + p.chunk < p.nredtot ? p.chunk : p.nredtot - (int64_t)s * p.chunk)) : 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        for (int d = kWave / 2; d >= p.cpw; d >>= 1) sums[k] += (uint32_t)__shfl_down((int)sums[k], d);
        words[(k * NW + wave) * kWave + lane] = sums[k];
      }
      __syncthreads();
      for (int k = wave; k < 8; k += NW) {
        if (lr != 0 || ncol != V) continue;
        uint32_t lo = 0, hi = 0;   // (at most sixteen halves each)
        for (int w = 0; w < NW; ++w) {
          const uint32_t x = words[(k * NW + w) * kWave + lane];
          lo += x & 0xffffu;
          hi += x >> 16;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int i = 4 * (k & 3) + (k >> 2) + 2 * h;
          if (i < skip) continue;
          const A x = (A)((uint64_t)(h ? hi : lo) - bias);
          if (p.split == 1) store_result<A>(p.out + off_o + (int64_t)i * p.kso[0], p.out_dtype, x, p.swap_o != 0);
          else reinterpret_cast<typename R::P *>(p.partial)[(int64_t)s * p.nout + (int64_t)other * p.nc + col0 + i] = to_storage<R::ACC>(x);
        }
      }
      return;
    }
    if (ncol == V) {
      packed_done = true;
      uint32_t even[4] = {0, 0, 0, 0}, odd[4] = {0, 0, 0, 0};  // bytes 0 and 2 / 1 and 3 of each word
      uint32_t pending = 0;                                    // rows added since the last spill
      auto spill = [&]() {
        const A bias = S == DT_I8 ? (A)128 * (A)pending : (A)0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          acc[4 * k + 0] += (A)(even[k] & 0xffffu) - bias;
          acc[4 * k + 1] += (A)(odd[k] & 0xffffu) - bias;
          acc[4 * k + 2] += (A)(even[k] >> 16) - bias;
          acc[4 * k + 3] += (A)(odd[k] >> 16) - bias;
          even[k] = odd[k] = 0;
        }
        pending = 0;
      };
      auto add_row = [&](const Pk &pk) {
        uint32_t w[4];
        __builtin_memcpy(w, &pk, 16);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t x = S == DT_I8 ? w[k] ^ 0x80808080u : w[k];
          even[k] += x & 0x00ff00ffu;
          odd[k] += (x >> 8) & 0x00ff00ffu;
        }
        if (++pending == 256) spill();
      };
      for (; r + (int64_t)(U - 1) * RS < r1; r += RS * U) {
        Pk pk[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          load_vec<St, V, NT>(p.a + off_a + row_offset(r + (int64_t)u * RS), pk[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) add_row(pk[u]);
      }
      for (; r < r1; r += RS) {
        Pk pk;
        load_vec<St, V, NT>(p.a + off_a + row_offset(r), pk);
        add_row(pk);
      }
      spill();
    }
  }
  // (any and all of bytes come here with fewer columns than a vector holds only)
  constexpr bool WHOLE = !(cols_bits<S, OP>() && V == 16);
  if (packed_done) {
    // (nothing left to add)
  } else if (WHOLE && ncol == V) {  // whole vectors of columns: no per-element conditions
    // (one loop per byte order: decided per row inside the loop, the reversal is computed for
    // every vector and selected away)
    auto rows = [&](auto swapped) {
      constexpr bool SW = decltype(swapped)::value;
      for (; r + (int64_t)(U - 1) * RS < r1; r += RS * U) {
        Pk pk[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
          load_vec<St, V, NT>(p.a + off_a + row_offset(r + (int64_t)u * RS), pk[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          order_pack<S>(SW, pk[u]);
#pragma unroll
          for (int i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(pk[u].v[i])));
        }
      }
      for (; r < r1; r += RS) {
        Pk pk;
        load_vec<St, V, NT>(p.a + off_a + row_offset(r), pk);
        order_pack<S>(SW, pk);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(pk.v[i])));
      }
    };
    if (p.swap_a) rows(std::true_type{});
    else rows(std::false_type{});
  } else if (ncol > 0) {  // fewer columns than a vector holds
    for (; r < r1; r += RS) {
      const char *src = p.a + off_a + row_offset(r);
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < ncol) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(load_one<S>(p.swap_a != 0, src + (int64_t)i * (int64_t)sizeof(St)))));
    }
  }
  // lanes of a wavefront that hold the same columns of different rows: fold onto the first
  if (RPW > 1) {
#pragma unroll
    for (int i = 0; i < V; ++i)
#pragma unroll
      for (int d = kWave / 2; d >= 1; d >>= 1)
        if (d >= p.cpw) acc[i] = R::combine(acc[i], shfl_down_any(acc[i], d));
  }
  // Combine the wavefronts (same columns, different rows): CH columns of the vector go through
  // LDS at a time, and wavefront c folds column c over all wavefronts, in wavefront order.  (One
  // column at a time, folded by the first wavefront alone, was four rounds of a barrier and a
  // chain of sixteen LDS reads and adds at the end of every workgroup - and the workgroups of
  // a split reduction all end together.)
  constexpr int CH = cols_lds_columns<A>() < V ? cols_lds_columns<A>() : V;
#pragma unroll
  for (int i0 = 0; i0 < V; i0 += CH) {
#pragma unroll
    for (int c = 0; c < CH; ++c) lds[((size_t)wave * CH + c) * kWave + lane] = acc[i0 + c];
    __syncthreads();
    if (wave < CH && lr == 0 && i0 + wave < ncol && i0 + wave >= skip) {
      const int c = wave, i = i0 + wave;
      A v = lds[(size_t)c * kWave + lane];
      for (int w = 1; w < NW; ++w) v = R::combine(v, lds[((size_t)w * CH + c) * kWave + lane]);
      if (p.split == 1) {
        store_result<A>(p.out + off_o + (int64_t)i * p.kso[0], p.out_dtype, v, p.swap_o != 0);
      } else {
        const int64_t olin = (int64_t)other * p.nc + col0 + i;
        reinterpret_cast<typename R::P *>(p.partial)[(int64_t)s * p.nout + olin] = to_storage<R::ACC>(v);
      }
    }
    if (i0 + CH < V) __syncthreads();
  }
}

// Columns whose last block would be mostly empty, in workgroups few enough that such blocks leave their
// CUs idle: the columns are cut into equal blocks of any number of lanes, and the workgroup's lanes
// are numbered through whole rows of its block, so that p.cpw lanes take a row and block / p.cpw rows
// go at a time (one reduced dim, vectors of columns, every lane folds its own rows, the rows meet in LDS).
// Float sums over the middle of [48, 1000, 777], 195 vectors per row: four blocks of 64 lanes, the last
// with three, made 144 of 192 workgroups do the work, 33.7 us; 240 blocks of 39 lanes 28.6 (30.3 before
// neighbouring blocks, whose rows end inside a line, went to one XCD), 5.2 TB/s.
template <int S, int OP, int V, bool NT, bool SW>
OCN_DEV void cols_flat_body(KRedArgs &p, typename Reducer<S, OP>::A *lds) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  const uint32_t tid = threadIdx.x, block = blockDim.x, lanes = (uint32_t)p.cpw;
  // (consecutive blocks on one XCD, which workgroups go to in turn: blocks of the same rows share lines)
  const uint32_t xcd = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds, more = gridDim.x % kXcds;
  const uint32_t b = xcd * per_xcd + (xcd < more ? xcd : more) + blockIdx.x / kXcds;
  const uint32_t other = rfastdiv(b, args_div(p.colblocks_div)), cb = b - other * p.colblocks_div.d;
  const uint32_t rpt = block / lanes;                         // rows per trip
  const uint32_t g = __umulhi(tid, p.cpw_m), l = tid - g * lanes;
  int64_t col0 = ((int64_t)cb * lanes + l) * V;
  const int64_t left = p.nc - col0;
  int ncol = left >= V ? V : (left > 0 ? (int)left : 0), skip = 0;
  if (ncol > 0 && ncol < V) {   // (as in cols_body: a whole vector that ends with the last column)
    skip = V - ncol;
    col0 -= skip;
    ncol = V;
  }
  int64_t off_a = col0 * (int64_t)sizeof(St), off_o = col0 * p.kso[0];
  {
    uint32_t o = other;
    const int nkept = p.nkept;
    for (int k = 1; k < nkept; ++k) {
      const uint32_t q = (k == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[k]));
      const uint32_t i = o - q * p.kdiv[k].d;
      o = q;
      off_a += (int64_t)i * p.ksa[k];
      off_o += (int64_t)i * p.kso[k];
    }
  }
  A acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = R::identity();
  constexpr int U = 4;
  struct alignas(16) Pk { St v[V]; };
  auto add = [&](Pk &pk) {
    order_pack<S>(SW, pk);
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(pk.v[i])));
  };
  if (ncol == V && g < rpt) {
    const int64_t rows = p.nredtot, step = (int64_t)rpt * p.rsa[0];
    const char *src = p.a + off_a + (int64_t)g * p.rsa[0];
    int64_t r = g;
    for (; r + (int64_t)(U - 1) * rpt < rows; r += (int64_t)U * rpt) {
      Pk pk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        load_vec<St, V, NT>(src, pk[u]);
        src += step;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) add(pk[u]);
    }
    for (; r < rows; r += rpt) {
      Pk pk;
      load_vec<St, V, NT>(src, pk);
      src += step;
      add(pk);
    }
  }
  // CH columns per barrier; lane c * lanes + l folds column c of column lane l over the rows of a trip
  constexpr int CH = cols_lds_columns<A>() < V ? cols_lds_columns<A>() : V;
  const uint32_t fc = g, fl = l;   // (the same division: lanes of a row fold one column each)
#pragma unroll
  for (int i0 = 0; i0 < V; i0 += CH) {
#pragma unroll
    for (int c = 0; c < CH; ++c) lds[(size_t)c * block + tid] = acc[i0 + c];
    __syncthreads();
    if (fc < (uint32_t)CH && ncol == V && i0 + (int)fc >= skip) {
      A v = lds[(size_t)fc * block + fl];
      for (uint32_t k = 1; k < rpt; ++k) v = R::combine(v, lds[(size_t)fc * block + k * lanes + fl]);
      store_result<A>(p.out + off_o + (int64_t)(i0 + (int)fc) * p.kso[0], p.out_dtype, v, p.swap_o != 0);
    }
    if (i0 + CH < V) __syncthreads();
  }
}

// Columns of a few rows each, many times over: a lane per vector of columns takes all of its rows, four in
// flight, and stores its results; neighbouring lanes take neighbouring vectors, then the next outputs.
// The forms above give a wavefront 64 / cpw rows and a workgroup four wavefronts: with five rows of
// fifteen complex columns 40 of 256 lanes had any, and 244044 workgroups a barrier each (471 us, 38 here,
// 4.6 TB/s).
template <int S, int OP, int V, bool SW>
OCN_DEV void cols_lane_body(KRedArgs &p) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  const uint32_t t = blockIdx.x * (uint32_t)kBlock + threadIdx.x;
  const uint32_t other = rfastdiv(t, args_div(p.colblocks_div)), l = t - other * p.colblocks_div.d;
  if (t >= (uint32_t)p.nvec) return;
  int64_t col0 = (int64_t)l * V;
  int skip = 0;
  if (V > 1 && p.nc - col0 < V) {   // (as in cols_body: a whole vector that ends with the last column)
    skip = V - (int)(p.nc - col0);
    col0 -= skip;
  }
  int64_t off_a = col0 * (int64_t)sizeof(St), off_o = col0 * p.kso[0];
  {
    uint32_t o = other;
    const int nkept = p.nkept;
    for (int k = 1; k < nkept; ++k) {
      const uint32_t q = (k == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[k]));
      const uint32_t i = o - q * p.kdiv[k].d;
      o = q;
      off_a += (int64_t)i * p.ksa[k];
      off_o += (int64_t)i * p.kso[k];
    }
  }
  A acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = R::identity();
  constexpr int U = 4;
  struct alignas(sizeof(St) * V >= 16 ? 16 : sizeof(St) * V) Pk { St v[V]; };
  const char *src = p.a + off_a;
  const int64_t step = p.rsa[0];
  const uint32_t rows = (uint32_t)p.nredtot;
  for (uint32_t r = 0; r < rows; r += U) {   // (past the last row it is loaded again and left out)
    Pk pk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) load_vec<St, V, false>(src + (int64_t)(r + u < rows ? r + u : rows - 1) * step, pk[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (r + u < rows) {
        order_pack<S>(SW, pk[u]);
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(pk[u].v[i])));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < V; ++i)
    if (i >= skip) store_result<A>(p.out + off_o + (int64_t)i * p.kso[0], p.out_dtype, acc[i], p.swap_o != 0);
}
template <int S, int OP> __global__ __launch_bounds__(kBlock) void red_cols_lane_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  constexpr int VF = 16 / (int)sizeof(storage_t<S>) > 0 ? 16 / (int)sizeof(storage_t<S>) : 1;
  if constexpr (VF > 1 && VF <= 8) {
    if (p.vec > 1) {
      if (p.swap_a) cols_lane_body<S, OP, VF, true>(p);
      else cols_lane_body<S, OP, VF, false>(p);
      return;
    }
  }
  if (p.swap_a) cols_lane_body<S, OP, 1, true>(p);
  else cols_lane_body<S, OP, 1, false>(p);
}

// (a kernel of its own: beside the other forms it cost those registers, 2 % of some sums)
template <int S, int OP> __global__ __launch_bounds__(kColsMaxWaves * kWave) void red_cols_flat_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using A = typename Reducer<S, OP>::A;
  constexpr int VF = 16 / (int)sizeof(storage_t<S>);
  extern __shared__ __align__(16) unsigned char red_cols_lds_raw[];
  A *lds = reinterpret_cast<A *>(red_cols_lds_raw);
  if (p.swap_a) {
    if (p.nt_load) cols_flat_body<S, OP, VF, true, true>(p, lds);
    else cols_flat_body<S, OP, VF, false, true>(p, lds);
  } else {
    if (p.nt_load) cols_flat_body<S, OP, VF, true, false>(p, lds);
    else cols_flat_body<S, OP, VF, false, false>(p, lds);
  }
}

template <int S, int OP> __global__ __launch_bounds__(kColsMaxWaves * kWave) void red_cols_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using A = typename Reducer<S, OP>::A;
  constexpr int VF = 16 / (int)sizeof(storage_t<S>) > 0 ? 16 / (int)sizeof(storage_t<S>) : 1;
  extern __shared__ __align__(16) unsigned char red_cols_lds_raw[];
  A *lds = reinterpret_cast<A *>(red_cols_lds_raw);
  if (p.vec > 1 && p.nred == 1) {
    if (p.nt_load) cols_body<S, OP, VF, (VF > 1), true>(p, lds);
    else cols_body<S, OP, VF, false, true>(p, lds);
  } else if (p.vec > 1) {
    cols_body<S, OP, VF, false, false>(p, lds);
  } else {
    cols_body<S, OP, 1, false, false>(p, lds);
  }
}

// Any and all over whole vectors of byte columns: a lane's sixteen columns in four registers, which also meet as
// such, with eight rows in flight (sixteen accumulators of a byte each took a shuffle and a round through LDS
// apiece: bool any over the rows of [3840, 72] 19.2 -> 8.3 us, of [222, 2382] 10.7 -> 8.2).  In a kernel of their own:
// beside the other body they took its registers from 69 to 128 and spilled.
template <int S, int OP, bool NT, bool SINGLE> OCN_DEV void cols_bits_body(KRedArgs &p, uint32_t *words) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  using Bits = BitFold<S, OP>;
  constexpr int V = 16, U = 8;
  struct alignas(16) Pk { St v[V]; };
  const ColsPlace k = cols_place<1, V>(p);
  uint32_t bits[4] = {Bits::kStart, Bits::kStart, Bits::kStart, Bits::kStart};
  if (k.ncol == V) {
    const char *base = p.a + k.off_a;
    auto add_row = [&](const Pk &pk) {
      uint32_t w[4];
      __builtin_memcpy(w, &pk, 16);
#pragma unroll
      for (int i = 0; i < 4; ++i) bits[i] = Bits::add(bits[i], w[i]);
    };
    int64_t r = k.r;
    for (; r + (int64_t)(U - 1) * k.rpw < k.r1; r += (int64_t)k.rpw * U) {
      Pk pk[U];
#pragma unroll
      for (int u = 0; u < U; ++u) load_vec<St, V, NT>(base + cols_row_offset<SINGLE>(p, r + (int64_t)u * k.rpw), pk[u]);
#pragma unroll
      for (int u = 0; u < U; ++u) add_row(pk[u]);
    }
    if (r < k.r1) {   // the last rows, all on their way together (the first of them again where there are fewer)
      Pk pk[U - 1];
#pragma unroll
      for (int u = 0; u < U - 1; ++u)
        load_vec<St, V, NT>(base + cols_row_offset<SINGLE>(p, r + (int64_t)u * k.rpw < k.r1 ? r + (int64_t)u * k.rpw : r), pk[u]);
#pragma unroll
      for (int u = 0; u < U - 1; ++u) add_row(pk[u]);
    }
  }
  // words[word of the vector][wavefront][lane]
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    for (int d = kWave / 2; d >= p.cpw; d >>= 1) bits[i] = Bits::combine(bits[i], (uint32_t)__shfl_down((int)bits[i], d));
    words[(i * k.waves + k.wave) * kWave + k.lane] = bits[i];
  }
  __syncthreads();
  if (k.lr != 0 || k.ncol != V) return;
  for (int i = k.wave; i < 4; i += k.waves) {
    uint32_t v = words[i * k.waves * kWave + k.lane];
    for (int w = 1; w < k.waves; ++w) v = Bits::combine(v, words[(i * k.waves + w) * kWave + k.lane]);
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int c = 4 * i + b;
      if (c < k.skip) continue;
      const A x = Bits::result(v, b);
      if (p.split == 1) store_result<A>(p.out + k.off_o + (int64_t)c * p.kso[0], p.out_dtype, x, p.swap_o != 0);
      else reinterpret_cast<typename R::P *>(p.partial)[(int64_t)k.split * p.nout + (int64_t)k.other * p.nc + k.col0 + c] = to_storage<R::ACC>(x);
    }
  }
}
template <int S, int OP> __global__ __launch_bounds__(kColsMaxWaves * kWave) void red_cols_bits_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  extern __shared__ __align__(16) unsigned char red_cols_lds_raw[];
  uint32_t *words = reinterpret_cast<uint32_t *>(red_cols_lds_raw);
  if (p.nred != 1) cols_bits_body<S, OP, false, false>(p, words);
  else if (p.nt_load) cols_bits_body<S, OP, true, true>(p, words);
  else cols_bits_body<S, OP, false, true>(p, words);
}

// ---------------------------------------------------------------------------------------
// generic
// ---------------------------------------------------------------------------------------

template <int S, int OP> __global__ __launch_bounds__(kBlock) void red_generic_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  // the grid is capped (a launch cannot have 2^32 lanes): more outputs than lanes loop
  for (int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x; o < p.nout; o += (int64_t)gridDim.x * kBlock) {
  // 64-bit decomposition over the kept dims (fastest first)
  int64_t off_a = 0, off_o = 0, t = o;
  for (int k = 0; k < p.nkept; ++k) {
    const int64_t n = p.ksize[k];
    const int64_t q = t / n;
    const int64_t i = t - q * n;
    t = q;
    off_a += i * p.ksa[k];
    off_o += i * p.kso[k];
  }
  A acc = R::identity();
  for (int64_t r = 0; r < p.nredtot; ++r) {
    int64_t off = 0, q = r;
    for (int k = 0; k < p.nred; ++k) {
      const int64_t n = p.rsize[k];
      const int64_t qq = q / n;
      off += (q - qq * n) * p.rsa[k];
      q = qq;
    }
    acc = R::combine(acc, R::lift(from_storage<S>(load_one<S>(p.swap_a != 0, p.a + off_a + off))));
  }
  store_result<A>(p.out + off_o, p.out_dtype, acc, p.swap_o != 0);
  }
}

#endif  // __HIPCC__

}  // namespace ocn
