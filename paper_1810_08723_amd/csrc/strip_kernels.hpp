// Reductions over dense blocks of narrow rows: [rows, width] elements one after the other in memory, as
// the leading, the middle or all but one of a tensor's axes leave them.  Two forms, each plain and fused
// with an elementwise operation:
//
//   strip columns  the rows are reduced (with `inner` > 1 also runs of `inner` columns).  A group of
//                  lanes walks the block front to back in 16-byte vectors, wherever rows end.  Their number
//                  is a multiple of width / gcd(width, vector), so that from one trip to the next a lane
//                  keeps its columns and folds them in registers; the lanes' columns meet in LDS.
//   strip rows     every row is reduced.  A workgroup copies whole rows to LDS in 16-byte vectors, wherever
//                  they end, and then gives each row to one or a few neighbouring lanes.
//
// Bound by HBM once every lane has whole vectors and four of them in flight.  The other forms give a row of
// columns, or a row of addends, a power of two of lanes: what a narrow row leaves idle, reads at its end
// element by element and waits for alone is most of their time.  96 MB of floats (14.8 us at 6.5 TB/s): sums
// over the middle of [72727, 33, 10] 181 -> 24 us, [24000, 100, 10] 72 -> 19.6, [2608, 400, 23] 24.9 -> 19.2, over
// the first axis of [1090909, 22] 27.7 -> 22.5 (17 and the second launch), of rows of 5 103 -> 26, of 22 37 -> 20,
// of 100 29 -> 20.7.
#pragma once

#include "red_kernels.hpp"

namespace ocn {

struct RedStripArgs {
  const char *a, *b;                // (b: second input of a fused call)
  char *out, *partial;
  int64_t kso;                      // byte stride of the columns' (rows: the rows') kept dim in the output
  int64_t rs;                       // fused columns: byte stride per row of an input that is one element per row; runs: of the rows
  uint32_t ngroups, nother;         // groups of lanes in all (blocks of rows times splits; runs: outputs); other kept dims
  uint32_t rows, chunk;             // rows of a block; rows per split
  uint32_t width, inner;            // elements per row; columns that go into one output
  uint32_t lanes, lanes_m, groups;  // lanes per group, ceil(2^32 / lanes), groups per workgroup
  uint32_t nog, parts;              // outputs per group; lanes that share an output's fold
  uint32_t rotate;                  // rows: lanes start their rows at different elements
  uint32_t flags;                   // kStrip*
  int32_t out_dtype;
  int64_t pstep, psplit;            // partial results: from one output to the next, from one split to the next
  FastDiv split_div, width_div, inner_div, nog_div, outs_div;   // (outs: groups * nog)
  int64_t osa[kMaxDims], osb[kMaxDims], oso[kMaxDims];          // other kept dims, fastest first
  FastDiv odiv[kMaxDims];
};
enum : uint32_t { kStripNt = 1, kStripSwapA = 2, kStripSwapO = 4 };

// LDS of the column form: the accumulators of every lane's vector (es: size of an element)
template <class A> OCN_HD constexpr size_t strip_cols_lds(int block, int es) { return (size_t)block * (size_t)(16 / es) * sizeof(A); }

#if defined(__HIPCC__)

using KStripArgs = const __attribute__((address_space(4))) RedStripArgs;

// byte offsets of a group's block in the inputs and the output, and its rows
struct StripBlock {
  int64_t a, b, o;
  uint32_t row0, rows, split, other;
};
OCN_DEV StripBlock strip_block(KStripArgs &p, uint32_t g) {
  StripBlock k;
  k.other = rfastdiv(g, args_div(p.split_div));
  k.split = g - k.other * p.split_div.d;
  k.row0 = k.split * p.chunk;
  k.rows = k.row0 + p.chunk < p.rows ? p.chunk : p.rows - k.row0;
  k.a = k.b = k.o = 0;
  uint32_t t = k.other;
  const uint32_t nother = p.nother;
  for (uint32_t d = 0; d < nother; ++d) {
    const uint32_t q = d + 1 == nother ? 0u : rfastdiv(t, args_div(p.odiv[d]));
    const int64_t i = t - q * p.odiv[d].d;
    t = q;
    k.a += i * p.osa[d];
    k.b += i * p.osb[d];
    k.o += i * p.oso[d];
  }
  return k;
}

// Vectors of a lane on their way at a time: four, but two where sixteen unsigned bytes are widened to 64 bits each, whose
// words take a lane past its 128 registers with four (sums and products of uint8 spilled 5 to 43; 200 calls 2831 -> 2695
// us, [300, 986, 16] 11.3 -> 10.5; of int8, which fit, 2215 and 2249).
template <int S, class A> constexpr uint32_t strip_ahead = S == DT_U8 && sizeof(A) == 8 ? 2 : 4;

// Vectors l, l + lanes, ... below n: U on their way at a time, and what is left together too.
// (load and add are told the number of the trip as well)
template <class Buf, uint32_t U = 4, class Load, class Add> OCN_DEV void strip_walk(uint32_t l, uint32_t lanes, uint32_t n, Load load, Add add) {
  uint32_t t = l, trip = 0;
  for (; t + (U - 1) * lanes < n; t += U * lanes, trip += U) {
    Buf v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) load(t + u * lanes, trip + u, v[u]);
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) add(trip + u, v[u]);
  }
  if (t < n) {
    Buf v[U - 1];
#pragma unroll
    for (uint32_t u = 0; u < U - 1; ++u)
      if (t + u * lanes < n) load(t + u * lanes, trip + u, v[u]);
#pragma unroll
    for (uint32_t u = 0; u < U - 1; ++u)
      if (t + u * lanes < n) add(trip + u, v[u]);
  }
}

// The columns of a workgroup's groups meet: lds[lane * V + i] is element lane * V + i of one trip's worth
// of rows.  p.parts lanes share an output, each folds every parts-th of its elements, the first of them
// what the others have found.
template <class R> OCN_DEV void strip_fold(KStripArgs &p, typename R::A *lds, uint32_t per_group) {
  using A = typename R::A;
  const uint32_t tid = threadIdx.x, outs = p.outs_div.d, nog = p.nog, inner = p.inner, parts = p.parts, width = p.width;
  const uint32_t addends = rfastdiv(per_group, args_div(p.nog_div));   // elements that go into one output
  auto fold = [&](uint32_t part, uint32_t o) -> A {
    const uint32_t g = rfastdiv(o, args_div(p.nog_div)), j = o - g * nog;
    const A *src = lds + g * per_group + j * inner;
    A v = R::identity();
    if (inner == 1) {
#pragma clang loop vectorize(disable) interleave(disable) unroll_count(4)
      for (uint32_t e = part; e < addends; e += parts) v = R::combine(v, src[e * width]);
    } else {
#pragma clang loop vectorize(disable) interleave(disable) unroll_count(4)
      for (uint32_t e = part; e < addends; e += parts) {
        const uint32_t q = rfastdiv(e, args_div(p.inner_div));
        v = R::combine(v, src[q * width + (e - q * inner)]);
      }
    }
    return v;
  };
  auto put = [&](uint32_t o, A v) {
    const uint32_t g = rfastdiv(o, args_div(p.nog_div)), j = o - g * nog, gi = blockIdx.x * p.groups + g;
    if (gi >= p.ngroups) return;
    const StripBlock k = strip_block(p, gi);
    if (p.split_div.d == 1) store_result<A>(p.out + k.o + (int64_t)j * p.kso, p.out_dtype, v, (p.flags & kStripSwapO) != 0);
    else reinterpret_cast<typename R::P *>(p.partial)[(int64_t)k.split * p.psplit + ((int64_t)k.other * nog + j) * p.pstep] = to_storage<R::ACC>(v);
  };
  __syncthreads();
  if (parts == 1) {
    for (uint32_t o = tid; o < outs; o += blockDim.x) put(o, fold(0, o));
    return;
  }
  // (outs * parts is at most a workgroup's lanes)
  A v = R::identity();
  if (tid < outs * parts) {
    const uint32_t part = rfastdiv(tid, args_div(p.outs_div));
    v = fold(part, tid - part * outs);
  }
  __syncthreads();
  lds[tid] = v;
  __syncthreads();
  if (tid < outs) {
    for (uint32_t q = 1; q < parts; ++q) v = R::combine(v, lds[q * outs + tid]);
    put(tid, v);
  }
}

template <int S, int OP, bool NT, bool SW> OCN_DEV void strip_cols_body(KStripArgs &p, typename Reducer<S, OP>::A *lds) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  constexpr uint32_t V = 16 / sizeof(St);
  struct alignas(16) Pk { St v[V]; };
  const uint32_t tid = threadIdx.x, lanes = p.lanes;
  const uint32_t gl = __umulhi(tid, p.lanes_m), l = tid - gl * lanes, g = blockIdx.x * p.groups + gl;
  if constexpr (cols_bits<S, OP>()) {   // sixteen columns in four registers
    using Bits = BitFold<S, OP>;
    uint32_t bits[4] = {Bits::kStart, Bits::kStart, Bits::kStart, Bits::kStart};
    if (gl < p.groups && g < p.ngroups) {
      const StripBlock k = strip_block(p, g);
      const uint32_t n = k.rows * p.width, full = n / V;
      const char *base = p.a + k.a + (int64_t)k.row0 * (int64_t)p.width;
      auto add = [&](uint32_t, Pk &v) {
        uint32_t w[4];
        __builtin_memcpy(w, &v, 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) bits[i] = Bits::add(bits[i], w[i]);
      };
      strip_walk<Pk>(l, lanes, full, [&](uint32_t t, uint32_t, Pk &v) { load_vec<St, V, NT>(base + (uint64_t)t * 16u, v); }, add);
      if (full * V < n && full % lanes == l) {   // the elements behind the last whole vector
        Pk v;
#pragma unroll
        for (uint32_t i = 0; i < V; ++i) {
          const St x = *reinterpret_cast<const St *>(base + (full * V + i < n ? full * V + i : n - 1));
          v.v[i] = full * V + i < n ? x : (St)(Bits::kNeutral & 0xffu);
        }
        add(0, v);
      }
    }
#pragma unroll
    for (uint32_t i = 0; i < V; ++i) lds[tid * V + i] = Bits::result(bits[i / 4], (int)(i % 4));
    strip_fold<R>(p, lds, lanes * V);
    return;
  }
  A acc[V];
#pragma unroll
  for (uint32_t i = 0; i < V; ++i) acc[i] = R::identity();
  if (gl < p.groups && g < p.ngroups) {
    const StripBlock k = strip_block(p, g);
    const uint32_t n = k.rows * p.width, full = n / V;
    const char *base = p.a + k.a + (int64_t)k.row0 * (int64_t)(p.width * sizeof(St));
    strip_walk<Pk, strip_ahead<S, A>>(
        l, lanes, full, [&](uint32_t t, uint32_t, Pk &v) { load_vec<St, V, NT>(base + (uint64_t)t * 16u, v); },
        [&](uint32_t, Pk &v) {
          order_pack<S>(SW, v);
#pragma unroll
          for (uint32_t i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(v.v[i])));
        });
    if (V > 1 && full * V < n && full % lanes == l) {   // the elements behind the last whole vector, all on their way together
      St v[V];
#pragma unroll
      for (uint32_t i = 0; i < V - 1; ++i) v[i] = *reinterpret_cast<const St *>(base + (uint64_t)(full * V + i < n ? full * V + i : n - 1) * sizeof(St));
#pragma unroll
      for (uint32_t i = 0; i < V - 1; ++i)
        if (full * V + i < n) {
          order_pack<S>(SW, v[i]);
          acc[i] = R::combine(acc[i], R::lift(from_storage<S>(v[i])));
        }
    }
  }
#pragma unroll
  for (uint32_t i = 0; i < V; ++i) lds[tid * V + i] = acc[i];
  strip_fold<R>(p, lds, lanes * V);
}

template <int S, int OP> __global__ __launch_bounds__(kStripLanes) void red_strip_cols_kernel(const RedStripArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KStripArgs &p = *(KStripArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  using A = typename Reducer<S, OP>::A;
  extern __shared__ __align__(16) unsigned char strip_lds[];
  A *lds = reinterpret_cast<A *>(strip_lds);
  const uint32_t flags = p.flags;
  if (flags & kStripSwapA) {
    strip_cols_body<S, OP, false, true>(p, lds);
  } else if (flags & kStripNt) {
    strip_cols_body<S, OP, true, false>(p, lds);
  } else {
    strip_cols_body<S, OP, false, false>(p, lds);
  }
}

// Whole rows from LDS: p.parts neighbouring lanes (a power of two) take a row each element in turn.
template <class R, class Get> OCN_DEV void strip_rows_fold(KStripArgs &p, const StripBlock &k, Get get) {
  using A = typename R::A;
  const uint32_t parts = p.parts, part = threadIdx.x & (parts - 1), width = p.width, step = (uint32_t)kBlock / parts, rotate = p.rotate;
  __syncthreads();
  for (uint32_t r0 = 0; r0 < k.rows; r0 += step) {    // (the same trips for all lanes: they fold together)
    const uint32_t r = r0 + threadIdx.x / parts;
    A v = R::identity();
    if (r < k.rows) {
      const uint32_t e0 = r * width;
      uint32_t c = part + (rotate ? (r & (rotate - 1)) * parts : 0u);
#pragma clang loop vectorize(disable) interleave(disable) unroll_count(4)
      for (uint32_t i = part; i < width; i += parts) {
        v = R::combine(v, get(e0 + c));
        c = c + parts < width ? c + parts : part;
      }
    }
    v = group_fold<R>(v, (int)parts);
    if (r < k.rows && part == 0)
      store_result<A>(p.out + k.o + (int64_t)(k.row0 + r) * p.kso, p.out_dtype, v, (p.flags & kStripSwapO) != 0);
  }
}

// Runs of columns in an output where rows are too long for the forms above ([rows, outputs, run], rows any distance
// apart): a workgroup owns p.nog whole outputs, p.lanes lanes take their columns of a row in 16-byte vectors,
// p.groups rows go at a time; the runs meet in LDS.  Lanes that share an output read its run, a piece of every
// row, by themselves otherwise, each in lines of its own.
template <int S, int OP, bool NT, bool SW> OCN_DEV void strip_runs_body(KStripArgs &p, typename Reducer<S, OP>::A *lds) {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  using St = storage_t<S>;
  constexpr uint32_t V = 16 / sizeof(St);
  struct alignas(16) Pk { St v[V]; };
  const uint32_t tid = threadIdx.x, lanes = p.lanes, inner = p.inner, groups = p.groups;
  const uint32_t g = __umulhi(tid, p.lanes_m), l = tid - g * lanes;
  const uint32_t cb = rfastdiv(blockIdx.x, args_div(p.split_div)), split = blockIdx.x - cb * p.split_div.d;
  const uint32_t row0 = split * p.chunk, rows = row0 + p.chunk < p.rows ? p.chunk : p.rows - row0;
  const uint32_t o0 = cb * p.nog, outs = o0 + p.nog < p.ngroups ? p.nog : p.ngroups - o0, cw = outs * inner;
  if (g < groups && l * V < cw) {
    // (the last vector ends with the last column; its first elements, a neighbour's, are dropped)
    const int skip = l * V + V > cw ? (int)(l * V + V - cw) : 0;
    const int64_t rs = p.rs, col = (int64_t)o0 * inner + (int64_t)(l * V) - skip;
    const char *base = p.a + col * (int64_t)sizeof(St) + (int64_t)row0 * rs;
    A acc[V];
    auto load = [&](uint32_t t, uint32_t, Pk &v) { load_vec<St, V, NT>(base + (int64_t)t * rs, v); };
    if constexpr (cols_bits<S, OP>()) {
      using Bits = BitFold<S, OP>;
      uint32_t bits[4] = {Bits::kStart, Bits::kStart, Bits::kStart, Bits::kStart};
      strip_walk<Pk>(g, groups, rows, load, [&](uint32_t, Pk &v) {
        uint32_t w[4];
        __builtin_memcpy(w, &v, 16);
#pragma unroll
        for (int i = 0; i < 4; ++i) bits[i] = Bits::add(bits[i], w[i]);
      });
#pragma unroll
      for (uint32_t i = 0; i < V; ++i) acc[i] = Bits::result(bits[i / 4], (int)(i % 4));
    } else {
#pragma unroll
      for (uint32_t i = 0; i < V; ++i) acc[i] = R::identity();
      strip_walk<Pk, strip_ahead<S, A>>(g, groups, rows, load, [&](uint32_t, Pk &v) {
        order_pack<S>(SW, v);
#pragma unroll
        for (uint32_t i = 0; i < V; ++i) acc[i] = R::combine(acc[i], R::lift(from_storage<S>(v.v[i])));
      });
    }
    A *dst = lds + g * cw + l * V;
#pragma unroll
    for (int i = 0; i < (int)V; ++i)
      if (i >= skip) dst[i - skip] = acc[i];
  }
  __syncthreads();
  const uint32_t parts = p.parts, part = tid & (parts - 1), step = blockDim.x / parts;
  for (uint32_t first = 0; first < outs; first += step) {   // (the same trips for all lanes: they fold together)
    const uint32_t o = first + tid / parts;
    A v = R::identity();
    if (o < outs)
      for (uint32_t q = 0; q < groups; ++q) {
        const A *src = lds + q * cw + o * inner;
#pragma clang loop vectorize(disable) interleave(disable) unroll_count(4)
        for (uint32_t j = part; j < inner; j += parts) v = R::combine(v, src[j]);
      }
    v = group_fold<R>(v, (int)parts);
    if (o < outs && part == 0) {
      if (p.split_div.d == 1) store_result<A>(p.out + (int64_t)(o0 + o) * p.kso, p.out_dtype, v, (p.flags & kStripSwapO) != 0);
      else reinterpret_cast<typename R::P *>(p.partial)[(int64_t)split * p.psplit + (int64_t)(o0 + o) * p.pstep] = to_storage<R::ACC>(v);
    }
  }
}
template <int S, int OP> __global__ __launch_bounds__(kStripLanes) void red_strip_runs_kernel(const RedStripArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KStripArgs &p = *(KStripArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  extern __shared__ __align__(16) unsigned char strip_lds[];
  auto *lds = reinterpret_cast<typename Reducer<S, OP>::A *>(strip_lds);
  const uint32_t flags = p.flags;
  if (flags & kStripSwapA) strip_runs_body<S, OP, false, true>(p, lds);
  else if (flags & kStripNt) strip_runs_body<S, OP, true, false>(p, lds);
  else strip_runs_body<S, OP, false, false>(p, lds);
}

// A lane's fold over one-byte elements, four at a time; kNeutral changes nothing.
template <int S, int OP> struct WordFold {
  using R = Reducer<S, OP>;
  using A = typename R::A;
  static constexpr bool kBits = cols_bits<S, OP>(), kDot = OP == R_SUM && (S == DT_I8 || S == DT_U8);
  static constexpr uint32_t kNeutral = kBits         ? BitFold<S, OP>::kNeutral
                                       : OP == R_SUM ? 0u
                                       : OP == R_MIN ? (S == DT_I8 ? 0x7f7f7f7fu : ~0u)
                                       : OP == R_MAX ? (S == DT_I8 ? 0x80808080u : 0u)
                                                     : 0x01010101u;
  // extremes compare two bytes at a time, each the high one of 16 bits (what lies below only breaks ties)
  static constexpr bool kPairs = !kBits && (OP == R_MIN || OP == R_MAX);
  using Half = std::conditional_t<S == DT_I8, int16_t, uint16_t>;
  using Pair = Half __attribute__((ext_vector_type(2)));
  static constexpr int kKind = kPairs ? 0 : kBits || kDot ? 1 : 2;
  struct Pairs { Pair even, odd; };
  std::conditional_t<kKind == 0, Pairs, std::conditional_t<kKind == 1, uint32_t, A>> acc;
  OCN_DEV static Pair extreme(Pair x, uint32_t w) {
    const Pair y = __builtin_bit_cast(Pair, w);
    return OP == R_MAX ? __builtin_elementwise_max(x, y) : __builtin_elementwise_min(x, y);
  }
  OCN_DEV void init() {
    if constexpr (kPairs) acc.even = acc.odd = __builtin_bit_cast(Pair, kNeutral);
    else if constexpr (kBits) acc = BitFold<S, OP>::kStart;
    else if constexpr (kDot) acc = 0u;
    else acc = R::identity();
  }
  OCN_DEV void add(uint32_t w) {
    if constexpr (kPairs) {
      acc.even = extreme(acc.even, w << 8);
      acc.odd = extreme(acc.odd, w);
    } else if constexpr (kBits) acc = BitFold<S, OP>::add(acc, w);
    else if constexpr (kDot && S == DT_I8) acc = (uint32_t)__builtin_amdgcn_sdot4((int)w, 0x01010101, (int)acc, false);
    else if constexpr (kDot) acc = __builtin_amdgcn_udot4(w, 0x01010101u, acc, false);
    else {
#pragma unroll
      for (int b = 0; b < 4; ++b) acc = R::combine(acc, R::lift(from_storage<S>((storage_t<S>)(uint8_t)(w >> (8 * b)))));
    }
  }
  OCN_DEV A result() {
    if constexpr (kPairs) {
      const Pair v = extreme(acc.even, __builtin_bit_cast(uint32_t, acc.odd));
      const Half x = OP == R_MAX ? (v.x > v.y ? v.x : v.y) : (v.x < v.y ? v.x : v.y);
      return (A)(x >> 8);
    } else if constexpr (kBits) return BitFold<S, OP>::whole(acc);
    else if constexpr (kDot && S == DT_I8) return (A)(int32_t)acc;   // (rows of 1024 bytes at most)
    else if constexpr (kDot) return (A)acc;
    else return acc;
  }
};

// Rows of bytes come from LDS in the aligned words that cover them, with the neighbours' bytes in the first
// and the last word replaced.  Byte by byte the reads and their addresses were the time of rows of 32 and more,
// which therefore stayed with lanes that load their row's vectors themselves and take its last bytes one by one:
// 100 MB of int8 sums in rows of 33 63 -> 25.5 us, of 156 62.5 -> 22.9, of 1000 40 -> 21.7 (15.4 at 6.5 TB/s), of 17 (byte by byte before) 37 -> 32.
template <int S, int OP> OCN_DEV void strip_byte_rows_fold(KStripArgs &p, const StripBlock &k, const uint32_t *lds) {
  using F = WordFold<S, OP>;
  using R = typename F::R;
  using A = typename R::A;
  const uint32_t parts = p.parts, part = threadIdx.x & (parts - 1), width = p.width, step = (uint32_t)kBlock / parts, rotate = p.rotate;
  __syncthreads();
  for (uint32_t r0 = 0; r0 < k.rows; r0 += step) {    // (the same trips for all lanes: they fold together)
    const uint32_t r = r0 + threadIdx.x / parts;
    F f;
    f.init();
    if (r < k.rows) {
      const uint32_t e0 = r * width, e1 = e0 + width, w0 = e0 / 4, nw = (e1 + 3) / 4 - w0;
      const uint32_t head = ~0u << (8 * (e0 & 3)), tail = ~0u >> (8 * ((0u - e1) & 3));
      uint32_t c = part + (rotate ? (r & (rotate - 1)) * parts : 0u);
#pragma clang loop vectorize(disable) interleave(disable) unroll_count(4)
      for (uint32_t i = part; i < nw; i += parts) {
        const uint32_t m = (c == 0 ? head : ~0u) & (c + 1 == nw ? tail : ~0u);
        f.add((lds[w0 + c] & m) | (F::kNeutral & ~m));
        c = c + parts < nw ? c + parts : part;
      }
    }
    const A v = group_fold<R>(f.result(), (int)parts);
    if (r < k.rows && part == 0)
      store_result<A>(p.out + k.o + (int64_t)(k.row0 + r) * p.kso, p.out_dtype, v, (p.flags & kStripSwapO) != 0);
  }
}

template <int S, int OP> __global__ __launch_bounds__(kBlock) void red_strip_rows_kernel(const RedStripArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KStripArgs &p = *(KStripArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  using R = Reducer<S, OP>;
  using St = storage_t<S>;
  constexpr uint32_t V = 16 / sizeof(St);
  struct alignas(16) Pk { St v[V]; };
  extern __shared__ __align__(16) unsigned char strip_lds[];
  St *lds = reinterpret_cast<St *>(strip_lds);
  const StripBlock k = strip_block(p, blockIdx.x);
  const uint32_t n = k.rows * p.width, full = n / V, tid = threadIdx.x;
  const char *base = p.a + k.a + (int64_t)k.row0 * (int64_t)(p.width * sizeof(St));
  const bool nt = (p.flags & kStripNt) != 0, sw = (p.flags & kStripSwapA) != 0;
  auto keep = [&](uint32_t trip, Pk &v) {
    order_pack<S>(sw, v);
    reinterpret_cast<Pk *>(strip_lds)[tid + trip * (uint32_t)kBlock] = v;
  };
  if (nt) strip_walk<Pk>(tid, kBlock, full, [&](uint32_t t, uint32_t, Pk &v) { load_vec<St, V, true>(base + (uint64_t)t * 16u, v); }, keep);
  else strip_walk<Pk>(tid, kBlock, full, [&](uint32_t t, uint32_t, Pk &v) { load_vec<St, V, false>(base + (uint64_t)t * 16u, v); }, keep);
  if (full * V + tid < n) lds[full * V + tid] = load_one<S>(sw, base + (uint64_t)(full * V + tid) * sizeof(St));
  if constexpr (sizeof(St) == 1) strip_byte_rows_fold<S, OP>(p, k, reinterpret_cast<const uint32_t *>(strip_lds));
  else strip_rows_fold<R>(p, k, [&](uint32_t e) { return R::lift(from_storage<S>(lds[e])); });
}

#endif  // __HIPCC__

}  // namespace ocn
