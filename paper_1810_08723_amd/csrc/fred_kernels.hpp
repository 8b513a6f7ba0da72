// Fused elementwise+reduce kernels for gfx950: out = reduce(op, g(a, b)) without the
// intermediate tensor (sections 3.2 and 5 of the paper: elementwise functions followed by a
// reduction along axes, e.g. the inner product and norm of the QR example).
//
// Each element is produced exactly as the elementwise kernels would store it - converted to
// the intermediate type - and then folded exactly as the reduction kernels would fold it, so
// the result equals the two-step computation up to the order of a floating-point sum.  The
// three layouts and the launch geometry are those of red_kernels.hpp; split reductions write
// partial results that a plain second launch folds.
#pragma once

#include "ew_kernels.hpp"
#include "red_kernels.hpp"
#include "strip_kernels.hpp"

namespace ocn {

#if defined(__HIPCC__)

// input byte offsets (a and b) of reduced index q over the reduced dims from `first` upward
OCN_DEV void reduced_offset2(KRedArgs &p, uint32_t q, int first, int64_t &oa, int64_t &ob) {
  oa = 0;
  ob = 0;
  const int nred = p.nred;
  for (int k = first; k < nred; ++k) {
    const uint32_t qq = (k == nred - 1) ? 0u : rfastdiv(q, args_div(p.rdiv[k]));
    const uint32_t i = q - qq * p.rdiv[k].d;
    q = qq;
    oa += (int64_t)i * p.rsa[k];
    ob += (int64_t)i * p.rsb[k];
  }
}

// byte offsets of output number `o` in a, b and out
OCN_DEV void kept_offsets2(KRedArgs &p, uint32_t o, int64_t &off_a, int64_t &off_b, int64_t &off_o) {
  off_a = off_b = off_o = 0;
  const int nkept = p.nkept;
  for (int k = 0; k < nkept; ++k) {
    const uint32_t q = (k == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[k]));
    const uint32_t i = o - q * p.kdiv[k].d;
    o = q;
    off_a += (int64_t)i * p.ksa[k];
    off_b += (int64_t)i * p.ksb[k];
    off_o += (int64_t)i * p.kso[k];
  }
}

// V consecutive elements of one input, or V copies of one element where it is broadcast
template <class S, int V> OCN_DEV void fused_load(const char *src, bool bcast, Pack<S, V> &dst) {
  if (bcast) {
    const S s = *reinterpret_cast<const S *>(src);
#pragma unroll
    for (int i = 0; i < V; ++i) dst.v[i] = s;
  } else {
    load_vec<S, V, false>(src, dst);
  }
}

template <class G, int OP> struct FusedFold {
  static constexpr int E = G::SO_DT;  // type of the intermediate elements
  using R = Reducer<E, OP>;
  using A = typename R::A;
  OCN_DEV static A add(A acc, typename G::SAt a, typename G::SBt b) {
    return R::combine(acc, R::lift(from_storage<E>(G::eval(a, b))));
  }
};

// ---------------------------------------------------------------------------------------
// rows: the reduced axis is the fastest of the inputs
// ---------------------------------------------------------------------------------------

template <class G, int OP, int V>
OCN_DEV typename FusedFold<G, OP>::A fred_rows_accumulate(KRedArgs &p, const char *pa, const char *pb,
                                                          int64_t t0, int64_t t1, int lane, int lanes) {
  using F = FusedFold<G, OP>;
  using A = typename F::A;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
#ifndef OCN_FRED_U
#define OCN_FRED_U 2
#endif
  constexpr int U = OCN_FRED_U;
  A acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = F::R::identity();
  const bool single = p.nred == 1;
  const bool abc = p.a_bcast, bbc = p.b_bcast;
  // vectors below t_full are known to be whole
  int64_t t_full = t0;
  if (p.n0 % V == 0) t_full = t1;
  else if (single) t_full = p.n0 / V < t1 ? p.n0 / V : t1;
  auto address = [&](int64_t tt, int64_t &e0, const char *&qa, const char *&qb) {
    int64_t oa = 0, ob = 0, iv = tt;
    if (!single) {
      const uint32_t q = rfastdiv((uint32_t)tt, args_div(p.vpr_div));
      iv = (uint32_t)tt - q * p.vpr_div.d;
      reduced_offset2(p, q, 1, oa, ob);
    }
    e0 = iv * V;
    qa = pa + oa + (abc ? 0 : e0 * (int64_t)sizeof(SAt));
    qb = pb + ob + (bbc ? 0 : e0 * (int64_t)sizeof(SBt));
  };
  int64_t t = t0;
  for (; t + (int64_t)lanes * U <= t_full; t += (int64_t)lanes * U) {
    Pack<SAt, V> va[U];
    Pack<SBt, V> vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int64_t e0;
      const char *qa, *qb;
      address(t + (int64_t)u * lanes + lane, e0, qa, qb);
      fused_load<SAt, V>(qa, abc, va[u]);
      fused_load<SBt, V>(qb, bbc, vb[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < V; ++i) acc[u] = F::add(acc[u], va[u].v[i], vb[u].v[i]);
  }
  for (int64_t tt = t + lane; tt < t1; tt += lanes) {
    int64_t e0;
    const char *qa, *qb;
    address(tt, e0, qa, qb);
    const int64_t left = p.n0 - e0;
    const int n = left >= V ? V : (int)left;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      if (i < n) {
        const SAt x = reinterpret_cast<const SAt *>(qa)[abc ? 0 : i];
        const SBt y = reinterpret_cast<const SBt *>(qb)[bbc ? 0 : i];
        acc[0] = F::add(acc[0], x, y);
      }
    }
  }
  A r = acc[0];
#pragma unroll
  for (int u = 1; u < U; ++u) r = F::R::combine(r, acc[u]);
  return r;
}

template <class G, int OP> __global__ __launch_bounds__(kBlock) void fred_rows_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using A = typename F::A;
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
    int64_t off_a, off_b;
    kept_offsets2(p, (uint32_t)o, off_a, off_b, off_o);
    const int lanes = per_block ? kBlock : width;
    if (p.vec > 1) acc = fred_rows_accumulate<G, OP, G::V>(p, p.a + off_a, p.b + off_b, t0, t1, lane, lanes);
    else acc = fred_rows_accumulate<G, OP, 1>(p, p.a + off_a, p.b + off_b, t0, t1, lane, lanes);
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
    if (p.split == 1) store_result<A>(p.out + off_o, p.out_dtype, acc);
    else reinterpret_cast<typename R::P *>(p.partial)[o * p.split + s] = to_storage<R::ACC>(acc);
  }
}

// The common fused row reduction - one reduced dim along which both inputs are contiguous and
// read in whole 16-byte vectors, at most one kept dim (along which either input may be
// broadcast), a wavefront or a workgroup per output or per split of it, everything below 2^31 -
// without the index decomposition and the 64-bit bookkeeping of the general kernel, and with
// every load a single 16-byte piece per lane, so that a wavefront's instruction covers whole
// lines of its input (the access shape streaming loads need; the general kernel reads 64 bytes
// per lane and input when the intermediate type is bool).
template <class G, int OP, bool NT>
OCN_DEV typename FusedFold<G, OP>::A fred_lean_fold(const char *pa, const char *pb, uint32_t t0, uint32_t t1,
                                                    uint32_t lane, uint32_t lanes) {
  using F = FusedFold<G, OP>;
  using A = typename F::A;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  static_assert(sizeof(SAt) == sizeof(SBt) && sizeof(SAt) <= 16, "equal input widths of at most 16 bytes");
  constexpr int V = 16 / (int)sizeof(SAt);
  // Vectors in flight of each input.  (Four spill complex sums under the 64 registers of OCN_ROWS_OCC, complex
  // double products of [16384, 1000] 116 us where two take 76, and lose 5 to 15 % of halves and of rows of
  // 50000 doubles.  Products of four-byte elements win: float [16384, 1000] 21.2 -> 19.9, [20000, 600] with a row
  // 10.7 -> 10.0.)
  constexpr int U = sizeof(SAt) == 4 && G::SO_DT == G::SA_DT ? 4 : 2;
  // Trips are counted for all lanes alike: with the count of each lane its own, a row of 250 vectors is
  // three round trips of a wavefront, for the lanes with four vectors and those with three.  (Except for moduli
  // of complex elements, where that spills: [3000, 4096] 34 us, 30 so.)
  constexpr bool OWN = dt_kind(G::SA_DT) == K_CPLX && G::EW == B_ABSGT;
  constexpr int T = OWN ? 1 : U;   // vectors in flight of what is left
  A acc[U];
#pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = F::R::identity();
  const uint32_t ahead = OWN ? 0u : lane;
  uint32_t t = OWN ? t0 + lane : t0;
  for (; OWN ? t + (U - 1) * lanes < t1 : t + U * lanes <= t1; t += U * lanes) {
    Pack<SAt, V> va[U];
    Pack<SBt, V> vb[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load_vec<SAt, V, NT>(pa + (uint64_t)(t + u * lanes + ahead) * 16u, va[u]);
      load_vec<SBt, V, NT>(pb + (uint64_t)(t + u * lanes + ahead) * 16u, vb[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < V; ++i) acc[u] = F::add(acc[u], va[u].v[i], vb[u].v[i]);
  }
  for (; t < t1; t += T * lanes) {   // what is left, fewer than U per lane: lanes past the end load the last vector and drop it
    Pack<SAt, V> va[T];
    Pack<SBt, V> vb[T];
#pragma unroll
    for (int u = 0; u < T; ++u) {
      if (t + u * lanes < t1) {
        const uint32_t tt = t + u * lanes + ahead < t1 ? t + u * lanes + ahead : t1 - 1;
        load_vec<SAt, V, NT>(pa + (uint64_t)tt * 16u, va[u]);
        load_vec<SBt, V, NT>(pb + (uint64_t)tt * 16u, vb[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < T; ++u) {
      if (t + u * lanes + ahead < t1) {
#pragma unroll
        for (int i = 0; i < V; ++i) acc[u] = F::add(acc[u], va[u].v[i], vb[u].v[i]);
      }
    }
  }
  A r = acc[0];
#pragma unroll
  for (int u = 1; u < U; ++u) r = F::R::combine(r, acc[u]);
  return r;
}

template <class G, int OP> __global__ __launch_bounds__(kLeanWaves * kWave) OCN_ROWS_OCC void fred_rows_lean_kernel(const RedLeanArgs p) {
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using A = typename F::A;
  __shared__ A lds[kLeanWaves];
  const uint32_t tid = threadIdx.x, lane_in_wave = tid & (kWave - 1), wave = tid / kWave;
  const bool per_block = p.group > kWave;
  const uint32_t gidx = per_block ? blockIdx.x : blockIdx.x * (kBlock / kWave) + wave;
  const bool active = gidx < p.nout * p.split;
  const uint32_t lane = per_block ? tid : lane_in_wave;
  uint32_t o = gidx, sp = 0, t0 = 0, t1 = p.nvec;
  A acc = R::identity();
  if (active) {
    if (p.split != 1) {
      o = gidx / p.split;
      sp = gidx - o * p.split;
      t0 = sp * p.chunk;
      t1 = t0 + p.chunk < p.nvec ? t0 + p.chunk : p.nvec;
    }
    const char *pa = p.a + (int64_t)o * p.ksa;
    const char *pb = p.b + (int64_t)o * p.ksb;
    const uint32_t lanes = (uint32_t)p.group;
    if (p.nt_load) acc = fred_lean_fold<G, OP, true>(pa, pb, t0, t1, lane, lanes);
    else acc = fred_lean_fold<G, OP, false>(pa, pb, t0, t1, lane, lanes);
    // the elements behind the last whole vector: one lane of the last split
    if (p.tail && lane == 0 && sp + 1 == p.split) {
      const typename G::SAt *qa = reinterpret_cast<const typename G::SAt *>(pa + (uint64_t)p.nvec * 16u);
      const typename G::SBt *qb = reinterpret_cast<const typename G::SBt *>(pb + (uint64_t)p.nvec * 16u);
      for (uint32_t i = 0; i < p.tail; ++i) acc = F::add(acc, qa[i], qb[i]);
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
    if (p.split == 1) store_result<A>(p.out + (int64_t)o * p.kso, p.out_dtype, acc);
    else reinterpret_cast<typename R::P *>(p.partial)[(uint64_t)o * p.split + sp] = to_storage<R::ACC>(acc);
  }
}

// Rows of at most one vector per lane of their group, a single reduced dim, no split: the same
// groups, loads and fold order as fred_rows_kernel without its loops and 64-bit bookkeeping.
template <class G, int OP, int V>
OCN_DEV typename FusedFold<G, OP>::A fred_short_row(KRedArgs &p, const char *pa, const char *pb, uint32_t lane) {
  using F = FusedFold<G, OP>;
  using A = typename F::A;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  A acc = F::R::identity();
  if (lane < (uint32_t)p.nvec) {
    const bool abc = p.a_bcast, bbc = p.b_bcast;
    const uint32_t e0 = lane * V;
    const char *qa = pa + (abc ? 0 : (int64_t)e0 * (int64_t)sizeof(SAt));
    const char *qb = pb + (bbc ? 0 : (int64_t)e0 * (int64_t)sizeof(SBt));
    const uint32_t left = (uint32_t)p.n0 - e0;
    if (left >= (uint32_t)V) {
      Pack<SAt, V> va;
      Pack<SBt, V> vb;
      fused_load<SAt, V>(qa, abc, va);
      fused_load<SBt, V>(qb, bbc, vb);
#pragma unroll
      for (int i = 0; i < V; ++i) acc = F::add(acc, va.v[i], vb.v[i]);
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < (int)left)
          acc = F::add(acc, reinterpret_cast<const SAt *>(qa)[abc ? 0 : i], reinterpret_cast<const SBt *>(qb)[bbc ? 0 : i]);
    }
  }
  return acc;
}

template <class G, int OP> __global__ __launch_bounds__(kBlock) void fred_rows_short_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using A = typename F::A;
  const uint32_t width = (uint32_t)p.group;
  const uint32_t gl = blockIdx.x * kBlock + threadIdx.x;
  const uint32_t o = gl >> (__ffs(p.group) - 1), lane = gl & (width - 1);
  const bool active = o < (uint32_t)p.nout;
  A acc = R::identity();
  int64_t off_o = 0;
  if (active) {
    int64_t off_a, off_b;
    kept_offsets2(p, o, off_a, off_b, off_o);
    if (p.vec > 1) acc = fred_short_row<G, OP, G::V>(p, p.a + off_a, p.b + off_b, lane);
    else acc = fred_short_row<G, OP, 1>(p, p.a + off_a, p.b + off_b, lane);
  }
  acc = group_fold<R>(acc, (int)width);
  if (active && lane == 0) store_result<A>(p.out + off_o, p.out_dtype, acc);
}

// ---------------------------------------------------------------------------------------
// cols: a kept axis is the fastest of the inputs; lanes own output columns
// ---------------------------------------------------------------------------------------

// NT: inputs that are not broadcast are read with streaming loads (one 16-byte piece per lane each).
// BC: the input that is broadcast along the columns (1: a, 2: b, 0: neither); -1: told at run time, for
// several reduced dims and for columns taken one per lane.  With one reduced dim, row r lies r strides
// further on (no index decomposition).
//
// Bound by how many rows a wavefront has in flight.  A broadcast input lands in the first slot of its
// vector and is spread out once all loads of the trip are issued: spread right away, in a branch on
// a flag, every row's loads were waited for before the next row's were issued (fp32 [16384, 1000] times
// a column 18.0 -> 14.4 us, double [31614, 512] 36.7 -> 26.7, fp32 [1712, 22] 12.4 -> 6.7; 4.5 TB/s at the
// first).
template <class G, int OP, int V, bool NT, int BC>
OCN_DEV void fred_cols_body(KRedArgs &p, typename FusedFold<G, OP>::A *lds) {
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using A = typename F::A;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1);
  const int wave = tid / kWave;
  const int NW = (int)blockDim.x / kWave;
  const bool abc = BC >= 0 ? BC == 1 : p.a_bcast != 0, bbc = BC >= 0 ? BC == 2 : p.b_bcast != 0;

  uint32_t b = blockIdx.x;
  const uint32_t per_split = (uint32_t)(p.colblocks_div.d * (uint32_t)(p.nout / p.nc));
  const uint32_t s = b / per_split;
  b -= s * per_split;
  const uint32_t other = rfastdiv(b, args_div(p.colblocks_div));
  const uint32_t cb = b - other * p.colblocks_div.d;
  // p.cpw lanes (a power of two) cover one row of columns; with fewer than 64 of them a
  // wavefront takes 64 / cpw rows at a time
  const int cpw_log2 = __ffs(p.cpw) - 1;
  const int lc = lane & (p.cpw - 1), lr = lane >> cpw_log2;
  const int RPW = kWave >> cpw_log2;
  int64_t col0 = ((int64_t)cb * p.cpw + lc) * V;
  const int64_t left = p.nc - col0;
  int ncol = left >= V ? V : (left > 0 ? (int)left : 0);
  int skip = 0;   // columns of the last lane's vector that are its neighbour's (as in red_cols_kernel)
  if (ncol > 0 && ncol < V && p.nc >= V) {
    skip = V - ncol;
    col0 -= skip;
    ncol = V;
  }

  int64_t off_a = abc ? 0 : col0 * (int64_t)sizeof(SAt), off_b = bbc ? 0 : col0 * (int64_t)sizeof(SBt);
  int64_t off_o = col0 * p.kso[0];
  {
    uint32_t o = other;
    const int nkept = p.nkept;
    for (int k = 1; k < nkept; ++k) {
      const uint32_t q = (k == nkept - 1) ? 0u : rfastdiv(o, args_div(p.kdiv[k]));
      const uint32_t i = o - q * p.kdiv[k].d;
      o = q;
      off_a += (int64_t)i * p.ksa[k];
      off_b += (int64_t)i * p.ksb[k];
      off_o += (int64_t)i * p.kso[k];
    }
  }
  A acc[V];
#pragma unroll
  for (int i = 0; i < V; ++i) acc[i] = R::identity();
  const int64_t r0 = (int64_t)s * p.chunk;
  int64_t r1 = r0 + p.chunk;
  if (r1 > p.nredtot) r1 = p.nredtot;
  // each wavefront takes one contiguous run of the workgroup's rows, RPW rows at a time (as in
  // red_cols_kernel: rows dealt out in turn measured 10 % slower there)
  const int RS = RPW;
  const int64_t per_wave = (((r1 - r0) + NW - 1) / NW + RPW - 1) / RPW * RPW;
  const int64_t w0 = r0 + (int64_t)wave * per_wave;
  if (w0 + per_wave < r1) r1 = w0 + per_wave;
  int64_t r = w0 + lr;
  if constexpr (BC >= 0) {
    if (ncol == V) {
      // Rows in flight (eight of 16 bytes: the same).  Counts take 16 columns per lane, four pieces or more
      // per row and input that share lines; rows of two such inputs go one at a time (== over floats
      // [3000, 4096] 35 us with two, 25 so).
      constexpr int W = V * (int)(sizeof(SAt) > sizeof(SBt) ? sizeof(SAt) : sizeof(SBt)), U = W <= 16 ? 4 : BC == 0 ? 1 : 2;
      const int64_t sa = (int64_t)RS * p.rsa[0], sb = (int64_t)RS * p.rsb[0];
      const char *qa = p.a + off_a + r * p.rsa[0], *qb = p.b + off_b + r * p.rsb[0];
      auto load = [&](const char *ra, const char *rb, Pack<SAt, V> &va, Pack<SBt, V> &vb) {
        if constexpr (BC == 1) va.v[0] = *reinterpret_cast<const SAt *>(ra);
        else load_vec<SAt, V, NT && sizeof(SAt) * V == 16>(ra, va);
        if constexpr (BC == 2) vb.v[0] = *reinterpret_cast<const SBt *>(rb);
        else load_vec<SBt, V, NT && sizeof(SBt) * V == 16>(rb, vb);
      };
      auto add = [&](const Pack<SAt, V> &va, const Pack<SBt, V> &vb) {
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = F::add(acc[i], va.v[BC == 1 ? 0 : i], vb.v[BC == 2 ? 0 : i]);
      };
      for (; r + (int64_t)(U - 1) * RS < r1; r += RS * U) {
        Pack<SAt, V> va[U];
        Pack<SBt, V> vb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          load(qa, qb, va[u], vb[u]);
          qa += sa;
          qb += sb;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) add(va[u], vb[u]);
      }
      for (; r < r1; r += RS) {
        Pack<SAt, V> va;
        Pack<SBt, V> vb;
        load(qa, qb, va, vb);
        qa += sa;
        qb += sb;
        add(va, vb);
      }
    }
  } else if (ncol == V) {
    constexpr int U = 2;
    for (; r + (int64_t)(U - 1) * RS < r1; r += RS * U) {
      Pack<SAt, V> va[U];
      Pack<SBt, V> vb[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        int64_t oa, ob;
        reduced_offset2(p, (uint32_t)(r + (int64_t)u * RS), 0, oa, ob);
        fused_load<SAt, V>(p.a + off_a + oa, abc, va[u]);
        fused_load<SBt, V>(p.b + off_b + ob, bbc, vb[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < V; ++i) acc[i] = F::add(acc[i], va[u].v[i], vb[u].v[i]);
    }
  }
  if (ncol > 0) {  // remaining rows, and fewer columns than a vector holds
    for (; r < r1; r += RS) {
      int64_t oa, ob;
      reduced_offset2(p, (uint32_t)r, 0, oa, ob);
      const char *qa = p.a + off_a + oa, *qb = p.b + off_b + ob;
#pragma unroll
      for (int i = 0; i < V; ++i)
        if (i < ncol)
          acc[i] = F::add(acc[i], reinterpret_cast<const SAt *>(qa)[abc ? 0 : i],
                          reinterpret_cast<const SBt *>(qb)[bbc ? 0 : i]);
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
  // combine the wavefronts: CH columns per barrier, wavefront c folds column c (as red_cols_kernel)
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
        store_result<A>(p.out + off_o + (int64_t)i * p.kso[0], p.out_dtype, v);
      } else {
        const int64_t olin = (int64_t)other * p.nc + col0 + i;
        reinterpret_cast<typename R::P *>(p.partial)[(int64_t)s * p.nout + olin] = to_storage<R::ACC>(v);
      }
    }
    if (i0 + CH < V) __syncthreads();
  }
}

// A kernel per form (BC and NT as above): in one kernel each form paid for the registers of the others, and
// counts of comparisons spilled up to 52 (== over floats [4000, 333] 31 -> 27 us, |a| > |b| over complex floats
// [16384, 1000] against a row 37 -> 29).  Seven are spilled still where such moduli are compared with a
// column; the form for several dims, which spills none, takes 19.8 us for [65536, 37], 16.9 so.
// Elements of 16 bytes gain from the forms only where one input is broadcast (complex double
// products of [4000, 333] with a column 12.3 -> 11.3 us; of two matrices [800, 20000] 94 -> 103).
template <class G, int BC> constexpr bool fred_cols_form() { return G::V > 1 || BC > 0; }
template <class G, int OP, int BC, bool NT = false> __global__ __launch_bounds__(kColsMaxWaves * kWave) void fred_cols_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using A = typename FusedFold<G, OP>::A;
  extern __shared__ __align__(16) unsigned char fred_cols_lds_raw[];
  A *lds = reinterpret_cast<A *>(fred_cols_lds_raw);
  if constexpr (BC >= 0) fred_cols_body<G, OP, G::V, NT, BC>(p, lds);
  else if (p.vec > 1) fred_cols_body<G, OP, G::V, false, -1>(p, lds);
  else fred_cols_body<G, OP, 1, false, -1>(p, lds);
}

// ---------------------------------------------------------------------------------------
// strips: dense blocks of narrow rows (strip_kernels.hpp)
// ---------------------------------------------------------------------------------------

// BC: the input that is one element per row (1: a, 2: b); 0: both are dense blocks.  A vector lies in
// one row or two (rows hold at least a vector where an input is one element per row).
template <class G, int OP, int BC> __global__ __launch_bounds__(kStripLanes) void fred_strip_cols_kernel(const RedStripArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KStripArgs &p = *(KStripArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using A = typename F::A;
  using St = typename G::SAt;
  static_assert(sizeof(typename G::SAt) == sizeof(typename G::SBt), "equal input types");
  constexpr uint32_t V = 16 / sizeof(St);
  struct Buf { Pack<St, V> a, b; };   // (of an input with one element per row: the elements of the vector's first row and of the next)
  extern __shared__ __align__(16) unsigned char strip_lds[];
  A *lds = reinterpret_cast<A *>(strip_lds);
  const uint32_t tid = threadIdx.x, lanes = p.lanes;
  const uint32_t gl = __umulhi(tid, p.lanes_m), l = tid - gl * lanes, g = blockIdx.x * p.groups + gl;
  A acc[V];
#pragma unroll
  for (uint32_t i = 0; i < V; ++i) acc[i] = R::identity();
  if (gl < p.groups && g < p.ngroups) {
    const StripBlock k = strip_block(p, g);
    const uint32_t width = p.width, n = k.rows * width, full = n / V;
    const uint32_t ro = rfastdiv(l * V, args_div(p.width_div)), cut = (ro + 1) * width - l * V, per_trip = rfastdiv(lanes * V, args_div(p.width_div));
    const int64_t skip = (int64_t)k.row0 * (int64_t)(width * sizeof(St));
    const char *pa = p.a + k.a + (BC == 1 ? (int64_t)k.row0 * p.rs : skip), *pb = p.b + k.b + (BC == 2 ? (int64_t)k.row0 * p.rs : skip);
    auto per_row = [&](const char *src, uint32_t trip, Pack<St, V> &v) {
      const uint32_t r = trip * per_trip + ro;
      v.v[0] = *reinterpret_cast<const St *>(src + (int64_t)r * p.rs);
      if constexpr (V > 1) v.v[1] = *reinterpret_cast<const St *>(src + (int64_t)(r + 1 < k.rows ? r + 1 : r) * p.rs);
    };
    auto add = [&](uint32_t i, const Buf &v) {
      const uint32_t at = V > 1 && i >= cut ? 1 : 0;
      acc[i] = F::add(acc[i], v.a.v[BC == 1 ? at : i], v.b.v[BC == 2 ? at : i]);
    };
    strip_walk<Buf>(
        l, lanes, full,
        [&](uint32_t t, uint32_t trip, Buf &v) {
          if constexpr (BC == 1) per_row(pa, trip, v.a);
          else load_vec<St, V, false>(pa + (uint64_t)t * 16u, v.a);
          if constexpr (BC == 2) per_row(pb, trip, v.b);
          else load_vec<St, V, false>(pb + (uint64_t)t * 16u, v.b);
        },
        [&](uint32_t, Buf &v) {
#pragma unroll
          for (uint32_t i = 0; i < V; ++i) add(i, v);
        });
    if (V > 1 && full * V < n && full % lanes == l) {   // the elements behind the last whole vector
      Buf v;
      const uint32_t trip = full / lanes;
      if constexpr (BC == 1) per_row(pa, trip, v.a);
      if constexpr (BC == 2) per_row(pb, trip, v.b);
#pragma unroll
      for (uint32_t i = 0; i < V - 1; ++i) {
        const uint64_t at = (uint64_t)(full * V + i < n ? full * V + i : n - 1) * sizeof(St);
        if constexpr (BC != 1) v.a.v[i] = *reinterpret_cast<const St *>(pa + at);
        if constexpr (BC != 2) v.b.v[i] = *reinterpret_cast<const St *>(pb + at);
      }
#pragma unroll
      for (uint32_t i = 0; i < V - 1; ++i)
        if (full * V + i < n) add(i, v);
    }
  }
#pragma unroll
  for (uint32_t i = 0; i < V; ++i) lds[tid * V + i] = acc[i];
  strip_fold<R>(p, lds, lanes * V);
}

// BC: the input that has one row for all rows (1: a, 2: b), whose elements a lane keeps: it has the same
// columns on every trip; 0: both are dense blocks.
template <class G, int OP, int BC> __global__ __launch_bounds__(kBlock) void fred_strip_rows_kernel(const RedStripArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KStripArgs &p = *(KStripArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  using F = FusedFold<G, OP>;
  using R = typename F::R;
  using St = typename G::SAt;
  using Mt = typename G::SOt;
  constexpr uint32_t V = 16 / sizeof(St);
  struct Buf { Pack<St, V> a, b; };
  extern __shared__ __align__(16) unsigned char strip_lds[];
  Mt *lds = reinterpret_cast<Mt *>(strip_lds);
  const StripBlock k = strip_block(p, blockIdx.x);
  const uint32_t width = p.width, n = k.rows * width, full = n / V, tid = threadIdx.x, lanes = p.lanes;
  const int64_t skip = (int64_t)k.row0 * (int64_t)(width * sizeof(St));
  const char *pa = p.a + k.a + (BC == 1 ? 0 : skip), *pb = p.b + k.b + (BC == 2 ? 0 : skip);
  Pack<St, V> row;
  if constexpr (BC != 0) {
#pragma unroll
    for (uint32_t i = 0; i < V; ++i) {
      const uint32_t e = tid * V + i, c = e - rfastdiv(e, args_div(p.width_div)) * width;
      row.v[i] = reinterpret_cast<const St *>(BC == 1 ? pa : pb)[c];
    }
  }
  auto eval = [&](uint32_t i, const Buf &v) { return G::eval(BC == 1 ? row.v[i] : v.a.v[i], BC == 2 ? row.v[i] : v.b.v[i]); };
  if (tid < lanes) {
    strip_walk<Buf>(
        tid, lanes, full,
        [&](uint32_t t, uint32_t, Buf &v) {
          if constexpr (BC != 1) load_vec<St, V, false>(pa + (uint64_t)t * 16u, v.a);
          if constexpr (BC != 2) load_vec<St, V, false>(pb + (uint64_t)t * 16u, v.b);
        },
        [&](uint32_t trip, Buf &v) {
          Pack<Mt, V> m;
#pragma unroll
          for (uint32_t i = 0; i < V; ++i) m.v[i] = eval(i, v);
          reinterpret_cast<Pack<Mt, V> *>(strip_lds)[tid + trip * lanes] = m;
        });
  }
  if (V > 1 && full * V + tid < n) {   // the elements behind the last whole vector
    const uint32_t e = full * V + tid, c = e - rfastdiv(e, args_div(p.width_div)) * width;
    lds[e] = G::eval(reinterpret_cast<const St *>(pa)[BC == 1 ? c : e], reinterpret_cast<const St *>(pb)[BC == 2 ? c : e]);
  }
  strip_rows_fold<R>(p, k, [&](uint32_t e) { return R::lift(from_storage<G::SO_DT>(lds[e])); });
}

// ---------------------------------------------------------------------------------------
// generic: any layout, one output per lane
// ---------------------------------------------------------------------------------------

template <class G, int OP> __global__ __launch_bounds__(kBlock) void fred_generic_kernel(const RedArgs by_value) {
  (void)by_value;  // read through the kernarg segment, which can be indexed at run time
  KRedArgs &p = *(KRedArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  if (p.warm) warm_arguments<RedArgs>();
  using F = FusedFold<G, OP>;
  using A = typename F::A;
  using SAt = typename G::SAt;
  using SBt = typename G::SBt;
  // the grid is capped (a launch cannot have 2^32 lanes): more outputs than lanes loop
  for (int64_t o = (int64_t)blockIdx.x * kBlock + threadIdx.x; o < p.nout; o += (int64_t)gridDim.x * kBlock) {
  int64_t off_a = 0, off_b = 0, off_o = 0, t = o;
  for (int k = 0; k < p.nkept; ++k) {
    const int64_t n = p.ksize[k];
    const int64_t q = t / n;
    const int64_t i = t - q * n;
    t = q;
    off_a += i * p.ksa[k];
    off_b += i * p.ksb[k];
    off_o += i * p.kso[k];
  }
  A acc = F::R::identity();
  for (int64_t r = 0; r < p.nredtot; ++r) {
    int64_t oa = 0, ob = 0, q = r;
    for (int k = 0; k < p.nred; ++k) {
      const int64_t n = p.rsize[k];
      const int64_t qq = q / n;
      oa += (q - qq * n) * p.rsa[k];
      ob += (q - qq * n) * p.rsb[k];
      q = qq;
    }
    acc = F::add(acc, *reinterpret_cast<const SAt *>(p.a + off_a + oa), *reinterpret_cast<const SBt *>(p.b + off_b + ob));
  }
  store_result<A>(p.out + off_o, p.out_dtype, acc);
  }
}

#endif  // __HIPCC__

}  // namespace ocn
