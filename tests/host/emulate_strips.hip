// Host-side emulation of the strip kernels' arithmetic (no GPU needed): reductions over dense blocks of narrow
// rows, plain and fused, as plan_reduce and plan_binary_reduce hand them to strip columns, strip rows and runs.
//
// For random calls of every element size - one block or many, other kept dims in any order, reversed, stepped or
// broadcast, outputs permuted, reversed and with gaps, bases off by a few elements, a lowered launch limit - it
// replays every workgroup, lane and trip with the arguments that the launch gets.  An element is stood for by a
// hash of its address (of a fused call: of both), an output by the sum of its elements', and it checks that
//   * every output is written once and holds what the tensors' sizes and strides say it does,
//   * whole vectors and single elements are read inside the tensor, streamed ones on their boundary,
//   * LDS is addressed inside what the launch asks for, and that is what a workgroup may have,
//   * every partial result is written once, inside the workspace, and the second launch's plan reads it.
// Exit code 0 when every case passes and every form has been met.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <vector>

#include "../../paper_1810_08723_amd/csrc/red_launch.hpp"

using namespace ocn;

static uint64_t rng_state = 0x13198A2E03707344ull;
static uint32_t rnd() {
  rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)(rng_state >> 33);
}
static int rnd_in(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }
static int64_t rnd_log(double lo, double hi) { return (int64_t)(lo * std::exp(std::log(hi / lo) * (rnd() % 10000) / 10000.0)); }

static uint64_t mix(uint64_t x) {
  x *= 0x9E3779B97F4A7C15ull;
  return (x ^ (x >> 29)) * 0xBF58476D1CE4E5B9ull;
}

// bytes of the accumulators in registers and LDS
template <int... I> static size_t acc_bytes(int op, int dt, std::integer_sequence<int, I...>) {
  size_t r = 0;
  ((I == op * DT_COUNT + dt ? (void)(r = [] {
    constexpr int o = I / DT_COUNT, s = I % DT_COUNT;
    if constexpr (red_supported(o, s)) return sizeof(typename Reducer<s, o>::A);
    else return (size_t)0;
  }()) : (void)0), ...);
  return r;
}
static size_t acc_bytes(int op, int dt) { return acc_bytes(op, dt, std::make_integer_sequence<int, R_COUNT * DT_COUNT>{}); }

struct Extent { int64_t lo, hi; };   // bytes that a view's elements lie in
static Extent extent(const ocn_tensor &t) {
  Extent e{(int64_t)(intptr_t)t.base + t.offset, (int64_t)(intptr_t)t.base + t.offset + dt_size(t.dtype)};
  for (int d = 0; d < t.ndim; ++d) (t.stride[d] < 0 ? e.lo : e.hi) += (t.size[d] - 1) * t.stride[d];
  return e;
}

using Written = std::vector<std::pair<int64_t, uint64_t>>;   // address, value

struct Replay {
  const RedPlan &p;
  const RedStripArgs &q;
  Extent a, b;
  size_t lds_bytes, abytes;
  Written outs, partials;
  const char *fault = nullptr;
  int es, V, mes;

  bool check(bool ok, const char *what) {
    if (!ok && !fault) fault = what;
    return ok;
  }
  uint64_t read(const char *at, int n, const Extent &e, bool nt) {   // n elements from `at` on
    const int64_t x = (int64_t)(intptr_t)at;
    check(x >= e.lo && x + n * es <= e.hi, "a read outside the tensor");
    check(!nt || x % 16 == 0, "a streamed vector off its boundary");
    return (uint64_t)x;
  }
  uint64_t value(uint64_t xa, uint64_t xb) const { return p.fused ? mix(xa + 3 * mix(xb)) : mix(xa); }

  struct Block { const char *a, *b; int64_t o; uint32_t row0, rows, split, other; };
  Block block(uint32_t g) const {
    Block k;
    k.other = fastdiv_host(g, q.split_div);
    k.split = g - k.other * q.split_div.d;
    k.row0 = k.split * q.chunk;
    k.rows = k.row0 + q.chunk < q.rows ? q.chunk : q.rows - k.row0;
    k.a = q.a;
    k.b = q.b;
    k.o = 0;
    uint32_t t = k.other;
    for (uint32_t d = 0; d < q.nother; ++d) {
      const uint32_t r = d + 1 == q.nother ? 0u : fastdiv_host(t, q.odiv[d]);
      const int64_t i = t - r * q.odiv[d].d;
      t = r;
      k.a += i * q.osa[d];
      k.b += i * q.osb[d];
      k.o += i * q.oso[d];
    }
    return k;
  }
  void put(int64_t o, uint32_t split, int64_t lin, uint64_t v) {
    if (q.split_div.d == 1) outs.push_back({(int64_t)(intptr_t)q.out + o, v});
    else partials.push_back({(int64_t)split * q.psplit + lin * q.pstep, v});
  }

  void cols() {
    const bool nt = (q.flags & kStripNt) && !(q.flags & kStripSwapA);
    const uint32_t nl = (uint32_t)p.block, per_group = q.lanes * (uint32_t)V;
    std::vector<uint64_t> lds((size_t)nl * V);
    check(lds.size() * abytes <= lds_bytes, "LDS of the columns");
    for (int64_t wg = 0; wg < p.grid && !fault; ++wg) {
      std::fill(lds.begin(), lds.end(), 0);
      for (uint32_t tid = 0; tid < nl; ++tid) {
        const uint32_t gl = (uint32_t)(((uint64_t)tid * q.lanes_m) >> 32), l = tid - gl * q.lanes, g = (uint32_t)wg * q.groups + gl;
        check(l < q.lanes, "a lane beyond its group");
        if (!(gl < q.groups && g < q.ngroups)) continue;
        const Block k = block(g);
        const uint32_t n = k.rows * q.width, full = n / V;
        const uint32_t ro = fastdiv_host(l * V, q.width_div), cut = (ro + 1) * q.width - l * V, per_trip = fastdiv_host(per_group, q.width_div);
        const int64_t skip = (int64_t)k.row0 * q.width * es;
        const char *pa = k.a + (q_bc() == 1 ? (int64_t)k.row0 * q.rs : skip), *pb = k.b + (q_bc() == 2 ? (int64_t)k.row0 * q.rs : skip);
        auto element = [&](uint32_t t, uint32_t trip, uint32_t i, bool single) {
          auto one = [&](const char *src, bool per_row, const Extent &e, bool stream) {
            if (!per_row) return (single ? read(src + ((int64_t)t * V + i) * es, 1, e, false) : read(src + (int64_t)t * 16, V, e, stream) + (uint64_t)i * es);
            const uint32_t r = trip * per_trip + ro;
            const uint32_t at = V > 1 && i >= cut ? (r + 1 < k.rows ? r + 1 : r) : r;
            read(src + (int64_t)r * q.rs, 1, e, false);
            return read(src + (int64_t)at * q.rs, 1, e, false);
          };
          const uint64_t xa = one(pa, q_bc() == 1, a, nt), xb = p.fused ? one(pb, q_bc() == 2, b, false) : 0;
          lds[(size_t)tid * V + i] += value(xa, xb);
        };
        uint32_t trip = 0;
        for (uint32_t t = l; t < full; t += q.lanes, ++trip)
          for (uint32_t i = 0; i < (uint32_t)V; ++i) element(t, trip, i, false);
        if (V > 1 && full * V < n && full % q.lanes == l)
          for (uint32_t i = 0; full * V + i < n; ++i) element(full, full / q.lanes, i, true);
      }
      // the fold
      const uint32_t outs_n = q.outs_div.d, addends = fastdiv_host(per_group, q.nog_div);
      auto fold = [&](uint32_t part, uint32_t o) {
        const uint32_t g = fastdiv_host(o, q.nog_div), j = o - g * q.nog;
        uint64_t v = 0;
        for (uint32_t e = part; e < addends; e += q.parts) {
          const uint32_t x = q.inner == 1 ? e * q.width : fastdiv_host(e, q.inner_div) * q.width + e % q.inner;
          const size_t at = (size_t)g * per_group + j * q.inner + x;
          if (check(at < lds.size(), "the fold reads beyond LDS")) v += lds[at];
        }
        return v;
      };
      check(q.parts == 1 || outs_n * q.parts <= nl, "more parts than lanes");
      for (uint32_t o = 0; o < outs_n; ++o) {
        uint64_t v = 0;
        for (uint32_t part = 0; part < q.parts; ++part) v += fold(part, o);
        const uint32_t g = fastdiv_host(o, q.nog_div), j = o - g * q.nog, gi = (uint32_t)wg * q.groups + g;
        if (gi >= q.ngroups) continue;
        const Block k = block(gi);
        put(k.o + (int64_t)j * q.kso, k.split, (int64_t)k.other * q.nog + j, v);
      }
    }
  }

  void rows() {
    const bool nt = (q.flags & kStripNt) != 0;
    const uint32_t lanes = p.fused ? q.lanes : (uint32_t)kBlock, width = q.width;
    std::vector<uint64_t> lds(lds_bytes / mes);
    std::vector<char> filled(lds.size());
    check(lds_bytes % 16 == 0 && lanes <= (uint32_t)kBlock, "LDS of the rows");
    for (int64_t wg = 0; wg < p.grid && !fault; ++wg) {
      std::fill(filled.begin(), filled.end(), 0);
      const Block k = block((uint32_t)wg);
      const uint32_t n = k.rows * width, full = n / V;
      const int64_t skip = (int64_t)k.row0 * width * es;
      const char *pa = k.a + (q_bc() == 1 ? 0 : skip), *pb = k.b + (q_bc() == 2 ? 0 : skip);
      auto store = [&](size_t at, uint64_t v) {
        if (check(at < lds.size() && !filled[at], "a row's element beyond LDS or twice")) lds[at] = v, filled[at] = 1;
      };
      for (uint32_t tid = 0; tid < lanes; ++tid)
        for (uint32_t t = tid, trip = 0; t < full; t += lanes, ++trip)
          for (uint32_t i = 0; i < (uint32_t)V; ++i) {
            const uint32_t c = (tid * V + i) % width;    // of an input with one row for all: what the lane keeps
            const uint64_t xa = q_bc() == 1 ? read(pa + (int64_t)c * es, 1, a, false) : read(pa + (int64_t)t * 16, V, a, nt) + (uint64_t)i * es;
            const uint64_t xb = !p.fused ? 0 : q_bc() == 2 ? read(pb + (int64_t)c * es, 1, b, false) : read(pb + (int64_t)t * 16, V, b, false) + (uint64_t)i * es;
            store((size_t)(tid + trip * lanes) * V + i, value(xa, xb));
          }
      for (uint32_t e = full * V; e < n; ++e) {
        check(e - full * V < (uint32_t)kBlock, "more last elements than lanes");
        const uint32_t c = e - fastdiv_host(e, q.width_div) * width;
        store(e, value(read(pa + (int64_t)(q_bc() == 1 ? c : e) * es, 1, a, false), p.fused ? read(pb + (int64_t)(q_bc() == 2 ? c : e) * es, 1, b, false) : 0));
      }
      check((q.parts & (q.parts - 1)) == 0 && q.parts <= (uint32_t)kWave && (q.rotate & (q.rotate - 1)) == 0, "parts and rotation");
      auto get = [&](size_t e) { return check(e < lds.size() && filled[e], "an element that was never stored") ? lds[e] : 0; };
      for (uint32_t r = 0; r < k.rows; ++r) {
        uint64_t v = 0;
        const uint32_t e0 = r * width, e1 = e0 + width, w0 = e0 / 4, nw = (e1 + 3) / 4 - w0;
        const bool words = es == 1 && !p.fused;
        const uint32_t units = words ? nw : width;
        for (uint32_t part = 0; part < q.parts; ++part) {
          uint32_t c = part + (q.rotate ? (r & (q.rotate - 1)) * q.parts : 0u);
          for (uint32_t i = part; i < units; i += q.parts) {
            if (!check(c < units, "a rotated lane beyond its row")) return;
            if (!words) v += get(e0 + c);
            else {
              const uint32_t m = (c == 0 ? ~0u << (8 * (e0 & 3)) : ~0u) & (c + 1 == nw ? ~0u >> (8 * ((0u - e1) & 3)) : ~0u);
              check((size_t)(w0 + c) * 4 + 4 <= lds_bytes, "a word beyond LDS");
              for (int x = 0; x < 4; ++x)
                if ((m >> (8 * x)) & 0xffu) v += get((size_t)(w0 + c) * 4 + x);
            }
            c = c + q.parts < units ? c + q.parts : part;
          }
        }
        outs.push_back({(int64_t)(intptr_t)q.out + k.o + (int64_t)(k.row0 + r) * q.kso, v});
      }
    }
  }

  void runs() {
    const bool nt = (q.flags & kStripNt) && !(q.flags & kStripSwapA);
    const uint32_t nl = (uint32_t)p.block;
    std::vector<uint64_t> lds((size_t)nl * V);
    check(lds.size() * abytes <= lds_bytes && q.groups * q.lanes <= nl, "LDS of the runs");
    for (int64_t wg = 0; wg < p.grid && !fault; ++wg) {
      std::fill(lds.begin(), lds.end(), 0);
      const uint32_t cb = fastdiv_host((uint32_t)wg, q.split_div), split = (uint32_t)wg - cb * q.split_div.d;
      const uint32_t row0 = split * q.chunk, rows = row0 + q.chunk < q.rows ? q.chunk : q.rows - row0;
      const uint32_t o0 = cb * q.nog, outs_n = o0 + q.nog < q.ngroups ? q.nog : q.ngroups - o0, cw = outs_n * q.inner;
      for (uint32_t tid = 0; tid < nl; ++tid) {
        const uint32_t g = (uint32_t)(((uint64_t)tid * q.lanes_m) >> 32), l = tid - g * q.lanes;
        if (!(g < q.groups && l * V < cw)) continue;
        const int skip = l * V + V > cw ? (int)(l * V + V - cw) : 0;
        const char *base = q.a + ((int64_t)o0 * q.inner + (int64_t)l * V - skip) * es + (int64_t)row0 * q.rs;
        for (uint32_t t = g; t < rows; t += q.groups) {
          const uint64_t x = read(base + (int64_t)t * q.rs, V, a, nt);
          for (int i = skip; i < V; ++i) {
            const size_t at = (size_t)g * cw + l * V + i - skip;
            if (check(at < lds.size(), "a run beyond LDS")) lds[at] += value(x + (uint64_t)i * es, 0);
          }
        }
      }
      check((q.parts & (q.parts - 1)) == 0 && q.parts <= (uint32_t)kWave, "parts of a run");
      for (uint32_t o = 0; o < outs_n; ++o) {
        uint64_t v = 0;
        for (uint32_t g = 0; g < q.groups; ++g)
          for (uint32_t j = 0; j < q.inner; ++j) v += lds[(size_t)g * cw + o * q.inner + j];
        put((int64_t)(o0 + o) * q.kso, split, o0 + o, v);
      }
    }
  }
  int q_bc() const { return p.strip_bc; }

  // the second launch, by its plan: elements of the workspace at a_ptr + strides (the workspace is at `ws`)
  void second(char *ws) {
    const size_t n = (size_t)p.nout * (size_t)p.split;
    std::vector<uint64_t> at(n);
    std::vector<char> filled(n);
    for (const auto &w : partials) {
      if (!check(w.first >= 0 && (size_t)w.first < n && !filled[w.first], "a partial result outside its place or twice")) return;
      at[w.first] = w.second;
      filled[w.first] = 1;
    }
    check(partials.size() == n, "a partial result is missing");
    check(p.workspace_bytes >= n * dt_size(p.acc_dtype), "the workspace is too small");
    RedPlan s;
    plan_second_pass(p, ws, &s);
    const int pes = dt_size(p.acc_dtype);
    check(s.nout == p.nout && s.nredtot == p.split, "the second launch's sizes");
    if (s.fold) check(!p.partial_rows && s.nkept == 1 && s.kstride_a[0] == pes && (s.nred == 0 || s.rstride_a[0] == p.nout * pes), "the fold's layout");
    for (int64_t o = 0; o < s.nout && !fault; ++o) {
      int64_t ka = 0, ko = 0, rem = o;
      for (int d = s.nkept - 1; d >= 0; --d) {
        ka += rem % s.ksize[d] * s.kstride_a[d];
        ko += rem % s.ksize[d] * s.kstride_o[d];
        rem /= s.ksize[d];
      }
      uint64_t v = 0;
      for (int64_t r = 0; r < s.nredtot; ++r) {
        int64_t x = s.a_ptr - ws + ka, rr = r;
        for (int d = s.nred - 1; d >= 0; --d) {
          x += rr % s.rsize[d] * s.rstride_a[d];
          rr /= s.rsize[d];
        }
        if (!check(x >= 0 && x % pes == 0 && (size_t)(x / pes) < n, "the second launch reads outside the workspace")) return;
        v += at[x / pes];
      }
      outs.push_back({(int64_t)(intptr_t)s.out_ptr + ko, v});
    }
  }
};

// A view of the sizes whose dims lie in memory in the given order (slowest first); of `gap` dims only every second
// index is in the view, and `reversed` ones run backwards.
static ocn_tensor make_view(int dt, int ndim, const int64_t *sizes, const int *order, unsigned gap, unsigned reversed, uint64_t base) {
  ocn_tensor t;
  std::memset(&t, 0, sizeof t);
  const int64_t es = dt_size(dt);
  t.base = (void *)base;
  t.dtype = dt;
  t.ndim = ndim;
  t.offset = rnd() % 2 ? 0 : es * rnd_in(1, 17);
  int64_t acc = es;
  for (int k = ndim - 1; k >= 0; --k) {
    const int d = order[k];
    if (gap >> d & 1) acc *= 2;
    t.size[d] = sizes[d];
    t.stride[d] = acc;
    acc *= sizes[d];
    if (reversed >> d & 1) {
      t.offset += (sizes[d] - 1) * t.stride[d];
      t.stride[d] = -t.stride[d];
    }
  }
  return t;
}

static int g_seen[4][3], g_split, g_partial_rows, g_rotate, g_swap, g_parts, g_words;

static int one_case(int case_no) {
  static const int kinds[] = {DT_BOOL, DT_I8, DT_U8, DT_I16, DT_F16, DT_I32, DT_F32, DT_F64, DT_I64, DT_C16, DT_C32, DT_C64};
  const bool fused = case_no && rnd() % 3 == 0;
  static const int fused_kinds[] = {DT_I32, DT_I64, DT_F16, DT_F32, DT_F64, DT_C32, DT_C64};
  const int dt = fused ? fused_kinds[rnd() % 7] : case_no ? kinds[rnd() % 12] : (int)DT_I8, es = dt_size(dt);
  const int bytes_small = es == 1 && !fused;
  set_max_launch_blocks(case_no && rnd() % 6 == 0 ? rnd_log(40, 4000) : 0);
  // sizes: dims 0.. of other blocks, then the block
  int ndim = 0, axes_n = 0, shape = case_no ? rnd_in(0, 5) : 2;
  int64_t size[8];
  int32_t axes[8];
  int order[8], narrow_from = 0;
  if (fused && shape >= 4) shape -= 3;
  int64_t total = rnd_log((bytes_small ? 2.1 : 0.3) * (1 << 20), 5 * (double)(1 << 20)) / es;
  int64_t width = shape == 5 ? rnd_log(32 * (16 / es) + 1, 6000) : rnd() % 3 ? rnd_log(2, 120) : rnd_log(2, 1100);
  if (shape == 2 && (case_no == 0 || (rnd() % 8 == 0 && es >= 4))) {   // rows in whole vectors, a multiple of eight LDS banks apart
    width = 32 / es * rnd_in(1, 16);
    total = (es == 1 ? (int64_t)49 << 20 : (int64_t)12700 << 10) / es;
  }
  if (shape == 5) total = std::max<int64_t>(total, (es == 1 ? (int64_t)4200 << 10 : (int64_t)2100 << 10) / es);
  auto add = [&](int64_t n, bool reduced) {
    if (reduced) axes[axes_n++] = ndim;
    size[ndim] = std::max<int64_t>(1, n);
    return ndim++;
  };
  switch (shape) {
    case 0: add(total / width, true); narrow_from = ndim - 1; add(width, false); break;                                    // columns of one block
    case 1: {                                                                                                          // ... of many
      const int64_t rows = rnd_log(2, std::max<double>(3, total / width / 2));
      if (rnd() % 3 == 0) add(rnd_in(2, 5), false);
      add(total / width / rows / (ndim ? size[0] : 1), false);
      narrow_from = add(rows, true);
      add(width, false);
      break;
    }
    case 2: {                                                                                                          // rows
      const int64_t w = std::min<int64_t>(width, 1100 / es);
      if (rnd() % 3 == 0) add(rnd_in(2, 7), false);
      const int64_t rows = ndim ? rnd_log(5, 3000) : total / w;
      if (ndim) add(total / w / rows / size[0], false);
      narrow_from = add(rows, false);
      add(w, true);
      break;
    }
    case 3: {                                                                                                          // runs of columns
      const int64_t inner = rnd_in(2, 40), kept = std::max<int64_t>(2, width / inner);
      narrow_from = add(total / (inner * kept), true);
      add(kept, false);
      add(inner, true);
      break;
    }
    case 4: {                                                                                                          // an axis of one element
      add(rnd_in(1, 5), false);
      narrow_from = add(total / size[0], false);
      add(1, true);
      break;
    }
    default: {                                                                                                         // runs of long rows
      const int64_t inner = rnd_in(2, 66), kept = width / inner + 2;
      narrow_from = add(std::max<int64_t>(rnd() % 4 ? 301 : 140, total / (inner * kept)), true);
      add(kept, false);
      add(inner, true);
    }
  }
  for (int d = 0; d < ndim; ++d) order[d] = d;
  if (narrow_from > 1 && rnd() % 2) std::swap(order[0], order[1]);
  // dims before the block keep any distance, the block's own are dense (the rows of runs too may lie apart)
  const unsigned loose = ((1u << narrow_from) - 1) | (shape == 5 ? 1u : 0u);
  const unsigned gap = rnd() % 3 ? 0 : rnd() & loose, reversed = rnd() % 3 ? 0 : rnd() & ((1u << ndim) - 1);
  ocn_tensor a = make_view(dt, ndim, size, order, gap, reversed, 0x100000000000ull), b;
  int ew = B_MUL, mid = dt;
  static const int ops[] = {R_SUM, R_SUM, R_MAX, R_ANY, R_PROD, R_MIN, R_ALL};
  int op = fused ? R_SUM : ops[rnd() % 7];
  if (fused) {
    if (rnd() % 3 == 0 && dt_kind(dt) != K_CPLX) {
      ew = B_LT;
      mid = DT_BOOL;
      op = rnd() % 2 ? R_SUM : R_ANY;
    }
    b = make_view(dt, ndim, size, order, gap, reversed, 0x200000000000ull);
    const int lone = rnd_in(0, 2);   // both dense, one element per row, one row for all
    if (lone) {
      int64_t bs[8];
      const int drop = lone == 1 ? ndim - 1 : narrow_from;
      for (int d = 0; d < ndim; ++d) bs[d] = d == drop || (d < narrow_from && rnd() % 2) ? 1 : size[d];
      b = make_view(dt, ndim, bs, order, 0, 0, 0x200000000000ull);
      for (int d = 0; d < ndim; ++d)
        if (bs[d] == 1) b.stride[d] = 0;
    }
    if (rnd() % 2) std::swap(a, b);
  } else if (es > 1 && rnd() % 5 == 0) {
    a.byteswapped = 1;
  }
  if (!red_supported(op, mid)) return 0;
  int64_t osize[8];
  int on = 0, oorder[8];
  for (int d = 0; d < ndim; ++d)
    if (std::find(axes, axes + axes_n, d) == axes + axes_n) osize[on++] = size[d];
  for (int d = 0; d < on; ++d) oorder[d] = d;
  if (rnd() % 4 == 0)
    for (int d = on - 1; d > 0; --d) std::swap(oorder[d], oorder[rnd() % (d + 1)]);
  ocn_tensor out = make_view(reduce_acc_dtype(op, mid), on, osize, oorder, rnd() % 4 ? 0 : rnd() & 7, rnd() % 4 ? 0 : rnd() & 7, 0x300000000000ull);

  RedPlan p;
  char *ws = (char *)0x400000000000ull;
  if (fused) {
    FusedPlan f;
    const int rc = plan_binary_reduce(ew, op, &a, &b, axes, axes_n, &out, mid, ws, &f);
    if (rc != OCN_OK) { std::printf("case %d: fused plan rc=%d\n", case_no, rc); return 1; }
    if (f.unfused) return 0;
    p = f.red;
  } else {
    const int rc = plan_reduce(op, &a, axes, axes_n, &out, &p);
    if (rc != OCN_OK) { std::printf("case %d: plan rc=%d\n", case_no, rc); return 1; }
  }
  if (!p.strip) return 0;
  const RedStripArgs q = make_red_strip_args(p, ws);
  const size_t abytes = acc_bytes(op, mid), lds = p.strip == 2 ? p.strip_lds : (size_t)p.block * (size_t)(16 / es) * abytes;
  Extent ea = extent(a), eb{0, 0};
  if (fused) eb = extent(b);
  Replay r{p, q, ea, eb, lds, abytes, {}, {}, nullptr, es, 16 / es, fused ? dt_size(mid) : es};
  r.check(abytes > 0 && lds <= 65536 && p.block <= (p.strip == 2 ? kBlock : kStripLanes) && p.grid <= max_launch_blocks(), "the launch");
  r.check(fused || p.workspace_bytes <= (size_t)OCN_REDUCE_SCRATCH_BYTES, "more partial results than a call without a workspace has room for");
  if (p.strip == 1) r.cols();
  else if (p.strip == 2) r.rows();
  else r.runs();
  if (!r.fault && p.split > 1) r.second(ws);
  // what the sizes and strides say
  int64_t numel = 1, obase = (int64_t)(intptr_t)out.base + out.offset;
  for (int d = 0; d < ndim; ++d) numel *= size[d];
  Written want;
  std::vector<uint64_t> sums((size_t)p.nout, 0);
  std::vector<int64_t> addr((size_t)p.nout, 0);
  int64_t idx[8] = {0}, xa = (int64_t)(intptr_t)a.base + a.offset, xb = fused ? (int64_t)(intptr_t)b.base + b.offset : 0, lin[8] = {0}, ostride[8] = {0};
  for (int d = ndim - 1, k = on - 1, l = 1; d >= 0; --d)
    if (std::find(axes, axes + axes_n, d) == axes + axes_n) {
      lin[d] = l;
      ostride[d] = out.stride[k];
      l *= (int)osize[k--];
    }
  int64_t ol = 0, oa = obase;
  for (int64_t e = 0; e < numel; ++e) {
    sums[ol] += r.value((uint64_t)xa, (uint64_t)xb);
    addr[ol] = oa;
    for (int d = ndim - 1; d >= 0; --d) {
      ++idx[d];
      xa += a.stride[d];
      if (fused) xb += b.stride[d];
      ol += lin[d];
      oa += ostride[d];
      if (idx[d] < size[d]) break;
      xa -= size[d] * a.stride[d];
      if (fused) xb -= size[d] * b.stride[d];
      ol -= size[d] * lin[d];
      oa -= size[d] * ostride[d];
      idx[d] = 0;
    }
  }
  for (int64_t o = 0; o < p.nout; ++o) want.push_back({addr[o], sums[o]});
  std::sort(want.begin(), want.end());
  std::sort(r.outs.begin(), r.outs.end());
  r.check(want == r.outs, "an output is missing, written twice or not the sum of its elements");
  if (r.fault) {
    std::printf("case %d: %s; form %d, op %d of type %d, fused %d (b %d), split %ld, block %d, sizes", case_no, r.fault, p.strip, op, dt, (int)fused, p.strip_bc, (long)p.split, p.block);
    for (int d = 0; d < ndim; ++d) std::printf(" %ld", (long)size[d]);
    std::printf("\n");
    return 1;
  }
  g_seen[p.strip][fused ? 1 + (p.strip_bc != 0) : 0]++;
  g_split += p.split > 1;
  g_partial_rows += p.split > 1 && p.partial_rows;
  g_rotate += p.strip == 2 && p.strip_rotate > 1;
  g_words += p.strip == 2 && es == 1;
  g_parts += p.strip_parts > 1;
  g_swap += p.swap_a;
  return 0;
}

int main(int argc, char **argv) {
  const int ncases = argc > 1 ? std::atoi(argv[1]) : 300;
  for (int c = 0; c < ncases; ++c)
    if (one_case(c)) return 1;
  std::printf("ok: %d cases; columns %d, fused %d + %d, rows %d, fused %d + %d, runs %d; split %d (%d side by side), words %d, rotated %d, parts %d, other byte order %d\n",
              ncases, g_seen[1][0], g_seen[1][1], g_seen[1][2], g_seen[2][0], g_seen[2][1], g_seen[2][2], g_seen[3][0], g_split, g_partial_rows, g_words, g_rotate, g_parts, g_swap);
  const bool met = g_seen[1][0] && g_seen[1][1] && g_seen[1][2] && g_seen[2][0] && g_seen[2][1] && g_seen[2][2] && g_seen[3][0] > 5 && g_split > g_partial_rows && g_partial_rows &&
                   g_words && g_rotate > 5 && g_parts && g_swap;
  return met ? 0 : 1;
}
