// Host-side emulation of the index arithmetic of ew_rows_kernel (no GPU needed).
//
// For random rows of any length and alignment - inputs contiguous along with the output,
// broadcast along rows or columns, with rows reversed, stepped or in another order, outputs
// contiguous or with gaps, bases off by a few elements - it replays every vector of the launch
// through the kernel's own helpers and the host-built arguments, and checks that
//   * every output element is written exactly once and nothing else is,
//   * every element read belongs to that output position,
//   * a vector moved in one piece is contiguous in that operand and inside its range.
// Rows of more than 2^31 elements (under outer dims) are replayed around columns 2^31 and 2^32 and
// at their ends only.
// Exit code 0 when every case passes.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <vector>

#include "../../paper_1810_08723_amd/csrc/ew_launch.hpp"

using namespace ocn;

static uint64_t rng_state = 0x243F6A8885A308D3ull;
static uint32_t rnd() {
  rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)(rng_state >> 33);
}
static int rnd_in(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }

// An operand whose last dim is contiguous (or broadcast): outer dims in any order and direction,
// with gaps, broadcast dims, and a base that is a multiple of the element size only.
static ocn_tensor make_rows(int dt, int ndim, const int64_t *sizes, char *base, bool is_out) {
  ocn_tensor t;
  std::memset(&t, 0, sizeof t);
  const int es = dt_size(dt);
  t.base = base;
  t.dtype = dt;
  t.ndim = ndim;
  t.offset = (int64_t)es * (rnd() % 3 == 0 ? 0 : rnd_in(0, 17));
  int order[8];
  for (int i = 0; i < ndim; ++i) order[i] = i;
  const int kind = rnd_in(0, 3);
  if (kind == 1 && ndim > 2) std::swap(order[rnd_in(0, ndim - 2)], order[rnd_in(0, ndim - 2)]);
  int64_t acc = es;
  for (int k = ndim - 1; k >= 0; --k) {
    const int d = order[k];
    t.size[d] = sizes[d];
    t.stride[d] = acc;
    acc *= sizes[d];
    if (kind == 2 && rnd() % 2) acc += (int64_t)es * rnd_in(1, 5);   // rows with gaps
  }
  if (!is_out)
    for (int d = 0; d < ndim; ++d) {
      if (rnd() % 4 == 0) { t.size[d] = 1; t.stride[d] = 0; }        // broadcast
      else if (d < ndim - 1 && rnd() % 5 == 0) {                      // reversed
        t.offset += (t.size[d] - 1) * t.stride[d];
        t.stride[d] = -t.stride[d];
      }
    }
  return t;
}

static int g_flat, g_rowform, g_crossing, g_partial, g_linear;

template <int V> static int replay(const EwPlan &p, const RowsArgs &q, int64_t grid, int case_no) {
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), dt_size(p.b.dtype)};
  // canonical plan: output address -> addresses of the inputs
  std::map<int64_t, std::pair<int64_t, int64_t>> want;
  std::vector<int64_t> idx(p.ndim, 0);
  for (int64_t e = 0; e < p.numel; ++e) {
    int64_t o = 0, a = 0, b = 0, rem = e;
    for (int d = p.ndim - 1; d >= 0; --d) {
      const int64_t i = rem % p.size[d];
      rem /= p.size[d];
      o += i * p.out.stride[d];
      a += i * p.a.stride[d];
      b += i * p.b.stride[d];
    }
    want[o] = {a, b};
  }
  const bool flat = q.flags & kRowsFlat, lin[3] = {flat, (q.flags & kRowsALinear) != 0, (q.flags & kRowsBLinear) != 0};
  const bool bc[3] = {false, (q.flags & kRowsABcast) != 0, (q.flags & kRowsBBcast) != 0};
  (flat ? g_flat : g_rowform)++;
  g_linear += lin[1] + lin[2];
  size_t written = 0;
#define FAIL(msg) do { std::printf("case %d: %s (vector %ld element %d)\n", case_no, msg, (long)g, i); return 1; } while (0)
  for (int64_t g = 0; g < grid * q.block * p.unroll; ++g) {
    if (g >= q.nvec) continue;   // the kernel's own condition
    RowsPlace r = rows_place<V>(q, g, es[0], es[1], es[2]);
    const RowsPlace start = r;
    const bool whole = r.hi - r.lo == V;
    if (!whole) ++g_partial;
    if (!r.inrow) ++g_crossing;
    bool piece[3];
    for (int x = 0; x < 3; ++x) piece[x] = x == 0 ? whole : whole && (lin[x] || r.inrow);
    const int nops = p.nin + 1;
    for (int i = 0; i < V; ++i) {
      if (i < r.lo || i >= r.hi) continue;
      int64_t off[3];
      for (int x = 0; x < nops; ++x) {
        if (piece[x]) off[x] = rows_offset(start, x, 0, es[x], lin[x], bc[x]) + (bc[x] && !lin[x] ? 0 : (int64_t)i * es[x]);
        else if (x == 0) off[x] = rows_offset(start, 0, 0, es[0], flat, false) + (int64_t)i * es[0];
        else off[x] = rows_offset(r, x, i, es[x], lin[x], bc[x]);
      }
      auto it = want.find(off[0]);
      if (it == want.end()) FAIL("an output position written twice or outside the output");
      if (it->second.first != off[1]) FAIL("wrong element of a");
      if (p.nin == 2 && it->second.second != off[2]) FAIL("wrong element of b");
      want.erase(it);
      ++written;
      rows_next(q, r);
    }
  }
#undef FAIL
  if (!want.empty() || written != (size_t)p.numel) { std::printf("case %d: %zu of %ld elements written\n", case_no, written, (long)p.numel); return 1; }
  return 0;
}

static int check_case(int nin, int op, int da, int db, int dout, int ndim, const int64_t *sizes, int case_no) {
  ocn_tensor a = make_rows(da, ndim, sizes, (char *)0x100000000ull, false), b = make_rows(db, ndim, sizes, (char *)0x200000000ull, false);
  ocn_tensor o = make_rows(dout, ndim, sizes, (char *)0x300000000ull, true);
  EwPlan p;
  const int rc = plan_elementwise(nin, op, &a, nin == 2 ? &b : nullptr, &o, 0, &p);
  if (rc != OCN_OK) { std::printf("case %d: plan rc=%d\n", case_no, rc); return 1; }
  if (p.kernel != OCN_KERNEL_EW_ROWS) return 0;
  RowsSlimArgs slim;
  int64_t grid;
  if (make_rows_slim_args(p, kSlimBlock, &slim, &grid) && rnd() % 4) return 0;   // (some of the aligned ones too)
  const RowsArgs q = make_rows_args(p, &grid);
  switch (p.vec) {
    case 1: return replay<1>(p, q, grid, case_no);
    case 2: return replay<2>(p, q, grid, case_no);
    case 4: return replay<4>(p, q, grid, case_no);
    case 8: return replay<8>(p, q, grid, case_no);
    case 16: return replay<16>(p, q, grid, case_no);
    default: std::printf("case %d: vector of %d\n", case_no, p.vec); return 1;
  }
}

// A row's vectors around columns 0, 2^31 and 2^32 and at its end: they hold the row's elements in
// order, each once, none behind the row.  (No memory stands behind the addresses.)
template <int V> static int replay_long(const EwPlan &p, const RowsArgs &q, int case_no) {
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), dt_size(p.b.dtype)};
  const int64_t n0 = p.size[p.ndim - 1], vpr = (n0 + V - 1) / V, nrows = p.numel / n0;
  const bool bc[3] = {false, (q.flags & kRowsABcast) != 0, (q.flags & kRowsBBcast) != 0};
  if (q.flags & kRowsFlat || q.nvec != vpr * nrows) { std::printf("long %d: not the row form\n", case_no); return 1; }
  for (int64_t row = 0; row < nrows; ++row) {
    int64_t want[3] = {0, 0, 0}, rem = row;
    for (int d = p.ndim - 2; d >= 0; --d) {
      want[0] += rem % p.size[d] * p.out.stride[d];
      want[1] += rem % p.size[d] * p.a.stride[d];
      want[2] += rem % p.size[d] * p.b.stride[d];
      rem /= p.size[d];
    }
    for (const int64_t around : {(int64_t)0, (int64_t)1 << 31, (int64_t)1 << 32, n0})
      for (int64_t c = std::max<int64_t>(0, around / V - 3); c < std::min(vpr, around / V + 3); ++c) {
        RowsPlace r = rows_place<V>(q, row * vpr + c, es[0], es[1], es[2]);
        const int n = (int)std::min<int64_t>(V, n0 - c * V);
        if (r.lo != 0 || r.hi != n || !r.inrow) {
          std::printf("long %d: row %ld vector %ld holds %d..%d, not 0..%d\n", case_no, (long)row, (long)c, r.lo, r.hi, n);
          return 1;
        }
        const int64_t first = rows_offset(r, 0, 0, es[0], false, false);
        for (int i = 0; i < n; ++i) {
          for (int x = 0; x <= p.nin; ++x) {
            const int64_t off = x == 0 ? first + (int64_t)i * es[0] : rows_offset(r, x, i, es[x], false, bc[x]);
            if (off != want[x] + (bc[x] ? 0 : (c * V + i) * es[x])) {
              std::printf("long %d: row %ld column %ld operand %d\n", case_no, (long)row, (long)(c * V + i), x);
              return 1;
            }
          }
          rows_next(q, r);
        }
      }
  }
  return 0;
}

static int check_long_rows() {
  const int64_t G = (int64_t)1 << 31;
  // outer sizes, row length, elements between rows, b broadcast along the rows (1) or over them (2)
  const struct { int nin, op, a, b, o; int64_t outer[2], n0, gap; int bcast; } cases[] = {
      {2, B_ADD, DT_U8, DT_U8, DT_U8, {1, 2}, G + 5, 0, 1},    {2, B_ADD, DT_U8, DT_U8, DT_U8, {1, 2}, G + 13, 0, 2},
      {1, U_IDENT, DT_U8, DT_U8, DT_U8, {2, 2}, G + 16, 16, 0}, {1, U_IDENT, DT_U8, DT_U8, DT_U8, {2, 3}, 2 * G + 21, 5, 0},
      {2, B_ADD, DT_F32, DT_F32, DT_F32, {1, 3}, G + 3, 4, 1},  {2, B_GT, DT_F16, DT_F16, DT_BOOL, {1, 2}, 2 * G + 9, 1, 0},
      {1, U_IDENT, DT_U8, DT_U8, DT_U8, {1, 2}, G - 1, 3, 0},  {2, B_ADD, DT_U8, DT_U8, DT_U8, {1, 5}, G - 15, 1, 1}};
  int case_no = 0;
  for (const auto &c : cases) {
    ocn_tensor t[3];   // out, a, b
    const int dts[3] = {c.o, c.a, c.b};
    for (int x = 0; x < 3; ++x) {
      std::memset(&t[x], 0, sizeof t[x]);
      const int64_t es = dt_size(dts[x]), row = (c.n0 + c.gap) * es;
      t[x].base = (char *)((uint64_t)(x + 1) << 44);
      t[x].dtype = dts[x];
      t[x].ndim = 3;
      const int64_t size[3] = {c.outer[0], c.outer[1], c.n0}, stride[3] = {2 * row * c.outer[1], row, es};
      for (int d = 0; d < 3; ++d) { t[x].size[d] = size[d]; t[x].stride[d] = stride[d]; }
      if (x == 2 && c.bcast == 1) { t[x].size[2] = 1; t[x].stride[2] = 0; }
      if (x == 2 && c.bcast == 2) t[x].size[1] = 1;
    }
    EwPlan p;
    const int rc = plan_elementwise(c.nin, c.op, &t[1], c.nin == 2 ? &t[2] : nullptr, &t[0], 0, &p);
    if (rc != OCN_OK || p.kernel != OCN_KERNEL_EW_ROWS) { std::printf("long %d: plan %d, kernel %d\n", case_no, rc, p.kernel); return 1; }
    int64_t grid;
    const RowsArgs q = make_rows_args(p, &grid);
    int bad = 1;
    switch (p.vec) {
      case 1: bad = replay_long<1>(p, q, case_no); break;
      case 2: bad = replay_long<2>(p, q, case_no); break;
      case 4: bad = replay_long<4>(p, q, case_no); break;
      case 8: bad = replay_long<8>(p, q, case_no); break;
      case 16: bad = replay_long<16>(p, q, case_no); break;
    }
    if (bad) return 1;
    ++case_no;
  }
  return 0;
}

int main(int argc, char **argv) {
  if (check_long_rows()) return 1;
  const int ncases = argc > 1 ? std::atoi(argv[1]) : 1000;
  const struct { int nin, op, a, b, o; } kinds[] = {
      {2, B_ADD, DT_F32, DT_F32, DT_F32}, {2, B_MUL, DT_I32, DT_F32, DT_F32}, {2, B_MUL, DT_F16, DT_F32, DT_F32},
      {2, B_GT, DT_F64, DT_F64, DT_BOOL}, {2, B_ADD, DT_U8, DT_U8, DT_U8}, {2, B_MUL, DT_C64, DT_C64, DT_C64},
      {1, U_IDENT, DT_F64, DT_F64, DT_I16}, {1, U_IDENT, DT_U8, DT_U8, DT_F32}, {1, U_NEG, DT_F16, DT_F16, DT_F16},
      {1, U_IDENT, DT_C32, DT_C32, DT_F32}};
  for (int c = 0; c < ncases; ++c) {
    const int ndim = rnd_in(1, 5);
    int64_t sizes[8], total = 1;
    for (int i = 0; i < ndim; ++i) {
      sizes[i] = i == ndim - 1 ? rnd_in(1, 1 << rnd_in(1, 7)) : rnd_in(1, 7);
      if (total * sizes[i] > 4000) sizes[i] = 1;
      total *= sizes[i];
    }
    const auto &k = kinds[rnd() % (sizeof kinds / sizeof kinds[0])];
    if (check_case(k.nin, k.op, k.a, k.b, k.o, ndim, sizes, c)) {
      std::printf("FAILED case %d: types %d %d %d sizes", c, k.a, k.b, k.o);
      for (int i = 0; i < ndim; ++i) std::printf(" %ld", (long)sizes[i]);
      std::printf("\n");
      return 1;
    }
  }
  std::printf("ok: %d cases; flat form %d, row form %d, inputs along with the output %d, vectors across rows %d, partial vectors %d\n",
              ncases, g_flat, g_rowform, g_linear, g_crossing, g_partial);
  return g_flat > 100 && g_rowform > 100 && g_crossing > 100 && g_partial > 100 ? 0 : 1;
}
