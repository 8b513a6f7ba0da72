// Host-side emulation of ew_tiled_any_kernel's index arithmetic (no GPU needed): the tiled kernel
// for clipped tiles and operands aligned to their elements only.
//
// For random permuted, stepped and broadcast operands of several type combinations, with bases
// off by a few elements, it replays every lane and pass of every workgroup through the kernel's
// own helpers and the host-built tables, and checks that every access stays inside its operand,
// that LDS elements are written once and inside the budget, and that every output element is
// written exactly once from the input elements that belong to it.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "../../paper_1810_08723_amd/csrc/ew_launch.hpp"

using namespace ocn;

static uint64_t rng_state = 0x13198A2E03707344ull;
static uint32_t rnd() {
  rng_state = rng_state * 6364136223846793005ull + 1442695040888963407ull;
  return (uint32_t)(rng_state >> 33);
}
static int rnd_in(int lo, int hi) { return lo + (int)(rnd() % (uint32_t)(hi - lo + 1)); }

struct HostTensor { ocn_tensor t; int64_t lo, hi; };

static int g_odd;

// dims permuted over a dense buffer, perhaps stepped along one axis, inputs perhaps broadcast, complex
// inputs perhaps with rows that lie an odd number of scalars apart (apart or as overlapping windows)
static HostTensor make_view(int dt, int ndim, const int64_t *sizes, char *base, bool input) {
  HostTensor h;
  std::memset(&h, 0, sizeof h);
  const int es = dt_size(dt);
  int perm[8];
  for (int i = 0; i < ndim; ++i) perm[i] = i;
  for (int i = ndim - 1; i > 0; --i) std::swap(perm[i], perm[rnd() % (uint32_t)(i + 1)]);
  const int step_axis = rnd() % 4 == 0 ? rnd_in(0, ndim - 1) : -1;
  h.t.base = base;
  h.t.dtype = dt;
  h.t.ndim = ndim;
  h.t.offset = (int64_t)es * (rnd() % 2 ? 0 : rnd_in(0, 9));
  h.lo = h.t.offset;
  int64_t acc = es;
  for (int k = ndim - 1; k >= 0; --k) {
    const int ax = perm[k];
    const int64_t step = ax == step_axis && (input || k < ndim - 1) ? 2 : 1;
    h.t.size[ax] = sizes[ax];
    h.t.stride[ax] = acc * step;
    acc *= sizes[ax] * step;
  }
  h.hi = h.lo + acc;
  const int sc = dt_size(dt_real_of(dt));
  if (input && sc < es && ndim > 1 && rnd() % 3 == 0) {
    const int slow = perm[rnd_in(0, ndim - 2)];
    h.t.stride[slow] = rnd() % 2 ? (int64_t)sc * rnd_in(1, 9) : h.t.stride[slow] + sc;
    h.t.offset += sc * (int)(rnd() % 2);
    h.lo = h.t.offset;
    h.hi = h.lo + es;
    for (int d = 0; d < ndim; ++d) h.hi += (h.t.size[d] - 1) * h.t.stride[d];
    ++g_odd;
  }
  if (input)
    for (int d = 0; d < ndim; ++d)
      if (rnd() % 10 == 0) { h.t.size[d] = 1; h.t.stride[d] = 0; }
  return h;
}

static int g_back, g_any, g_clipped, g_staged[2], g_element_orders, g_strided, g_dims[5];

// offset of the element that ends up as element i of the vector a lane loads at src; -1 if the load
// leaves the operand
static int64_t loaded(const HostTensor &h, int es, int V, const char *src, const char *end, uint32_t s0, int i) {
  const char *base = (const char *)h.t.base;
  int64_t off;
  if (s0 == (uint32_t)es) {   // one access of V elements
    int back, lg = 0;
    while ((1 << lg) < es) ++lg;
    const char *at = any_address(src, end - V * es, lg, back);
    if (back) ++g_back;
    if (at - base < h.lo || at - base + V * es > h.hi || end - base > h.hi) return -1;
    off = at - base + (int64_t)(i + back) * es;
  } else {
    off = src - base + (int64_t)i * s0;
  }
  return off < h.lo || off + es > h.hi ? -1 : off;
}

static int replay(const EwPlan &p, const HostTensor *h, int case_no) {
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), dt_size(p.b.dtype)};
  const AnyTiledArgs f = make_any_tiled_args(p, es[1]);
  const int nin = p.nin;
  ++g_any;
  ++g_dims[f.nord];
  std::vector<uint8_t> written((h[0].hi - h[0].lo) / es[0], 0);
  std::vector<int64_t> lds((size_t)p.lds_bytes);   // byte offset in the operand, at the LDS byte an element starts at
  int64_t count = 0;
#define FAIL(msg) do { std::printf("case %d: %s (tile %ld)\n", case_no, msg, (long)blk); return 1; } while (0)
  for (int64_t blk = 0; blk < p.total_tiles; ++blk) {
    int64_t base[3];
    const uint64_t lim = any_tile(f, (uint32_t)blk, base);
    const bool full = lim == f.whole;
    if (!full) ++g_clipped;
    std::fill(lds.begin(), lds.end(), INT64_MIN);
    for (int y = 0; y < nin; ++y) {
      if (!(y == 0 ? f.stage_a : f.stage_b)) continue;
      ++g_staged[y];
      const AnyOrder &g = f.ord[y + 1];
      const int V = std::max(1, 16 / es[y + 1]);
      if ((1 << g.vecw) != V) FAIL("staging vector length");
      if (f.stage_stride[y] != (uint32_t)es[y + 1]) ++g_element_orders;
      const char *gbase = (y == 0 ? f.a : f.b) + base[y + 1];
      for (uint32_t tid = 0; tid < f.block; ++tid) {
        const AnyLane l = any_lane(g, f.nord, tid);
        const uint32_t la = (swizzle(l.slot, f.swz[y]) << f.es_log2[y]) | f.lds_base[y];
        for (int j = 0; j < g.niter; ++j) {
          int n = 0;
          if (tid + (uint32_t)j * f.block < g.nvec) n = full ? V : any_inside(g, f.nord, l, lim, g.hi_c[j], V);
          for (int i = 0; i < n; ++i) {
            const int64_t off = loaded(h[y + 1], es[y + 1], V, gbase + g.hi_off[y + 1][j] + l.off[y + 1], f.end[y], f.stage_stride[y], i);
            if (off < 0) FAIL("staging load out of range");
            const uint32_t addr = la ^ f.st_hi[y][j] ^ f.st_el[y][i];
            if (addr % es[y + 1] || (int64_t)addr + es[y + 1] > p.lds_bytes) FAIL("LDS write out of range");
            if (lds[addr] != INT64_MIN) FAIL("LDS element written twice");
            lds[addr] = off;
          }
        }
      }
    }
    const AnyOrder &g = f.ord[0];
    const int V = rows_vec(es[0], std::max({es[0], es[1], nin == 2 ? es[2] : 1}));
    if ((1 << g.vecw) != V) FAIL("compute vector length");
    for (uint32_t tid = 0; tid < f.block; ++tid) {
      const AnyLane l = any_lane(g, f.nord, tid);
      uint32_t r[2];
      for (int y = 0; y < 2; ++y) r[y] = (swizzle(tid * (uint32_t)V, f.swz[y]) << f.es_log2[y]) | f.lds_base[y];
      for (int j = 0; j < g.niter; ++j) {
        int n = 0;
        if (tid + (uint32_t)j * f.block < g.nvec) n = full ? V : any_inside(g, f.nord, l, lim, g.hi_c[j], V);
        for (int i = 0; i < n; ++i) {
          const int64_t oo = (f.out + base[0] + g.hi_off[0][j] + l.off[0] + (int64_t)i * es[0]) - (char *)h[0].t.base;
          if (oo < h[0].lo || oo + es[0] > h[0].hi) FAIL("store out of range");
          if (written[(oo - h[0].lo) / es[0]]++) FAIL("output element written twice");
          ++count;
          int64_t want[2] = {p.off_a, p.off_b}, rem = oo - p.off_out;
          for (int d = 0; d < p.ndim; ++d) {
            const int64_t c = rem / p.out.stride[d];
            rem -= c * p.out.stride[d];
            want[0] += c * p.a.stride[d];
            want[1] += c * p.b.stride[d];
          }
          if (rem) FAIL("store between elements");
          for (int y = 0; y < nin; ++y) {
            int64_t got;
            if (y == 0 ? f.stage_a : f.stage_b) {
              const int EP = std::min(std::max(1, 16 / es[y + 1]), V), c = i / EP * EP;
              const uint32_t at = r[y] ^ f.rd_hi[y][j] ^ f.rd_el[y][c];
              if (at % ((uint32_t)EP * es[y + 1])) FAIL("misaligned LDS read");
              if ((int64_t)at + EP * es[y + 1] > p.lds_bytes) FAIL("LDS read out of range");
              got = lds[at + (uint32_t)(i - c) * es[y + 1]];
            } else {
              const uint32_t s0 = y == 0 ? f.sa0 : f.sb0;
              if (s0 != 0 && s0 != (uint32_t)es[y + 1]) ++g_strided;
              got = loaded(h[y + 1], es[y + 1], V, (y == 0 ? f.a : f.b) + base[y + 1] + g.hi_off[y + 1][j] + l.off[y + 1], f.end[y], s0, i);
              if (got < 0) FAIL("direct read out of range");
            }
            if (got != want[y]) FAIL(y == 0 ? "wrong element of a" : "wrong element of b");
          }
        }
      }
    }
  }
#undef FAIL
  if (count != p.numel) { std::printf("case %d: %ld of %ld elements written\n", case_no, (long)count, (long)p.numel); return 1; }
  return 0;
}

// A launch stays below 2^32 lanes, and below the bound set, whatever the lanes per workgroup.
static int check_launch_sizes() {
  const struct { int dt; int64_t n, m; } shapes[] = {
      {DT_F16, 10000001, 17}, {DT_F32, 140000003, 9}, {DT_F32, 8388607, 17}, {DT_U8, 16777215, 17}, {DT_F32, 1000, 17}};
  int taken = 0;
  for (const int64_t bound : {(int64_t)0, (int64_t)1500})
    for (const auto &s : shapes) {
      const int64_t es = dt_size(s.dt);
      ocn_tensor a, o;
      std::memset(&a, 0, sizeof a);
      a.dtype = s.dt;
      a.ndim = 3;
      a.size[0] = s.n;
      a.size[1] = a.size[2] = s.m;
      a.stride[0] = s.m * s.m * es;
      a.stride[1] = s.m * es;
      a.stride[2] = es;
      o = a;
      a.base = (char *)((uint64_t)1 << 44);
      o.base = (char *)((uint64_t)2 << 44);
      std::swap(a.stride[1], a.stride[2]);
      set_max_launch_blocks(bound);
      EwPlan p;
      const int rc = plan_elementwise(1, U_NEG, &a, nullptr, &o, 0, &p);
      const int64_t most = max_launch_blocks() * kBlock;
      set_max_launch_blocks(0);
      if (rc != OCN_OK) { std::printf("launch sizes: plan rc=%d\n", rc); return 1; }
      if (p.kernel != kKernelTiledAny) continue;
      ++taken;
      if (p.grid * p.block > most || p.grid * p.block >= (int64_t)1 << 32) {
        std::printf("launch sizes: %ld x %ld x %ld goes out with %ld workgroups of %d lanes\n", (long)s.n, (long)s.m, (long)s.m,
                    (long)p.grid, p.block);
        return 1;
      }
    }
  return taken >= 4 ? 0 : 1;
}

int main(int argc, char **argv) {
  if (check_launch_sizes()) return 1;
  const int ncases = argc > 1 ? std::atoi(argv[1]) : 1000;
  const struct { int nin, op, a, b, o; } kinds[] = {
      {2, B_ADD, DT_F32, DT_F32, DT_F32}, {2, B_MUL, DT_C32, DT_C32, DT_C32}, {2, B_ABSGT, DT_C32, DT_C32, DT_BOOL},
      {2, B_MUL, DT_I32, DT_F64, DT_F64}, {2, B_ADD, DT_U8, DT_U8, DT_U8}, {2, B_MUL, DT_C64, DT_C64, DT_C64},
      {1, U_IDENT, DT_F64, DT_F64, DT_I16}, {1, U_IDENT, DT_U8, DT_U8, DT_F32}, {1, U_NEG, DT_F16, DT_F16, DT_F16},
      {1, U_IDENT, DT_F32, DT_F32, DT_U8}, {2, B_LT, DT_I64, DT_I64, DT_BOOL}, {2, B_ADD, DT_C16, DT_C16, DT_C16},
      {2, B_MUL, DT_F32, DT_C32, DT_C32}};
  for (int c = 0; c < ncases; ++c) {
    const int ndim = rnd_in(2, 5);
    int64_t sizes[8], total = 1;
    for (int i = 0; i < ndim; ++i) {
      const int kind = rnd_in(0, 3);
      sizes[i] = kind == 0 ? rnd_in(2, 4) : kind == 1 ? rnd_in(5, 20) : kind == 2 ? 1 << rnd_in(2, 6) : rnd_in(21, 130);
      if (total * sizes[i] > 100000) sizes[i] = 2;
      total *= sizes[i];
    }
    const auto &k = kinds[rnd() % (sizeof kinds / sizeof kinds[0])];
    const HostTensor h[3] = {make_view(k.o, ndim, sizes, (char *)0x300000000ull, false), make_view(k.a, ndim, sizes, (char *)0x100000000ull, true),
                             make_view(k.b, ndim, sizes, (char *)0x200000000ull, true)};
    EwPlan p;
    const int rc = plan_elementwise(k.nin, k.op, &h[1].t, k.nin == 2 ? &h[2].t : nullptr, &h[0].t, 0, &p);
    int bad = rc != OCN_OK;
    if (bad) std::printf("case %d: plan rc=%d\n", c, rc);
    else if (p.kernel == kKernelTiledAny) bad = replay(p, h, c);
    if (bad) {
      std::printf("FAILED case %d: types %d %d %d sizes", c, k.a, k.b, k.o);
      for (int i = 0; i < ndim; ++i) std::printf(" %ld", (long)sizes[i]);
      std::printf("\n");
      return 1;
    }
  }
  std::printf("ok: %d cases, %d in this form (tiled dims 1: %d, 2: %d, 3: %d, 4: %d); clipped tiles %d, staged a %d, b %d, element orders %d, strided reads %d, moved back %d, complex inputs with odd strides %d\n",
              ncases, g_any, g_dims[1], g_dims[2], g_dims[3], g_dims[4], g_clipped, g_staged[0], g_staged[1], g_element_orders, g_strided, g_back, g_odd);
  return g_any > 300 && g_clipped > 100 && g_staged[0] > 100 && g_staged[1] > 100 && g_element_orders > 20 && g_strided > 20 && g_back > 20 && g_odd > 200 ? 0 : 1;
}
