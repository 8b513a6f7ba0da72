// Host-side emulation of ew_box_kernel's index arithmetic (no GPU needed): boxes of any extents.
//
// For random permuted, stepped and broadcast operands of several type combinations, with bases
// off by a few elements, it replays every lane and pass of every workgroup through the kernel's
// own helpers and the host-built arguments, and checks that every access stays inside its operand,
// that LDS accesses stay inside the budget and are aligned, and that every output element is
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

static int g_boxes, g_full, g_clipped, g_how[2], g_back, g_dims[5], g_runs[4], g_broadcast, g_carry;

static int replay(const EwPlan &p, const HostTensor *h, int case_no) {
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), dt_size(p.b.dtype)};
  const BoxArgs f = make_box_args(p);
  const int nin = p.nin;
  ++g_boxes;
  int64_t elems = 1;
  for (int d = 0; d < p.ndim; ++d) elems *= p.box[d];
  if (elems >= 1500 && es[0] >= 4) ++g_full;   // (boxes are halved until there are enough of them)
  ++g_dims[p.nord];
  ++g_runs[f.o.nrun];
  std::vector<uint8_t> written((h[0].hi - h[0].lo) / es[0], 0);
  std::vector<int64_t> lds((size_t)p.lds_bytes + 16);   // byte offset in the operand, at the LDS byte an element starts at
  std::vector<uint8_t> taken((size_t)p.total_tiles, 0);
  int64_t count = 0;
  auto lg = [](int e) { int l = 0; while ((1 << l) < e) ++l; return l; };
  const char *origin[3] = {f.out, f.a, f.b};
#define FAIL(msg) do { std::printf("case %d: %s (box %ld)\n", case_no, msg, (long)blk); return 1; } while (0)
  for (int64_t blk = 0; blk < p.total_tiles; ++blk) {
    int64_t base[3];
    const uint32_t number = box_number(f, (uint32_t)blk);
    if (number >= p.total_tiles || taken[number]++) FAIL("box number");
    const uint64_t lims = box_origin(f, number, base);
    if (lims != f.inner) ++g_clipped;
    std::fill(lds.begin(), lds.end(), INT64_MIN);
    for (int y = 0; y < nin; ++y) {
      const BoxInput &in = f.in[y];
      ++g_how[in.how];
      if (in.how == kBoxInPlace) continue;
      const int e = es[y + 1];
      const int V = std::max(1, 16 / e);
      if (in.epv != (uint32_t)V) FAIL("vector length");
      if (in.nvec >= 65536) FAIL("too many vectors");
      const char *src = origin[y + 1] + base[y + 1];
      const bool at_end = f.end[y] - src < (int64_t)in.reach;
      for (uint32_t tid = 0; tid < f.block; ++tid) {
        BoxLane l = box_lane(in, tid);
        for (uint32_t k = 0; k < in.niter; ++k, box_advance(in, f.block, l)) {
          if (l.t != tid + k * f.block) FAIL("vector number");
          if (l.t >= in.nvec || (lims != f.inner && !box_exists(in, lims, l))) continue;
          const uint32_t back = at_end ? box_back(l.off, box_room(f.end[y], src, 16), lg(e)) : 0;
          if (back) ++g_back;
          if (l.off < kBoxSlack || l.off < back * e) FAIL("offset");
          const int64_t at = src + (int64_t)l.off - kBoxSlack - (int64_t)back * e - (char *)h[y + 1].t.base;
          if (at < h[y + 1].lo || at + V * e > h[y + 1].hi) FAIL("load out of range");
          if (l.lds % 16 || (int64_t)l.lds + V * e > p.lds_bytes) FAIL("LDS write out of range");
          for (int i = 0; i + (int)back < V; ++i) {
            if (lds[l.lds + i * e] != INT64_MIN) FAIL("LDS element written twice");
            lds[l.lds + i * e] = at + (int64_t)(i + back) * e;
          }
        }
      }
    }
    const int es_max = std::max({es[0], es[1], nin == 2 ? es[2] : 1});
    const int V = box_vec_len(es[0], es_max);
    auto walk = [&](auto width) -> int {
      constexpr int W = decltype(width)::value;
      if (f.o.nvec >= 65536) FAIL("too many vectors");
      for (uint32_t tid = 0; tid < f.block; ++tid) {
        BoxVec v = box_vec(f.o, tid);
        for (uint32_t k = 0; k < f.o.niter; ++k, box_advance_out(f.o, f.block, v)) {
          if (v.t != tid + k * f.block) FAIL("vector number");
          const int n = box_count<W>(f.o, lims, lims != f.inner, v);
          if (n <= 0) continue;
          const int64_t at = f.out + base[0] + v.off - (char *)h[0].t.base;
          uint32_t pos[2] = {v.pos[0], v.pos[1]};
          BoxRun run{};
          if (f.o.nrun > 1) run = box_run<W>(f.o, v, pos);
          for (int i = 0; i < W; ++i) {
            for (int y = 0; y < nin; ++y)
              if (f.in[y].how != kBoxInPlace && (pos[y] % es[y + 1] || (int64_t)pos[y] + es[y + 1] > p.lds_bytes)) FAIL("LDS read out of range");
            if (i < n) {
              const int64_t oo = at + (int64_t)i * es[0];
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
                const char *src = origin[y + 1] + base[y + 1];
                if (f.in[y].how != kBoxInPlace) {
                  got = lds[pos[y]];
                } else if (f.o.run[y] == 0) {
                  ++g_broadcast;
                  got = src + (int64_t)v.pos[y] - kBoxSlack - (char *)h[y + 1].t.base;
                } else {
                  const uint32_t back = f.end[y] - src < (int64_t)f.in[y].reach ? box_back(v.pos[y], box_room(f.end[y], src, W * es[y + 1]), lg(es[y + 1])) : 0;
                  const int64_t from = src + (int64_t)v.pos[y] - kBoxSlack - (int64_t)back * es[y + 1] - (char *)h[y + 1].t.base;
                  if (back) ++g_back;
                  if (from < h[y + 1].lo || from + W * es[y + 1] > h[y + 1].hi) FAIL("read in place out of range");
                  got = from + (int64_t)(i + back) * es[y + 1];
                }
                if (got != want[y]) FAIL(y == 0 ? "wrong element of a" : "wrong element of b");
              }
            }
            if (i + 1 < n) {
              if (f.o.nrun > 1) {
                const uint32_t c0 = run.c[0];
                box_next<W>(f.o, run, pos);
                if (run.c[0] < c0) ++g_carry;
              } else {
                for (int y = 0; y < 2; ++y) pos[y] += f.o.run[y] / W;
              }
            }
          }
        }
      }
      return 0;
    };
    const int rc = V == 1 ? walk(std::integral_constant<int, 1>{}) : V == 2 ? walk(std::integral_constant<int, 2>{})
                 : V == 4 ? walk(std::integral_constant<int, 4>{}) : V == 8 ? walk(std::integral_constant<int, 8>{})
                 : V == 16 ? walk(std::integral_constant<int, 16>{}) : 1;
    if (rc) return 1;
  }
#undef FAIL
  if (count != p.numel) { std::printf("case %d: %ld of %ld elements written\n", case_no, (long)count, (long)p.numel); return 1; }
  return 0;
}

int main(int argc, char **argv) {
  const int ncases = argc > 1 ? std::atoi(argv[1]) : 1000;
  const struct { int nin, op, a, b, o; } kinds[] = {
      {2, B_ADD, DT_F32, DT_F32, DT_F32}, {2, B_MUL, DT_C32, DT_C32, DT_C32}, {2, B_ABSGT, DT_C32, DT_C32, DT_BOOL},
      {2, B_MUL, DT_I32, DT_F64, DT_F64}, {2, B_ADD, DT_U8, DT_U8, DT_U8}, {2, B_MUL, DT_C64, DT_C64, DT_C64},
      {1, U_IDENT, DT_F64, DT_F64, DT_I16}, {1, U_IDENT, DT_U8, DT_U8, DT_F32}, {1, U_NEG, DT_F16, DT_F16, DT_F16},
      {1, U_IDENT, DT_F32, DT_F32, DT_U8}, {2, B_LT, DT_I64, DT_I64, DT_BOOL}, {2, B_ADD, DT_C16, DT_C16, DT_C16},
      {2, B_MUL, DT_F32, DT_C32, DT_C32}, {2, B_ADD, DT_F16, DT_F16, DT_F16}};
  for (int c = 0; c < ncases; ++c) {
    const bool large = c % 80 == 79;   // boxes of full size
    const int ndim = rnd_in(2, large ? 4 : 6);
    int64_t sizes[8], total = 1;
    for (int i = 0; i < ndim; ++i) {
      const int kind = rnd_in(0, 3);
      sizes[i] = kind == 0 ? rnd_in(2, 4) : kind == 1 ? rnd_in(5, 20) : kind == 2 ? 1 << rnd_in(2, 6) : rnd_in(21, 130);
      if (total * sizes[i] > 100000) sizes[i] = 2;
      total *= sizes[i];
    }
    if (large) sizes[rnd_in(0, ndim - 1)] *= (1200000 + total - 1) / total;
    const auto &k = kinds[rnd() % (sizeof kinds / sizeof kinds[0])];
    const HostTensor h[3] = {make_view(k.o, ndim, sizes, (char *)0x300000000ull, false), make_view(k.a, ndim, sizes, (char *)0x100000000ull, true),
                             make_view(k.b, ndim, sizes, (char *)0x200000000ull, true)};
    EwPlan p;
    const int rc = plan_elementwise(k.nin, k.op, &h[1].t, k.nin == 2 ? &h[2].t : nullptr, &h[0].t, 0, &p);
    int bad = rc != OCN_OK;
    if (bad) std::printf("case %d: plan rc=%d\n", c, rc);
    else if (p.kernel == kKernelBox) bad = replay(p, h, c);
    if (bad) {
      std::printf("FAILED case %d: types %d %d %d sizes", c, k.a, k.b, k.o);
      for (int i = 0; i < ndim; ++i) std::printf(" %ld", (long)sizes[i]);
      std::printf("\n");
      return 1;
    }
  }
  std::printf("ok: %d cases, %d in boxes (dims 1: %d, 2: %d, 3: %d, 4: %d; runs along 1: %d, 2: %d, 3: %d); clipped %d, staged %d, in place %d, broadcast %d, moved back %d, carries %d, complex inputs with odd strides %d, of full size %d\n",
              ncases, g_boxes, g_dims[1], g_dims[2], g_dims[3], g_dims[4], g_runs[1], g_runs[2], g_runs[3], g_clipped, g_how[0], g_how[1],
              g_broadcast, g_back, g_carry, g_odd, g_full);
  return g_boxes > 300 && g_full * 1000 >= ncases && g_dims[3] && g_dims[4] && g_runs[1] && g_runs[2] && g_runs[3] && g_clipped > 100 && g_how[0] > 100 && g_how[1] > 100 && g_broadcast > 20 && g_back > 20 && g_carry > 100 ? 0 : 1;
}
