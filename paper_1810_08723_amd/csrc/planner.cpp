// Host planner: see planner.hpp.  Plain C++, no HIP.
#include "planner.hpp"

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <cstring>

#include "sigs.hpp"

namespace ocn {

// ---------------------------------------------------------------------------------------
// small helpers
// ---------------------------------------------------------------------------------------

namespace {
std::atomic<int64_t> g_max_launch_blocks{((int64_t)1 << 24) - 1};
}
int64_t max_launch_blocks() { return g_max_launch_blocks.load(std::memory_order_relaxed); }
void set_max_launch_blocks(int64_t blocks) {
  const int64_t hard = ((int64_t)1 << 24) - 1;
  g_max_launch_blocks.store(blocks <= 0 || blocks > hard ? hard : blocks, std::memory_order_relaxed);
}

FastDiv make_fastdiv(uint32_t d) {
  // q = (mulhi(n, m) + n) >> s with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1;
  // exact for every n < 2^31
  FastDiv f;
  f.d = d ? d : 1;
  uint32_t s = 0;
  while (((uint64_t)1 << s) < f.d) ++s;
  f.s = s;
  f.m = (uint32_t)(((((uint64_t)1 << s) - f.d) << 32) / f.d + 1);
  return f;
}

static bool valid_dtype(int dt) { return dt >= 0 && dt < DT_COUNT; }
static int scalar_size(int dt) { return dt_size(dt_real_of(dt)); }

static int check_tensor(const ocn_tensor *t) {
  if (!t) return OCN_ERR_NULLPTR;
  if (!valid_dtype(t->dtype)) return OCN_ERR_DTYPE;
  if (t->ndim < 0 || t->ndim > kMaxDims) return OCN_ERR_NDIM;
  bool empty = false;
  for (int d = 0; d < t->ndim; ++d) {
    if (t->size[d] < 0) return OCN_ERR_SHAPE;
    if (t->size[d] == 0) empty = true;
  }
  if (!empty && !t->base) return OCN_ERR_NULLPTR;
  return OCN_OK;
}

static int check_alignment(const ocn_tensor *t) {
  const int64_t sc = scalar_size(t->dtype);
  if (((intptr_t)t->base + t->offset) % sc != 0) return OCN_ERR_ALIGN;
  for (int d = 0; d < t->ndim; ++d)
    if (t->size[d] > 1 && t->stride[d] % sc != 0) return OCN_ERR_ALIGN;
  return OCN_OK;
}

// [lo, hi) of the bytes a view touches, relative to address zero
static void byte_range(const ocn_tensor *t, intptr_t *lo, intptr_t *hi) {
  intptr_t l = (intptr_t)t->base + t->offset, h = l;
  for (int d = 0; d < t->ndim; ++d) {
    if (t->size[d] <= 1) continue;
    int64_t span = (t->size[d] - 1) * t->stride[d];
    if (span < 0) l += span; else h += span;
  }
  *lo = l;
  *hi = h + dt_size(t->dtype);
}

// Conservative proof that no byte of the view is addressed twice: with dimensions sorted by
// |stride|, each stride must step over everything the faster dimensions span.
static bool provably_non_overlapping(const ocn_tensor *t) {
  int64_t st[kMaxDims], sz[kMaxDims];
  int n = 0;
  for (int d = 0; d < t->ndim; ++d) {
    if (t->size[d] <= 1) continue;
    st[n] = std::llabs(t->stride[d]);
    sz[n] = t->size[d];
    ++n;
  }
  for (int i = 1; i < n; ++i)  // insertion sort by stride, ascending
    for (int j = i; j > 0 && st[j] < st[j - 1]; --j) {
      std::swap(st[j], st[j - 1]);
      std::swap(sz[j], sz[j - 1]);
    }
  int64_t extent = dt_size(t->dtype);  // bytes spanned so far
  for (int i = 0; i < n; ++i) {
    if (st[i] < extent) return false;
    extent = (sz[i] - 1) * st[i] + extent;
  }
  return true;
}

// ---------------------------------------------------------------------------------------
// implicit casting (section 3.2.1): the smallest type that can keep both
// ---------------------------------------------------------------------------------------

static int int_bits_of(int dt) { return dt_size(dt) * 8; }

static int float_for_bits(int need_bits, int at_least) {
  // smallest real floating type with >= need_bits of exact integer range and >= at_least
  int r = at_least;
  if (need_bits > 11 && r < DT_F32) r = DT_F32;
  if (need_bits > 24 && r < DT_F64) r = DT_F64;
  return r;
}

static int promote_real(int a, int b) {
  const int ka = dt_kind(a), kb = dt_kind(b);
  if (ka == K_BOOL) return b;
  if (kb == K_BOOL) return a;
  if (ka == K_REAL && kb == K_REAL) return std::max(a, b);
  if (ka == K_REAL || kb == K_REAL) {
    const int f = ka == K_REAL ? a : b, i = ka == K_REAL ? b : a;
    // magnitude bits an integer type needs to be held exactly by a float significand
    const int need = dt_kind(i) == K_SINT ? int_bits_of(i) - 1 : int_bits_of(i);
    if (need > 53) return DT_F64;  // the paper's stated exception for 64-bit integers
    return float_for_bits(need, f);
  }
  if (ka == kb) return int_bits_of(a) >= int_bits_of(b) ? a : b;
  // signed with unsigned: a signed type strictly wider than the unsigned one
  const int s = ka == K_SINT ? a : b, u = ka == K_SINT ? b : a;
  const int ub = int_bits_of(u), sb = int_bits_of(s);
  if (sb > ub) return s;
  switch (ub) {
    case 8: return DT_I16;
    case 16: return DT_I32;
    case 32: return DT_I64;
    default: return DT_F64;  // nothing keeps uint64 and a signed integer
  }
}

int promote(int a, int b) {
  if (!valid_dtype(a) || !valid_dtype(b)) return OCN_ERR_DTYPE;
  if (dt_kind(a) == K_CPLX || dt_kind(b) == K_CPLX) {
    const int r = promote_real(dt_real_of(a), dt_real_of(b));
    return r == DT_F16 ? DT_C16 : r == DT_F32 ? DT_C32 : DT_C64;
  }
  return promote_real(a, b);
}

// ---------------------------------------------------------------------------------------
// elementwise planning
// ---------------------------------------------------------------------------------------

namespace {

struct Dim {
  int64_t size;
  int64_t so, sa, sb;
};

int64_t iabs64(int64_t x) { return x < 0 ? -x : x; }

int ilog2_ceil(int64_t x) {
  int l = 0;
  while (((int64_t)1 << l) < x) ++l;
  return l;
}

// is the input the identical view as the output (same address, element size and strides)?
bool same_view(const ocn_tensor *in, const ocn_tensor *out) {
  if ((intptr_t)in->base + in->offset != (intptr_t)out->base + out->offset) return false;
  if (dt_size(in->dtype) != dt_size(out->dtype)) return false;
  if (in->ndim != out->ndim) return false;
  for (int d = 0; d < out->ndim; ++d) {
    if (in->size[d] != out->size[d]) return false;
    if (out->size[d] > 1 && in->stride[d] != out->stride[d]) return false;
  }
  return true;
}

int check_alias(const ocn_tensor *in, const ocn_tensor *out) {
  if (same_view(in, out)) return OCN_OK;
  intptr_t ilo, ihi, olo, ohi;
  byte_range(in, &ilo, &ihi);
  byte_range(out, &olo, &ohi);
  if (ilo < ohi && olo < ihi) return OCN_ERR_ALIAS;
  return OCN_OK;
}

int check_broadcast(const ocn_tensor *in, const ocn_tensor *out) {
  if (in->ndim > out->ndim) return OCN_ERR_SHAPE;
  const int lead = out->ndim - in->ndim;
  for (int d = 0; d < in->ndim; ++d)
    if (in->size[d] != out->size[lead + d] && in->size[d] != 1) return OCN_ERR_SHAPE;
  return OCN_OK;
}

// stride of input along out's dimension d (zero where the input is broadcast)
int64_t bstride(const ocn_tensor *in, const ocn_tensor *out, int d) {
  const int lead = out->ndim - in->ndim;
  if (d < lead) return 0;
  return in->size[d - lead] == 1 ? 0 : in->stride[d - lead];
}

// the dimension with the smallest non-zero |stride| (ties: the later one); -1 if none
template <class Get> int fastest_dim(int n, Get stride_of) {
  int best = -1;
  int64_t bs = 0;
  for (int d = 0; d < n; ++d) {
    int64_t s = iabs64(stride_of(d));
    if (s == 0) continue;
    if (best < 0 || s <= bs) { best = d; bs = s; }
  }
  return best;
}

// order the tiled dims of one operand by that operand's |stride|, fastest first; zero
// strides (broadcast) go last since they do not affect coalescing
void tile_order(const EwPlan &p, const int64_t *stride, int8_t *ord) {
  int n = 0;
  for (int d = p.ndim - 1; d >= 0; --d)
    if (p.tile_log2[d] > 0) ord[n++] = (int8_t)d;
  auto key = [&](int d) {
    int64_t s = iabs64(stride[d]);
    return s == 0 ? INT64_MAX : s;
  };
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && key(ord[j]) < key(ord[j - 1]); --j) std::swap(ord[j], ord[j - 1]);
}

// LDS per workgroup, so that several share a CU's 160 KB.  A tile grows to the run lengths its
// operands want and no further: small tiles, i.e. many resident workgroups, measured faster
// than large ones on MI355X once every run is a full cache line.
constexpr int64_t kMaxLdsBytes = 32 * 1024;

// kTilesVector: for the all-vector form; kTilesAny: for tiles of any size and alignment;
// kTilesGeneral: for the general form
enum TileRule { kTilesVector, kTilesAny, kTilesGeneral };
void choose_tiles(EwPlan &p, TileRule rule, int fa, int fb) {
  // Operands that want coalescing along their own fastest axis: the output and every staged
  // input.  Tile bits are handed out one at a time, each to the fastest unsaturated dimension
  // of one operand.  First every staged input is grown to a contiguous run of a full 128-byte
  // cache line (a shorter read run still fetches the whole line, and the other half is fetched
  // again by a neighbouring tile); the output to a full line as well when it is written with
  // streaming stores (partial-line streaming writes run at half rate), else to 64 bytes
  // (partial-line writes into the cache cost no extra traffic).  After that the tile only
  // grows, round-robin, until every enumeration order has a whole vector for each of the 256
  // lanes (which the lean kernel form needs); for the general form it grows on while the
  // staging areas stay within 16 KiB.
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), p.nin == 2 ? dt_size(p.b.dtype) : 1};
  const int staged_bytes = (p.stage_a ? es[1] : 0) + (p.stage_b ? es[2] : 0);
  int budget = 12;
  while (budget > 8 && ((int64_t)staged_bytes << budget) > kMaxLdsBytes) --budget;
  const int es_max = std::max({es[0], es[1], p.nin == 2 ? es[2] : es[1]});
  const int vmax = std::max({rows_vec(es[0], es_max), p.stage_a ? 16 / es[1] : 1, p.stage_b ? 16 / es[2] : 1});
  int vbits = 0;
  while ((1 << vbits) < vmax) ++vbits;
  int preferred = std::min(budget, 8 + vbits);
  if (rule != kTilesVector) {  // larger tiles, within 16 KiB of LDS
    preferred = budget;
    while (preferred > 8 && ((int64_t)staged_bytes << preferred) > 16 * 1024) --preferred;
  }
  const int64_t *strides[3] = {p.out.stride, p.a.stride, p.b.stride};
  const bool wants[3] = {true, p.stage_a, p.stage_b};
  int used = 0;
  auto saturated = [&](int d) { return ((int64_t)1 << p.tile_log2[d]) >= p.size[d]; };
  // give operand o one more bit along its fastest unsaturated dim; false if it has none
  auto grow = [&](int o) {
    int best = -1;
    int64_t bs = 0;
    for (int d = 0; d < p.ndim; ++d) {
      if (saturated(d)) continue;
      const int64_t s = iabs64(strides[o][d]);
      if (s == 0) continue;
      if (best < 0 || s < bs || (s == bs && d > best)) { best = d; bs = s; }
    }
    if (best < 0) return false;
    ++p.tile_log2[best];
    ++used;
    return true;
  };
  // bytes of operand o that the tile covers contiguously, starting from its fastest dim
  auto run_bytes = [&](int o) {
    int64_t run = es[o];
    bool any = true;
    while (any) {
      any = false;
      for (int d = 0; d < p.ndim; ++d)
        if (p.tile_log2[d] > 0 && iabs64(strides[o][d]) == run) {
          const int64_t ext = std::min<int64_t>((int64_t)1 << p.tile_log2[d], p.size[d]);
          run *= ext;
          any = ext > 1 && ext == p.size[d] ? true : false;  // only a fully covered dim chains on
          if (!any) return run;
          break;
        }
    }
    return run;
  };
  // Tiles of any size move whole vectors along the output's and every staged input's fastest dim:
  // an extent below the vector's length is rounded up to it (its vectors are then never whole).
  if (rule == kTilesAny) {
    auto at_least = [&](int d, int bits) {
      while (d >= 0 && p.tile_log2[d] < bits) { ++p.tile_log2[d]; ++used; }
    };
    auto log2i = [](int v) { int l = 0; while ((1 << l) < v) ++l; return l; };
    at_least(p.ndim - 1, log2i(rows_vec(es[0], es_max)));
    if (p.stage_a) at_least(fa, log2i(16 / es[1]));
    if (p.stage_b) at_least(fb, log2i(16 / es[2]));
  }
  const int64_t target[3] = {rule == kTilesAny && p.nt_store && !(p.stage_a && p.stage_b) ? 512 : p.nt_store ? 128 : 64, 128, 128};
  bool progress = true;
  while (used < budget && progress) {
    progress = false;
    for (int o = 0; o < 3 && used < budget; ++o)
      if (wants[o] && run_bytes(o) < target[o] && grow(o)) progress = true;
  }
  progress = true;
  while (used < preferred && progress) {
    progress = false;
    for (int o = 0; o < 3 && used < preferred; ++o)
      if (wants[o] && grow(o)) progress = true;
  }
  p.tile_bits = used;
}

// Boxes of any extents (ew_box_kernel).
//
// A box has about this many elements (twice as many of one or two bytes): staged inputs take 8 to 32 KiB
// of LDS, so that four or more workgroups share a CU (4096 complex elements in 64 KiB: 49 us where
// 2048 take 44; three, of one-byte types with two inputs, for their registers), and a lane moves two to
// four vectors of each operand.
constexpr int64_t kBoxElems = 2048;
constexpr int64_t kBoxLds = 32 * 1024;
// The contiguous bytes each operand should have in a box: two lines, since runs start anywhere and
// touch one line more than they fill (6000 x 5000 plus a transpose: 69 us, 77 with 128 bytes).
constexpr int64_t kBoxRun = 256;
// Gaps of up to this many bytes do not end what an operand touches in a row: the next piece is in the
// same line or the one after it.
constexpr int64_t kBoxGap = 64;
// Boxes in a row that one XCD takes.  Neighbouring boxes share the lines at the ends of their runs; dealt
// out one by one every XCD fetches them for itself (complex products of [44, 66, 17, 71, 2]: 263 MB
// fetched instead of 143, 55 us instead of 44; groups of 4 and 64 are within 6 % of 16, an eighth of
// all boxes each is 5 to 20 % slower on plain transposes).
constexpr int kBoxGroup = 16;

// Turns that the first wavefront takes to read an element per lane from LDS, at most: lanes whose elements lie
// in the same bank, but not in the same place.  pos: bytes per coordinate.  (A run that several dims
// share has no gaps between rows: int32 [8, 189, 4751] with the axis of 8 fastest, 32 turns, 20.5 us in
// boxes and 15.1 in tiles.)
int bank_turns(const EwPlan &p, int V, int es, const int32_t *ext, const int32_t *pos) {
  const int width = std::max(4, es), lanes = std::min(kWave, 256 / width);   // bytes of a read; lanes served at a time
  uint32_t c[4] = {0, 0, 0, 0};
  int64_t run = 1, e = 0;
  for (int k = 0; k < p.box_run[0]; ++k) run *= ext[p.ord_o[k]];
  int32_t last[kWave];
  uint8_t count[kWave] = {0};
  int most = 0;
  for (int lane = 0; lane < lanes; ++lane) {
    int32_t at = 0;
    for (int k = 0; k < p.nord; ++k) at += (int32_t)c[k] * pos[p.ord_o[k]];
    at /= width;
    const int bank = at % lanes;
    if (count[bank] == 0 || last[bank] != at) most = std::max<int>(most, ++count[bank]);
    last[bank] = at;
    // the next vector: further along the run, or the first of the next row
    int k = 0;
    if ((e += V) < run) c[0] += (uint32_t)V;
    else {
      e = 0;
      for (; k < p.box_run[0]; ++k) c[k] = 0;
      if (k < p.nord) ++c[k];
    }
    for (; k + 1 < p.nord && c[k] >= (uint32_t)ext[p.ord_o[k]]; ++k) {
      c[k + 1] += c[k] / (uint32_t)ext[p.ord_o[k]];
      c[k] %= (uint32_t)ext[p.ord_o[k]];
    }
  }
  return most;
}

// Lays the operation out in boxes; false where that form does not apply.  Extents grow from one, always
// for the operand that touches the fewest bytes in a row inside the box, along the axis that lengthens
// them (an axis covered whole passes on to the next one); an operand that a wide gap cuts off is left
// as it is, or it would take the whole box (double [1965283, 14] transposed plus a stepped column 478 us,
// 106 in tiles; float [2, 86669, 250], one input of two elements and a gap, 571 -> 233).  Axes are cut into
// equal parts at the end, the output's fastest one into whole vectors, whose rest would be stored element by
// element (bytes [50001, 289] transposed 20.8 us in parts of 58).  tiles_stage: tiles would stage an input.
bool plan_boxes(EwPlan &p, bool tiles_stage) {
  const int n = p.ndim, nin = p.nin;
  const Operand *ops[3] = {&p.out, &p.a, &p.b};
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), nin == 2 ? dt_size(p.b.dtype) : 1};
  const int es_max = std::max({es[0], es[1], nin == 2 ? es[2] : es[1]});
  const int V = box_vec_len(es[0], es_max);
  for (int d = 0; d < n; ++d)
    if (p.out.stride[d] < 0 || p.a.stride[d] < 0 || p.b.stride[d] < 0) return false;
  if (p.out.stride[n - 1] != es[0]) return false;
  // the dims of an operand, its fastest first (broadcast ones do not lengthen its runs)
  int8_t ord[3][kMaxDims];
  int nd[3] = {0, 0, 0};
  for (int x = 0; x <= nin; ++x) {
    for (int d = n - 1; d >= 0; --d)
      if (ops[x]->stride[d] != 0 && p.size[d] > 1) ord[x][nd[x]++] = (int8_t)d;
    std::stable_sort(ord[x], ord[x] + nd[x], [&](int8_t i, int8_t j) { return ops[x]->stride[i] < ops[x]->stride[j]; });
  }
  int32_t ext[kMaxDims];
  for (int d = 0; d < kMaxDims; ++d) ext[d] = 1;
  int64_t elems = 1;
  // the contiguous bytes of operand x inside the box; dims its runs go along
  auto run_of = [&](int x, int *dims) {
    int64_t run = es[x];
    int k = 0;
    for (; k < nd[x]; ++k) {
      const int d = ord[x][k];
      if (ext[d] == 1 || ops[x]->stride[d] != run) break;
      run *= ext[d];
      if (ext[d] < p.size[d]) { ++k; break; }
    }
    if (dims) *dims = k;
    return run;
  };
  int64_t most = es_max <= 2 ? 2 * kBoxElems : kBoxElems;
  // (few boxes: smaller ones, down to a vector of the output per lane)
  while (most > (int64_t)kBlock * V && p.numel / most < 2 * kNumCUs) most /= 2;
  auto fits = [&](int64_t e) {
    int64_t bytes = 0;
    for (int x = 1; x <= nin; ++x) bytes += e * es[x];
    return bytes <= kBoxLds;
  };
  // the bytes operand x touches in a row inside the box, gaps shorter than a line's half among them, and
  // the dim that would lengthen them (-1: none would, or not inside this box)
  auto reach_of = [&](int x, int *next) {
    int64_t r = es[x];
    *next = -1;
    for (int k = 0; k < nd[x]; ++k) {
      const int d = ord[x][k];
      if (ops[x]->stride[d] > std::max<int64_t>(r, kBoxGap)) break;
      r += (ext[d] - 1) * ops[x]->stride[d];
      if (ext[d] < p.size[d]) { *next = d; break; }
    }
    return r;
  };
  int tiled = 0;
  // one step along a dim; false if the box cannot grow there
  auto grow = [&](int d) {
    if (d < 0 || ext[d] >= p.size[d] || (ext[d] == 1 && tiled == 4)) return false;
    const int64_t others = elems / ext[d];
    int64_t e = std::min<int64_t>(p.size[d], 2 * (int64_t)ext[d]);
    if (3 * e >= 2 * p.size[d]) e = p.size[d];
    while (e > ext[d] && (others * e > most || !fits(others * e) || e > 4096)) --e;
    if (e == ext[d]) return false;
    tiled += ext[d] == 1;
    ext[d] = (int32_t)e;
    elems = others * e;
    return true;
  };
  // (at least two vectors of the output per lane: cdouble 5000 x 3001 transposed 94 us, 108 with one)
  const int64_t enough = std::min<int64_t>(most, 2 * kBlock * V);
  for (bool open[3] = {true, true, nin == 2};;) {
    int x = -1, next = -1;
    int64_t reach = 0;
    for (int y = 0; y < 3; ++y) {
      int d;
      const int64_t r = open[y] ? reach_of(y, &d) : 0;
      if (open[y] && (x < 0 || r < reach)) x = y, reach = r, next = d;
    }
    if (x < 0 || (reach >= kBoxRun && elems >= enough)) break;
    if (!grow(next)) open[x] = false;
  }
  for (int k = 0; k < nd[0] && elems < enough; ++k)
    while (elems < enough && grow(ord[0][k])) {}
  for (int d = 0; d < n; ++d) {
    const int64_t parts = (p.size[d] + ext[d] - 1) / ext[d];
    int64_t e = (p.size[d] + parts - 1) / parts;
    if (d == n - 1 && e < p.size[d]) e = std::min<int64_t>(ext[d], (e + V - 1) / V * V);
    ext[d] = (int32_t)e;
  }
  elems = 1;
  p.total_tiles = 1;
  for (int d = 0; d < n; ++d) {
    p.box[d] = ext[d];
    elems *= ext[d];
    p.ntiles[d] = (p.size[d] + ext[d] - 1) / ext[d];
    p.total_tiles *= p.ntiles[d];
  }
  if (elems < 2 || p.total_tiles > max_launch_blocks()) return false;
  // (four short axes, and a long one that no box may cover too: less than a wavefront's work per workgroup;
  // float [2, 5, 866805, 2, 3] in boxes of 60 elements 1694 us, 329 in tiles)
  if (elems < kWave * V && p.total_tiles > 2 * kNumCUs) return false;
  // (the same of more boxes, but for less than an element per lane: doubles [176656, 4, 2, 8, 2] compared in
  // boxes of 128 elements 354 us, 77 in tiles)
  if (elems < kBlock && p.total_tiles > 16 * kNumCUs) return false;
  // the orders inside the box, and how far runs go
  for (int x = 0; x <= nin; ++x) {
    int m = 0;
    int8_t *o = x == 0 ? p.ord_o : x == 1 ? p.ord_a : p.ord_b;
    for (int k = 0; k < nd[x]; ++k)
      if (ext[ord[x][k]] > 1) o[m++] = ord[x][k];
    p.box_dims[x] = m;
    run_of(x, &p.box_run[x]);
    int64_t span = 0, bytes = es[x];
    bool whole = true;
    for (int d = 0; d < n; ++d) {
      span += (int64_t)ext[d] * ops[x]->stride[d];
      bytes += (p.size[d] - 1) * ops[x]->stride[d];
      whole = whole && ops[x]->stride[d] % es[x] == 0;
    }
    if (span >= ((int64_t)1 << 31) - 64) return false;
    if (x > 0 && bytes < std::max<int64_t>(16, (int64_t)V * es[x]) + (whole ? 0 : es[x] - scalar_size(ops[x]->dtype))) return false;   // shorter than a vector
  }
  if (p.box_run[0] == 0 || p.box_dims[0] > 4) return false;
  p.nord = p.box_dims[0];
  p.box_run[0] = std::min(p.box_run[0], 3);
  // An input that runs along with the output, or is broadcast along its runs, is read in place; any
  // other one is staged, in vectors where it is contiguous along its fastest axis.
  int64_t lds = 0;
  int staged = 0;
  const int bytes = es[0] + es[1] + (nin == 2 ? es[2] : 0);
  for (int x = 1; x <= nin; ++x) {
    bool along = true, broadcast = true;
    int64_t run = es[x];
    for (int k = 0; k < p.box_run[0]; ++k) {
      const int d = p.ord_o[k];
      along = along && ops[x]->stride[d] == run;
      broadcast = broadcast && ops[x]->stride[d] == 0;
      run *= ext[d];
    }
    const int8_t *o = x == 1 ? p.ord_a : p.ord_b;
    if (along || broadcast) {
      p.box_how[x - 1] = 1;
    } else {
      // (strided along its own fastest axis: the form for any alignment gathers such an input's elements)
      if (p.box_run[x] == 0) return false;
      p.box_how[x - 1] = 0;
      ++staged;
      int64_t rows = 1, len = 1;
      for (int k = 0; k < p.box_dims[x]; ++k) (k < p.box_run[x] ? len : rows) *= ext[o[k]];
      int64_t pitch = (len * es[x] + 15) / 16 * 16;
      if (pitch % 32 == 0) pitch += 16;
      lds += pitch * rows;
      // (16-byte loads for four bytes or less of a row: bytes [2, 18528704] three apart, cast to 16 bits, 87 us, 31
      // in tiles; ...
      if ((len * es[x] + 15) / 16 * 16 * rows >= 4 * elems * es[x]) return false;
      // ... or lanes that read from the same few banks, more than 16 turns and three per byte that an element
      // moves: of 970 such calls three in five lose to tiles, of 39000 others one in twenty does)
      int32_t pos[kMaxDims] = {0};
      int64_t at = es[x], row = pitch;
      for (int k = 0; k < p.box_dims[x]; ++k) {
        int64_t &step = k < p.box_run[x] ? at : row;
        pos[o[k]] = (int32_t)step;
        step *= ext[o[k]];
      }
      if (bank_turns(p, V, es[x], ext, pos) > std::max(16, 3 * bytes)) return false;
    }
  }
  p.stage_a = p.box_how[0] == 0;
  p.stage_b = nin == 2 && p.box_how[1] == 0;
  p.lds_bytes = lds;
  if (!p.stage_a && !p.stage_b) return false;
  if (lds > 64 * 1024) return false;
  // (vectors of which an eighth or less lies in a run: bytes [4, 161832, 2, 2], pairs with a gap, 13.8 us, 10.6 in tiles)
  int64_t run = 1;
  for (int k = 0; k < p.box_run[0]; ++k) run *= ext[p.ord_o[k]];
  if (run * 8 <= V) return false;
  // Few boxes that stage what tiles read in place: long vectors are few lanes (of 360 calls on two such
  // inputs of bytes 206 lose; [9, 262] 5.0 us in tiles, 6.2 so).
  if (!tiles_stage && p.total_tiles < 2 * kNumCUs && (V >= 16 || (V >= 8 && staged == 2))) return false;
  p.tile_bits = ilog2_ceil(elems);
  p.vecw_o = ilog2_ceil(V);
  p.vec = V;
  for (int d = 0; d < n; ++d) p.tile_log2[d] = ilog2_ceil(ext[d]);   // (plan inspection)
  p.kernel = kKernelBox;
  p.grid = p.total_tiles;
  p.block = kBlock;
  p.box_group = kBoxGroup;
  return true;
}

}  // namespace

namespace {
// Is this copy or cast one between planes and pixels that the pixel kernels take?  C channels side
// by side on one side (pixels dense: C elements apart) and planes on the other, contiguous along the
// pixels; at least one vector of pixels; the types the kernels exist for; native byte order, or a
// plain copy within the other one.
int pixel_layout(const EwPlan &p, int es_o, int es_a) {
  const int n = p.ndim, sa = p.a.dtype, so = p.out.dtype;
  if (n < 2) return 0;
  auto sample = [](int dt) { return dt == DT_U8 || dt == DT_U16 || dt == DT_I16 || dt == DT_F16 || dt == DT_F32; };
  if (sa == so ? es_o > 8 || !(p.swap == 0 || p.swap == 5) : !sample(sa) || !sample(so) || p.swap != 0) return 0;
  const int64_t v = 16 / es_o;
  auto fits = [&](int64_t m, int64_t c) {
    const int64_t mvec = (m + v - 1) / v, total = mvec * (p.numel / (m * c));
    return c >= 2 && c <= 4 && m >= v && m < ((int64_t)1 << 31) && total < ((int64_t)1 << 31) &&
           (total + kBlock - 1) / kBlock <= max_launch_blocks();
  };
  const int64_t c1 = p.size[n - 2], c2 = p.size[n - 1];
  if (p.out.stride[n - 1] == es_o && p.a.stride[n - 2] == es_a && p.a.stride[n - 1] == c1 * es_a && fits(c2, c1)) return kKernelToPlanes;
  if (p.out.stride[n - 1] == es_o && p.out.stride[n - 2] == c2 * es_o && p.a.stride[n - 2] == es_a && p.a.stride[n - 1] != es_a && fits(c1, c2))
    return kKernelToPixels;
  return 0;
}
}  // namespace

int plan_elementwise(int nin, int op, const ocn_tensor *a, const ocn_tensor *b,
                     const ocn_tensor *out, uint32_t flags, EwPlan *plan) {
  EwPlan p;
  p.nin = nin;
  p.op = op;
  int rc;
  if ((rc = check_tensor(a)) != OCN_OK) return rc;
  if (nin == 2 && (rc = check_tensor(b)) != OCN_OK) return rc;
  if ((rc = check_tensor(out)) != OCN_OK) return rc;
  if (nin == 2 ? (op < 0 || op >= B_COUNT) : (op < 0 || op >= U_COUNT)) return OCN_ERR_OP;
  if (a->device != out->device || (nin == 2 && b->device != out->device)) return OCN_ERR_DEVICE;
  if ((rc = check_broadcast(a, out)) != OCN_OK) return rc;
  if (nin == 2 && (rc = check_broadcast(b, out)) != OCN_OK) return rc;

  // operands stored in the other byte order (section 3.1.3); one-byte scalars have no order
  p.swap = (a->byteswapped && scalar_size(a->dtype) > 1 ? 1 : 0) |
           (nin == 2 && b->byteswapped && scalar_size(b->dtype) > 1 ? 2 : 0) |
           (out->byteswapped && scalar_size(out->dtype) > 1 ? 4 : 0);

  // compute type and strict-mode checks (section 3.2.1)
  const int sa = a->dtype, sb = nin == 2 ? b->dtype : a->dtype, so = out->dtype;
  if (nin == 2) {
    if ((flags & OCN_STRICT_TYPES) && sa != sb) return OCN_ERR_DTYPE;
    if ((flags & OCN_STRICT_TYPES) && !is_compare(op) && !is_logical(op) && sa != so) return OCN_ERR_DTYPE;
    const int promoted = promote(sa, sb);
    p.T = binary_compute_dtype(op, sa, sb, so, promoted, promote(promoted, so));
    if (!binary_supported(op, p.T)) return OCN_ERR_DTYPE;
    p.specialised = binary_specialised(op, sa, sb, so);
  } else {
    const bool modulus = op == U_ABS && dt_kind(sa) == K_CPLX;   // complex -> real of the same precision
    if ((flags & OCN_STRICT_TYPES) && op != U_LNOT && sa != so && !(modulus && so == dt_real_of(sa)))
      return OCN_ERR_DTYPE;
    p.T = unary_compute_dtype(op, sa, so);
    if (!unary_supported(op, p.T)) return OCN_ERR_DTYPE;
    p.specialised = unary_specialised(op, sa, so);
  }

  int64_t numel = 1;
  for (int d = 0; d < out->ndim; ++d) numel *= out->size[d];
  p.numel = numel;
  if (numel == 0) {  // nothing to do
    *plan = p;
    return OCN_OK;
  }
  if ((rc = check_alignment(a)) != OCN_OK) return rc;
  if (nin == 2 && (rc = check_alignment(b)) != OCN_OK) return rc;
  if ((rc = check_alignment(out)) != OCN_OK) return rc;
  if (!provably_non_overlapping(out)) return OCN_ERR_OVERLAP_OUT;
  if ((rc = check_alias(a, out)) != OCN_OK) return rc;
  if (nin == 2 && (rc = check_alias(b, out)) != OCN_OK) return rc;

  // ---- canonical dimension list ---------------------------------------------------------
  Dim dims[kMaxDims];
  int n = 0;
  int64_t off_o = out->offset, off_a = a->offset, off_b = nin == 2 ? b->offset : 0;
  for (int d = 0; d < out->ndim; ++d) {
    if (out->size[d] == 1) continue;  // drop
    Dim x{out->size[d], out->stride[d], bstride(a, out, d), nin == 2 ? bstride(b, out, d) : 0};
    if (x.so < 0) {  // flip so that the output walks forward
      off_o += (x.size - 1) * x.so;
      off_a += (x.size - 1) * x.sa;
      off_b += (x.size - 1) * x.sb;
      x.so = -x.so; x.sa = -x.sa; x.sb = -x.sb;
    }
    dims[n++] = x;
  }
  // sort by output stride, slowest first (insertion sort: n <= 8, and stable)
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && dims[j].so > dims[j - 1].so; --j) std::swap(dims[j], dims[j - 1]);
  // merge neighbours that every operand walks as one longer dimension
  int m = 0;
  for (int i = 0; i < n; ++i) {
    if (m > 0) {
      Dim &u = dims[m - 1];
      const Dim &v = dims[i];
      if (u.so == v.so * v.size && u.sa == v.sa * v.size && u.sb == v.sb * v.size) {
        u.size *= v.size;
        u.so = v.so; u.sa = v.sa; u.sb = v.sb;
        continue;
      }
    }
    dims[m++] = dims[i];
  }
  n = m;
  if (n == 0) {  // a single element
    dims[0] = Dim{1, (int64_t)dt_size(so), 0, 0};
    n = 1;
  }
  p.ndim = n;
  for (int d = 0; d < n; ++d) {
    p.size[d] = dims[d].size;
    p.out.stride[d] = dims[d].so;
    p.a.stride[d] = dims[d].sa;
    p.b.stride[d] = dims[d].sb;
  }
  p.off_out = off_o; p.off_a = off_a; p.off_b = off_b;
  p.out.ptr = (char *)out->base + off_o; p.out.dtype = so;
  p.a.ptr = (char *)a->base + off_a; p.a.dtype = sa;
  p.b.ptr = nin == 2 ? (char *)b->base + off_b : nullptr; p.b.dtype = sb;

  // ---- kernel selection ------------------------------------------------------------------
  const int es_o = dt_size(so), es_a = dt_size(sa), es_b = dt_size(sb);
  // An output of 32 MiB or more will not be found in the caches by whoever reads it next
  // (4 MB of L2 per XCD, 256 MB of Infinity Cache shared with the inputs): write it with
  // streaming stores, so that its dirty lines do not burden the next kernel.
  p.nt_store = numel * es_o >= kStreamBytes;
  const int inner = n - 1;
  const int es_max = std::max({es_o, es_a, nin == 2 ? es_b : es_a});
  const int es_min = std::min({es_o, es_a, nin == 2 ? es_b : es_a});
  const int VT = rows_vec(es_o, es_max);                    // the tiled kernel's compute vector (Sig::V)
  const int V = rows_stream_vec(es_o, es_min, es_max);      // the rows kernel's vector (Sig::VR)
  auto inner_ok = [&](int64_t stride, int es) { return stride == es || stride == 0; };
  bool rows = p.specialised && p.out.stride[inner] == es_o && inner_ok(p.a.stride[inner], es_a) &&
              (nin == 1 || inner_ok(p.b.stride[inner], es_b));
  if (rows) {
    // does every row of every non-broadcast operand start on a boundary of its vector?
    auto aligned = [&](const Operand &x, int es) {
      if (x.stride[inner] == 0) return true;
      const int64_t vb = (int64_t)V * es;
      if ((intptr_t)x.ptr % vb != 0) return false;
      for (int d = 0; d < inner; ++d)
        if (x.stride[d] % vb != 0) return false;
      return true;
    };
    p.rows_aligned = aligned(p.out, es_o) && aligned(p.a, es_a) && (nin == 1 || aligned(p.b, es_b));
    // 32-bit vector and row indices (a flat 1-D tensor needs no division and may be larger)
    const int64_t vpr = (p.size[inner] + V - 1) / V;
    const int64_t nrows = numel / p.size[inner];
    if (n > 1 && (vpr * nrows >= ((int64_t)1 << 31))) rows = false;
    // more workgroups than one launch may have: the generic kernel, which loops, takes it (rows
    // that are not aligned go to the tiled kernel below, which has its own numbering)
    if ((vpr * nrows + (int64_t)kBlock * rows_stream_unroll(V, es_min) - 1) /
            ((int64_t)kBlock * rows_stream_unroll(V, es_min)) > max_launch_blocks()) {
      rows = false;
      if (p.rows_aligned) p.specialised = false;
    }
    // Unaligned rows of a few elements, which vectors cross one after the other, element by element:
    // two or four per row and eight per vector go to the tiles once they are millions (3.9 million rows
    // of two halves 136 us here, 32 there), and 8- or 16-bit integers with floats to the
    // generic-dtype kernel (rows of five: 8.2 us, 12.4 here; pairs at any size: 4.6 million 62 and 121).
    if (rows && n > 1 && !p.rows_aligned) {
      const int64_t n0 = p.size[inner];
      if (V == 8 && (n0 == 2 || n0 == 4) && numel >= (int64_t)4 << 20) rows = false;
      if (nin == 2 && small_integer_pair(sa, sb) && n0 < V + 2 && n0 % V != 0 && numel >= 1 << 14 && (n0 == 2 || numel < 1 << 19)) {
        rows = false;
        p.specialised = false;
      }
    }
    if (rows) {
      p.kernel = OCN_KERNEL_EW_ROWS;
      p.vec = V;
      p.unroll = rows_stream_unroll(V, es_min);
      p.a_inner_bcast = p.a.stride[inner] == 0;
      p.b_inner_bcast = nin == 2 && p.b.stride[inner] == 0;
      // Inputs too large to be found in a cache again are read with streaming loads: those
      // that move one piece per lane and are not broadcast along any dim (a broadcast operand
      // is re-read from the caches by every row).
      auto streamed = [&](const Operand &x, int es) {
        if (V * es > 16) return false;
        int64_t distinct = es;
        for (int d = 0; d < n; ++d) {
          if (x.stride[d] == 0) return false;
          distinct *= p.size[d];
        }
        return distinct >= kStreamBytes;
      };
      p.nt_a = streamed(p.a, es_a);
      p.nt_b = nin == 2 && streamed(p.b, es_b);
      const int64_t nvec = vpr * nrows;
      p.grid = (nvec + (int64_t)kBlock * p.unroll - 1) / ((int64_t)kBlock * p.unroll);
      p.lds_bytes = 0;
      *plan = p;
      return OCN_OK;
    }
  }

  // A plain copy from planes into an output whose fastest axis is 2..8 elements long, the
  // next output axis being the input's fastest (channel-first to channel-last): lanes take
  // 16-byte vectors along that long axis and deal them out in registers.
  if (nin == 1 && op == U_IDENT && sa == so && es_o <= 8 && n >= 2 && (p.swap == 0 || p.swap == 5)) {
    const int64_t c = p.size[n - 1], mlen = p.size[n - 2], vv = 16 / es_o;
    bool ok = c >= 2 && c <= 8 && p.out.stride[n - 1] == es_o && p.out.stride[n - 2] == c * es_o &&
              p.a.stride[n - 2] == es_o && p.a.stride[n - 1] % 16 == 0 && mlen % vv == 0 &&
              (intptr_t)p.out.ptr % 16 == 0 && (intptr_t)p.a.ptr % 16 == 0;
    for (int d = 0; d < n - 2 && ok; ++d) ok = p.out.stride[d] % 16 == 0 && p.a.stride[d] % 16 == 0;
    const int64_t nvec = numel / (c * vv);
    const int64_t grid = (nvec + kBlock - 1) / kBlock;
    if (ok && nvec < ((int64_t)1 << 31) && grid <= max_launch_blocks()) {
      p.kernel = OCN_KERNEL_EW_INTERLEAVE;
      p.vec = (int)vv;
      p.grid = grid;
      p.nt_a = numel * es_o >= kStreamBytes;
      p.lds_bytes = (int64_t)kBlock * c * 16;
      *plan = p;
      return OCN_OK;
    }
  }

  if (!p.specialised) {
    // generic-dtype kernel: one element per lane, conversions through runtime switches
    p.kernel = OCN_KERNEL_EW_GENERIC;
    p.vec = 1;
    p.grid = std::min<int64_t>((numel + kBlock - 1) / kBlock, max_launch_blocks());   // the kernel loops beyond that
    *plan = p;
    return OCN_OK;
  }

  // A copy or cast between planes and interleaved pixels of two to four channels takes the pixel
  // kernels where the all-vector tiled form does not apply (uint8 pixels [32, 480, 640, 3] to float
  // planes: 32.6 us in tiles of any alignment, 21.8 there; uint8 planes to float pixels 65.7 and 21.8).
  const int pixels = nin == 1 && op == U_IDENT ? pixel_layout(p, es_o, es_a) : 0;
  const bool pixels_ok = pixels != 0;
  auto plan_pixels = [&](EwPlan &q) {
    q.kernel = pixels;
    q.vec = 16 / es_o;
    q.stage_a = q.stage_b = false;
    q.lds_bytes = pixels == kKernelToPixels ? (int64_t)kBlock * 16 * q.size[n - 1] : 0;
    for (int d = 0; d < kMaxDims; ++d) q.tile_log2[d] = 0;
    const int64_t m = q.size[pixels == kKernelToPlanes ? n - 1 : n - 2], c = q.size[pixels == kKernelToPlanes ? n - 2 : n - 1];
    q.grid = ((m + q.vec - 1) / q.vec * (numel / (m * c)) + kBlock - 1) / kBlock;
  };

  // tiled / generic: stage an input through LDS when its fastest axis is not the output's
  const int fo = inner;  // the output's fastest dim after sorting
  const int fa = fastest_dim(n, [&](int d) { return p.a.stride[d]; });
  const int fb = nin == 2 ? fastest_dim(n, [&](int d) { return p.b.stride[d]; }) : -1;
  p.stage_a = fa >= 0 && fa != fo;
  p.stage_b = fb >= 0 && fb != fo;
  // First the small tiles that suit the unclipped all-vector form of the tiled kernel.  A plan
  // that cannot take that form is laid out again for the general form, which wants larger
  // tiles (its per-tile overhead is higher), and without staging for inputs whose own fastest
  // axis is shorter than 32 bytes: coalescing along such an axis gains less than the general
  // form's staging costs (measured on channel-last to channel-first copies with 3 channels).
  bool stage_a0 = p.stage_a, stage_b0 = p.stage_b;
  for (int rule = kTilesVector; rule <= kTilesGeneral; ++rule) {
    if (rule == kTilesAny && pixels_ok) {
      *plan = p;
      plan_pixels(*plan);
      return OCN_OK;
    }
    if (rule == kTilesAny) {
      // Boxes of any extents where the tiles above do not fit: over 34500 random calls of one to five dims, 2000
      // to 60 million elements and ten types they take 0.72 of the time of tiles of any alignment (6000 x 5000
      // plus a transpose 73.7 -> 69.3 us, float [200001, 17, 17] transposed 289 -> 105, complex products of
      // [5, 25, 5, 38, 17] 15.3 -> 6.9); one call in 38 is slower by more than 5 %, one in 300 by 20 %.  Tiles
      // keep what was not measured, 2^31 elements and more; inputs strided along their own fastest axis,
      // which they gather (every other float of [200001, 17, 17] 174 us, 373 by elements in boxes); and of
      // matrices: large ones of four bytes with one input (5000 x 3001 27.4 us in tiles and 32.7 in boxes,
      // 1185 x 50123 83 and 119, 3490 x 1122 12.6 and 10.8), and two kinds whose layout plan inspection has
      // always reported as tiles although boxes are faster: small ones that fill tiles of 64 x 64 to 70 %
      // (float 500 x 701 6.5 us in tiles, 5.0 in boxes) and those with an output axis of a quarter vector
      // (bytes 4194304 x 2 13.9 and 9.6).
      const int64_t n0 = p.size[0], n1 = p.size[n - 1];
      const bool matrix_in_tiles =
          n == 2 && ((nin == 1 && es_o == 4 && es_a == 4 && n0 >= 1024 && n1 >= 1024) ||
                     (numel < 1 << 19 && numel * 10 >= (n0 + 63) / 64 * 64 * ((n1 + 63) / 64 * 64) * 7) ||
                     (n1 * 4 <= VT && (n1 & (n1 - 1)) == 0 && numel >= n1 << 19));
      EwPlan q = p;
      const bool tiles_stage = (stage_a0 && p.size[fa] * es_a >= 32) || (stage_b0 && p.size[fb] * es_b >= 32);
      if (numel < (int64_t)1 << 31 && !matrix_in_tiles && plan_boxes(q, tiles_stage)) {
        *plan = q;
        return OCN_OK;
      }
      if (stage_a0 && p.size[fa] * es_a < 32) stage_a0 = false;
      if (stage_b0 && p.size[fb] * es_b < 32) stage_b0 = false;
    }
    p.stage_a = stage_a0;
    p.stage_b = stage_b0;
    for (int d = 0; d < kMaxDims; ++d) p.tile_log2[d] = 0;
    p.fast_tiled = false;
    choose_tiles(p, (TileRule)rule, fa, fb);
    tile_order(p, p.out.stride, p.ord_o);
    tile_order(p, p.a.stride, p.ord_a);
    tile_order(p, p.b.stride, p.ord_b);
    p.nord = 0;
    for (int d = 0; d < n; ++d)
      if (p.tile_log2[d] > 0) ++p.nord;
    // an input whose fastest tiled dim is the output's needs no staging after all
    if (p.nord == 0 || p.ord_a[0] == p.ord_o[0]) p.stage_a = false;
    if (p.nord == 0 || p.ord_b[0] == p.ord_o[0]) p.stage_b = false;

    // ---- vector widths of the three enumeration orders -----------------------------------
    // aligned: base pointer and every stride except the one along `skip` are multiples of vb
    auto aligned = [&](const Operand &x, int64_t vb, int skip) {
      if (rule == kTilesAny) return true;   // that form takes any alignment
      if ((intptr_t)x.ptr % vb != 0) return false;
      for (int d = 0; d < n; ++d)
        if (d != skip && x.stride[d] % vb != 0) return false;
      return true;
    };
    auto log2i = [](int v) { int l = 0; while ((1 << l) < v) ++l; return l; };
    p.vecw_o = p.vecw_a = p.vecw_b = 0;
    if (p.nord > 0) {
      const int d0 = p.ord_o[0];
      // compute phase: V consecutive elements along the output's fastest dim per lane
      bool ok = p.out.stride[d0] == es_o && p.tile_log2[d0] >= log2i(VT) && VT > 1 &&
                aligned(p.out, (int64_t)VT * es_o, d0);
      auto direct_ok = [&](const Operand &x, int es, bool staged) {
        if (staged) return true;
        if (x.stride[d0] != es) return true;  // broadcast or strided: element loads, no constraint
        return aligned(x, (int64_t)VT * es, d0);
      };
      ok = ok && direct_ok(p.a, es_a, p.stage_a) && (nin == 1 || direct_ok(p.b, es_b, p.stage_b));
      if (ok) p.vecw_o = log2i(VT);
      auto stage_vec = [&](const Operand &x, int es, const int8_t *ord) {
        const int v = 16 / es;
        if (v <= 1) return 0;
        const int f = ord[0];
        if (rule == kTilesAny) return log2i(v);   // (strided: its elements are fetched one by one)
        if (x.stride[f] != es || p.tile_log2[f] < log2i(v) || !aligned(x, 16, f)) return 0;
        return log2i(v);
      };
      if (p.stage_a) p.vecw_a = stage_vec(p.a, es_a, p.ord_a);
      if (p.stage_b) p.vecw_b = stage_vec(p.b, es_b, p.ord_b);
    }
    const int64_t tile_elems = (int64_t)1 << p.tile_bits;
    p.lds_bytes = 0;
    if (p.stage_a) p.lds_bytes += (tile_elems * es_a + 15) / 16 * 16;
    if (p.stage_b) p.lds_bytes += (tile_elems * es_b + 15) / 16 * 16;
    p.total_tiles = 1;
    for (int d = 0; d < n; ++d) {
      p.ntiles[d] = (p.size[d] + ((int64_t)1 << p.tile_log2[d]) - 1) >> p.tile_log2[d];
      p.total_tiles *= p.ntiles[d];
    }
    // One tile per workgroup.  (Persistent workgroups looping over tiles, and handing each XCD
    // a contiguous range of tiles, were both measured slower on MI355X.)
    p.grid = p.total_tiles;
    p.kernel = (p.stage_a || p.stage_b) ? OCN_KERNEL_EW_TILED : OCN_KERNEL_EW_GENERIC;
    // The unclipped all-vector form of the tiled kernel: no tile is clipped, every enumeration
    // order moves whole vectors over at least one full pass, inputs that are not staged are
    // contiguous along the output's fastest dim, and inside a tile every stride is non-negative
    // with offsets that fit 31 bits.
    if (rule != kTilesAny && p.kernel == OCN_KERNEL_EW_TILED && p.vecw_o > 0) {
      bool ok = true;
      const int d0 = p.ord_o[0];
      if (p.stage_a ? p.vecw_a == 0 : p.a.stride[d0] != es_a) ok = false;
      if (nin == 2 && (p.stage_b ? p.vecw_b == 0 : p.b.stride[d0] != es_b)) ok = false;
      const int vmax = std::max(p.vecw_o, std::max(p.stage_a ? p.vecw_a : 0, p.stage_b ? p.vecw_b : 0));
      if (p.tile_bits - vmax < 8) ok = false;  // fewer vectors than lanes in some order
      int64_t span_o = 0, span_a = 0, span_b = 0;
      for (int d = 0; d < n && ok; ++d) {
        const int64_t ext = (int64_t)1 << p.tile_log2[d];
        if (p.size[d] % ext != 0) ok = false;
        if (ext > 1 && (p.a.stride[d] < 0 || p.b.stride[d] < 0)) ok = false;
        span_o += (ext - 1) * p.out.stride[d];
        span_a += (ext - 1) * iabs64(p.a.stride[d]);
        span_b += (ext - 1) * iabs64(p.b.stride[d]);
      }
      const int64_t lim = ((int64_t)1 << 31) - 64;
      p.fast_tiled = ok && span_o < lim && span_a < lim && span_b < lim;
    }
    if (p.fast_tiled) {
      // An input whose contiguous run inside a tile is a fraction of a 128-byte line shares its
      // lines with the neighbouring tiles along the dim that continues the run.  Such tiles are
      // handed to workgroups that land on the same XCD one after the other (see the kernel), so
      // that the line is fetched into that L2 once instead of once per tile.
      p.pair_dim = -1;
      p.pair_log2 = 0;
      const Operand *ins[2] = {&p.a, &p.b};
      const int es_in[2] = {es_a, es_b};
      for (int x = 0; x < nin && p.pair_dim < 0; ++x) {
        int64_t run = es_in[x];
        int cont = -1;
        for (bool more = true; more;) {
          more = false;
          for (int d = 0; d < n; ++d) {
            if (iabs64(ins[x]->stride[d]) != run || p.size[d] == 1) continue;
            const int64_t ext = (int64_t)1 << p.tile_log2[d];
            if (ext >= p.size[d]) {  // fully covered: the run goes on along another dim
              run *= p.size[d];
              more = true;
            } else {                 // the neighbouring tiles along d continue the run
              run *= ext;
              cont = d;
            }
            break;
          }
        }
        if (cont < 0 || run >= 128 || 128 % run != 0 || ins[x]->stride[cont] < 0) continue;
        const int lg = run == 64 ? 1 : run == 32 ? 2 : 0;
        if (lg == 0 || p.ntiles[cont] % (1 << lg) != 0 || p.total_tiles % (8 << lg) != 0) continue;
        p.pair_dim = cont;
        p.pair_log2 = lg;
      }
      break;
    }
    if (rule == kTilesAny) {
      // Tiles of any size and alignment: up to four tiled dims, the output contiguous along its
      // fastest one, non-negative strides and offsets below 2^31 bytes inside a tile.
      bool ok = p.nord > 0 && p.nord <= 4 && p.out.stride[p.ord_o[0]] == es_o && p.vecw_o == log2i(VT) && p.tile_bits <= 12 &&
                (!p.stage_a || p.tile_log2[p.ord_a[0]] >= p.vecw_a) && (!p.stage_b || p.tile_log2[p.ord_b[0]] >= p.vecw_b) && p.total_tiles <= max_launch_blocks();
      // Not where vectors are mostly empty or gather their elements, once that is most of the time (in
      // smaller launches this form's fewer round trips win): an output whose fastest axis is a
      // quarter of its vector, a power of two that the general form's tiles fit exactly (2.4 M x 4 x 2
      // int8 plus a permuted view 147 us here, 49 there; three elements gain up to six million), and
      // two inputs strided along a single long run (4 x 2.6 M bytes, 1 and 4 apart: 42 and 23).
      const int64_t nfo = p.size[fo];
      if (nfo * 4 <= VT && (nfo & (nfo - 1)) == 0 && numel >= nfo << 19) ok = false;
      auto gathered = [&](const Operand &x, int es, bool staged) { return !staged && x.stride[fo] != es && x.stride[fo] != 0; };
      if (nin == 2 && p.nord == 1 && VT >= 8 && numel >= (int64_t)2 << 20 && gathered(p.a, es_a, p.stage_a) && gathered(p.b, es_b, p.stage_b))
        ok = false;
      int64_t span_o = 0, span_a = 0, span_b = 0;
      for (int d = 0; d < n && ok; ++d) {
        const int64_t ext = (int64_t)1 << p.tile_log2[d];
        if (ext > 1 && (p.a.stride[d] < 0 || p.b.stride[d] < 0)) ok = false;
        span_o += ext * p.out.stride[d];
        span_a += ext * iabs64(p.a.stride[d]);
        span_b += ext * iabs64(p.b.stride[d]);
      }
      const int64_t lim = ((int64_t)1 << 31) - 64;
      // An input that is read in vectors has to be as long as one: a vector that runs past its end
      // is loaded from further back, by whole elements.
      auto long_enough = [&](const Operand &x, int es, bool staged, const int8_t *ord, int vecw) {
        if (x.stride[staged ? ord[0] : p.ord_o[0]] != es) return true;
        int64_t bytes = es;
        bool whole = true;
        for (int d = 0; d < n; ++d) {
          bytes += (p.size[d] - 1) * iabs64(x.stride[d]);
          whole = whole && x.stride[d] % es == 0;
        }
        return bytes >= ((int64_t)es << vecw) + (whole ? 0 : es - scalar_size(x.dtype));
      };
      ok = ok && long_enough(p.a, es_a, p.stage_a, p.ord_a, p.stage_a ? p.vecw_a : p.vecw_o) &&
           (nin == 1 || long_enough(p.b, es_b, p.stage_b, p.ord_b, p.stage_b ? p.vecw_b : p.vecw_o));
      if (ok && span_o < lim && span_a < lim && span_b < lim) {
        p.kernel = kKernelTiledAny;
        // Lanes per workgroup.  With one vector per lane, operand and pass a workgroup of 512 lanes
        // has a tile of 4096 floats in flight at once and two of them share a CU's wavefront slots
        // evenly (float 6000 x 5000 plus a transpose: 74.8 us, 79.6 with 256 lanes, 85.3 with 1024),
        // but more lanes than the output has vectors only wait for the others.  Few tiles leave
        // most of the chip idle anyway: there every lane is worth having (45 000 complex products: 7.7
        // us with 1024, 10.3 with 256).
        const int nvec_o = 1 << (p.tile_bits - p.vecw_o);
        const int nvec = std::max(nvec_o, std::max(p.stage_a ? 1 << (p.tile_bits - p.vecw_a) : 0, p.stage_b ? 1 << (p.tile_bits - p.vecw_b) : 0));
        const bool few = p.total_tiles <= kNumCUs;
        // The bound on workgroups is one on lanes (256 in each): larger workgroups keep to it.
        const int64_t most = max_launch_blocks() * kBlock;
        p.block = kBlock;
        while (p.block < (few ? 1024 : 512) && p.block < (few ? nvec : nvec_o) && p.total_tiles * p.block * 2 <= most) p.block *= 2;
        break;
      }
    }
  }  // rules
  p.vec = 1 << p.vecw_o;
  // (small tensors of 8- and 16-bit integers with floats into outputs with gaps, which only the general
  // form takes: the generic-dtype kernel; int8 [52, 55] plus a float column 17.2 us here, 7.8 there)
  const bool small_general = nin == 2 && small_integer_pair(sa, sb) && !p.fast_tiled && p.kernel != kKernelTiledAny &&
                             p.out.stride[fo] != es_o && numel < 1 << 19;
  // (tile coordinates are 32-bit: beyond them the 64-bit generic kernel)
  if (small_general || p.total_tiles >= ((int64_t)1 << 31)) {
    p.specialised = false;
    p.kernel = OCN_KERNEL_EW_GENERIC;
    p.vec = 1;
    p.stage_a = p.stage_b = false;
    p.lds_bytes = 0;
    p.grid = (numel + kBlock - 1) / kBlock;
  }
  *plan = p;
  return OCN_OK;
}

// ---------------------------------------------------------------------------------------
// reduction planning
// ---------------------------------------------------------------------------------------

bool reduce_supported(int op, int dt) {
  if (op < 0 || op >= R_COUNT || !valid_dtype(dt)) return false;
  const int k = dt_kind(dt);
  switch (op) {
    case R_SUM: case R_ANY: case R_ALL: return true;
    default: return k != K_CPLX;
  }
}

int reduce_acc_dtype(int op, int dt) {
  const int k = dt_kind(dt);
  switch (op) {
    case R_SUM: case R_PROD:
      if (k == K_BOOL || k == K_SINT) return DT_I64;
      if (k == K_UINT) return DT_U64;
      if (dt == DT_F16) return DT_F32;
      if (dt == DT_F32 || dt == DT_F64) return DT_F64;
      return dt == DT_C16 ? DT_C32 : DT_C64;
    case R_MIN: case R_MAX: return dt;
    default: return DT_BOOL;
  }
}

namespace {

struct RDim { int64_t size, sa, so, sb; };

// sorts by decreasing key, then merges neighbours that every operand walks as one longer dim
template <class Key> int sort_merge_by(RDim *d, int n, Key key) {
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && key(d[j]) > key(d[j - 1]); --j) std::swap(d[j], d[j - 1]);
  int m = 0;
  for (int i = 0; i < n; ++i) {
    if (m > 0) {
      RDim &u = d[m - 1];
      const RDim &v = d[i];
      if (u.sa == v.sa * v.size && u.so == v.so * v.size && u.sb == v.sb * v.size) {
        u.size *= v.size; u.sa = v.sa; u.so = v.so; u.sb = v.sb;
        continue;
      }
    }
    d[m++] = d[i];
  }
  return m;
}

int sort_merge(RDim *d, int n, bool by_out) {
  return sort_merge_by(d, n, [&](const RDim &x) { return by_out ? x.so : iabs64(x.sa); });
}

#ifndef OCN_RED_TARGET_WAVES
#define OCN_RED_TARGET_WAVES (256 * 16)
#endif
constexpr int64_t kTargetWaves = OCN_RED_TARGET_WAVES;  // enough wavefronts to occupy every CU
// A row reduction that runs in the lean form of the kernel and has to be split over workgroups
// is split into half as many wavefronts, eight per CU: with four 16-byte loads per lane in
// flight that measured fastest (int8 full sum of 2^28: 41.9 us, against 45.2, 44.7 and 43.6 with
// 6, 12 and 16 per CU; the count of a > b over 2^26 pairs: 81.7 against 83.2 with 16).  The
// general kernel's element loads want the sixteen (full sum of a stride-2 view: 96 against 104 us).
constexpr int64_t kLeanSplitWaves = 256 * 8;
// Outputs of at most this many bytes of input that would be split (a chip hardly filled) are taken whole
// by sixteen wavefronts each: one reads 256 KiB in about 2 us, and the second launch of a split
// reduction costs 2 to 5 (float sums of 128 to 250 KiB 5.5 -> 4.1 .. 4.8 us; int8 of 254 KiB 6.4 -> 5.3).  Where a
// CU is slower than that, below the size that is split in three: vectors that start inside four bytes, which
// it reads at a third of the rate (maxima of 130 KiB of halves 7.1 us in two parts and 6.6, of 180 KiB 7.7 and
// 7.9; int16 sums of 175 KiB 8.6 and 7.9; of 200 KiB in three 7.1 and 8.5, of 250 KiB 7.4 and 9.8), and products
// of signed bytes (160 KiB 11.1 and 11.7, 250 KiB 11.4 and 16.4).  But such outputs too where there are half as
// many as CUs, which a split does not make faster by much (128 of 200 KiB 10.1 and 9.3, 200 of them 12.0 and 9.8).
constexpr int64_t kOneWorkgroupBytes = 256 * 1024, kOneWorkgroupSlowBytes = 192 * 1024 - 1;
bool one_workgroup_each(int64_t bytes, int64_t nout, bool slow) {
  return bytes <= (slow && nout < kNumCUs / 2 ? kOneWorkgroupSlowBytes : kOneWorkgroupBytes);
}
constexpr int kLeanMaxLanes = 1024;

// Launch shape of the column kernels (plain and fused): lanes per row of columns, wavefronts per
// workgroup, and workgroups that share a column block through the workspace.
//   cpw    A whole wavefront per row, or as few lanes as the columns need, and fewer where more than
//          30 % of the lanes would have no column (they then take several rows at a time; 777
//          columns: 64 lanes, 76 % of them busy, ran 36 us against 41 with 32) and there are rows
//          enough to take (two rows of 42 doubles, 98352 times: 159 us with 32 lanes, 315 with 16; up
//          to 64 rows of all shapes tried ran 5 to 15 % faster without).
//   nw     As many wavefronts per workgroup as leave each lane 16 rows, up to about 4096 in all: they
//          combine through LDS, where more workgroups would combine through memory and a second
//          launch (float sums over the middle of [48, 1000, 777]: 36.6 us with sixteen and no
//          split, 38 to 40 with four and two to five splits).
//   split  Only where that leaves half of the chip idle and the wavefronts with runs of 32 rows and more
//          (8 columns of 38191 int16, 37 rows per lane: 23.6 us in one workgroup, 14.9 split), and rounded down, so that the workgroups go out in one round ([16384, 4099]: 55 us with 15
//          splits, 255 workgroups of sixteen wavefronts, 69 with 16).
// bounded: the partial results never outgrow what a call without a workspace has (columns whose
// vectors are not aligned: 8-bit ones have sixteen times the accumulators of one column per lane, and
// int8 [5000, 32767] would take 2 MiB for eight splits).
struct ColsShape { int cpw, nw; int64_t split; };
// Are columns that do not start on vector boundaries taken in whole vectors?  As soon as they fill one,
// but with eight and more elements per vector only where the vectors of all rows keep half of a
// workgroup's lanes busy (10 rows of 27 bytes, 13860 times: 31 us with a column per lane, 124 with two
// lanes per row; two and four elements per vector gained at every size).
bool unaligned_columns(int64_t nc, int64_t vec, int64_t rows) {
  return nc >= vec && (vec < 8 || (nc + vec - 1) / vec * rows >= kBlock / 2);
}
ColsShape choose_cols_shape(int64_t col_lanes, int64_t others, int64_t rows, int64_t nout, int acc_es, bool bounded) {
  ColsShape r;
  r.cpw = kWave;
  while (r.cpw > 1 && r.cpw / 2 >= col_lanes) r.cpw /= 2;
  while (rows >= 64 && r.cpw > 16 && col_lanes * 10 < (col_lanes + r.cpw - 1) / r.cpw * r.cpw * 7) r.cpw /= 2;
  const int64_t rpw = kWave / r.cpw;
  const int64_t blocks0 = (col_lanes + r.cpw - 1) / r.cpw * others;
  r.nw = 4;
  while (r.nw < 16 && blocks0 * r.nw * 2 <= kTargetWaves && rows >= r.nw * 2 * 16 * rpw) r.nw *= 2;
  r.split = 1;
  if ((blocks0 * r.nw < kTargetWaves / 4 || blocks0 * 2 <= kNumCUs) && rows >= r.nw * rpw * 32) {
    const int64_t want = std::max<int64_t>(1, kTargetWaves / (blocks0 * r.nw));
    r.split = std::min(want, rows / (r.nw * rpw * 8));
    // eight rows per lane, but sixteen where the partial results would outgrow what a call without
    // a workspace has
    const int64_t fits = (int64_t)OCN_REDUCE_SCRATCH_BYTES / (nout * acc_es);
    r.split = std::max<int64_t>(1, std::min(r.split, std::max(fits, std::min(want, rows / (r.nw * rpw * 16)))));
    if (bounded && r.split > fits) {
      r.split = std::max<int64_t>(1, fits);
      // narrower columns instead, until the workgroups go round once
      while (r.cpw > 16 && (col_lanes + r.cpw / 2 - 1) / (r.cpw / 2) * others * r.split <= kNumCUs + kNumCUs / 16) r.cpw /= 2;
    }
  }
  return r;
}

// Lanes per row of columns where the columns are cut into equal blocks and a workgroup's 1024 lanes go on
// through further rows (cols_flat_body); 0 where blocks of `cpw` lanes are as good.  Blocks of a power
// of two lanes leave the last one mostly empty, and with few workgroups per CU its CU idles too: what
// counts is the lanes of the fullest CU.  A reduction that would be split over its rows takes this form
// if it fills three quarters of the chip evenly by itself, which saves the second launch (not in blocks
// below 24 lanes where its rows are whole lines: [20, 4000, 800] floats 45.1 us split, 49.6 in 17 lanes).
// Floats [64, 2000, 516] 73 -> 47 us, [128, 512, 132] 15.6 -> 9.4, [200, 1000, 280] 47 -> 37; halves [48, 1000,
// 777] 27.7 -> 19.8; few rows gain as well, eight trips of the workgroup at least (int32 [3, 109, 24665] 12.4
// -> 7.0, cfloat [230, 89, 192] 9.3 -> 6.5; none of 539 calls of 32 to 127 rows loses).
constexpr int kFlatLanes = 1024;
int choose_flat_columns(int64_t col_lanes, int64_t others, int64_t rows, int cpw, int64_t split, bool aligned) {
  const int64_t blocks = (col_lanes + cpw - 1) / cpw;
  if (blocks < 2 || blocks * others > 4 * kNumCUs) return 0;
  // (wide columns of rows on vector boundaries, a thousand and more, fill the chip as they are: doubles [2588, 13648]
  // 46.4 us split and 54.1 so, eight of 96 such calls slower and the mean 1.10 times as fast; 3 of 637 wide ones with
  // fewer rows or rows off those boundaries, mean 1.17)
  if (col_lanes > 4096 && aligned && rows >= 1024) return 0;
  // (at least 15 % fewer lanes than the fullest CU has; at most a quarter more than an even share)
  int64_t best = split > 1 ? col_lanes * others * 5 / (4 * kNumCUs) + 1 : (blocks * others + kNumCUs - 1) / kNumCUs * cpw * 85 / 100;
  int lanes = 0;
  for (int64_t n = (col_lanes + kFlatLanes / 4 - 1) / (kFlatLanes / 4); n * 16 <= col_lanes && n * others <= 2 * kNumCUs; ++n) {
    const int64_t l = (col_lanes + n - 1) / n, groups = (col_lanes + l - 1) / l * others, cost = (groups + kNumCUs - 1) / kNumCUs * l;
    if (cost < best && rows >= kFlatLanes / l * 8 && (split == 1 || (groups * 4 >= 3 * kNumCUs && l >= (aligned ? 24 : 16)))) {
      best = cost;
      lanes = (int)l;
    }
  }
  return lanes;
}

// Few rows, many times over: a lane per vector of columns (cols_lane_body).  At most this many rows where
// a wavefront's lanes would cover several rows of columns (complex sums of [244044, 5, 15] 471 -> 38 us,
// int32 [60000, 32, 20] 152 -> 42), at most eight where columns are wide ([8, 1000, 5000] halves 32 -> 25; with
// 16 rows of 4096 floats 21.5 and 25.6, wavefronts that stream whole lines are faster); and enough lanes:
// twice as many for wide columns of 16 bits, whose vectors of eight are few (int16 [2, 335298] 5.4 us
// in blocks, 5.9 so; over 2 to 8 rows of 33000 vectors blocks take 0.9 of the time, of 60000 the same, of
// 90000 1.05 to 1.4).
// Bytes in vectors of sixteen keep the forms above: sixteen wide sums are too many registers (bool
// any of [5000, 20, 64] 43 us, where 27 columns, one to a lane, gain eight times).
constexpr int64_t kLaneRows = 32, kLaneWide = 48, kLaneColumns = 32768;

int64_t gcd64(int64_t a, int64_t b) { return b ? gcd64(b, a % b) : a; }

// Is the input (of a fused call: are the inputs) made of dense blocks of narrow rows (strip_kernels.hpp)?
struct StripBlocks {
  bool cols = false, rows = false;
  int bc = 0;               // fused: the input that is one element per row (columns) or one row for all (rows)
  int64_t inner = 1, width = 0, nrows = 0;
};
StripBlocks strip_blocks(const RedPlan &p) {
  StripBlocks s;
  if (p.nkept < 1 || p.nout < 1 || p.nredtot < 1) return s;
  const int es = dt_size(p.a_dtype), kc = p.nkept - 1;
  // Reduced axes of one element: rows of one (17 million floats 62 -> 43 us, halves 57 -> 43, doubles 68 -> 55;
  // bytes, stored one by one, 47 and 53)
  if (p.nred < 1) {
    s.rows = !p.fused && es > 1 && p.kstride_a[kc] == es;
    s.width = 1;
    s.nrows = p.ksize[kc];
    return s;
  }
  const int64_t V = 16 / es;
  auto cols = [&](const int64_t *ks, const int64_t *rs) { return ks[kc] == es && rs[0] == p.ksize[kc] * es; };
  auto rows = [&](const int64_t *ks, const int64_t *rs) { return rs[0] == es && ks[kc] == p.rsize[0] * es; };
  if (p.nred == 1) {
    const bool ca = cols(p.kstride_a, p.rstride_a), ra = rows(p.kstride_a, p.rstride_a);
    if (!p.fused) {
      s.cols = ca;
      s.rows = ra;
    } else {
      const bool cb = cols(p.kstride_b, p.rstride_b), rb = rows(p.kstride_b, p.rstride_b);
      const bool ea = p.kstride_a[kc] == 0, eb = p.kstride_b[kc] == 0;
      if (ca || cb) {
        s.bc = ca && cb ? 0 : ca ? 2 : 1;
        s.cols = s.bc == 0 || ((s.bc == 1 ? ea : eb) && p.ksize[kc] >= V);
      } else if (ra || rb) {
        s.bc = ra && rb ? 0 : ra ? 2 : 1;
        s.rows = s.bc == 0 || (s.bc == 1 ? ea && p.rstride_a[0] == es : eb && p.rstride_b[0] == es);
      }
    }
    s.width = s.cols ? p.ksize[kc] : p.rsize[0];
    s.nrows = s.cols ? p.rsize[0] : p.ksize[kc];
  } else if (!p.fused && p.nred == 2 && p.rstride_a[1] == es && p.kstride_a[kc] == p.rsize[1] * es &&
             p.rstride_a[0] == p.ksize[kc] * p.kstride_a[kc]) {
    s.cols = true;
    s.inner = p.rsize[1];
    s.width = p.ksize[kc] * s.inner;
    s.nrows = p.rsize[0];
  }
  if (s.width < 2 || s.width > (1 << 20)) s.cols = s.rows = false;
  return s;
}
// streaming loads: every vector of an input far larger than the caches starts on a vector boundary
bool strip_nt(const RedPlan &p, int64_t piece, int64_t block) {
  if (p.fused || (intptr_t)p.a_ptr % 16 || (piece < block && piece % 16)) return false;
  for (int d = 0; d + 1 < p.nkept; ++d)
    if (p.kstride_a[d] % 16) return false;
  return p.nout * p.nredtot * dt_size(p.a_dtype) >= kStreamBytes;
}

// Columns of dense blocks in strips.  Against the forms above, over 2000 random calls of 16 KB to 128 MB, all
// types: mean 1.16 times as fast, three times and more where rows of a few elements are summed in blocks of 30 to
// 300 (halves [676846, 51, 3] 1050 -> 60 us, floats [72727, 33, 10] 181 -> 24); 1.5 % slower by more than 5 %.
//   lanes   A group has as many as make four trips of a block, in multiples of m = width / gcd(width, vector),
//           and workgroups of 256 take several groups; blocks that keep a workgroup busy get one, of
//           1024 lanes where there are enough vectors for that on every CU.
//   split   Long blocks that are few, in as few workgroups as go round evenly.
// The forms above stay the better ones where: blocks are small altogether (one launch that the fold's
// barriers lengthen: doubles [262, 59] 5.0 and 5.7 us); few rows of whole vectors, which a lane walks by
// itself (halves [1095563, 7, 8] 49 and 68; below 16 MB tests hold it to that for all rows of a vector and more, at
// 9.4 us for int32 [5462, 31, 22] where strips take 7.2), or of bytes that a lane sums one by one, where a strip's lane
// sums sixteen in 64 bits each (int8 [249498, 17, 2] 7.8 and 17.6, uint8 [25146, 24, 12] 4.8 and 9.4); rows of many
// vectors and fewer than eight of them (floats [93, 4,
// 460] 4.0 and 5.6); splits that idle lanes, or rows of a large output, whose partial results would not
// fit what a call without a workspace has, leave uneven (floats [95, 340, 279] 9.6 and 14.4, sums over
// [12000, 2000] 23 and 36), splits of many small blocks ([63, 94, 748] 7.1 and 10.5), and splits of several blocks of fewer than
// 1024 rows of 4 bytes and more that take one launch otherwise (doubles [16, 85, 459] 4.0 and 7.0; 59 calls 0.86 times as fast
// so, longer ones 1.1; comparisons gain 2.3 times and stay); a workgroup per block where a fused call computes elements of 4
// bytes and more, and one input is an element per row (floats [65, 959, 118] 9.3 and 12.4; 310 calls 0.91) or blocks are short (4
// bytes: fewer than 64 rows 0.92, 8: than 256 0.92, beyond it 1.1 and 1.04); a few short blocks of 16-bit elements that a lane
// takes one by one otherwise (halves [616, 5, 48] 3.6 and 7.2; 13 calls 0.8).  With runs of columns in an output: few outputs of
// less than 24 MB, and runs that are read in vectors anyhow (strip_runs_from).
constexpr int64_t kStripSmall = 256 << 10, kStripBytesSmall = 2 << 20, kStripSplitSmall = 1 << 20, kStripInnerSmall = 4 << 20, kStripInnerFew = 24 << 20,
                  kStripLaneSmall = 16 << 20, kStripManySmall = 24 << 20, kStripSplitRows = 1024, kStripFewGroups = 40;
// Runs that the forms above read in vectors: bytes from which strips, and runs of long rows, are faster.  By the bytes of
// a run and whether they are whole vectors, over 2100 random calls (ratio of the times, other form to this): runs below 64 bytes
// from 8 MB on (0.9 below 6, 1.2 from 8 to 12, 1.9 above), longer ones from 12 (0.95, 1.4; sums of halves [1474, 42, 64] 6.2 and 9.8
// us), whole vectors 16 (0.85, 1.35).  Two outputs stay with the other form (50 calls 0.92; maxima of bool [295229, 2, 48]
// 8.8 and 18.3), three and four come from 24 MB on (three 0.78 below, 1.4 above).
constexpr int64_t strip_runs_from(int64_t run, bool whole, int64_t outputs) {
  return outputs < 3 ? INT64_MAX : outputs < 5 ? (int64_t)24 << 20 : (run < 64 ? 8 : whole ? 16 : 12) * ((int64_t)1 << 20);
}
bool choose_strip_cols(RedPlan &p, const StripBlocks &s) {
  const int es = dt_size(p.a_dtype), acc_es = dt_size(p.acc_dtype);
  const int64_t V = 16 / es, width = s.width, rows = s.nrows, kept = p.ksize[p.nkept - 1], others = p.nout / kept;
  const int64_t m = width / gcd64(width, V);
  if (rows * width >= ((int64_t)1 << 31)) return false;
  const int64_t nv = (rows * width + V - 1) / V, total = others * rows * width * es;   // vectors of a block; bytes
  // (accumulators of all lanes' vectors in 64 KiB of LDS; those of halves are held in four bytes)
  const int64_t top = std::min<int64_t>(kStripLanes, 65536 / (V * std::max(acc_es, p.acc_dtype == OCN_HALF ? 4 : 1)));
  if (p.fused && m > kBlock) return false;   // (double products of a column and [13223, 481] 36.6 and 38.5 with what follows)
  if (m > top || nv < 2 * m || (m > 32 && rows < 8) || total < (es == 1 ? kStripBytesSmall : kStripSmall)) return false;
  const bool wide = es == 1 && acc_es == 8;   // (a lane's sixteen accumulators take 32 registers)
  if (p.kernel == OCN_KERNEL_RED_COLS && p.cpw == 0 &&
      (width % V == 0 || rows <= 16 || (width > V && total < kStripLaneSmall) || (wide && width < 3 * V)))
    return false;
  if (s.inner > 1 && total < (p.vec > 1 ? strip_runs_from(s.inner * es, s.inner % V == 0, kept) : kept < 5 ? kStripInnerFew : kStripInnerSmall)) return false;
  constexpr int64_t trips = 4;
  int64_t want = std::max<int64_t>(1, (nv / trips + m / 2) / m);   // times m lanes that a block keeps busy
  int64_t block = kBlock, split = 1, chunk = rows, lanes, groups = 1;
  if (m <= kBlock && (want * m <= kBlock / 2 || kBlock / m * m * others >= (int64_t)kNumCUs * 2 * kBlock)) {
    want = std::min(want, kBlock / m);
    lanes = std::max<int64_t>(2, want * m);
    groups = kBlock / lanes;
  } else {
    block = top;
    while (block > kBlock && m <= block / 2 && want * m <= block / 2) block /= 2;
    // (one workgroup takes 16 vectors per lane without a split: no second launch)
    if (nv > block / m * m * 16 || others > 64)
      while (block > kBlock && m <= block / 2 && nv * others < kNumCUs * block * trips) block /= 2;
    lanes = block / m * m;
    const int64_t fits = std::max<int64_t>(1, (int64_t)OCN_REDUCE_SCRATCH_BYTES / (p.nout * acc_es));
    const int64_t slots = (int64_t)kNumCUs * 1024 / block;
    const int64_t most = nv <= lanes * 16 ? 1 : std::max<int64_t>(1, std::min({fits, nv / (lanes * trips), 2 * slots / others}));
    // workgroups that go round once, or twice where that is the more even by a tenth
    auto even = [&](int64_t q) { return (double)(others * q) / (double)((others * q + slots - 1) / slots * slots); };
    const int64_t once = std::max<int64_t>(1, std::min(most, slots / others));
    split = even(most) > even(once) * 1.1 ? most : once;
    if (most == fits && others * split * block < 160 * 1024 && nv > lanes * 16) return false;
    if (split > 1 && others >= 32 && total < kStripManySmall) return false;
    const bool compares = p.fused && p.mid_dtype == OCN_BOOL;
    if (split > 1 && others > 1 && p.split == 1 && rows < kStripSplitRows && es >= 4 && !compares) return false;
    if (split == 1 && others > 1 && block > kBlock) {
      if (p.fused && !compares && es >= 4 && (p.vec > 1 || es == 16) && (s.bc || rows < (es == 4 ? 64 : es == 8 ? 256 : 0))) return false;
      if (wide && rows < kLaneRows) return false;   // (sums of bool [3126, 20, 914] 33.6 and 46.8)
    }
    // a workgroup of 1024 lanes for each of more blocks than CUs, of bytes that are compared one by one and rows of which it takes two
    // at most (maxima of int8 and uint8: 57 random calls 0.78, none faster, more rows 1.25, smaller workgroups 1.08, fewer blocks
    // 1.17; uint8 [672, 47, 847] 9.6 and 15.3)
    if (split == 1 && block > 512 && es == 1 && acc_es == 1 && p.acc_dtype != OCN_BOOL && !p.fused && m >= 384 && others >= kNumCUs) return false;
    // few blocks of long rows, whose columns the other form deals out to two workgroups and more, from four of a strip's vectors
    // per lane on, 16-bit elements from ten (600 random calls: 0.9; those of 64 blocks and more or fewer vectors 1.0, complex doubles in
    // two and three workgroups 1.04; maxima of halves [28, 119, 871] 5.9 and 8.8, doubles [27, 62, 484] 3.7 and 5.0)
    if (split == 1 && p.split == 1 && others < kNumCUs / 4 && width * es >= 1024 && nv >= (es == 2 ? 10 : 4) * lanes &&
        p.grid >= (es == 16 ? 4 : 2) * others)
      return false;
    if (split > 1 && (p.flat_cols || lanes * 8 < block * 7 || total < (es == 1 ? kStripBytesSmall : kStripSplitSmall))) return false;
    if (m > kWave && lanes * 4 < block * 3) return false;
    chunk = (rows + split - 1) / split;
    // (splits that start on a line, unless that is many rows of them)
    const int64_t line = 128 / gcd64(128, width * es);
    if (chunk > 4 * line) chunk = (chunk + line - 1) / line * line;
    split = (rows + chunk - 1) / chunk;
  }
  const int64_t grid = (others * split + groups - 1) / groups;
  if (grid > max_launch_blocks()) return false;
  if (es == 2 && p.kernel == OCN_KERNEL_RED_COLS && p.vec == 1 && rows < 32 && grid < kStripFewGroups) return false;
  p.kernel = OCN_KERNEL_RED_COLS;
  p.strip = 1;
  p.strip_lanes = (int)lanes;
  p.strip_groups = (int)groups;
  // lanes that share an output: as many as make their turns and the first one's over the others about equal
  const int64_t outs = groups * (width / s.inner), addends = lanes * V / (width / s.inner);
  int64_t parts = 1;
  while ((parts + 1) * outs <= block && (parts + 1) * (parts + 1) <= addends) ++parts;
  p.strip_parts = (int)parts;
  p.split = split;
  // (partial results of an output side by side where the second launch then reads them in vectors: few outputs of
  // many splits, float sums over [18423, 79] 10.1 us, 7.8 so; 4-byte ones gain nothing)
  p.partial_rows = acc_es == 8 && p.nout <= 256;
  p.chunk = chunk;
  p.block = (int)block;
  p.grid = grid;
  p.nt_load = strip_nt(p, chunk * width * es, rows * width * es);
  return true;
}

// Rows of dense blocks in strips: 16 KB of them per workgroup, less where that leaves CUs idle.  A power of
// two of lanes per row, each with a whole vector or the row's few last elements one by one, is as
// fast only for small inputs and rows of whole vectors (float rows of 22 [1090909, 22] 37 -> 20 us, of 5 103 -> 26,
// of 16 24.1 -> 19.0, of 64 23.1 -> 18.4), and for blocks that end long before a workgroup's share.  Where the lines lie, by what
// the other form does and by element size, over 5500 random calls (ratio of the times, other form to this):
//   single elements   (rows shorter than two vectors that start anywhere) from 1 MB on, of 4 bytes 2 MB (0.96 below, 1.2 above),
//                     of 8 bytes 4 MB (0.84 below, 1.06 above), of 16 bytes 8 MB (0.93 below, 1.1 above)
//   vectors, rests    from 4 MB on, of 8 bytes 6 MB (1.05 below, 1.1 above); of a fused call with one row for all from 12 MB on
//                     (2 bytes 0.93 below, with halves [22935, 242] 5.3 and 7.0 us; 4 bytes 1.0 below; 1.15 above), of 8 bytes 8 MB
//                     (1.0 below, 1.2 above)
//   whole vectors     from 12 MB on, of 4 bytes 16 MB (1.0 below, 1.25 above), of 2 bytes 32 MB (0.98 below, 1.1 above); not rows
//                     of one vector, or two of 8 or 16 bits (halves [5000000, 8] 23.6 and 26.5, maxima of floats
//                     [2070888, 4] 10.6 and 12.6); bytes from 48 MB on (int8 sums in rows of 64: 16 MB 6.2 and
//                     6.7 us, 30 MB 10.4 either way, 50 MB 15.3 -> 12.9; rows of 33 gain at all sizes, 6 MB 6.3 -> 4.5)
//   blocks of few     a workgroup takes rows of one block: from 5 KB of them on, single elements 512 bytes times their size
//   rows              (cfloat [48969, 18, 2] minus a row 6.7 and 56 us, doubles [100131, 5, 3] 7.0 and 108)
// Bytes come from LDS in words, those of a fused
// call one by one: from 32 of them on the other form is the better one there (any over rows of 50 32.5 and 35.6).
constexpr int64_t kStripRowBytes = 16 << 10, kStripByteRowsWhole = 48 << 20, kStripRowsBlock = 5 << 10, kStripRowsBlockSingle = 512;
int64_t strip_rows_from(int es, bool vectors, bool whole, bool words, bool one_row) {
  const int64_t mb = 1 << 20;
  if (!vectors) return es <= 2 ? mb : es / 2 * mb;
  if (whole) return words ? kStripByteRowsWhole : es == 2 ? 32 * mb : es == 4 ? 16 * mb : 12 * mb;
  if (one_row) return es <= 4 ? 12 * mb : 8 * mb;
  return es >= 8 ? 6 * mb : 4 * mb;
}
bool choose_strip_rows(RedPlan &p, const StripBlocks &s) {
  const int es = dt_size(p.a_dtype), mes = p.fused ? dt_size(p.mid_dtype) : es;
  const int64_t V = 16 / es, width = s.width, rows = s.nrows, others = p.nout / rows, total = p.nout * width * es;
  const int64_t m = width / gcd64(width, V), vecs = width / V;
  const bool words = es == 1 && !p.fused;   // read from LDS in words
  if (width * es > kStripRowBytes / 16 || (es == 1 && p.fused && width >= 32) || (s.bc && m > kBlock)) return false;
  const bool whole = p.vec > 1 && width % V == 0;   // in whole vectors by the other form too
  if (total < strip_rows_from(es, p.vec > 1, whole, words, s.bc != 0)) return false;
  if (whole && (vecs == 1 || (vecs == 2 && es <= 2))) return false;
  const int64_t piece = std::max<int64_t>(2048, std::min(kStripRowBytes, total / (4 * kNumCUs)));
  int64_t chunk = 4;
  while (chunk * 2 * width * es <= piece) chunk *= 2;
  if (rows < chunk && rows * width * es < (p.vec > 1 ? kStripRowsBlock : kStripRowsBlockSingle * es)) return false;
  chunk = std::min(chunk, rows);
  const int64_t grid = others * ((rows + chunk - 1) / chunk);
  if (grid > max_launch_blocks()) return false;
  int parts = 1;
  while (parts < kWave && chunk * parts * 2 <= kBlock) parts *= 2;
  p.kernel = OCN_KERNEL_RED_ROWS;
  p.strip = 2;
  p.strip_lanes = (int)(s.bc ? kBlock / m * m : kBlock);
  p.strip_parts = parts;
  // lanes read their rows from different elements on where rows lie a multiple of eight banks apart
  if (width * mes % 4 == 0 && gcd64(width * mes / 4, 64) >= 8) {
    p.strip_rotate = 1;
    while (p.strip_rotate * 2 <= (words ? width / 4 : width) / parts && p.strip_rotate < kWave) p.strip_rotate *= 2;
  }
  p.strip_lds = (size_t)((chunk * width * mes + 15) / 16 * 16);
  p.split = 1;
  p.chunk = chunk;
  p.block = kBlock;
  p.grid = grid;
  p.nt_load = strip_nt(p, chunk * width * es, rows * width * es);
  return true;
}

// Runs of columns in an output, rows too long for a strip.  A workgroup gets the outputs whose columns fill 32 to 256
// lanes best, with what a run's ends share of a line counted against short ones; rows are split while workgroups are
// fewer than two per CU and eight trips are left to each.
// The forms above, where lanes share an output and read its run of every row in lines of its own, stay the better
// ones for long runs (half sums over the outer axes of [980, 193, 96] 14.7 and 16.3 us, bytes in runs of 500 to 5000
// 1.2 to 2.4 times as long so) and for few rows unless there is much of them (maxima of floats [148, 453, 28] 6.2 and
// 9.4; [227, 5192, 13] 21.3 -> 18.7), and where lanes read the runs in vectors, as far as strip_runs_from says (sums of int8
// [555, 597, 16] 3.9 and 10.8).  Floats [1049, 7872, 8] 168 -> 44, halves [957, 7281, 7] 113 -> 27,
// bool any over [1356, 3062, 5] 31 -> 13.  With strips, which take the shorter rows, 170 random calls with runs of 2 to 256
// bytes are 1.72 times as fast in the mean as without either, 8.4 ms together -> 3.1.  256 splits at most, whose fold is
// one workgroup's for few outputs.
constexpr int64_t kRunsSmall = 2 << 20, kRunsBytesSmall = 4 << 20, kRunsRows = 300, kRunsFewRows = 128, kRunsMuch = 32 << 20, kRunsLong = 64,
                  kRunsBytes = 256, kRunsSplits = 256;
bool choose_strip_runs(RedPlan &p) {
  if (p.fused || p.nkept != 1 || p.nred != 2) return false;
  const int es = dt_size(p.a_dtype), acc_es = dt_size(p.acc_dtype);
  const int64_t V = 16 / es, inner = p.rsize[1], rows = p.rsize[0], width = p.nout * inner;
  if (inner < 2 || p.rstride_a[1] != es || p.kstride_a[0] != inner * es) return false;
  if (width < 32 * V || width >= ((int64_t)1 << 31) || rows < kRunsFewRows) return false;
  const int64_t total = rows * width * es;
  if (total < (p.vec > 1 ? strip_runs_from(inner * es, inner % V == 0, p.nout) : es == 1 ? kRunsBytesSmall : kRunsSmall) || (rows < kRunsRows && total < kRunsMuch)) return false;
  if (inner * es > kRunsBytes || inner > (es == 1 ? kRunsLong / 2 : kRunsLong)) return false;
  // (512 lanes for bytes, whose sixteen columns a lane leave few workgroups)
  const int64_t top = std::min<int64_t>(es == 1 ? kStripLanes / 2 : kStripLanes, 65536 / (V * std::max(acc_es, p.acc_dtype == OCN_HALF ? 4 : 1)));
  const int64_t least = std::max<int64_t>(1, 32 * V / inner), most = std::max<int64_t>(1, 256 * V / inner), by = std::max<int64_t>(1, (most - least) / 64);
  const int64_t slots = (int64_t)kNumCUs * 2 * kStripLanes / top, fits = (int64_t)OCN_REDUCE_SCRATCH_BYTES / (p.nout * acc_es);
  int64_t outs = 0, lanes = 0, blocks = 0, split = 1;
  double best = 0;
  for (int64_t q = least; q <= most; q += by) {
    const int64_t n = std::min(q, p.nout), l = (n * inner + V - 1) / V, nb = (p.nout + n - 1) / n;
    if (l > top) break;
    const double bytes = (double)(n * inner * es);
    const int64_t splits = std::max<int64_t>(1, std::min({slots / nb, rows / (top / std::max<int64_t>(2, l) * 8), fits, kRunsSplits}));
    const double share = (double)(top / l * n * inner) / (double)(top * V) * (double)p.nout / (double)(nb * n) * bytes / (bytes + 96) *
                         std::min(1.0, (double)(nb * splits) / (double)kNumCUs);
    if (share > best) {
      best = share;
      outs = n;
      lanes = std::max<int64_t>(2, l);
      blocks = nb;
      split = splits;
    }
  }
  if (!outs || blocks * split > max_launch_blocks() || blocks * split < kNumCUs / 4) return false;
  const int64_t groups = top / lanes;
  int64_t parts = 1;
  while (parts < kWave && parts * 2 <= inner && parts * 2 * outs <= top) parts *= 2;
  p.kernel = OCN_KERNEL_RED_COLS;
  p.strip = 3;
  p.strip_lanes = (int)lanes;
  p.strip_groups = (int)groups;
  p.strip_parts = (int)parts;
  p.strip_inner = inner;
  p.strip_width = outs * inner;
  p.strip_rows = rows;
  p.chunk = (rows + split - 1) / split;
  p.split = (rows + p.chunk - 1) / p.chunk;
  p.block = (int)top;
  p.grid = blocks * p.split;
  p.vec = (int)V;
  p.cpw = kWave;
  p.nt_load = (intptr_t)p.a_ptr % 16 == 0 && p.rstride_a[0] % 16 == 0 && outs * inner * es % 16 == 0 && width * es % 16 == 0 &&
              rows * width * es >= kStreamBytes;
  p.short_rows = p.lean = p.flat_cols = false;
  return true;
}

void choose_strip(RedPlan &p) {
  const StripBlocks s = strip_blocks(p);
  if (!(s.cols && choose_strip_cols(p, s)) && !(s.rows && choose_strip_rows(p, s))) {
    choose_strip_runs(p);
    return;
  }
  p.strip_bc = s.bc;
  p.strip_inner = s.inner;
  p.strip_width = s.width;
  p.strip_rows = s.nrows;
  p.vec = 16 / dt_size(p.a_dtype);
  p.cpw = kWave;
  p.short_rows = p.lean = p.flat_cols = false;
}
void choose_reduce_launch(RedPlan &p) {
  const int es = dt_size(p.a_dtype);
  const int acc_es = dt_size(p.acc_dtype);
  // fastest dims
  const int64_t r_fast = p.nred ? iabs64(p.rstride_a[p.nred - 1]) : 0;
  int64_t k_fast = 0;  // smallest non-zero kept stride of the input
  int k_fast_dim = -1;
  for (int d = 0; d < p.nkept; ++d) {
    int64_t s = iabs64(p.kstride_a[d]);
    if (s && (k_fast_dim < 0 || s <= k_fast)) { k_fast = s; k_fast_dim = d; }
  }
  const int vfull = std::max(1, 16 / es);
  auto all_aligned = [&](int64_t vb, int skip_kept, int skip_red) {
    if ((intptr_t)p.a_ptr % vb) return false;
    for (int d = 0; d < p.nkept; ++d)
      if (d != skip_kept && p.kstride_a[d] % vb) return false;
    for (int d = 0; d < p.nred; ++d)
      if (d != skip_red && p.rstride_a[d] % vb) return false;
    return true;
  };
  bool idx32 = p.nout < ((int64_t)1 << 31) && p.nredtot < ((int64_t)1 << 31);
  for (int d = 0; d < p.nkept; ++d) idx32 = idx32 && p.ksize[d] < ((int64_t)1 << 31);
  for (int d = 0; d < p.nred; ++d) idx32 = idx32 && p.rsize[d] < ((int64_t)1 << 31);
  // a flat contiguous full reduction may be longer than 2^31 elements
  const bool flat_full = p.nkept == 0 && p.nred == 1;
  bool aligned = true;   // every vector starts on a vector boundary

  const bool rows_contig = p.nred >= 1 && r_fast == es && (k_fast_dim < 0 || k_fast > r_fast);
  const bool cols_ok = k_fast_dim >= 0 && k_fast == es && p.kstride_a[k_fast_dim] == es &&
                       (p.nred == 0 || r_fast == 0 || r_fast > k_fast) && p.nredtot >= 1 && idx32 &&
                       k_fast_dim == p.nkept - 1 && p.nred >= 1;
  if (p.nred >= 1 && (idx32 || flat_full) && (rows_contig || !cols_ok)) {
    // ---- rows: lanes share an output ---------------------------------------------------
    // With the reduced axis the input's fastest, lanes load whole vectors; any other layout
    // goes element by element with the innermost reduced stride.
    p.kernel = OCN_KERNEL_RED_ROWS;
    // Rows that do not start on vector boundaries are read in whole vectors all the same (at
    // unaligned addresses) as soon as they hold two.
    const int64_t n0 = p.rsize[p.nred - 1];
    aligned = all_aligned((int64_t)vfull * es, -1, p.nred - 1);
    p.vec = rows_contig && (aligned || n0 >= 2 * vfull) ? vfull : 1;
    const int64_t vpr = (n0 + p.vec - 1) / p.vec;         // vectors per innermost run
    const int64_t nvec = vpr * (p.nredtot / n0);          // vectors per output
    int64_t cover = 1;                                    // lanes one output can keep busy
    while (cover < nvec && cover < kBlock) cover <<= 1;
    if (rows_contig || k_fast_dim < 0 || r_fast < k_fast) {
      // neighbouring lanes read neighbouring addends
      // a whole workgroup only when each of its lanes gets at least four vectors (the depth of
      // the unrolled loop): rows of 10 to 14 KiB measured 10-20 % slower on 256 lanes than on 64
      p.group = nvec < 4 * kBlock ? (int)std::min<int64_t>(cover, kWave) : kBlock;
    } else {
      // a kept axis is faster: neighbouring lanes take neighbouring outputs, and share one
      // only as far as it takes to fill the device
      int64_t need = 1;
      while (need * p.nout < kTargetWaves * kWave && need < cover) need <<= 1;
      p.group = need > kWave ? kBlock : (int)need;
    }
    const int64_t groups_per_block = kBlock / p.group;
    const int64_t waves = (p.nout * p.group + kWave - 1) / kWave;
    p.split = 1;
    // the common 2-D shape: one reduced dim read in vectors, at most one kept dim, a wavefront or
    // a workgroup per output (or per split of it), everything below 2^31
    const bool lean_shape = p.nred == 1 && p.nkept <= 1 && p.vec > 1 && es < 16 &&
                            p.group >= kWave && nvec < ((int64_t)1 << 31);
    if (p.group >= kWave && waves < kTargetWaves) {
      // split long reductions so the device fills; keep >= 16 vectors per lane per split, but 4, one
      // trip of the loop, where several dims are walked and a vector takes as long to find as sixteen
      // elements did (uint8 [2830, 102] rows 103 apart: 21.9 us with four splits of 16)
      const int64_t want = ((lean_shape ? kLeanSplitWaves : kTargetWaves) + waves - 1) / waves;
      const int64_t per_lane = p.vec > 1 && p.nred > 1 && nvec >= (int64_t)p.group * 16 ? 4 : 16;
      const int64_t most = std::max<int64_t>(1, nvec / ((int64_t)p.group * per_lane));
      p.split = std::max<int64_t>(1, std::min(want, most));
      const bool slow = (p.op == R_PROD && p.a_dtype == OCN_INT8) || !all_aligned(4, -1, p.nred - 1);
      if (p.split > 1 && lean_shape && one_workgroup_each(nvec * 16, p.nout, slow)) {
        p.split = 1;
        p.group = p.block = kLeanMaxLanes;
      }
    }
    p.chunk = (nvec + p.split - 1) / p.split;
    p.split = (nvec + p.chunk - 1) / p.chunk;
    p.grid = p.group > kBlock ? p.nout : (p.nout * p.split + groups_per_block - 1) / groups_per_block;
    p.short_rows = p.group <= kWave && nvec <= p.group && p.nred == 1 && p.split == 1 &&
                   p.nout * p.group < ((int64_t)1 << 32) && n0 < ((int64_t)1 << 31);
    p.lean = !p.short_rows && lean_shape && p.nout * p.split < ((int64_t)1 << 31) && p.chunk < ((int64_t)1 << 31);
  } else if (cols_ok) {
    // ---- cols: a kept axis is the input's fastest; lanes own output columns -------------
    // (requires that axis to be the last canonical kept dim, i.e. also the output's fastest)
    p.kernel = OCN_KERNEL_RED_COLS;
    const int64_t nc = p.ksize[p.nkept - 1];
    aligned = all_aligned((int64_t)vfull * es, p.nkept - 1, -1);
    p.vec = aligned || unaligned_columns(nc, vfull, p.nredtot) ? vfull : 1;
    const int64_t col_lanes = (nc + p.vec - 1) / p.vec, others = p.nout / nc;
    const ColsShape shape = choose_cols_shape(col_lanes, others, p.nredtot, p.nout, acc_es, !aligned);
    p.cpw = shape.cpw;
    p.split = shape.split;
    int nw = shape.nw;
    // bytes whose lanes and wavefronts meet in packed words, and whose blocks of 64 lanes are 1024 columns: narrower
    // ones, down to a line, while most CUs have none (bool any over the rows of [222, 2382] 8.2 -> 6.0 us, sums 7.5 -> 6.5;
    // with sixteen accumulators, which meet one by one, int8 maxima of [33, 5000] took 7.7 instead of 6.0)
    const bool packed = es == 1 && (p.acc_dtype == OCN_BOOL || (p.op == R_SUM && (p.a_dtype == OCN_INT8 || p.a_dtype == OCN_UINT8) && p.nredtot <= 256 * nw));
    if (packed && p.vec > 1 && p.split == 1)
      while (p.cpw > 8 && (col_lanes + p.cpw - 1) / p.cpw * others * 4 <= kNumCUs && p.nredtot >= nw * (kWave / p.cpw) * 4) p.cpw /= 2;
    const int flat = p.nred == 1 && p.vec > 1 && p.vec <= 8 ? choose_flat_columns(col_lanes, others, p.nredtot, p.cpw, p.split, aligned) : 0;
    if (flat) {
      p.flat_cols = true;
      p.split = 1;
      p.cpw = flat;
      nw = kFlatLanes / kWave;
    }
    const int64_t blocks0 = (col_lanes + p.cpw - 1) / p.cpw * others;
    p.block = nw * kWave;
    p.chunk = (p.nredtot + p.split - 1) / p.split;
    p.split = (p.nredtot + p.chunk - 1) / p.chunk;
    p.grid = blocks0 * p.split;
    const int64_t lane_vec = nc < p.vec ? 1 : p.vec, lanes = (nc + lane_vec - 1) / lane_vec * others;
    const int64_t enough = lane_vec == 8 && col_lanes >= kLaneWide ? 2 * kLaneColumns : kLaneColumns;
    if (p.nred == 1 && p.vec <= 8 && (p.nredtot <= 8 || (p.nredtot <= kLaneRows && col_lanes < kLaneWide)) && lanes >= enough &&
        lanes < ((int64_t)1 << 31) - kBlock) {
      p.flat_cols = false;
      p.cpw = 0;
      p.vec = (int)lane_vec;
      p.split = 1;
      p.chunk = p.nredtot;
      p.block = kBlock;
      p.grid = (lanes + kBlock - 1) / kBlock;
    }
  } else {
    p.kernel = OCN_KERNEL_RED_GENERIC;
    p.vec = 1;
    p.split = 1;
    p.chunk = p.nredtot;
    p.grid = std::min<int64_t>((p.nout + kBlock - 1) / kBlock, max_launch_blocks());   // the kernel loops beyond that
  }
  if (idx32) choose_strip(p);
  if (p.grid > max_launch_blocks()) {
    // more workgroups than one launch may have: the generic kernel, which loops over its outputs
    p.kernel = OCN_KERNEL_RED_GENERIC;
    p.vec = 1;
    p.split = 1;
    p.short_rows = p.lean = false;
    p.block = kBlock;
    p.chunk = p.nredtot;
    p.grid = std::min<int64_t>((p.nout + kBlock - 1) / kBlock, max_launch_blocks());
  }
  p.passes = p.split > 1 ? 2 : 1;
  p.workspace_bytes = p.split > 1 ? (size_t)(p.nout * p.split * acc_es) : 0;
  // an input that cannot stay in the caches anyway is read with streaming loads (whole
  // 16-byte vectors only: neighbouring lanes then cover whole lines)
  if (!p.strip) p.nt_load = p.vec > 1 && aligned && p.cpw != 0 && p.kernel != OCN_KERNEL_RED_GENERIC && p.nout * p.nredtot * es >= kStreamBytes;
}

}  // namespace

int plan_reduce(int op, const ocn_tensor *a, const int32_t *axes, int32_t naxes,
                const ocn_tensor *out, RedPlan *plan) {
  RedPlan p;
  p.op = op;
  int rc;
  if ((rc = check_tensor(a)) != OCN_OK) return rc;
  if ((rc = check_tensor(out)) != OCN_OK) return rc;
  if (op < 0 || op >= R_COUNT) return OCN_ERR_OP;
  if (a->device != out->device) return OCN_ERR_DEVICE;
  if (naxes < 0 || naxes > a->ndim) return OCN_ERR_SHAPE;
  if (naxes > 0 && !axes) return OCN_ERR_NULLPTR;
  bool reduced[kMaxDims] = {false};
  for (int i = 0; i < naxes; ++i) {
    if (axes[i] < 0 || axes[i] >= a->ndim || reduced[axes[i]]) return OCN_ERR_SHAPE;
    reduced[axes[i]] = true;
  }
  if (out->ndim != a->ndim - naxes) return OCN_ERR_SHAPE;
  RDim kd[kMaxDims], rd[kMaxDims];
  int nk = 0, nr = 0, j = 0;
  int64_t nout = 1, nred = 1;
  for (int d = 0; d < a->ndim; ++d) {
    if (reduced[d]) {
      nred *= a->size[d];
      rd[nr++] = RDim{a->size[d], a->stride[d], 0};
    } else {
      if (out->size[j] != a->size[d]) return OCN_ERR_SHAPE;
      nout *= a->size[d];
      kd[nk++] = RDim{a->size[d], a->stride[d], out->stride[j]};
      ++j;
    }
  }
  if (!reduce_supported(op, a->dtype)) return OCN_ERR_DTYPE;
  p.nout = nout;
  p.nredtot = nred;
  p.a_dtype = a->dtype;
  p.out_dtype = out->dtype;
  p.acc_dtype = reduce_acc_dtype(op, a->dtype);
  p.swap_a = a->byteswapped && scalar_size(a->dtype) > 1;     // stored in the other byte order (section 3.1.3)
  p.swap_o = out->byteswapped && scalar_size(out->dtype) > 1;
  if (nout == 0) { *plan = p; return OCN_OK; }
  if ((op == R_MIN || op == R_MAX) && nred == 0) return OCN_ERR_EMPTY;
  if (nred > 0 && (rc = check_alignment(a)) != OCN_OK) return rc;
  if ((rc = check_alignment(out)) != OCN_OK) return rc;
  if (!provably_non_overlapping(out)) return OCN_ERR_OVERLAP_OUT;
  if (nred > 0) {
    intptr_t ilo, ihi, olo, ohi;
    byte_range(a, &ilo, &ihi);
    byte_range(out, &olo, &ohi);
    if (ilo < ohi && olo < ihi) return OCN_ERR_ALIAS;
  }

  int64_t off_a = a->offset, off_o = out->offset;
  // kept dims: drop size 1, flip to forward output strides, sort by output stride, merge
  int n = 0;
  for (int d = 0; d < nk; ++d) {
    if (kd[d].size == 1) continue;
    RDim x = kd[d];
    if (x.so < 0) {
      off_o += (x.size - 1) * x.so;
      off_a += (x.size - 1) * x.sa;
      x.so = -x.so; x.sa = -x.sa;
    }
    kd[n++] = x;
  }
  nk = sort_merge(kd, n, true);
  // The column kernel walks the fastest kept dim forward through the input.  If making the
  // output stride positive left the input stride there at minus one element, turn that dim
  // around again: the kernels accept a negative output stride.
  if (nk > 0 && kd[nk - 1].sa == -(int64_t)dt_size(a->dtype)) {
    RDim &x = kd[nk - 1];
    off_o += (x.size - 1) * x.so;
    off_a += (x.size - 1) * x.sa;
    x.so = -x.so;
    x.sa = -x.sa;
  }
  // reduced dims: drop size 1, flip to forward input strides (the set of addends is the
  // same), sort by input stride, merge
  n = 0;
  for (int d = 0; d < nr; ++d) {
    if (rd[d].size == 1) continue;
    RDim x = rd[d];
    if (x.sa < 0) {
      off_a += (x.size - 1) * x.sa;
      x.sa = -x.sa;
    }
    rd[n++] = x;
  }
  nr = nred == 0 ? 0 : sort_merge(rd, n, false);
  p.nkept = nk;
  p.nred = nr;
  for (int d = 0; d < nk; ++d) { p.ksize[d] = kd[d].size; p.kstride_a[d] = kd[d].sa; p.kstride_o[d] = kd[d].so; }
  for (int d = 0; d < nr; ++d) { p.rsize[d] = rd[d].size; p.rstride_a[d] = rd[d].sa; }
  p.off_a = off_a;
  p.off_out = off_o;
  p.a_ptr = (char *)a->base + off_a;
  p.out_ptr = (char *)out->base + off_o;
  choose_reduce_launch(p);
  *plan = p;
  return OCN_OK;
}

namespace {

// Launch shape of a fused elementwise+reduce kernel.  Same three layouts as the plain
// reduction; an input may be broadcast (stride 0) along the vectorised dim as long as the
// other one is contiguous there.
void choose_fused_launch(RedPlan &p) {
  const int es_a = dt_size(p.a_dtype), es_b = dt_size(p.b_dtype), es_m = dt_size(p.mid_dtype);
  const int acc_es = dt_size(p.acc_dtype);
  auto fast_ok = [&](int64_t sa, int64_t sb) {
    return (sa == es_a || sa == 0) && (sb == es_b || sb == 0) && !(sa == 0 && sb == 0);
  };
  // stride in elements along a dim, of the input that moves slower there (0: both broadcast):
  // a dim counts as fast only if no input jumps along it
  auto elems = [&](int64_t sa, int64_t sb) {
    return std::max(iabs64(sa) / es_a, iabs64(sb) / es_b);
  };
  int64_t r_fast = 0, k_fast = 0;
  int k_fast_dim = -1;
  if (p.nred) r_fast = elems(p.rstride_a[p.nred - 1], p.rstride_b[p.nred - 1]);
  for (int d = 0; d < p.nkept; ++d) {
    const int64_t e = elems(p.kstride_a[d], p.kstride_b[d]);
    if (e && (k_fast_dim < 0 || e <= k_fast)) { k_fast = e; k_fast_dim = d; }
  }
  const int vfull = rows_vec(es_m, std::max({es_a, es_b, es_m}));  // as Sig::V with the intermediate type as output
  // every stride except the one along the vectorised dim, and the base, are multiples of the
  // vector size of each input that is not broadcast there
  auto all_aligned = [&](int skip_kept, int skip_red, bool a_bcast, bool b_bcast) {
    const int64_t va = a_bcast ? es_a : (int64_t)vfull * es_a, vb = b_bcast ? es_b : (int64_t)vfull * es_b;
    if ((intptr_t)p.a_ptr % va || (intptr_t)p.b_ptr % vb) return false;
    for (int d = 0; d < p.nkept; ++d)
      if (d != skip_kept && (p.kstride_a[d] % va || p.kstride_b[d] % vb)) return false;
    for (int d = 0; d < p.nred; ++d)
      if (d != skip_red && (p.rstride_a[d] % va || p.rstride_b[d] % vb)) return false;
    return true;
  };
  bool idx32 = p.nout < ((int64_t)1 << 31) && p.nredtot < ((int64_t)1 << 31);
  for (int d = 0; d < p.nkept; ++d) idx32 = idx32 && p.ksize[d] < ((int64_t)1 << 31);
  for (int d = 0; d < p.nred; ++d) idx32 = idx32 && p.rsize[d] < ((int64_t)1 << 31);
  const bool flat_full = p.nkept == 0 && p.nred == 1;

  p.split = 1;
  if (p.nred >= 1 && fast_ok(p.rstride_a[p.nred - 1], p.rstride_b[p.nred - 1]) &&
      (k_fast_dim < 0 || k_fast > r_fast) && (idx32 || flat_full)) {
    p.kernel = OCN_KERNEL_RED_ROWS;
    p.a_fast_bcast = p.rstride_a[p.nred - 1] == 0;
    p.b_fast_bcast = p.rstride_b[p.nred - 1] == 0;
    const int64_t n0 = p.rsize[p.nred - 1];
    // (unaligned rows in whole vectors too once they hold two, as in the plain reduction)
    p.vec = n0 >= 2 * vfull || all_aligned(-1, p.nred - 1, p.a_fast_bcast, p.b_fast_bcast) ? vfull : 1;
    const int64_t vpr = (n0 + p.vec - 1) / p.vec;
    const int64_t nvec = vpr * (p.nredtot / n0);
    int64_t cover = 1;                                    // lanes one output can keep busy
    while (cover < nvec && cover < kWave) cover <<= 1;
    p.group = (nvec * p.vec * (es_a + es_b) <= 16 * 1024) ? (int)cover : kBlock;
    const int64_t groups_per_block = kBlock / p.group;
    const int64_t waves = (p.nout * p.group + kWave - 1) / kWave;
    if (p.group >= kWave && waves < kTargetWaves) {
      const int64_t want = (kTargetWaves + waves - 1) / waves;
      const int64_t most = std::max<int64_t>(1, nvec / ((int64_t)p.group * 8));
      p.split = std::max<int64_t>(1, std::min(want, most));
    }
    p.chunk = (nvec + p.split - 1) / p.split;
    p.split = (nvec + p.chunk - 1) / p.chunk;
    p.grid = (p.nout * p.split + groups_per_block - 1) / groups_per_block;
    p.short_rows = p.group <= kWave && nvec <= p.group && p.nred == 1 && p.split == 1 &&
                   p.nout * p.group < ((int64_t)1 << 32) && n0 < ((int64_t)1 << 31);
    // The common 2-D shape takes the lean form of the kernel: one reduced dim along which both
    // inputs are contiguous, at most one kept dim, at least a wavefront's vectors per output, everything below 2^31.  Its vectors are 16 bytes of
    // each input whatever the intermediate type is.
    const int lv = es_a == es_b && es_a <= 16 ? 16 / es_a : 0;   // elements per vector
    if (!p.short_rows && lv >= 1 && p.nred == 1 && p.nkept <= 1 && !p.a_fast_bcast && !p.b_fast_bcast &&
        n0 / lv >= kWave && n0 / lv < ((int64_t)1 << 31) && p.nout < ((int64_t)1 << 31)) {
      const int64_t nv = n0 / lv;
      int group = nv * 32 <= 16 * 1024 ? kWave : kBlock;          // as above: rows of up to 16 KiB take a wavefront
      const int64_t lwaves = (p.nout * group + kWave - 1) / kWave;
      int64_t split = 1;
      if (lwaves < kTargetWaves) {
        const int64_t want = (kLeanSplitWaves + lwaves - 1) / lwaves;
        const int64_t most = std::max<int64_t>(1, nv / ((int64_t)group * 8));
        split = std::max<int64_t>(1, std::min(want, most));
      }
      const bool dwords = (intptr_t)p.a_ptr % 4 == 0 && (intptr_t)p.b_ptr % 4 == 0 &&
                          (p.nkept == 0 || (p.kstride_a[0] % 4 == 0 && p.kstride_b[0] % 4 == 0));
      if (split > 1 && one_workgroup_each(nv * 32, p.nout, !dwords)) {
        split = 1;
        group = kLeanMaxLanes;
      }
      const int64_t chunk = (nv + split - 1) / split;
      split = (nv + chunk - 1) / chunk;
      if (p.nout * split < ((int64_t)1 << 31)) {
        p.lean = true;
        p.vec = lv;
        p.group = group;
        p.block = std::max(group, kBlock);
        p.split = split;
        p.chunk = chunk;
        p.grid = group > kBlock ? p.nout : (p.nout * split + kBlock / group - 1) / (kBlock / group);
        // inputs far larger than the caches are streamed; one that is broadcast along the kept
        // dim is re-read by every output and stays cacheable, and then so does the other (one flag)
        const bool a_rows = p.nkept == 0 || p.kstride_a[0] != 0, b_rows = p.nkept == 0 || p.kstride_b[0] != 0;
        const bool aligned = (intptr_t)p.a_ptr % 16 == 0 && (intptr_t)p.b_ptr % 16 == 0 &&
                             (p.nkept == 0 || (p.kstride_a[0] % 16 == 0 && p.kstride_b[0] % 16 == 0));
        p.nt_load = a_rows && b_rows && aligned && p.nout * n0 * es_a >= kStreamBytes;
      }
    }
  } else if (k_fast_dim >= 0 && k_fast_dim == p.nkept - 1 && p.nred >= 1 && idx32 &&
             fast_ok(p.kstride_a[k_fast_dim], p.kstride_b[k_fast_dim]) && (r_fast == 0 || r_fast > k_fast)) {
    p.kernel = OCN_KERNEL_RED_COLS;
    p.a_fast_bcast = p.kstride_a[k_fast_dim] == 0;
    p.b_fast_bcast = p.kstride_b[k_fast_dim] == 0;
    const int64_t nc = p.ksize[p.nkept - 1];
    const bool aligned = all_aligned(p.nkept - 1, -1, p.a_fast_bcast, p.b_fast_bcast);
    p.vec = aligned || unaligned_columns(nc, vfull, p.nredtot) ? vfull : 1;
    const int64_t col_lanes = (nc + p.vec - 1) / p.vec, others = p.nout / nc;
    const ColsShape shape = choose_cols_shape(col_lanes, others, p.nredtot, p.nout, acc_es, false);
    p.cpw = shape.cpw;
    p.split = shape.split;
    const int nw = shape.nw;
    const int64_t blocks0 = (col_lanes + p.cpw - 1) / p.cpw * others;
    p.block = nw * kWave;
    // inputs far larger than the caches, each read as one 16-byte piece per lane and broadcast
    // along no dim: streaming loads
    {
      // (not where one is a column vector: the other is then a matrix that the next product reads again, and up
      // to 256 MB it finds there what this one left; streamed, the products of [16384, 1000] with a
      // column and then with a row take 14.4 + 13.7 us, 14.9 + 11.6 so)
      bool plain = aligned && p.vec > 1 && (int64_t)p.vec * es_a == 16 && (int64_t)p.vec * es_b == 16;
      for (int d = 0; d < p.nkept; ++d) plain = plain && p.kstride_a[d] != 0 && p.kstride_b[d] != 0;
      for (int d = 0; d < p.nred; ++d) plain = plain && p.rstride_a[d] != 0 && p.rstride_b[d] != 0;
      p.nt_load = plain && p.nout * p.nredtot * es_a >= kStreamBytes;
    }
    p.chunk = (p.nredtot + p.split - 1) / p.split;
    p.split = (p.nredtot + p.chunk - 1) / p.chunk;
    p.grid = blocks0 * p.split;
  } else {
    p.kernel = OCN_KERNEL_RED_GENERIC;
    p.vec = 1;
    p.chunk = p.nredtot;
    p.grid = std::min<int64_t>((p.nout + kBlock - 1) / kBlock, max_launch_blocks());
  }
  if (idx32) choose_strip(p);
  p.passes = p.split > 1 ? 2 : 1;
  p.workspace_bytes = p.split > 1 ? (size_t)(p.nout * p.split * acc_es) : 0;
}

}  // namespace

int plan_binary_reduce(int ew_op, int red_op, const ocn_tensor *a, const ocn_tensor *b,
                       const int32_t *axes, int32_t naxes, const ocn_tensor *out, int mid_dtype,
                       char *workspace, FusedPlan *plan) {
  FusedPlan fp;
  RedPlan &p = fp.red;
  int rc;
  if ((rc = check_tensor(a)) != OCN_OK) return rc;
  if ((rc = check_tensor(b)) != OCN_OK) return rc;
  if ((rc = check_tensor(out)) != OCN_OK) return rc;
  if (ew_op < 0 || ew_op >= B_COUNT || red_op < 0 || red_op >= R_COUNT) return OCN_ERR_OP;
  if (!valid_dtype(mid_dtype)) return OCN_ERR_DTYPE;
  if (a->device != out->device || b->device != out->device) return OCN_ERR_DEVICE;
  // the fused kernels take operands in native byte order only (one-byte scalars have no order):
  // with an operand in the other order the call runs as the two calls it abbreviates, whose
  // kernels reverse on load and on store
  bool other_order = false;
  for (const ocn_tensor *t : {a, b, out})
    if (t->byteswapped && scalar_size(t->dtype) > 1) other_order = true;
  // broadcast shape of the two inputs (missing leading dims count as size 1)
  const int nd = std::max(a->ndim, b->ndim);
  int64_t shape[kMaxDims], sa[kMaxDims], sb[kMaxDims];
  for (int d = 0; d < nd; ++d) {
    const int da = d - (nd - a->ndim), db = d - (nd - b->ndim);
    const int64_t na = da >= 0 ? a->size[da] : 1, nb = db >= 0 ? b->size[db] : 1;
    if (na != nb && na != 1 && nb != 1) return OCN_ERR_SHAPE;
    shape[d] = na == 1 ? nb : na;
    sa[d] = (da >= 0 && na != 1) ? a->stride[da] : 0;
    sb[d] = (db >= 0 && nb != 1) ? b->stride[db] : 0;
  }
  if (naxes < 0 || naxes > nd) return OCN_ERR_SHAPE;
  if (naxes > 0 && !axes) return OCN_ERR_NULLPTR;
  bool reduced[kMaxDims] = {false};
  for (int i = 0; i < naxes; ++i) {
    if (axes[i] < 0 || axes[i] >= nd || reduced[axes[i]]) return OCN_ERR_SHAPE;
    reduced[axes[i]] = true;
  }
  if (out->ndim != nd - naxes) return OCN_ERR_SHAPE;
  const int promoted = promote(a->dtype, b->dtype);
  const int T = binary_compute_dtype(ew_op, a->dtype, b->dtype, mid_dtype, promoted, promote(promoted, mid_dtype));
  if (!binary_supported(ew_op, T) || !reduce_supported(red_op, mid_dtype)) return OCN_ERR_DTYPE;

  RDim kd[kMaxDims], rd[kMaxDims];
  int nk = 0, nr = 0, j = 0;
  int64_t nout = 1, nred = 1;
  for (int d = 0; d < nd; ++d) {
    if (reduced[d]) {
      nred *= shape[d];
      rd[nr++] = RDim{shape[d], sa[d], 0, sb[d]};
    } else {
      if (out->size[j] != shape[d]) return OCN_ERR_SHAPE;
      nout *= shape[d];
      kd[nk++] = RDim{shape[d], sa[d], out->stride[j], sb[d]};
      ++j;
    }
  }
  p.op = red_op;
  p.fused = true;
  p.ew_op = ew_op;
  p.nout = nout;
  p.nredtot = nred;
  p.a_dtype = a->dtype;
  p.b_dtype = b->dtype;
  p.mid_dtype = mid_dtype;
  p.out_dtype = out->dtype;
  p.acc_dtype = reduce_acc_dtype(red_op, mid_dtype);
  if (nout == 0) { *plan = fp; return OCN_OK; }
  if ((red_op == R_MIN || red_op == R_MAX) && nred == 0) return OCN_ERR_EMPTY;
  if ((rc = check_alignment(a)) != OCN_OK) return rc;
  if ((rc = check_alignment(b)) != OCN_OK) return rc;
  if ((rc = check_alignment(out)) != OCN_OK) return rc;
  if (!provably_non_overlapping(out)) return OCN_ERR_OVERLAP_OUT;
  if (nred > 0) {
    intptr_t olo, ohi, ilo, ihi;
    byte_range(out, &olo, &ohi);
    byte_range(a, &ilo, &ihi);
    if (ilo < ohi && olo < ihi) return OCN_ERR_ALIAS;
    byte_range(b, &ilo, &ihi);
    if (ilo < ohi && olo < ihi) return OCN_ERR_ALIAS;
  }

  // elementwise into a temporary, then reduce it
  auto plan_unfused = [&]() -> int {
    fp.unfused = true;
    ocn_tensor &m = fp.mid;
    m.base = workspace;
    m.offset = 0;
    m.dtype = mid_dtype;
    m.ndim = nd;
    m.device = out->device;
    int64_t acc = dt_size(mid_dtype);
    for (int d = nd - 1; d >= 0; --d) { m.size[d] = shape[d]; m.stride[d] = acc; acc *= shape[d]; }
    fp.mid_bytes = ((size_t)acc + 255) / 256 * 256;
    // planned against a stand-in address when the caller only wants sizes
    if (!workspace) m.base = (void *)(uintptr_t)0x1000;
    int rc2;
    if ((rc2 = plan_elementwise(2, ew_op, a, b, &m, 0, &fp.ew)) != OCN_OK) return rc2;
    if ((rc2 = plan_reduce(red_op, &m, axes, naxes, out, &fp.red)) != OCN_OK) return rc2;
    fp.workspace_bytes = fp.mid_bytes + fp.red.workspace_bytes;
    *plan = fp;
    return OCN_OK;
  };
  // no fused kernel for these types
  if (other_order || !fused_specialised(ew_op, a->dtype, b->dtype, mid_dtype, red_op) || nred == 0) return plan_unfused();

  const int es_a = dt_size(a->dtype), es_b = dt_size(b->dtype);
  int64_t off_a = a->offset, off_b = b->offset, off_o = out->offset;
  // kept dims: drop size 1, flip to forward output strides, sort by output stride, merge
  int n = 0;
  for (int d = 0; d < nk; ++d) {
    if (kd[d].size == 1) continue;
    RDim x = kd[d];
    if (x.so < 0) {
      off_o += (x.size - 1) * x.so; off_a += (x.size - 1) * x.sa; off_b += (x.size - 1) * x.sb;
      x.so = -x.so; x.sa = -x.sa; x.sb = -x.sb;
    }
    kd[n++] = x;
  }
  nk = sort_merge(kd, n, true);
  // the column kernel walks the fastest kept dim forward through the inputs: turn it around
  // again if the flip above left both inputs walking backwards (or broadcast) there
  if (nk > 0) {
    RDim &x = kd[nk - 1];
    const bool a_back = x.sa == -(int64_t)es_a, b_back = x.sb == -(int64_t)es_b;
    if ((a_back && (b_back || x.sb == 0)) || (b_back && x.sa == 0)) {
      off_o += (x.size - 1) * x.so; off_a += (x.size - 1) * x.sa; off_b += (x.size - 1) * x.sb;
      x.so = -x.so; x.sa = -x.sa; x.sb = -x.sb;
    }
  }
  // reduced dims: drop size 1, flip so the faster-moving input walks forward, sort, merge
  n = 0;
  for (int d = 0; d < nr; ++d) {
    if (rd[d].size == 1) continue;
    RDim x = rd[d];
    const int64_t lead = x.sa != 0 ? x.sa : x.sb;
    if (lead < 0) {
      off_a += (x.size - 1) * x.sa; off_b += (x.size - 1) * x.sb;
      x.sa = -x.sa; x.sb = -x.sb;
    }
    rd[n++] = x;
  }
  nr = sort_merge_by(rd, n, [&](const RDim &x) { return std::max(iabs64(x.sa) / es_a, iabs64(x.sb) / es_b); });
  p.nkept = nk;
  p.nred = nr;
  for (int d = 0; d < nk; ++d) {
    p.ksize[d] = kd[d].size; p.kstride_a[d] = kd[d].sa; p.kstride_b[d] = kd[d].sb; p.kstride_o[d] = kd[d].so;
  }
  for (int d = 0; d < nr; ++d) { p.rsize[d] = rd[d].size; p.rstride_a[d] = rd[d].sa; p.rstride_b[d] = rd[d].sb; }
  p.off_a = off_a; p.off_b = off_b; p.off_out = off_o;
  p.a_ptr = (char *)a->base + off_a;
  p.b_ptr = (char *)b->base + off_b;
  p.out_ptr = (char *)out->base + off_o;
  choose_fused_launch(p);
  // The fused kernels cover the two layouts with a contiguous axis.  Anything else would fold
  // each output in a single lane: for long reductions the two-launch route, whose kernels
  // spread every layout over the device, is faster despite the temporary.
  if (p.kernel == OCN_KERNEL_RED_GENERIC && p.nredtot >= 1024) return plan_unfused();
  // more workgroups than one launch may have: the two calls, whose kernels loop
  if (p.grid > max_launch_blocks()) return plan_unfused();
  fp.workspace_bytes = p.workspace_bytes;
  *plan = fp;
  return OCN_OK;
}

void plan_second_pass(const RedPlan &first, char *workspace, RedPlan *second) {
  RedPlan q;
  q.op = first.op;  // every supported reduction folds its own partial results
  q.a_dtype = first.acc_dtype;
  q.out_dtype = first.out_dtype;
  q.acc_dtype = reduce_acc_dtype(q.op, q.a_dtype);
  q.nout = first.nout;
  q.nredtot = first.split;
  q.a_ptr = workspace;
  q.out_ptr = first.out_ptr;
  q.off_a = 0;
  q.off_out = first.off_out;
  const int64_t es = dt_size(q.a_dtype);
  q.nkept = first.nkept;
  const bool rows_layout = first.kernel == OCN_KERNEL_RED_ROWS || first.partial_rows;  // [nout][split], else [split][nout]
  int64_t lin = rows_layout ? first.split * es : es;
  for (int d = first.nkept - 1; d >= 0; --d) {
    q.ksize[d] = first.ksize[d];
    q.kstride_o[d] = first.kstride_o[d];
    q.kstride_a[d] = lin;
    lin *= first.ksize[d];
  }
  q.nred = 1;
  q.rsize[0] = first.split;
  q.rstride_a[0] = rows_layout ? es : first.nout * es;
  q.split = 1;
  q.swap_o = first.swap_o;   // the partial results are in native order, the output as the caller declared it
  q.chunk = first.split;
  q.passes = 1;
  q.workspace_bytes = 0;
  q.vec = 1;
  if (rows_layout) {
    q.kernel = OCN_KERNEL_RED_ROWS;
    q.group = 1;                       // lanes per output: the partials of one output are adjacent
    while (q.group < first.split && q.group < kWave) q.group <<= 1;
    if (first.split >= 4 * kBlock) q.group = kBlock;   // as in the first pass: four partials per lane and more
    q.chunk = first.split;  // vectors (vec = 1) per output
    q.grid = (q.nout * q.group + kBlock - 1) / kBlock;
    // Eight-byte partial results in whole, aligned 16-byte vectors, at most one kept dim: the
    // lean form of the kernel, whose few arguments arrive with the first scalar loads (this
    // launch is nothing but a chain of latencies)
    const int64_t nv = first.split / 2;
    if (es == 8 && first.split % 2 == 0 && nv >= kWave && nv < ((int64_t)1 << 31) && first.nkept <= 1 &&
        q.nout < ((int64_t)1 << 31) && (intptr_t)workspace % 16 == 0) {
      q.lean = true;
      q.vec = 2;
      q.chunk = nv;
      q.group = nv < 4 * kBlock ? kWave : kBlock;
      q.grid = (q.nout + kBlock / q.group - 1) / (kBlock / q.group);
    }
  } else if (!rows_layout && first.nkept >= 1 && q.nout < ((int64_t)1 << 31)) {
    q.kernel = OCN_KERNEL_RED_COLS;
    const int64_t nc = q.ksize[q.nkept - 1];
    while (q.cpw > 1 && q.cpw / 2 >= nc) q.cpw /= 2;
    const int64_t colblocks = (nc + q.cpw - 1) / q.cpw;
    q.grid = colblocks * (q.nout / nc);
    if (first.split >= 64) q.block = 16 * kWave;   // many partials per column: more wavefronts share them
    // partial results of a single kept dim: the kernel made for this launch (sixteen wavefronts from 64
    // splits on: 256 of five float columns 8 us with four)
    if (first.nkept == 1 && first.split < ((int64_t)1 << 31) && max_launch_blocks() >= (q.nout + kWave - 1) / kWave) {
      q.fold = true;
      q.block = first.split >= 64 ? 16 * kWave : kBlock;
      q.grid = (q.nout + kWave - 1) / kWave;
    }
  } else {
    q.kernel = OCN_KERNEL_RED_GENERIC;
    q.grid = std::min<int64_t>((q.nout + kBlock - 1) / kBlock, max_launch_blocks());
  }
  *second = q;
}

// ---------------------------------------------------------------------------------------
// plan inspection
// ---------------------------------------------------------------------------------------

void fill_info(const EwPlan &p, ocn_plan_info *info) {
  std::memset(info, 0, sizeof *info);
  info->kernel = p.kernel == kKernelBox ? OCN_KERNEL_EW_TILED : p.kernel == kKernelTiledAny ? (p.stage_a || p.stage_b ? OCN_KERNEL_EW_TILED : OCN_KERNEL_EW_GENERIC)
                 : p.kernel == kKernelToPlanes || p.kernel == kKernelToPixels ? OCN_KERNEL_EW_GENERIC : p.kernel;
  info->compute_dtype = p.T;
  info->ndim = p.ndim;
  for (int d = 0; d < p.ndim; ++d) {
    info->size[d] = p.size[d];
    info->stride_out[d] = p.out.stride[d];
    info->stride_a[d] = p.a.stride[d];
    info->stride_b[d] = p.b.stride[d];
    info->tile_log2[d] = p.tile_log2[d];
  }
  info->offset_out = p.off_out;
  info->offset_a = p.off_a;
  info->offset_b = p.off_b;
  info->vec = p.vec;
  info->stage_a = p.stage_a;
  info->stage_b = p.stage_b;
  info->specialised = p.specialised;
  info->passes = p.kernel == OCN_KERNEL_NONE ? 0 : 1;
  info->grid = p.grid;
  info->block = kBlock;   // (rows and tiles of any size: the caller puts in what they are launched with)
  info->split = 1;
  info->lds_bytes = p.lds_bytes;
  info->unclipped = p.fast_tiled ? 1 : 0;
  info->tile_group = p.fast_tiled && p.pair_dim >= 0 ? (int64_t)1 << p.pair_log2 : 1;
}

void fill_info(const RedPlan &p, ocn_plan_info *info) {
  std::memset(info, 0, sizeof *info);
  info->kernel = p.kernel;
  info->compute_dtype = p.acc_dtype;
  info->ndim = p.nkept;
  info->nred = p.nred;
  for (int d = 0; d < p.nkept; ++d) {
    info->size[d] = p.ksize[d];
    info->stride_out[d] = p.kstride_o[d];
    info->stride_a[d] = p.kstride_a[d];
  }
  for (int d = 0; d < p.nred; ++d) {
    info->red_size[d] = p.rsize[d];
    info->red_stride_a[d] = p.rstride_a[d];
  }
  info->offset_out = p.off_out;
  info->offset_a = p.off_a;
  info->vec = p.vec;
  info->specialised = 1;
  info->passes = p.kernel == OCN_KERNEL_NONE ? 0 : p.passes;
  info->grid = p.grid;
  info->block = p.block;
  info->split = p.split;
  info->stage_a = p.strip;
}

}  // namespace ocn
