// Kernel-argument builders for the elementwise kernels (dtype independent).
#include "ew_launch.hpp"

#include <algorithm>
#include <cstdint>
#include <cstring>

namespace ocn {

EwLauncher g_binary_launchers[B_COUNT][DT_COUNT][DT_COUNT][DT_COUNT];
EwLauncher g_unary_launchers[U_COUNT][DT_COUNT][DT_COUNT];

RowsArgs make_rows_args(const EwPlan &p, int64_t *grid) {
  RowsArgs r;
  std::memset(&r, 0, sizeof r);
  r.out = p.out.ptr;
  r.a = p.a.ptr;
  r.b = p.b.ptr;
  r.numel = p.numel;
  const int inner = p.ndim - 1;
  const int64_t n0 = p.size[inner];
  const int es_o = dt_size(p.out.dtype), es_a = dt_size(p.a.dtype), es_b = dt_size(p.b.dtype);
  r.nouter = inner;
  for (int k = 0; k < inner; ++k) {  // fastest outer dim first
    const int d = inner - 1 - k;
    r.so[k] = p.out.stride[d];
    r.sa[k] = p.a.stride[d];
    r.sb[k] = p.b.stride[d];
    r.odiv[k] = make_fastdiv((uint32_t)p.size[d]);
  }
  // is the operand one contiguous run in the order of the dims?
  auto linear = [&](const Operand &x, int es) {
    int64_t expect = es;
    for (int d = inner; d >= 0; --d) {
      if (x.stride[d] != expect) return false;
      expect *= p.size[d];
    }
    return true;
  };
  r.flags = (p.a_inner_bcast ? kRowsABcast : 0u) | (p.b_inner_bcast ? kRowsBBcast : 0u) | (p.nt_store ? kRowsNtStore : 0u) |
            ((uint32_t)p.swap << kRowsSwapShift);
  // flat form: element numbers are split into row and column in 32 bits
  if (linear(p.out, es_o) && (inner == 0 || p.numel + 2 * p.vec < ((int64_t)1 << 31))) {
    r.flags |= kRowsFlat;
    // (not where the one vector more that a shift may take would be one workgroup too many)
    if ((intptr_t)p.out.ptr % es_o == 0 && p.numel / p.vec + 2 < max_launch_blocks() * kBlock * p.unroll)
      r.shift = (uint32_t)(((intptr_t)p.out.ptr / es_o) % p.vec);
    r.nvec = (p.numel + r.shift + p.vec - 1) / p.vec;
    r.inner = (uint32_t)n0;   // (below 2^31 with outer dims, unused without)
    r.rdiv = make_fastdiv(r.inner);
    // (the streaming hint only where the vectors of the input are aligned like the output's)
    auto aligned = [&](const Operand &x, int es) { return ((intptr_t)x.ptr - (int64_t)r.shift * es) % ((int64_t)p.vec * es) == 0; };
    if (linear(p.a, es_a)) r.flags |= kRowsALinear | (p.nt_a && aligned(p.a, es_a) ? kRowsNtA : 0u);
    if (p.nin == 2 && linear(p.b, es_b)) r.flags |= kRowsBLinear | (p.nt_b && aligned(p.b, es_b) ? kRowsNtB : 0u);
  } else {
    const int64_t vpr = (n0 + p.vec - 1) / p.vec;
    r.last = (uint32_t)(n0 - (vpr - 1) * p.vec);
    r.rdiv = make_fastdiv((uint32_t)(inner > 0 ? vpr : 1));
    r.nvec = vpr * (p.numel / n0);
  }
  // one-wavefront workgroups, four times fewer of four wavefronts where a launch cannot have as many
  r.block = kSlimBlock;
  *grid = (r.nvec + (int64_t)r.block * p.unroll - 1) / ((int64_t)r.block * p.unroll);
  if (*grid > max_launch_blocks()) {
    r.block = kBlock;
    *grid = (r.nvec + (int64_t)r.block * p.unroll - 1) / ((int64_t)r.block * p.unroll);
  }
  return r;
}

bool make_rows_slim_args(const EwPlan &p, int block, RowsSlimArgs *args, int64_t *grid) {
  const int inner = p.ndim - 1;
  if (inner < 0 || inner > 1) return false;
  const int64_t n0 = p.size[inner];
  // whole vectors; a one-dimensional tensor may end with part of one where a lane takes several (with
  // one vector per lane the kernel for rows of any length is as fast)
  const int64_t tail = n0 % p.vec;
  if (!p.rows_aligned || (tail != 0 && (inner == 1 || p.unroll == 1))) return false;
  const int64_t vpr = n0 / p.vec;
  const int64_t nvec = vpr * (inner == 1 ? p.size[0] : 1);
  const int64_t lanes = nvec + (tail != 0 ? 1 : 0);
  const int64_t g = (lanes + (int64_t)block * p.unroll - 1) / ((int64_t)block * p.unroll);
  // 32-bit vector numbers (including those of the lanes past the end), one launch
  if (nvec >= ((int64_t)1 << 31) || g * block * p.unroll >= ((int64_t)1 << 32) || g > max_launch_blocks() || g < 1)
    return false;
  RowsSlimArgs r;
  std::memset(&r, 0, sizeof r);
  r.out = p.out.ptr;
  r.a = p.a.ptr;
  r.b = p.b.ptr;
  if (inner == 1) {
    r.so = p.out.stride[0];
    r.sa = p.a.stride[0];
    r.sb = p.b.stride[0];
  }
  r.nvec = (uint32_t)nvec;
  // without an outer dim: row 0 for every vector
  r.vpr_div = make_fastdiv((uint32_t)std::max<int64_t>(vpr, 1));
  r.flags = (p.a_inner_bcast ? kSlimABcast : 0u) | (p.b_inner_bcast ? kSlimBBcast : 0u) | (p.nt_a ? kSlimNtA : 0u) |
            (p.nt_b ? kSlimNtB : 0u) | (p.nt_store ? kSlimNtStore : 0u) | ((uint32_t)p.swap << kSlimSwapShift) | ((uint32_t)tail << kSlimTailShift);
  *args = r;
  *grid = g;
  return true;
}

void ew_launch_shape(const EwPlan &p, int64_t *grid, int64_t *block) {
  *grid = p.grid;
  *block = p.kernel == kKernelTiledAny || p.kernel == kKernelBox ? p.block : kBlock;
  if (p.kernel != OCN_KERNEL_EW_ROWS) return;
  RowsSlimArgs slim;
  *block = kSlimBlock;
  if (!make_rows_slim_args(p, kSlimBlock, &slim, grid)) *block = make_rows_args(p, grid).block;
}

TiledArgs make_tiled_args(const EwPlan &p, int es_a) {
  TiledArgs t;
  std::memset(&t, 0, sizeof t);
  t.out = p.out.ptr;
  t.a = p.a.ptr;
  t.b = p.b.ptr;
  t.ndim = p.ndim;
  t.tile_bits = p.tile_bits;
  t.total_tiles = (uint32_t)p.total_tiles;
  for (int d = 0; d < p.ndim; ++d) {
    t.size[d] = p.size[d];
    t.so[d] = p.out.stride[d];
    t.sa[d] = p.a.stride[d];
    t.sb[d] = p.b.stride[d];
    t.tl[d] = p.tile_log2[d];
    t.ntdiv[d] = make_fastdiv((uint32_t)p.ntiles[d]);
  }
  t.stage_a = p.stage_a;
  t.stage_b = p.stage_b;
  t.nt_store = p.nt_store;
  t.swap = p.swap;
  const int64_t tile_elems = (int64_t)1 << p.tile_bits;
  t.lds_off_b = p.stage_a ? (uint32_t)((tile_elems * es_a + 15) / 16 * 16) : 0u;
  // bit position of each tiled dim in the output's enumeration order = its LDS slot shift
  int slot_shift[kMaxDims] = {0};
  int acc = 0;
  for (int k = 0; k < p.nord; ++k) {
    slot_shift[p.ord_o[k]] = acc;
    acc += p.tile_log2[p.ord_o[k]];
  }
  const int8_t *ords[3] = {p.ord_o, p.ord_a, p.ord_b};
  const int vecw[3] = {p.vecw_o, p.vecw_a, p.vecw_b};
  for (int x = 0; x < 3; ++x) {
    TileOrder &o = t.ord[x];
    o.nord = (int8_t)p.nord;
    o.vecw = (int8_t)vecw[x];
    for (int k = 0; k < p.nord; ++k) {
      const int d = ords[x][k];
      o.dim[k] = (int8_t)d;
      o.width[k] = (int8_t)p.tile_log2[d];
      o.lds_shift[k] = (int8_t)slot_shift[d];
      o.stride[0][k] = p.out.stride[d];
      o.stride[1][k] = p.a.stride[d];
      o.stride[2][k] = p.b.stride[d];
    }
    const int64_t nvec = tile_elems >> vecw[x];
    o.niter = (int32_t)((nvec + kBlock - 1) / kBlock);
    // contribution of the pass number (bits 8 and up of the vector index) to offsets and slot
    for (int j = 0; j < o.niter && j < kMaxTilePasses; ++j) {
      const LanePos hi = lane_pos(o, (uint32_t)j * kBlock);
      for (int y = 0; y < 3; ++y) o.hi_off[y][j] = hi.off[y];
      o.hi_slot[j] = hi.slot;
    }
  }
  // XOR swizzle of a staged operand's LDS slots: the vector index along the operand's own
  // fastest dim is folded into the low slot bits, at the granularity of one LDS access of the
  // compute phase (the elements of a vector, at most 16 bytes), over as many bits as it takes
  // to spread the accesses of a wavefront over 128 bytes of banks
  auto make_swizzle = [&](const TileOrder &o, int es) {
    TileSwizzle z{0, 0, 0};
    if (p.nord == 0) return z;
    const int w_f = o.width[0] - o.vecw;             // vector positions along the operand's dim
    const int w_0 = p.tile_log2[p.ord_o[0]];         // bits of the output's fastest dim
    int dst = 0, want = 5;
    if (p.vecw_o > 0) {
      while (dst < p.vecw_o && (2 << dst) * es <= 16) ++dst;   // keep the groups read at once intact
      want = 0;
      while (((es << dst) << want) < 128) ++want;
    }
    if (dst > w_0) dst = w_0;
    int bits = std::min(want, std::min(w_f, w_0 - dst));
    if (bits < 0) bits = 0;
    z.src = (uint32_t)(o.lds_shift[0] + o.vecw);
    z.mask = (1u << bits) - 1u;
    z.dst = (uint32_t)dst;
    return z;
  };
  if (p.stage_a) t.swz[0] = make_swizzle(t.ord[1], es_a);
  if (p.stage_b) t.swz[1] = make_swizzle(t.ord[2], dt_size(p.b.dtype));
  return t;
}

FastTiledArgs make_fast_tiled_args(const EwPlan &p, int es_a) {
  const TiledArgs t = make_tiled_args(p, es_a);
  FastTiledArgs f;
  std::memset(&f, 0, sizeof f);
  f.warm = p.total_tiles <= kWarmTiles;
  f.out = t.out;
  f.a = t.a;
  f.b = t.b;
  f.stage_a = t.stage_a;
  f.stage_b = t.stage_b;
  f.nt_store = t.nt_store;
  f.swap = t.swap;
  // tile grid: only dims with more than one tile, fastest (last canonical dim) first.  Where
  // neighbouring tiles along one dim share input lines, that dim's tile index is split: its low
  // part (the group of tiles sharing a line) varies fastest of all, its high part stays in place.
  f.pair_log2 = p.pair_dim >= 0 ? p.pair_log2 : 0;
  auto add_dim = [&](int d, int64_t count, int64_t mult) {
    const int j = f.ntd++;
    f.ntdiv[j] = make_fastdiv((uint32_t)count);
    f.step[0][j] = t.so[d] * ((int64_t)mult << t.tl[d]);
    f.step[1][j] = t.sa[d] * ((int64_t)mult << t.tl[d]);
    f.step[2][j] = t.sb[d] * ((int64_t)mult << t.tl[d]);
  };
  const int64_t group = (int64_t)1 << f.pair_log2;
  if (f.pair_log2) add_dim(p.pair_dim, group, 1);
  for (int d = p.ndim - 1; d >= 0; --d) {
    const bool paired = f.pair_log2 && d == p.pair_dim;
    const int64_t count = paired ? p.ntiles[d] / group : p.ntiles[d];
    if (count <= 1) continue;
    add_dim(d, count, paired ? group : 1);
  }
  const int es[2] = {es_a, p.nin == 2 ? dt_size(p.b.dtype) : 1};
  // An input too large to be found in a cache again is read with streaming loads where every
  // run of it inside a tile - along its own fastest axis if it is staged, along the output's
  // if it is read in place - is a whole number of 128-byte lines starting on a line boundary
  // (a streaming load of part of a line runs at a fraction of the rate of an ordinary one).
  auto whole_lines = [&](const Operand &x, int esz, int run_dim) {
    if (x.stride[run_dim] != esz || (((int64_t)esz << p.tile_log2[run_dim]) % 128) != 0) return false;
    if (((intptr_t)x.ptr % 128) != 0) return false;
    int64_t distinct = esz;
    for (int d = 0; d < p.ndim; ++d) {
      if (x.stride[d] == 0) return false;
      if (d != run_dim && x.stride[d] % 128 != 0) return false;
      distinct *= p.size[d];
    }
    return distinct >= kStreamBytes;
  };
  if (p.nord > 0) {
    f.nt_a = whole_lines(p.a, es[0], p.stage_a ? p.ord_a[0] : p.ord_o[0]) ? 1 : 0;
    f.nt_b = p.nin == 2 && whole_lines(p.b, es[1], p.stage_b ? p.ord_b[0] : p.ord_o[0]) ? 1 : 0;
  }
  auto log2i = [](int64_t v) { int l = 0; while (((int64_t)1 << l) < v) ++l; return l; };
  const int64_t tile_elems = (int64_t)1 << p.tile_bits;
  // the larger staging area goes first, so that the smaller one starts at a multiple of its own
  // (power-of-two) size and the base can be OR-ed into XOR-built addresses
  const int64_t bytes_a = p.stage_a ? tile_elems * es[0] : 0, bytes_b = p.stage_b ? tile_elems * es[1] : 0;
  if (bytes_a >= bytes_b) { f.lds_base[0] = 0; f.lds_base[1] = (uint32_t)bytes_a; }
  else { f.lds_base[1] = 0; f.lds_base[0] = (uint32_t)bytes_b; }
  f.swz[0] = t.swz[0];
  f.swz[1] = t.swz[1];
  f.es_log2[0] = (uint32_t)log2i(es[0]);
  f.es_log2[1] = (uint32_t)log2i(es[1]);
  f.vc_log2 = (uint32_t)p.vecw_o;
  for (int x = 0; x < 3; ++x) {
    const TileOrder &o = t.ord[x];
    FastOrder &g = f.ord[x];
    g.niter = o.niter;
    uint32_t shift = 0;
    for (int k = 0; k < o.nord && shift < 8; ++k) {
      const uint32_t vw = k == 0 ? (uint32_t)o.vecw : 0u;
      const uint32_t w = (uint32_t)o.width[k] - vw;
      const uint32_t wl = std::min(w, 8u - shift);  // bits of this dim's index held by the lane number
      if (wl > 0) {
        const int i = g.nlane++;
        g.shift[i] = shift;
        g.mask[i] = (1u << wl) - 1u;
        g.up[i] = vw;
        g.slot_shift[i] = (uint32_t)o.lds_shift[k];
        for (int y = 0; y < 3; ++y) g.stride[y][i] = (uint32_t)o.stride[y][k];
      }
      shift += w;
    }
    for (int j = 0; j < o.niter && j < kMaxTilePasses; ++j)
      for (int y = 0; y < 3; ++y) g.hi_off[y][j] = (uint32_t)o.hi_off[y][j];
  }
  for (int y = 0; y < 2; ++y) {
    if (!(y == 0 ? p.stage_a : p.stage_b)) continue;
    const TileOrder &o = t.ord[y + 1];
    const TileSwizzle &z = t.swz[y];
    const uint32_t sh = f.es_log2[y];
    for (int j = 0; j < o.niter && j < kMaxTilePasses; ++j) f.st_hi[y][j] = swizzle(o.hi_slot[j], z) << sh;
    for (int i = 0; i < (1 << o.vecw) && i < 16; ++i) f.st_el[y][i] = swizzle((uint32_t)i << o.lds_shift[0], z) << sh;
    const TileOrder &oc = t.ord[0];
    for (int j = 0; j < oc.niter && j < kMaxTilePasses; ++j)
      f.rd_hi[y][j] = swizzle(((uint32_t)j * kBlock) << p.vecw_o, z) << sh;
    const int epc = std::min(std::max(1, 16 / es[y]), 1 << p.vecw_o);
    for (int c = 0; c * epc < (1 << p.vecw_o) && c < 16; ++c) f.rd_ch[y][c] = swizzle((uint32_t)(c * epc), z) << sh;
  }
  return f;
}

AnyTiledArgs make_any_tiled_args(const EwPlan &p, int es_a) {
  const TiledArgs t = make_tiled_args(p, es_a);
  AnyTiledArgs f;
  std::memset(&f, 0, sizeof f);
  f.out = t.out;
  f.a = t.a;
  f.b = t.b;
  auto end_of = [&](const Operand &x) {
    const char *e = x.ptr + dt_size(x.dtype);
    for (int d = 0; d < p.ndim; ++d)
      if (x.stride[d] > 0) e += (p.size[d] - 1) * x.stride[d];
    return e;
  };
  f.end[0] = end_of(p.a);
  if (p.nin == 2) f.end[1] = end_of(p.b);
  f.warm = p.total_tiles <= kWarmTiles;
  f.block = (uint32_t)p.block;
  f.nord = p.nord;
  f.stage_a = t.stage_a;
  f.stage_b = t.stage_b;
  f.nt_store = t.nt_store;
  f.swap = t.swap;
  f.sa0 = (uint32_t)p.a.stride[p.ord_o[0]];
  f.sb0 = (uint32_t)p.b.stride[p.ord_o[0]];
  f.stage_stride[0] = (uint32_t)p.a.stride[p.ord_a[0]];
  f.stage_stride[1] = (uint32_t)p.b.stride[p.ord_b[0]];
  // packed limits: 16 bits per tiled dim, in the output's order
  int pos[kMaxDims];
  for (int d = 0; d < kMaxDims; ++d) pos[d] = -1;
  for (int k = 0; k < p.nord; ++k) {
    const int d = p.ord_o[k];
    pos[d] = k;
    f.inner |= (uint64_t)std::min<int64_t>((int64_t)1 << p.tile_log2[d], p.size[d]) << (16 * k);
    f.whole |= (uint64_t)1 << p.tile_log2[d] << (16 * k);
  }
  for (int d = p.ndim - 1; d >= 0; --d) {
    if (p.ntiles[d] <= 1) continue;
    const int j = f.ntd++;
    f.ntdiv[j] = make_fastdiv((uint32_t)p.ntiles[d]);
    f.step[0][j] = t.so[d] * ((int64_t)1 << t.tl[d]);
    f.step[1][j] = t.sa[d] * ((int64_t)1 << t.tl[d]);
    f.step[2][j] = t.sb[d] * ((int64_t)1 << t.tl[d]);
    f.dim_shift[j] = pos[d] >= 0 ? (uint32_t)(16 * pos[d]) : 64u;
    f.last[j] = (uint32_t)(p.size[d] - ((p.ntiles[d] - 1) << p.tile_log2[d]));
  }
  const int es[2] = {es_a, p.nin == 2 ? dt_size(p.b.dtype) : 1};
  const int64_t tile_elems = (int64_t)1 << p.tile_bits;
  const int64_t bytes_a = p.stage_a ? tile_elems * es[0] : 0, bytes_b = p.stage_b ? tile_elems * es[1] : 0;
  // the larger staging area first, so that each base can be OR-ed into XOR-built addresses
  if (bytes_a >= bytes_b) { f.lds_base[0] = 0; f.lds_base[1] = (uint32_t)bytes_a; }
  else { f.lds_base[1] = 0; f.lds_base[0] = (uint32_t)bytes_b; }
  for (int y = 0; y < 2; ++y) {
    f.swz[y] = t.swz[y];
    while ((1 << f.es_log2[y]) < es[y]) ++f.es_log2[y];
  }
  uint32_t hi_slot[3][kMaxTilePasses];
  const uint32_t lane_bits = f.block == 1024 ? 10 : f.block == 512 ? 9 : 8;
  for (int x = 0; x < 3; ++x) {
    const TileOrder &o = t.ord[x];
    AnyOrder &g = f.ord[x];
    g.vecw = o.vecw;
    g.nvec = (uint32_t)(tile_elems >> o.vecw);
    g.niter = (int32_t)((g.nvec + f.block - 1) / f.block);
    uint32_t shift = 0, upper[kAnyDims], above[kAnyDims];   // bits of each dim's index held by the pass number
    for (int k = 0; k < o.nord; ++k) {
      const uint32_t vw = k == 0 ? (uint32_t)o.vecw : 0u, w = (uint32_t)o.width[k] - vw;
      const uint32_t wl = shift < lane_bits ? std::min(w, lane_bits - shift) : 0u;   // bits held by the lane number
      g.shift[k] = std::min(shift, 31u);
      g.mask[k] = (1u << wl) - 1u;
      g.up[k] = vw;
      g.slot_shift[k] = (uint32_t)o.lds_shift[k];
      g.lim_shift[k] = (uint32_t)(16 * pos[o.dim[k]]);
      for (int y = 0; y < 3; ++y) g.stride[y][k] = (uint32_t)o.stride[y][k];
      upper[k] = w - wl;
      above[k] = vw + wl;
      shift += w;
    }
    for (int j = 0; j < g.niter; ++j) {
      const LanePos hi = lane_pos(o, (uint32_t)j * f.block);
      for (int y = 0; y < 3; ++y) g.hi_off[y][j] = (uint32_t)hi.off[y];
      hi_slot[x][j] = hi.slot;
      uint32_t rest = (uint32_t)j;
      for (int k = 0; k < o.nord; ++k) {
        const uint32_t c = (rest & ((1u << upper[k]) - 1u)) << above[k];
        rest >>= upper[k];
        g.hi_c[j] |= (uint64_t)c << (16 * k);
      }
    }
  }
  for (int y = 0; y < 2; ++y) {
    if (!(y == 0 ? p.stage_a : p.stage_b)) continue;
    const TileOrder &o = t.ord[y + 1];
    const TileSwizzle &z = t.swz[y];
    const uint32_t sh = f.es_log2[y];
    for (int j = 0; j < f.ord[y + 1].niter; ++j) f.st_hi[y][j] = swizzle(hi_slot[y + 1][j], z) << sh;
    for (int i = 0; i < (1 << o.vecw) && i < 16; ++i) f.st_el[y][i] = swizzle((uint32_t)i << o.lds_shift[0], z) << sh;
    for (int j = 0; j < f.ord[0].niter; ++j) f.rd_hi[y][j] = swizzle(((uint32_t)j * f.block) << p.vecw_o, z) << sh;
    for (int i = 0; i < (1 << p.vecw_o) && i < 16; ++i) f.rd_el[y][i] = swizzle((uint32_t)i, z) << sh;
  }
  return f;
}

BoxArgs make_box_args(const EwPlan &p) {
  BoxArgs f;
  std::memset(&f, 0, sizeof f);
  const Operand *ops[3] = {&p.out, &p.a, &p.b};
  const int es[3] = {dt_size(p.out.dtype), dt_size(p.a.dtype), p.nin == 2 ? dt_size(p.b.dtype) : 1};
  const int8_t *ords[3] = {p.ord_o, p.ord_a, p.ord_b};
  const uint32_t vec = 1u << p.vecw_o;
  f.out = p.out.ptr;
  f.a = p.a.ptr;
  f.b = p.b.ptr;
  for (int x = 1; x <= p.nin; ++x) {
    const char *e = ops[x]->ptr + es[x];
    int64_t reach = 0;
    for (int d = 0; d < p.ndim; ++d) {
      e += (p.size[d] - 1) * ops[x]->stride[d];
      reach += (p.box[d] - 1) * ops[x]->stride[d];
    }
    f.end[x - 1] = e;
    f.in[x - 1].reach = (uint32_t)(reach + std::max<int64_t>(16, (int64_t)vec * es[x]));
  }
  f.warm = p.total_tiles <= kWarmTiles;
  f.nt_store = p.nt_store;
  f.swap = p.swap;
  f.block = (uint32_t)p.block;
  auto inverse = [](uint32_t d) { return (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); };   // (d above one)
  // the limits: largest coordinates, in the output's order; the bits above them are zero, the limit of
  // a coordinate that is always zero
  uint32_t shift_of[kMaxDims];
  constexpr uint32_t kNone = 63;
  for (int d = 0; d < kMaxDims; ++d) shift_of[d] = kNone;
  for (int k = 0; k < p.nord; ++k) {
    shift_of[p.ord_o[k]] = (uint32_t)(16 * k);
    f.inner |= (uint64_t)(p.box[p.ord_o[k]] - 1) << (16 * k);
  }
  f.group = (uint32_t)p.box_group;
  f.group_div = make_fastdiv(std::max(1u, f.group * kXcds));
  f.regular = f.group > 1 ? (uint32_t)p.total_tiles / f.group_div.d * f.group_div.d : 0u;
  for (int j = 0; j < kMaxDims; ++j) f.ntdiv[j] = make_fastdiv(1);
  for (int d = p.ndim - 1; d >= 0; --d) {
    if (p.ntiles[d] <= 1) continue;
    const int j = f.ntd++;
    f.ntdiv[j] = make_fastdiv((uint32_t)p.ntiles[d]);
    for (int x = 0; x < 3; ++x) f.step[x][j] = ops[x]->stride[d] * p.box[d];
    if (p.box[d] > 1) f.cut[j] = (uint64_t)(p.box[d] - (p.size[d] - (p.ntiles[d] - 1) * p.box[d])) << shift_of[d];
  }
  uint32_t pos[2][kMaxDims] = {};   // bytes of an input per coordinate, where it is read
  uint32_t lds = 0;
  for (int y = 0; y < p.nin; ++y) {
    BoxInput &in = f.in[y];
    const Operand &x = *ops[y + 1];
    in.how = p.box_how[y];
    if (in.how == kBoxInPlace) {
      for (int d = 0; d < p.ndim; ++d) pos[y][d] = (uint32_t)x.stride[d];
      f.o.start[y] = kBoxSlack;
      continue;
    }
    const int nd = p.box_dims[y + 1], nrun = p.box_run[y + 1], nrow = nd - nrun;
    const int8_t *o = ords[y + 1];
    const uint32_t e = (uint32_t)es[y + 1];
    in.epv = 16u / e;
    uint32_t len = 1, rows = 1;
    for (int k = 0; k < nrun; ++k) {
      pos[y][o[k]] = len * e;
      len *= (uint32_t)p.box[o[k]];
    }
    in.unit = len / (uint32_t)p.box[o[nrun - 1]];
    in.lim_run = shift_of[o[nrun - 1]];
    in.vpr = (len + in.epv - 1) / in.epv;
    in.vpr_m = in.vpr > 1 ? inverse(in.vpr) : 0;
    in.pitch = (len * e + 15) / 16 * 16;
    if (in.pitch % 32 == 0) in.pitch += 16;
    in.base = f.o.start[y] = lds;
    uint32_t radix[3] = {in.vpr, 1u << 16, 1u << 16};
    for (int k = 0; k < kBoxRows; ++k) {
      in.lim[k] = kNone;
      if (k >= nrow) continue;
      const int d = o[nrun + k];
      const uint32_t ext = (uint32_t)p.box[d];
      if (k < 2 && k + 1 < nrow) {   // (the last coordinate is what is left)
        in.ext[k] = radix[k + 1] = ext;
        in.ext_m[k] = inverse(ext);
      }
      in.stride[k] = (uint32_t)x.stride[d];
      in.lim[k] = shift_of[d];
      pos[y][d] = rows * in.pitch;
      rows *= ext;
    }
    in.nvec = in.vpr * rows;
    in.niter = (in.nvec + f.block - 1) / f.block;
    lds += rows * in.pitch;
    uint32_t rest = f.block;
    for (int k = 0; k < 3; ++k) {
      in.wrap[k] = radix[k];
      in.add[k] = rest % radix[k];
      rest /= radix[k];
    }
    in.add_off = in.add[0] * 16u + in.add[1] * in.stride[0] + in.add[2] * in.stride[1] + rest * in.stride[2];
    in.add_c2 = rest;
    in.add_lds = in.add[0] * 16u + f.block / radix[0] * in.pitch;
    in.wrap_off[0] = in.stride[0] - radix[0] * 16u;
    in.wrap_off[1] = in.stride[1] - radix[1] * in.stride[0];
    in.wrap_off[2] = in.stride[2] - radix[2] * in.stride[1];
    in.wrap_lds = in.pitch - radix[0] * 16u;
  }
  BoxOutput &out = f.o;
  out.nrun = p.box_run[0];
  const int nrow = p.nord - out.nrun;
  uint32_t len = 1, rows = 1;
  for (int k = 0; k < out.nrun; ++k) len *= (uint32_t)p.box[p.ord_o[k]];
  const int last = p.ord_o[out.nrun - 1];
  out.unit = len / (uint32_t)p.box[last];
  out.lim_run = shift_of[last];
  out.vpr = (len + vec - 1) / vec;
  out.vpr_m = out.vpr > 1 ? inverse(out.vpr) : 0;
  out.step = vec * (uint32_t)es[0];
  for (int y = 0; y < 2; ++y) out.run[y] = vec * pos[y][p.ord_o[0]];
  for (int k = 0; k + 1 < kBoxRunDims; ++k) {
    out.run_ext[k] = 1u << 16;   // (never reached)
    if (k + 1 >= out.nrun) continue;
    const uint32_t ext = (uint32_t)p.box[p.ord_o[k]];
    out.run_ext[k] = ext;
    out.run_m[k] = inverse(ext);
    // what a step along the run's next dim adds to one along all of this dim
    for (int y = 0; y < 2; ++y) out.run_pos[y][k] = pos[y][p.ord_o[k + 1]] - ext * pos[y][p.ord_o[k]];
  }
  uint32_t radix[3] = {out.vpr, 1u << 16, 1u << 16};
  for (int k = 0; k < kBoxRows; ++k) {
    out.lim[k] = kNone;
    if (k >= nrow) continue;
    const int d = p.ord_o[out.nrun + k];
    const uint32_t ext = (uint32_t)p.box[d];
    if (k < 2 && k + 1 < nrow) {
      out.ext[k] = radix[k + 1] = ext;
      out.ext_m[k] = inverse(ext);
    }
    out.stride[k] = (uint32_t)p.out.stride[d];
    out.lim[k] = shift_of[d];
    for (int y = 0; y < 2; ++y) out.pos[y][k] = pos[y][d];
    rows *= ext;
  }
  out.nvec = out.vpr * rows;
  out.niter = (out.nvec + f.block - 1) / f.block;
  uint32_t rest = f.block;
  for (int k = 0; k < 3; ++k) {
    out.wrap[k] = radix[k];
    out.add[k] = rest % radix[k];
    rest /= radix[k];
  }
  out.add_c2 = rest;
  auto per_pass = [&](uint32_t step, const uint32_t (&per)[kBoxRows], uint32_t &add, uint32_t (&wrap)[3]) {
    add = out.add[0] * step + out.add[1] * per[0] + out.add[2] * per[1] + rest * per[2];
    wrap[0] = per[0] - radix[0] * step;
    wrap[1] = per[1] - radix[1] * per[0];
    wrap[2] = per[2] - radix[2] * per[1];
  };
  per_pass(out.step, out.stride, out.add_off, out.wrap_off);
  for (int y = 0; y < 2; ++y) per_pass(out.run[y], out.pos[y], out.add_pos[y], out.wrap_pos[y]);
  return f;
}

InterpArgs make_interp_args(const EwPlan &p) {
  InterpArgs a;
  std::memset(&a, 0, sizeof a);
  a.out = p.out.ptr;
  a.a = p.a.ptr;
  a.b = p.b.ptr;
  a.ndim = p.ndim;
  a.nin = p.nin;
  a.op = p.op;
  a.T = p.T;
  a.dt_a = p.a.dtype;
  a.dt_b = p.b.dtype;
  a.dt_o = p.out.dtype;
  for (int d = 0; d < p.ndim; ++d) {
    a.size[d] = p.size[d];
    a.so[d] = p.out.stride[d];
    a.sa[d] = p.a.stride[d];
    a.sb[d] = p.b.stride[d];
  }
  a.numel = p.numel;
  a.swap = p.swap;
  a.vec = 1;
  // Four elements per lane where the innermost dim allows it: contiguous in the output, contiguous
  // or broadcast in the inputs, and at least four long.  Alignment does not matter (one access of at
  // most 16 bytes per 16 bytes at any multiple of the scalar size).  Where the length is not a
  // multiple of four, a row's last group ends with the row and repeats elements of the one before
  // it - not in place, where those may have been overwritten by then.  The elementary functions
  // stay at one.
  const bool elementary = p.nin == 1 && ((p.op >= U_SIN && p.op <= U_LOG) || (p.op >= U_ASIN && p.op <= U_TANH));
  if (p.ndim >= 1 && !elementary) {
    const int last = p.ndim - 1;
    const int64_t n0 = p.size[last], es_o = dt_size(p.out.dtype);
    auto fits = [&](const Operand &x) { return x.stride[last] == 0 || x.stride[last] == dt_size(x.dtype); };
    const bool in_place = p.a.ptr == p.out.ptr || (p.nin == 2 && p.b.ptr == p.out.ptr);
    if (p.out.stride[last] == es_o && fits(p.a) && (p.nin == 1 || fits(p.b)) && n0 >= 4 && (n0 % 4 == 0 || !in_place)) {
      const int64_t groups = (n0 + 3) / 4, over = groups * 4 - n0;
      a.vec = 4;
      a.inner_a = p.a.stride[last] != 0;
      a.inner_b = p.nin == 2 && p.b.stride[last] != 0;
      a.back[0] = (int32_t)(over * p.out.stride[last]);
      a.back[1] = (int32_t)(over * p.a.stride[last]);
      a.back[2] = p.nin == 2 ? (int32_t)(over * p.b.stride[last]) : 0;
      a.nt_store = p.nt_store && es_o == 4;   // one 16-byte piece per lane
      a.size[last] = groups;
      a.so[last] *= 4;
      a.sa[last] *= 4;
      a.sb[last] *= 4;
      a.numel = a.numel / n0 * groups;
    }
  }
  a.idx32 = a.numel < ((int64_t)1 << 31);
  if (a.idx32)
    for (int d = 0; d < p.ndim; ++d) a.div[d] = make_fastdiv((uint32_t)a.size[d]);
  return a;
}

}  // namespace ocn
