// Kernel-argument builder for the reduction kernels (dtype independent).
#include "red_launch.hpp"

#include <algorithm>
#include <cstring>

namespace ocn {

RedLauncher g_reduce_launchers[R_COUNT][DT_COUNT];
RedLauncher g_fused_launchers[B_COUNT][DT_COUNT][R_COUNT];

RedArgs make_red_args(const RedPlan &p, char *partial) {
  RedArgs r;
  std::memset(&r, 0, sizeof r);
  r.a = p.a_ptr;
  r.out = p.out_ptr;
  r.partial = partial;
  r.warm = p.grid <= 1024;
  r.nkept = p.nkept;
  r.nred = p.nred;
  r.out_dtype = p.out_dtype;
  r.vec = p.vec;
  r.group = p.group;
  for (int k = 0; k < p.nkept; ++k) {  // fastest first
    const int d = p.nkept - 1 - k;
    r.ksa[k] = p.kstride_a[d];
    r.kso[k] = p.kstride_o[d];
    r.kdiv[k] = make_fastdiv((uint32_t)p.ksize[d]);
    r.ksize[k] = p.ksize[d];
    r.ksb[k] = p.kstride_b[d];
  }
  for (int k = 0; k < p.nred; ++k) {
    const int d = p.nred - 1 - k;
    r.rsa[k] = p.rstride_a[d];
    r.rdiv[k] = make_fastdiv((uint32_t)p.rsize[d]);
    r.rsize[k] = p.rsize[d];
    r.rsb[k] = p.rstride_b[d];
  }
  r.b = p.b_ptr;
  r.a_bcast = p.a_fast_bcast;
  r.b_bcast = p.b_fast_bcast;
  r.nout = p.nout;
  r.nredtot = p.nredtot;
  r.split = p.split;
  r.chunk = p.chunk;
  r.nt_load = p.nt_load ? 1 : 0;
  r.swap_a = p.swap_a ? 1 : 0;
  r.swap_o = p.swap_o ? 1 : 0;
  if (p.kernel == OCN_KERNEL_RED_ROWS) {
    r.n0 = p.rsize[p.nred - 1];
    const int64_t vpr = (r.n0 + p.vec - 1) / p.vec;
    r.vpr_div = make_fastdiv((uint32_t)(p.nred > 1 ? vpr : 1));
    r.nvec = vpr * (p.nredtot / r.n0);
  } else if (p.kernel == OCN_KERNEL_RED_COLS) {
    r.nc = p.ksize[p.nkept - 1];
    r.cpw = p.cpw;
    r.cpw_m = p.flat_cols ? (uint32_t)((((uint64_t)1 << 32) + p.cpw - 1) / p.cpw) : 0u;
    // (without lanes per row, one lane per vector of columns: a "block" is one lane's)
    const int64_t wide = (int64_t)std::max(1, p.cpw) * p.vec, colblocks = (r.nc + wide - 1) / wide;
    if (p.cpw == 0) r.nvec = colblocks * (p.nout / r.nc);
    r.colblocks_div = make_fastdiv((uint32_t)colblocks);
  }
  return r;
}

RedLeanArgs make_red_lean_args(const RedPlan &p, char *partial) {
  RedLeanArgs r;
  std::memset(&r, 0, sizeof r);
  r.a = p.a_ptr;
  r.out = p.out_ptr;
  r.partial = partial;
  r.b = p.b_ptr;
  r.ksa = p.nkept ? p.kstride_a[0] : 0;
  r.ksb = p.nkept ? p.kstride_b[0] : 0;
  r.kso = p.nkept ? p.kstride_o[0] : 0;
  r.nout = (uint32_t)p.nout;
  r.split = (uint32_t)p.split;
  r.nvec = (uint32_t)(p.nredtot / p.vec);
  r.tail = (uint32_t)(p.nredtot % p.vec);
  r.chunk = (uint32_t)p.chunk;
  r.out_dtype = p.out_dtype;
  r.group = p.group;
  r.nt_load = p.nt_load ? 1 : 0;
  r.swap_a = p.swap_a ? 1 : 0;
  r.swap_o = p.swap_o ? 1 : 0;
  return r;
}

RedStripArgs make_red_strip_args(const RedPlan &p, char *partial) {
  RedStripArgs r;
  std::memset(&r, 0, sizeof r);
  const int kc = p.nkept - 1;      // the columns' (rows: the rows') kept dim
  r.a = p.a_ptr;
  r.b = p.b_ptr;
  r.out = p.out_ptr;
  r.partial = partial;
  r.kso = p.kstride_o[kc];
  r.rs = p.strip_bc == 1 || p.strip == 3 ? p.rstride_a[0] : p.rstride_b[0];
  r.rows = (uint32_t)p.strip_rows;
  r.chunk = (uint32_t)p.chunk;
  r.width = (uint32_t)p.strip_width;
  r.inner = (uint32_t)p.strip_inner;
  r.lanes = (uint32_t)p.strip_lanes;
  r.lanes_m = (uint32_t)((((uint64_t)1 << 32) + r.lanes - 1) / r.lanes);
  r.groups = (uint32_t)p.strip_groups;
  r.parts = (uint32_t)p.strip_parts;
  r.rotate = (uint32_t)p.strip_rotate;
  const int64_t pieces = (p.strip_rows + p.chunk - 1) / p.chunk, others = p.nout / p.ksize[kc];
  r.ngroups = (uint32_t)(p.strip == 3 ? p.nout : others * pieces);
  r.nog = (uint32_t)(r.width / r.inner);
  r.flags = (p.nt_load ? kStripNt : 0u) | (p.swap_a ? kStripSwapA : 0u) | (p.swap_o ? kStripSwapO : 0u);
  r.out_dtype = p.out_dtype;
  r.pstep = p.partial_rows ? pieces : 1;
  r.psplit = p.partial_rows ? 1 : p.nout;
  r.split_div = make_fastdiv((uint32_t)pieces);
  r.width_div = make_fastdiv(r.width);
  r.inner_div = make_fastdiv(r.inner);
  r.nog_div = make_fastdiv(r.nog);
  r.outs_div = make_fastdiv(r.groups * r.nog);
  for (int d = kc - 1; d >= 0; --d) {
    const int k = (int)r.nother++;
    r.osa[k] = p.kstride_a[d];
    r.osb[k] = p.kstride_b[d];
    r.oso[k] = p.kstride_o[d];
    r.odiv[k] = make_fastdiv((uint32_t)p.ksize[d]);
  }
  return r;
}

}  // namespace ocn
