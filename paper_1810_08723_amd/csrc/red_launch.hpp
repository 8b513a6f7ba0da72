// Host side of the reduction kernels.
#pragma once

#include <hip/hip_runtime.h>

#include "red_kernels.hpp"
#include "strip_kernels.hpp"

namespace ocn {

using RedLauncher = hipError_t (*)(const RedPlan &, char *partial, hipStream_t);
extern RedLauncher g_reduce_launchers[R_COUNT][DT_COUNT];
// fused elementwise+reduce kernels: [elementwise op][input dtype (both inputs)][reduce op]
extern RedLauncher g_fused_launchers[B_COUNT][DT_COUNT][R_COUNT];

RedArgs make_red_args(const RedPlan &p, char *partial);
RedLeanArgs make_red_lean_args(const RedPlan &p, char *partial);
RedStripArgs make_red_strip_args(const RedPlan &p, char *partial);

// lanes per workgroup of the lean rows kernels
inline unsigned lean_block(const RedPlan &p) { return p.group > kBlock ? (unsigned)p.group : (unsigned)kBlock; }

#if defined(__HIPCC__)
template <int S, int OP> hipError_t launch_red(const RedPlan &p, char *partial, hipStream_t stream) {
  if (p.strip) {
    const RedStripArgs args = make_red_strip_args(p, partial);
    const size_t lds = p.strip != 2 ? strip_cols_lds<typename Reducer<S, OP>::A>((int)p.block, (int)sizeof(storage_t<S>)) : p.strip_lds;
    if (p.strip == 1) hipLaunchKernelGGL((red_strip_cols_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), lds, stream, args);
    else if (p.strip == 3) hipLaunchKernelGGL((red_strip_runs_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), lds, stream, args);
    else hipLaunchKernelGGL((red_strip_rows_kernel<S, OP>), dim3((unsigned)p.grid), dim3(kBlock), lds, stream, args);
    return hipGetLastError();
  }
  const RedArgs args = make_red_args(p, partial);
  switch (p.kernel) {
    case OCN_KERNEL_RED_ROWS:
      if (p.lean) {
        const RedLeanArgs lean = make_red_lean_args(p, partial);
        if (lean.tail) hipLaunchKernelGGL((red_rows_lean_kernel<S, OP, true>), dim3((unsigned)p.grid), dim3(lean_block(p)), 0, stream, lean);
        else hipLaunchKernelGGL((red_rows_lean_kernel<S, OP, false>), dim3((unsigned)p.grid), dim3(lean_block(p)), 0, stream, lean);
        break;
      }
      if (p.short_rows) {
        hipLaunchKernelGGL((red_rows_short_kernel<S, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
        break;
      }
      hipLaunchKernelGGL((red_rows_kernel<S, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
      break;
    case OCN_KERNEL_RED_COLS:
      if (p.fold) {
        RedFoldArgs f;
        f.partial = p.a_ptr;
        f.out = p.out_ptr;
        f.kso = p.kstride_o[0];
        f.nout = (uint32_t)p.nout;
        f.split = (uint32_t)p.nredtot;
        f.out_dtype = p.out_dtype;
        f.swap_o = p.swap_o ? 1 : 0;
        hipLaunchKernelGGL((red_fold_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), 0, stream, f);
        break;
      }
      {
        using A = typename Reducer<S, OP>::A;
        constexpr int VF = 16 / (int)sizeof(storage_t<S>) > 0 ? 16 / (int)sizeof(storage_t<S>) : 1;
        if constexpr (cols_bits<S, OP>()) {   // (a lane's last vector ends with the last column: sixteen of them at least)
          if (p.vec > 1 && p.ksize[p.nkept - 1] >= VF) {
            hipLaunchKernelGGL((red_cols_bits_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), (size_t)p.block * 16, stream, args);
            break;
          }
        }
        const size_t lds = cols_lds_bytes<A>((int)p.block, p.vec > 1 ? VF : 1);
        if constexpr (VF > 1 && VF <= 8) {
          if (p.flat_cols) {
            hipLaunchKernelGGL((red_cols_flat_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), lds, stream, args);
            break;
          }
        }
        if (p.cpw == 0) hipLaunchKernelGGL((red_cols_lane_kernel<S, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
        else hipLaunchKernelGGL((red_cols_kernel<S, OP>), dim3((unsigned)p.grid), dim3((unsigned)p.block), lds, stream, args);
      }
      break;
    default:
      hipLaunchKernelGGL((red_generic_kernel<S, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
      break;
  }
  return hipGetLastError();
}
#endif

}  // namespace ocn
