// Host side of the elementwise kernels: turns a plan into kernel arguments and launches.
#pragma once

#include <hip/hip_runtime.h>

#include "ew_kernels.hpp"

namespace ocn {

using EwLauncher = hipError_t (*)(const EwPlan &, hipStream_t);

// dispatch tables, filled once by the kernel translation units (see ew_register.cpp)
extern EwLauncher g_binary_launchers[B_COUNT][DT_COUNT][DT_COUNT][DT_COUNT];
extern EwLauncher g_unary_launchers[U_COUNT][DT_COUNT][DT_COUNT];

// arguments and grid of the kernel for rows of any length and alignment
RowsArgs make_rows_args(const EwPlan &p, int64_t *grid);
// arguments of the kernel for the common row shapes; false if the plan is not one of them
bool make_rows_slim_args(const EwPlan &p, int block, RowsSlimArgs *args, int64_t *grid);
// workgroups and lanes per workgroup that the plan goes out with (plan inspection)
void ew_launch_shape(const EwPlan &p, int64_t *grid, int64_t *block);
TiledArgs make_tiled_args(const EwPlan &p, int es_a);
FastTiledArgs make_fast_tiled_args(const EwPlan &p, int es_a);
AnyTiledArgs make_any_tiled_args(const EwPlan &p, int es_a);
BoxArgs make_box_args(const EwPlan &p);
InterpArgs make_interp_args(const EwPlan &p);
hipError_t launch_interp(const EwPlan &p, hipStream_t stream);
hipError_t launch_interleave(const EwPlan &p, hipStream_t stream);
hipError_t launch_pixels(const EwPlan &p, hipStream_t stream);

// Are there vectors of an input that go on into the next row, and are they taken in two whole pieces?  With two inputs of
// bytes not where rows are long and the output is large: vectors that cross are too few then for what the pieces cost all
// others (sums of int8 [54396, 1520] with reversed rows 43.1 us without them and 49.0 with; 28 calls 0.96 times as fast with
// them, rows of 16 to 1023 elements 1.2, longer ones below 8 million elements 1.1).
inline bool rows_in_pieces(const RowsArgs &p, int vec, bool two_of_bytes) {
  if (!(p.flags & kRowsFlat) || !p.nouter || p.inner < (uint32_t)vec) return false;
  if ((p.flags & kRowsALinear) && (p.flags & kRowsBLinear)) return false;
  return !two_of_bytes || p.inner < 64u * (uint32_t)vec || p.numel < ((int64_t)8 << 20);
}

#if defined(__HIPCC__)
template <int OP, int SA, int SB, int SO, int NIN>
hipError_t launch_ew(const EwPlan &p, hipStream_t stream) {
  using G = Sig<OP, SA, SB, SO, NIN>;
  if (p.kernel == OCN_KERNEL_EW_ROWS) {
    RowsSlimArgs slim;
    int64_t slim_grid;
    if (make_rows_slim_args(p, kSlimBlock, &slim, &slim_grid)) {
      hipLaunchKernelGGL((ew_rows_slim_kernel<G>), dim3((unsigned)slim_grid), dim3(kSlimBlock), 0, stream, slim);
    } else {
      const RowsArgs args = make_rows_args(p, &slim_grid);
      if constexpr (G::UR == 1) {   // (several vectors per lane: never in pieces)
        if (rows_in_pieces(args, G::VR, G::NIN2 && G::VR == 16)) {
          hipLaunchKernelGGL((ew_rows_kernel<G, true>), dim3((unsigned)slim_grid), dim3(args.block), 0, stream, args);
          return hipGetLastError();
        }
      }
      hipLaunchKernelGGL((ew_rows_kernel<G, false>), dim3((unsigned)slim_grid), dim3(args.block), 0, stream, args);
    }
  } else if (p.kernel == kKernelTiledAny) {
    const AnyTiledArgs args = make_any_tiled_args(p, (int)sizeof(typename G::SAt));
    hipLaunchKernelGGL((ew_tiled_any_kernel<G>), dim3((unsigned)p.grid), dim3(args.block), (size_t)p.lds_bytes, stream, args);
  } else if (p.kernel == kKernelBox) {
    const BoxArgs args = make_box_args(p);
    hipLaunchKernelGGL((ew_box_kernel<G>), dim3((unsigned)p.grid), dim3(args.block), (size_t)p.lds_bytes, stream, args);
  } else if (p.fast_tiled) {
    const FastTiledArgs args = make_fast_tiled_args(p, (int)sizeof(typename G::SAt));
    hipLaunchKernelGGL((ew_tiled_fast_kernel<G>), dim3((unsigned)p.grid), dim3(kBlock), (size_t)p.lds_bytes, stream, args);
  } else {
    const TiledArgs args = make_tiled_args(p, (int)sizeof(typename G::SAt));
    hipLaunchKernelGGL((ew_tiled_kernel<G>), dim3((unsigned)p.grid), dim3(kBlock), (size_t)p.lds_bytes, stream, args);
  }
  return hipGetLastError();
}
#endif

}  // namespace ocn
