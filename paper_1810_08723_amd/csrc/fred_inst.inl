// Instantiates one slice of the fused elementwise+reduce kernels and registers their
// launchers.  Included by fred_slice_*.hip with OCN_SLICE and OCN_NSLICES defined.
#include <type_traits>
#include <utility>

#include "fred_kernels.hpp"
#include "red_launch.hpp"

namespace ocn {
namespace {

template <class G, int OP> hipError_t launch_fred(const RedPlan &p, char *partial, hipStream_t stream) {
  if (p.strip) {
    const RedStripArgs args = make_red_strip_args(p, partial);
    const dim3 grid((unsigned)p.grid), block((unsigned)p.block);
    auto go = [&](auto bc) {
      constexpr int BC = decltype(bc)::value;
      using A = typename FusedFold<G, OP>::A;
      const size_t lds = p.strip == 1 ? strip_cols_lds<A>((int)p.block, (int)sizeof(typename G::SAt)) : p.strip_lds;
      if (p.strip == 1) hipLaunchKernelGGL((fred_strip_cols_kernel<G, OP, BC>), grid, block, lds, stream, args);
      else hipLaunchKernelGGL((fred_strip_rows_kernel<G, OP, BC>), grid, block, lds, stream, args);
    };
    if (p.strip_bc == 0) go(std::integral_constant<int, 0>{});
    else if (p.strip_bc == 1) go(std::integral_constant<int, 1>{});
    else go(std::integral_constant<int, 2>{});
    return hipGetLastError();
  }
  const RedArgs args = make_red_args(p, partial);
  switch (p.kernel) {
    case OCN_KERNEL_RED_ROWS:
      if (p.lean) {
        hipLaunchKernelGGL((fred_rows_lean_kernel<G, OP>), dim3((unsigned)p.grid), dim3(lean_block(p)), 0, stream,
                           make_red_lean_args(p, partial));
        break;
      }
      if (p.short_rows) {
        hipLaunchKernelGGL((fred_rows_short_kernel<G, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
        break;
      }
      hipLaunchKernelGGL((fred_rows_kernel<G, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
      break;
    case OCN_KERNEL_RED_COLS:
      {
        using A = typename FusedFold<G, OP>::A;
        const size_t lds = cols_lds_bytes<A>((int)p.block, p.vec > 1 ? G::V : 1);
        const dim3 grid((unsigned)p.grid), block((unsigned)p.block);
        auto form = [&](auto bc, auto nt) {
          constexpr int BC = fred_cols_form<G, decltype(bc)::value>() ? decltype(bc)::value : -1;
          hipLaunchKernelGGL((fred_cols_kernel<G, OP, BC, BC == 0 && decltype(nt)::value>), grid, block, lds, stream, args);
        };
        using std::integral_constant;
        if (p.vec != G::V || p.nred != 1) form(integral_constant<int, -1>{}, std::false_type{});
        else if (args.b_bcast) form(integral_constant<int, 2>{}, std::false_type{});
        else if (args.a_bcast) form(integral_constant<int, 1>{}, std::false_type{});
        else if (args.nt_load) form(integral_constant<int, 0>{}, std::true_type{});
        else form(integral_constant<int, 0>{}, std::false_type{});
      }
      break;
    default:
      hipLaunchKernelGGL((fred_generic_kernel<G, OP>), dim3((unsigned)p.grid), dim3(kBlock), 0, stream, args);
      break;
  }
  return hipGetLastError();
}

// index I enumerates (elementwise op, input dtype, reduce op)
template <int I> void register_fused() {
  constexpr int ew = I / (DT_COUNT * R_COUNT), t = (I / R_COUNT) % DT_COUNT, r = I % R_COUNT;
  constexpr int mid = is_compare(ew) ? (int)DT_BOOL : t;
  if constexpr (fused_specialised(ew, t, t, mid, r)) {
    // deal the instantiated signatures (not the sparse index space) round-robin to the slices
    constexpr int ord = ew * 7 + t + r;
    if constexpr (ord % OCN_NSLICES == OCN_SLICE)
      g_fused_launchers[ew][t][r] = &launch_fred<Sig<ew, t, t, mid, 2>, r>;
  }
}
template <int... I> void register_all_fused(std::integer_sequence<int, I...>) { (register_fused<I>(), ...); }

}  // namespace

#define OCN_CAT2(a, b) a##b
#define OCN_CAT(a, b) OCN_CAT2(a, b)
void OCN_CAT(register_fred_slice_, OCN_SLICE)() {
  register_all_fused(std::make_integer_sequence<int, B_COUNT * DT_COUNT * R_COUNT>{});
}

}  // namespace ocn
