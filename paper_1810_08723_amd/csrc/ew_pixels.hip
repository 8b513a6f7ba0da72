// Copies between planes and interleaved pixels of two to four channels, converting the samples
// (section 3.2.1 of the paper: a type cast fused into the copy), at any alignment and for any
// number of pixels:
//   to planes   out[c][m] = convert(in[m][c])  - images as they are stored, to channel-first
//   to pixels   out[m][c] = convert(in[c][m])
// Sorting and merging axes (section 4) leaves both with a dimension of C elements whose neighbours
// lie side by side on one side and a plane apart on the other; a tile through LDS would spend
// most of its time on that short axis, and reading it in place takes an access per sample.
//
// A lane takes V = 16 / (output element) consecutive pixels and deals their V * C samples out in
// registers.  To planes, it reads V * C consecutive samples and writes 16 bytes to each plane,
// neighbouring lanes side by side on both sides.  To pixels, it reads V samples of each plane and
// parks its 16 * C bytes in LDS, from where the wavefront stores runs of 64 consecutive 16-byte
// pieces, as ew_interleave_kernel does.  The last vector of a row ends with the row and overlaps
// the one before it: the same values are written twice.  uint8 pixels [32, 480, 640, 3] to float
// planes: 33.6 us with an access per sample, 21.8 here (6.8 TB/s); uint8 planes to float pixels: 92
// and 21.8; float pixels to planes: 67 and 40 (7.3 TB/s).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>

#include "ew_launch.hpp"

namespace ocn {
namespace {

struct PixelArgs {
  char *out;
  const char *a;
  int64_t plane;                        // bytes between planes, on the side that has them
  uint32_t nvec, m;                     // vectors in total; pixels per row
  FastDiv mvec_div;                     // vectors per row
  int32_t nouter;
  int32_t nt_store;
  FastDiv odiv[kMaxDims];               // outer dims, fastest first
  int64_t so[kMaxDims], sa[kMaxDims];
};

// a copy of elements of ES bytes made of scalars of AL bytes, whatever their type (but bool);
// AL: operands are aligned to their scalars only
template <int ES, int AL_ = ES> struct CopyOf {
  struct alignas(ES) Elem { unsigned char b[ES]; };
  using In = Elem;
  using Out = Elem;
  static constexpr int AL = AL_, ALO = AL_;
  OCN_DEV static Out cv(const In &x) { return x; }
  template <int N> OCN_DEV static void loaded(unsigned char (&)[N]) {}
};
// a copy of bools: whatever byte stands for true, 1 is written (four at a time, as they are loaded)
struct CopyOfBool : CopyOf<1> {
  template <int N> OCN_DEV static void loaded(unsigned char (&b)[N]) {
    static_assert(N % 4 == 0, "whole words");
#pragma unroll
    for (int i = 0; i < N; i += 4) {
      uint32_t w;
      __builtin_memcpy(&w, b + i, 4);
      w = bool_bytes(w);
      __builtin_memcpy(b + i, &w, 4);
    }
  }
};
template <int SA, int SO> struct CastOf {
  using In = storage_t<SA>;
  using Out = storage_t<SO>;
  static constexpr int AL = (int)sizeof(In), ALO = (int)sizeof(Out);
  OCN_DEV static Out cv(const In &x) { return to_storage<SO>(convert<SO>(from_storage<SA>(x))); }
  template <int N> OCN_DEV static void loaded(unsigned char (&)[N]) {}
};

// N consecutive bytes at an address that is a multiple of AL
template <int N, int AL> OCN_DEV void load_bytes(const char *src, unsigned char *dst) {
  using X = Unaligned<AL>;
  constexpr int n16 = N / 16 * 16, n8 = n16 + (N - n16) / 8 * 8, n4 = n8 + (N - n8) / 4 * 4, n2 = n4 + (N - n4) / 2 * 2;
#pragma unroll
  for (int i = 0; i < n16; i += 16) {
    const typename X::W4 w = *reinterpret_cast<const typename X::W4 *>(src + i);
    __builtin_memcpy(dst + i, &w, 16);
  }
  if constexpr (n8 > n16) {
    const typename X::W2 w = *reinterpret_cast<const typename X::W2 *>(src + n16);
    __builtin_memcpy(dst + n16, &w, 8);
  }
  if constexpr (n4 > n8) {
    const uint32_t w = *reinterpret_cast<const typename X::W1 *>(src + n8);
    __builtin_memcpy(dst + n8, &w, 4);
  }
  if constexpr (n2 > n4) {
    const uint16_t w = *reinterpret_cast<const typename X::H1 *>(src + n4);
    __builtin_memcpy(dst + n4, &w, 2);
  }
  if constexpr (N > n2) dst[n2] = *reinterpret_cast<const unsigned char *>(src + n2);
}

template <int AL> OCN_DEV void store16(char *dst, const void *v, bool nt) {
  using W4 = typename Unaligned<AL>::W4;
  W4 w;
  __builtin_memcpy(&w, v, 16);
  if (nt) {
    OCN_KEEP_BRANCH();
    __builtin_nontemporal_store(w, reinterpret_cast<W4 *>(dst));
    OCN_KEEP_BRANCH();
  } else {
    *reinterpret_cast<W4 *>(dst) = w;
  }
}

using KPixelArgs = const __attribute__((address_space(4))) PixelArgs;

// byte offsets of vector g: its row on both sides, and its first pixel
template <int V> OCN_DEV uint32_t pixel_place(KPixelArgs &p, uint32_t g, int64_t &off_o, int64_t &off_a) {
  const uint32_t d = p.mvec_div.d;
  uint32_t row = fastdiv(g, FastDiv{d, p.mvec_div.m, p.mvec_div.s});
  const uint32_t e = (g - row * d) * (uint32_t)V;
  off_o = off_a = 0;
  const int nouter = p.nouter;
  for (int k = 0; k < nouter; ++k) {
    const uint32_t od = p.odiv[k].d;
    const uint32_t q = k + 1 < nouter ? fastdiv(row, FastDiv{od, p.odiv[k].m, p.odiv[k].s}) : 0u;
    const int64_t i = (int64_t)(row - q * od);
    row = q;
    off_o += i * p.so[k];
    off_a += i * p.sa[k];
  }
  return e + (uint32_t)V <= p.m ? e : p.m - (uint32_t)V;
}

template <class F, int C> __global__ __launch_bounds__(kBlock) void to_planes_kernel(const PixelArgs by_value) {
  using In = typename F::In;
  using Out = typename F::Out;
  constexpr int V = 16 / (int)sizeof(Out);
  (void)by_value;
  KPixelArgs &p = *(KPixelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t g = blockIdx.x * (uint32_t)kBlock + threadIdx.x;
  if (g >= p.nvec) return;
  int64_t off_o, off_a;
  const uint32_t e = pixel_place<V>(p, g, off_o, off_a);
  union { unsigned char b[V * C * sizeof(In)]; In v[V * C]; } in;
  load_bytes<V * C * (int)sizeof(In), F::AL>(p.a + off_a + (int64_t)e * (C * (int)sizeof(In)), in.b);
  F::loaded(in.b);
  char *out = p.out + off_o + (int64_t)e * (int)sizeof(Out);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    Out o[V];
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = F::cv(in.v[i * C + c]);
    store16<F::ALO>(out + (int64_t)c * p.plane, o, p.nt_store != 0);
  }
}

template <class F, int C> __global__ __launch_bounds__(kBlock) void to_pixels_kernel(const PixelArgs by_value) {
  using In = typename F::In;
  using Out = typename F::Out;
  using Q = uint32_t __attribute__((ext_vector_type(4)));
  constexpr int V = 16 / (int)sizeof(Out);
  __shared__ Q parked[kBlock * C];
  (void)by_value;
  KPixelArgs &p = *(KPixelArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  const uint32_t tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const uint32_t g = blockIdx.x * (uint32_t)kBlock + tid;
  const bool valid = g < p.nvec;
  int64_t off_o = 0;
  if (valid) {
    int64_t off_a;
    const uint32_t e = pixel_place<V>(p, g, off_o, off_a);
    off_o += (int64_t)e * (16 * C / V);
    union { unsigned char b[V * sizeof(In)]; In v[V]; } in[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      load_bytes<V * (int)sizeof(In), F::AL>(p.a + off_a + (int64_t)c * p.plane + (int64_t)e * (int)sizeof(In), in[c].b);
      F::loaded(in[c].b);
    }
    Out o[V * C];
#pragma unroll
    for (int i = 0; i < V * C; ++i) o[i] = F::cv(in[i % C].v[i / C]);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      Q q;
      __builtin_memcpy(&q, reinterpret_cast<const char *>(o) + 16 * c, 16);
      parked[(wave * kWave + lane) * C + c] = q;
    }
  }
  __syncthreads();
  // piece k * 64 + lane of the wavefront's 64 * C pieces belongs to source lane (piece / C)
#pragma unroll
  for (int k = 0; k < C; ++k) {
    const uint32_t piece = (uint32_t)k * kWave + lane;
    const uint32_t from = piece / C, part = piece - from * C;
    const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)off_o, (int)from, kWave);
    const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)((uint64_t)off_o >> 32), (int)from, kWave);
    const int ok = __shfl(valid ? 1 : 0, (int)from, kWave);
    if (ok) {
      const Q q = parked[wave * kWave * C + piece];
      store16<F::ALO>(p.out + (int64_t)(((uint64_t)hi << 32) | lo) + (int64_t)part * 16, &q,
                                                       p.nt_store != 0);
    }
  }
}

template <class F> hipError_t launch_form(const PixelArgs &a, int c, bool to_planes, hipStream_t s) {
  const dim3 grid((unsigned)((a.nvec + kBlock - 1) / kBlock)), block(kBlock);
  switch (c) {
#define OCN_CASE(CC)                                                                            \
  case CC:                                                                                      \
    if (to_planes) hipLaunchKernelGGL((to_planes_kernel<F, CC>), grid, block, 0, s, a);         \
    else hipLaunchKernelGGL((to_pixels_kernel<F, CC>), grid, block, 0, s, a);                   \
    break;
    OCN_CASE(2) OCN_CASE(3) OCN_CASE(4)
#undef OCN_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// the planner's dims: [outer ..., C, M] to planes, [outer ..., M, C] to pixels
hipError_t launch_pixels(const EwPlan &p, hipStream_t stream) {
  const int n = p.ndim;
  const bool to_planes = p.kernel == kKernelToPlanes;
  const int dc = to_planes ? n - 2 : n - 1, dm = to_planes ? n - 1 : n - 2;
  PixelArgs a;
  std::memset(&a, 0, sizeof a);
  a.out = p.out.ptr;
  a.a = p.a.ptr;
  a.plane = to_planes ? p.out.stride[dc] : p.a.stride[dc];
  a.m = (uint32_t)p.size[dm];
  const int64_t mvec = (p.size[dm] + p.vec - 1) / p.vec;
  a.mvec_div = make_fastdiv((uint32_t)mvec);
  a.nouter = n - 2;
  int64_t rows = 1;
  for (int k = 0; k < n - 2; ++k) {   // fastest outer dim first
    const int d = n - 3 - k;
    a.odiv[k] = make_fastdiv((uint32_t)p.size[d]);
    a.so[k] = p.out.stride[d];
    a.sa[k] = p.a.stride[d];
    rows *= p.size[d];
  }
  a.nvec = (uint32_t)(rows * mvec);
  a.nt_store = p.nt_store;
  const int c = (int)p.size[dc];
  if (p.a.dtype == DT_BOOL && p.out.dtype == DT_BOOL) return launch_form<CopyOfBool>(a, c, to_planes, stream);
  if (p.a.dtype == p.out.dtype) {
    switch (dt_size(p.out.dtype)) {
      case 1: return launch_form<CopyOf<1>>(a, c, to_planes, stream);
      case 2: return launch_form<CopyOf<2>>(a, c, to_planes, stream);
      case 4:
        if (p.out.dtype == DT_C16) return launch_form<CopyOf<4, 2>>(a, c, to_planes, stream);
        return launch_form<CopyOf<4>>(a, c, to_planes, stream);
      case 8:
        if (p.out.dtype == DT_C32) return launch_form<CopyOf<8, 4>>(a, c, to_planes, stream);
        return launch_form<CopyOf<8>>(a, c, to_planes, stream);
      default: return hipErrorInvalidValue;
    }
  }
#define OCN_CAST(SA, SO) \
  if (p.a.dtype == SA && p.out.dtype == SO) return launch_form<CastOf<SA, SO>>(a, c, to_planes, stream);
#define OCN_FROM(SA)                                                                                             \
  if constexpr (SA != DT_U8) { OCN_CAST(SA, DT_U8) }                                                             \
  if constexpr (SA != DT_U16) { OCN_CAST(SA, DT_U16) }                                                           \
  if constexpr (SA != DT_I16) { OCN_CAST(SA, DT_I16) }                                                           \
  if constexpr (SA != DT_F16) { OCN_CAST(SA, DT_F16) }                                                           \
  if constexpr (SA != DT_F32) { OCN_CAST(SA, DT_F32) }
  OCN_FROM(DT_U8) OCN_FROM(DT_U16) OCN_FROM(DT_I16) OCN_FROM(DT_F16) OCN_FROM(DT_F32)
#undef OCN_FROM
#undef OCN_CAST
  return hipErrorInvalidValue;
}

}  // namespace ocn
