// Instantiation of the slab kernels for one activation type (SLAB_BF16) and frame kind (SLAB_RADIX:
// blocks applied directly, or in one radix-4 stage); the build compiles this file once for each.
#include "slab_kernels.h"

#if !defined(SLAB_BF16) || !defined(SLAB_RADIX)
#error "compile with -DSLAB_BF16=0|1 -DSLAB_RADIX=0|1"
#endif

namespace ff {
namespace slab {
namespace {

constexpr bool kBf = SLAB_BF16 != 0, kRad = SLAB_RADIX != 0;

// Contraction steps of a frame's MFMA matrix (up to 128 wide).
inline int steps_of(const FrameDev& f) { return kBf ? f.KT : f.KT4; }

#define SLAB_CASES(X)                                      \
  switch (steps_of(a.f)) {                                 \
    case 1: X(1); break;                                   \
    case 2: X(2); break;                                   \
    case 3: X(3); break;                                   \
    case 4: X(4); break;                                   \
    default: return hipErrorInvalidValue;                  \
  }

hipError_t analysis(const AnaArgs& a, dim3 grid, size_t lds, hipStream_t s) {
#define X(kt) hipLaunchKernelGGL((slab_analysis<kBf, kt, kRad>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

hipError_t fwd(const SlabArgs& a, dim3 grid, size_t lds, hipStream_t s) {
  const bool beta = a.beta != 0.f;
#define X(kt)                                                                                     \
  if (beta)                                                                                       \
    hipLaunchKernelGGL((slab_fwd<kBf, kt, kRad, true>), grid, dim3(kSlabThreads), lds, s, a);      \
  else                                                                                            \
    hipLaunchKernelGGL((slab_fwd<kBf, kt, kRad, false>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

hipError_t bwd(const SlabArgs& a, bool dx, bool dc, dim3 grid, size_t lds, hipStream_t s) {
  const bool beta = a.beta != 0.f;
#define X(kt)                                                                                              \
  if (dx && dc && beta)                                                                                    \
    hipLaunchKernelGGL((slab_bwd<kBf, kt, kRad, true, true, true>), grid, dim3(kSlabThreads), lds, s, a);   \
  else if (dx && dc)                                                                                       \
    hipLaunchKernelGGL((slab_bwd<kBf, kt, kRad, true, true, false>), grid, dim3(kSlabThreads), lds, s, a);  \
  else if (dx && beta)                                                                                     \
    hipLaunchKernelGGL((slab_bwd<kBf, kt, kRad, true, false, true>), grid, dim3(kSlabThreads), lds, s, a);  \
  else if (dx)                                                                                             \
    hipLaunchKernelGGL((slab_bwd<kBf, kt, kRad, true, false, false>), grid, dim3(kSlabThreads), lds, s, a); \
  else                                                                                                     \
    hipLaunchKernelGGL((slab_bwd<kBf, kt, kRad, false, true, false>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

template <int KT>
hipError_t allow() {
  hipError_t e = hipSuccess;
  for (const void* fn : {reinterpret_cast<const void*>(&slab_analysis<kBf, KT, kRad>),
                         reinterpret_cast<const void*>(&slab_fwd<kBf, KT, kRad, false>),
                         reinterpret_cast<const void*>(&slab_fwd<kBf, KT, kRad, true>),
                         reinterpret_cast<const void*>(&slab_bwd<kBf, KT, kRad, true, true, false>),
                         reinterpret_cast<const void*>(&slab_bwd<kBf, KT, kRad, true, true, true>),
                         reinterpret_cast<const void*>(&slab_bwd<kBf, KT, kRad, true, false, false>),
                         reinterpret_cast<const void*>(&slab_bwd<kBf, KT, kRad, true, false, true>),
                         reinterpret_cast<const void*>(&slab_bwd<kBf, KT, kRad, false, true, false>)}) {
    const hipError_t r = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (r != hipSuccess) e = r;
  }
  return e;
}

hipError_t configure() {
  hipError_t e = hipSuccess;
  for (const hipError_t r : {allow<1>(), allow<2>(), allow<3>(), allow<4>()})
    if (r != hipSuccess) e = r;
  return e;
}

}  // namespace

#if SLAB_BF16 && SLAB_RADIX
#define SLAB_NAME launch_bf16_radix
#elif SLAB_BF16
#define SLAB_NAME launch_bf16_direct
#endif
const SlabLaunch& SLAB_NAME() {
  static const SlabLaunch table = {analysis, fwd, bwd, configure};
  return table;
}

}  // namespace slab
}  // namespace ff
