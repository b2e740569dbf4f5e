// Instantiation of the slab kernels for one frame kind (SLAB_RADIX: blocks applied directly, or in one
// radix-4 stage); the build compiles this file once for each.
#include "slab_kernels.h"

#ifndef SLAB_RADIX
#error "compile with -DSLAB_RADIX=0|1"
#endif

namespace ff {
namespace slab {
namespace {

constexpr bool kRad = SLAB_RADIX != 0;

// Contraction steps of a frame's MFMA matrix (up to 128 wide).
inline int steps_of(const FrameDev& f) { return f.KT; }

#define SLAB_CASES(X)                                      \
  switch (steps_of(a.f)) {                                 \
    case 1: X(1); break;                                   \
    case 2: X(2); break;                                   \
    case 3: X(3); break;                                   \
    case 4: X(4); break;                                   \
    default: return hipErrorInvalidValue;                  \
  }

hipError_t analysis(const AnaArgs& a, dim3 grid, size_t lds, hipStream_t s) {
#define X(kt) hipLaunchKernelGGL((slab_analysis<kt, kRad>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

hipError_t fwd(const SlabArgs& a, dim3 grid, size_t lds, hipStream_t s) {
  const bool beta = a.beta != 0.f;
#define X(kt)                                                                                     \
  if (beta)                                                                                       \
    hipLaunchKernelGGL((slab_fwd<kt, kRad, true>), grid, dim3(kSlabThreads), lds, s, a);      \
  else                                                                                            \
    hipLaunchKernelGGL((slab_fwd<kt, kRad, false>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

hipError_t bwd(const SlabArgs& a, bool dx, bool dc, dim3 grid, size_t lds, hipStream_t s) {
  const bool beta = a.beta != 0.f;
#define X(kt)                                                                                              \
  if (dx && dc && beta)                                                                                    \
    hipLaunchKernelGGL((slab_bwd<kt, kRad, true, true, true>), grid, dim3(kSlabThreads), lds, s, a);   \
  else if (dx && dc)                                                                                       \
    hipLaunchKernelGGL((slab_bwd<kt, kRad, true, true, false>), grid, dim3(kSlabThreads), lds, s, a);  \
  else if (dx && beta)                                                                                     \
    hipLaunchKernelGGL((slab_bwd<kt, kRad, true, false, true>), grid, dim3(kSlabThreads), lds, s, a);  \
  else if (dx)                                                                                             \
    hipLaunchKernelGGL((slab_bwd<kt, kRad, true, false, false>), grid, dim3(kSlabThreads), lds, s, a); \
  else                                                                                                     \
    hipLaunchKernelGGL((slab_bwd<kt, kRad, false, true, false>), grid, dim3(kSlabThreads), lds, s, a)
  SLAB_CASES(X)
#undef X
  return hipGetLastError();
}

template <int KT>
hipError_t allow() {
  hipError_t e = hipSuccess;
  for (const void* fn : {reinterpret_cast<const void*>(&slab_analysis<KT, kRad>),
                         reinterpret_cast<const void*>(&slab_fwd<KT, kRad, false>),
                         reinterpret_cast<const void*>(&slab_fwd<KT, kRad, true>),
                         reinterpret_cast<const void*>(&slab_bwd<KT, kRad, true, true, false>),
                         reinterpret_cast<const void*>(&slab_bwd<KT, kRad, true, true, true>),
                         reinterpret_cast<const void*>(&slab_bwd<KT, kRad, true, false, false>),
                         reinterpret_cast<const void*>(&slab_bwd<KT, kRad, true, false, true>),
                         reinterpret_cast<const void*>(&slab_bwd<KT, kRad, false, true, false>)}) {
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

#if SLAB_RADIX
#define SLAB_NAME launch_radix
#else
#define SLAB_NAME launch_direct
#endif
const SlabLaunch& SLAB_NAME() {
  static const SlabLaunch table = {analysis, fwd, bwd, configure};
  return table;
}

}  // namespace slab
}  // namespace ff
