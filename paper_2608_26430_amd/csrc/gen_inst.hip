// Instantiation of one generic kernel (fwd_kernel or bwd_kernel, GEN_BWD) for one activation type
// (GEN_BF16), and for frames applied in several radix-4 stages or the others (GEN_MS): the build
// compiles this file once per combination in use, in parallel.  bf16 calls that come here are short
// (the slab kernels take the others) and have one chunk of input blocks.  Forwards run on token-grouped
// tiles where the frames allow them; the instantiation for several stages serves the rest.
#include "gen_kernels.h"

#if !defined(GEN_BWD) || !defined(GEN_BF16) || !defined(GEN_MS)
#error "compile with -DGEN_BWD=0|1 -DGEN_BF16=0|1 -DGEN_MS=0|1"
#endif

namespace ff {
namespace gen {

#if GEN_BWD
#define GEN_KERNEL bwd_kernel
#define GEN_ARGS BwdArgs
#if GEN_BF16
#define GEN_LAUNCH launch_bwd_bf16
#define GEN_CONFIGURE configure_bwd_bf16
#else
#define GEN_LAUNCH launch_bwd_f32
#define GEN_CONFIGURE configure_bwd_f32
#endif
#else
#define GEN_KERNEL fwd_kernel
#define GEN_ARGS FwdArgs
#if GEN_BF16
#define GEN_LAUNCH launch_fwd_bf16
#define GEN_CONFIGURE configure_fwd_bf16
#else
#define GEN_LAUNCH launch_fwd_f32
#define GEN_CONFIGURE configure_fwd_f32
#endif
#endif
#define GEN_CAT2(a, b) a##b
#define GEN_CAT(a, b) GEN_CAT2(a, b)
#define GEN_LAUNCH_MS GEN_CAT(GEN_LAUNCH, _ms)
#define GEN_CONFIGURE_MS GEN_CAT(GEN_CONFIGURE, _ms)

// The instantiation for frames applied in several radix-4 stages (GEN_MS=1, its own compile unit:
// one block per frame side there, so never input-side chunks), and the other two (GEN_MS=0).
hipError_t GEN_LAUNCH_MS(const GEN_ARGS& a, dim3 grid, size_t lds, hipStream_t s);
hipError_t GEN_CONFIGURE_MS();

#if GEN_BF16 && GEN_BWD
hipError_t GEN_LAUNCH(const GEN_ARGS& a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.nch > 1) return hipErrorInvalidValue;   // (not reached: the dispatch sends chunked calls to the slab kernels)
  return GEN_LAUNCH_MS(a, grid, lds, s);
}
hipError_t GEN_CONFIGURE() { return GEN_CONFIGURE_MS(); }
#endif

#if GEN_BF16 && !GEN_BWD && !GEN_MS
hipError_t GEN_LAUNCH(const GEN_ARGS& a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.nch > 1) return hipErrorInvalidValue;   // (not reached, as above)
  if (!a.g4) return GEN_LAUNCH_MS(a, grid, lds, s);
  hipLaunchKernelGGL((GEN_KERNEL<true, false, false, true>), grid, dim3(kFusedThreads), lds, s, a);
  return hipGetLastError();
}
hipError_t GEN_CONFIGURE() {
  const hipError_t e = GEN_CONFIGURE_MS();
  const hipError_t r = hipFuncSetAttribute(reinterpret_cast<const void*>(&GEN_KERNEL<true, false, false, true>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
  return r != hipSuccess ? r : e;
}
#elif GEN_MS
hipError_t GEN_LAUNCH_MS(const GEN_ARGS& a, dim3 grid, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL((GEN_KERNEL<GEN_BF16 != 0, false, true>), grid, dim3(kFusedThreads), lds, s, a);
  return hipGetLastError();
}

hipError_t GEN_CONFIGURE_MS() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&GEN_KERNEL<GEN_BF16 != 0, false, true>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
}
#else
hipError_t GEN_LAUNCH(const GEN_ARGS& a, dim3 grid, size_t lds, hipStream_t s) {
  if (a.fin.nst >= 2 || a.fout.nst >= 2) return GEN_LAUNCH_MS(a, grid, lds, s);
  if (a.nch > 1)
    hipLaunchKernelGGL((GEN_KERNEL<false, true>), grid, dim3(kFusedThreads), lds, s, a);
  else
    hipLaunchKernelGGL((GEN_KERNEL<false, false>), grid, dim3(kFusedThreads), lds, s, a);
  return hipGetLastError();
}

hipError_t GEN_CONFIGURE() {
  hipError_t e = GEN_CONFIGURE_MS();
  for (const void* fn : {reinterpret_cast<const void*>(&GEN_KERNEL<false, true>),
                         reinterpret_cast<const void*>(&GEN_KERNEL<false, false>)}) {
    const hipError_t r = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
    if (r != hipSuccess) e = r;
  }
  return e;
}
#endif

}  // namespace gen
}  // namespace ff
