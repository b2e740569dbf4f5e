// Host side of the slab kernels (slab_kernels.h): how a call is split over the workspace, and the
// launches of its two passes.
#include <algorithm>

#include "slab_kernels.h"

namespace ff {
namespace {

using namespace slab;

const SlabLaunch& kernels_for(const FrameDev& f) { return f.radix == 1 ? launch_direct() : launch_radix(); }

unsigned pad8(long n) { return (unsigned)((n + 7) / 8 * 8); }

void record(hipEvent_t ev, hipStream_t s) {
  if (ev) (void)hipEventRecord(ev, s);
}

// One side's tensors and the workspace of a pass, for the adapters and slabs of one launch.
struct Side {
  const FrameDev* f;
  ActPtrs A;
  int64_t ld;
};

// LDS of a workgroup: the tile of a group (and a spare row for lanes without one), then for directly
// applied blocks the stage; factored ones' windows and stage take the tile's place.
struct Lds {
  int stage;
  size_t bytes;
};
Lds lds_layout(const FrameDev& f, int nb) {
  const int rows = nb * f.W, S = Slab::S, vl = Slab::TC, cb = rows / vl;
  const int tile = (rows + 1) * kTileRow, stage = S * (cb | 1) * 16;
  if (f.radix == 1) return {tile, (size_t)(tile + stage)};
  const int windows = S * (4 * ((f.W2 + vl - 1) / vl) | 1) * 16;
  return {0, (size_t)std::max({tile, stage, windows})};
}

// dC partial rows of a call: slabs are taken sg at a time so that at most `rows` rows are needed.
void partial_rows(int T, int S, int rows, int* sg, int* nrows) {
  const int nslab = (T + S - 1) / S;
  *sg = std::max(1, (nslab + rows - 1) / rows);
  *nrows = (nslab + *sg - 1) / *sg;
}

// First pass over `count` adapters: slabs slab0 .. slab0 + nslab - 1 of `side`; `entries` on the
// launch that also writes the destination stream's entries.
hipError_t launch_analysis(const Side& side, const SlabStream& st, int count, int a0, int T, int slab0, int nslab,
                           unsigned char* ws, long ws_adapter, uint2* ent, long ent_adapter, bool entries,
                           const float* c, const float* const* cs, const SlabDesc* group, const int* tokens, int bwd,
                           int max_ent, hipStream_t s) {
  const FrameDev& f = *side.f;
  const bool ms = slab_ms_frame(f);
  const int threads = ms ? kMsThreads : kSlabThreads;
  AnaArgs a{};
  a.f = f;
  a.frag = f.wa16;
  a.T = T;
  a.slab0 = slab0;
  a.nslab = nslab;
  a.X = side.A.one;
  a.Xs = side.A.many ? side.A.many + a0 : nullptr;
  a.ld = (long)side.ld;
  a.ws = ws;
  a.ws_adapter = ws_adapter;
  a.word = st.word;
  a.coef = st.coef;
  a.nent = entries ? (group ? max_ent : 16 * (st.steps + kSlabPadSteps)) : 0;
  a.c = c;
  a.cs = cs ? cs + a0 : nullptr;
  a.ent = ent;
  a.ent_adapter = ent_adapter;
  a.group = group;
  a.tokens = tokens;
  a.bwd = bwd;
  const unsigned nprep = pad8((a.nent + threads - 1) / threads);
  if (ms) {
    a.nwork = (int)pad8((long)nslab * (Slab::S / kMsTok) * f.nblk);
    return launch_ms_analysis(a, dim3((unsigned)a.nwork + nprep, (unsigned)count), s);
  }
  // groups of at most 128 rows (wider ones leave fewer workgroups to hide the latencies), several per
  // workgroup where there is work enough
  a.nb = slab_group_blocks(f, std::min<int64_t>(2048, (int64_t)nslab * count * (((int64_t)f.nblk * f.W + 127) / 128)));
  a.ngroups = (f.nblk + a.nb - 1) / a.nb;
  a.gpw = (int)std::max<long>(1, std::min<long>(4, (long)nslab * a.ngroups * count / 2048));
  a.runs = (a.ngroups + a.gpw - 1) / a.gpw;
  a.nwork = (int)pad8((long)nslab * a.runs);
  const Lds l = lds_layout(f, a.nb);
  a.stage_off = l.stage;
  return kernels_for(f).analysis(a, dim3((unsigned)a.nwork + nprep, (unsigned)count), l.bytes, s);
}

// How a call of `count` adapters and nslab slabs uses a pool of `cap` slabs: `adapters` at a time with
// all their slabs, or one adapter with `slabs` of its slabs at a time.
struct Split {
  int adapters, slabs;
};
Split split_call(int count, int nslab, size_t pool_bytes, size_t slab_bytes) {
  const long cap = std::max<long>(1, (long)(pool_bytes / slab_bytes));
  if (nslab <= cap) return {(int)std::min<long>(count, cap / nslab), nslab};
  return {1, (int)cap};
}

// Arguments common to both directions; the work items and LDS of groups of at most nb blocks.
struct Launch {
  unsigned grid;
  size_t lds;   // (0: multi-stage)
};
Launch pass_args(SlabArgs& a, const FrameDev& dst, const FrameDev& src, const SlabStream& st, int T, int slab0,
                 int nslab, int sg, int nb, int ngroups) {
  a.f = dst;
  a.fa = dst.wa16;
  a.fs = dst.ws16;
  a.T = T;
  a.slab0 = slab0;
  a.nslab = nslab;
  a.sg = sg;
  a.nb = st.nb;
  a.ngroups = st.ngroups;
  a.nruns = (slab0 + nslab - 1) / sg - slab0 / sg + 1;
  a.src_slab = ((long)src.nblk * src.W + 1) * kSlabRowBytes;
  a.wstep = st.wstep;
  a.zptr = st.zptr;
  a.zrow = st.zrow;
  const unsigned grid = pad8((long)ngroups * a.nruns);
  if (slab_ms_frame(dst)) return {grid, 0};
  const Lds l = lds_layout(dst, nb);
  a.stage_off = l.stage;
  return {grid, l.bytes};
}

// Second pass of `count` adapters: a multi-stage destination is gathered into the workspace and then
// synthesised.  A backward pass writes dX if dx and dC partial rows if dc.
hipError_t launch_pass(const SlabArgs& a, const Launch& l, bool bwd, bool dx, bool dc, int count, hipStream_t s) {
  const dim3 grid(l.grid, (unsigned)count);
  if (!slab_ms_frame(a.f))
    return bwd ? kernels_for(a.f).bwd(a, dx, dc, grid, l.lds, s) : kernels_for(a.f).fwd(a, grid, l.lds, s);
  const hipError_t e = launch_ms_pass(a, bwd, dx, dc, grid, s);
  if (e != hipSuccess || !dx) return e;
  MsOutArgs o{};
  o.f = a.f;
  o.T = a.T;
  o.slab0 = a.slab0;
  o.nslab = a.nslab;
  o.nwork = (int)pad8((long)a.nslab * (Slab::S / kMsTok) * a.f.nblk);
  o.ws = a.wd;
  o.ws_adapter = a.ws_adapter;
  o.Y = a.Y;
  o.Ys = a.Ys;
  o.ldy = a.ldy;
  o.scale = a.scale;
  o.beta = a.beta;
  o.group = a.group;
  o.tokens = a.tokens;
  return launch_ms_synthesis(o, dim3((unsigned)o.nwork, (unsigned)count), s);
}

// Bytes of one slab of a side.
size_t side_bytes(const FrameDev& f) { return ((size_t)f.nblk * f.W + 1) * kSlabRowBytes; }
// Bytes a call keeps per slab: the source side's, and a multi-stage destination's.
size_t call_bytes(const FrameDev& src, const FrameDev& dst) {
  return side_bytes(src) + (slab_ms_frame(dst) ? side_bytes(dst) : 0);
}

}  // namespace

hipError_t configure_slab() {
  hipError_t e = hipSuccess;
  for (const SlabLaunch* l : {&launch_direct(), &launch_radix()}) {
    const hipError_t r = l->configure();
    if (r != hipSuccess) e = r;
  }
  const hipError_t r = configure_ms();
  return r != hipSuccess ? r : e;
}

hipError_t launch_fwd_slab(const ff_plan* p, int count, int T, ActPtrs X, int64_t ldx, const float* c,
                           const float* const* cs, float scale, float beta, ActPtrs Y, int64_t ldy, hipStream_t s) {
  hipEvent_t e0, e1;
  take_timing_events(&e0, &e1);
  const int S = Slab::S, nslab = (T + S - 1) / S;
  if (nslab == 0) return hipSuccess;
  const FrameDev &fi = p->fin->dev, &fo = p->fout->dev;
  const SlabStream& st = p->slab.fwd;
  const size_t slab_bytes = call_bytes(fi, fo);
  const Split sp = split_call(count, nslab, p->slab.pool_bytes, slab_bytes);
  const long ws_adapter = (long)slab_bytes * sp.slabs;
  record(e0, s);
  for (int a0 = 0; a0 < count; a0 += sp.adapters)
    for (int s0 = 0; s0 < nslab; s0 += sp.slabs) {
      const int na = std::min(sp.adapters, count - a0), ns = std::min(sp.slabs, nslab - s0);
      uint2* ent = p->slab.ent + (long)a0 * p->slab.ent_adapter;
      hipError_t e = launch_analysis({&fi, X, ldx}, st, na, a0, T, s0, ns, p->slab.pool, ws_adapter, ent,
                                     p->slab.ent_adapter, s0 == 0, c, cs, nullptr, nullptr, 0, 0, s);
      if (e != hipSuccess) return e;
      SlabArgs a{};
      const Launch l = pass_args(a, fo, fi, st, T, s0, ns, 1, st.nb, st.ngroups);
      a.ws = p->slab.pool;
      a.wd = p->slab.pool + (size_t)sp.slabs * side_bytes(fi);
      a.ws_adapter = ws_adapter;
      a.ent = ent;
      a.ent_adapter = p->slab.ent_adapter;
      a.Y = const_cast<void*>(Y.one);
      a.Ys = Y.many ? const_cast<void* const*>(Y.many) + a0 : nullptr;
      a.ldy = (long)ldy;
      a.scale = scale;
      a.beta = beta;
      e = launch_pass(a, l, false, true, false, na, s);
      if (e != hipSuccess) return e;
    }
  record(e1, s);
  return hipGetLastError();
}

hipError_t launch_bwd_slab(const ff_plan* p, int count, int T, ActPtrs X, int64_t ldx, ActPtrs G,
                           int64_t ldg, const float* c, const float* const* cs, float scale, float beta_dx, ActPtrs dX,
                           int64_t lddx, bool want_dx, int accumulate_dc, float* dC, float* const* dCs, bool want_dc,
                           hipStream_t s, const BwdScratch* ws) {
  hipEvent_t e0, e1;
  take_timing_events(&e0, &e1);
  const int S = Slab::S, nslab = (T + S - 1) / S;
  const FrameDev &fi = p->fin->dev, &fo = p->fout->dev;
  const SlabStream& st = p->slab.bwd;
  int sg = 1, nrows = 0;
  partial_rows(T, S, p->slab.rows, &sg, &nrows);
  const size_t slab_bytes = call_bytes(fo, fi);
  const long pstride = 16L * st.steps;
  unsigned char* pool = p->slab.pool;
  size_t pool_bytes = p->slab.pool_bytes;
  uint2* ents = p->slab.ent;
  float* partial = p->partial;
  if (ws) {   // the caller's scratch: entries, partial rows, then slabs
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t eb = up((size_t)16 * (st.steps + kSlabPadSteps) * sizeof(uint2));
    const size_t pb = up((size_t)nrows * (size_t)pstride * sizeof(float));
    const size_t have = ws->floats * sizeof(float);
    if (eb + pb + slab_bytes > have) return hipErrorInvalidValue;
    unsigned char* base = reinterpret_cast<unsigned char*>(ws->base);
    ents = reinterpret_cast<uint2*>(base);
    partial = reinterpret_cast<float*>(base + eb);
    pool = base + eb + pb;
    pool_bytes = have - eb - pb;
  }
  const Split sp = split_call(count, std::max(nslab, 1), pool_bytes, slab_bytes);
  const long ws_adapter = (long)slab_bytes * sp.slabs;
  record(e0, s);
  for (int a0 = 0; a0 < count && (want_dx || want_dc); a0 += sp.adapters)
    for (int s0 = 0; s0 < nslab; s0 += sp.slabs) {
      const int na = std::min(sp.adapters, count - a0), ns = std::min(sp.slabs, nslab - s0);
      uint2* ent = ents + (long)a0 * p->slab.ent_adapter;
      // a dC-only call reads no coefficients (its entries carry zeros)
      hipError_t e = launch_analysis({&fo, G, ldg}, st, na, a0, T, s0, ns, pool, ws_adapter, ent, p->slab.ent_adapter,
                                     s0 == 0, want_dx ? c : nullptr, want_dx ? cs : nullptr, nullptr, nullptr, 1, 0, s);
      if (e != hipSuccess) return e;
      unsigned char* wd = pool + (size_t)sp.slabs * side_bytes(fo);
      if (want_dc && slab_ms_frame(fi)) {
        e = launch_analysis({&fi, X, ldx}, st, na, a0, T, s0, ns, wd, ws_adapter, nullptr, 0, false, nullptr, nullptr,
                            nullptr, nullptr, 1, 0, s);
        if (e != hipSuccess) return e;
      }
      SlabArgs a{};
      const Launch l = pass_args(a, fi, fo, st, T, s0, ns, sg, st.nb, st.ngroups);
      a.ws = pool;
      a.wd = wd;
      a.ws_adapter = ws_adapter;
      a.ent = ent;
      a.ent_adapter = p->slab.ent_adapter;
      a.X = X.one;
      a.Xs = X.many ? X.many + a0 : nullptr;
      a.ldx = (long)ldx;
      a.Y = const_cast<void*>(dX.one);
      a.Ys = dX.many ? const_cast<void* const*>(dX.many) + a0 : nullptr;
      a.ldy = (long)lddx;
      a.scale = scale;
      a.beta = beta_dx;
      a.prows = nrows;
      a.pstride = pstride;
      a.partial = partial + (long)a0 * nrows * pstride;
      e = launch_pass(a, l, true, want_dx, want_dc, na, s);
      if (e != hipSuccess) return e;
    }
  record(e1, s);
  if (want_dc)
    return launch_dc_reduce(partial, nrows, (int)pstride, st.coef, p->dev.coef_pad, p->dev.ncoef_pad, scale,
                            accumulate_dc, dC, dCs, count, s);
  return hipGetLastError();
}

namespace {

// Group calls: dC from each adapter's own partial rows (those of its tokens), as dc_reduce.
constexpr int kRedWaves = 16, kRedBatch = 8;

__global__ void __launch_bounds__(64 * kRedWaves) slab_reduce_group(const SlabDesc* group, const GenDesc* gen,
                                                                    const int* tokens, int T, int S, int sg, float scale,
                                                                    int accumulate, float* const* dCs) {
  __shared__ float red[kRedWaves][64];
  const int bi = blockIdx.y, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const SlabDesc* d = group + bi;
  const GenDesc* gd = gen + bi;
  float* out = dCs[bi];
  const int len = 16 * d->bwd.steps, nmain = (len + 63) / 64;
  if ((int)blockIdx.x >= nmain) {
    const int j = ((int)blockIdx.x - nmain) * (int)blockDim.x + threadIdx.x;
    if (!accumulate && j < gd->ncoef_pad) gstore(out + gload(gd->coef_pad + j), 0.f);
    return;
  }
  const int Tb = group_tokens(tokens, T, bi);
  const int nrows = ((Tb + S - 1) / S + sg - 1) / sg;
  const int e = blockIdx.x * 64 + lane;
  const float* p = d->partial + min(e, len - 1);
  float sum = 0.f;
  for (int r0 = w; r0 < nrows; r0 += kRedWaves * kRedBatch) {
    float v[kRedBatch];
#pragma unroll
    for (int j = 0; j < kRedBatch; ++j) {
      const int r = r0 + j * kRedWaves;
      v[j] = r < nrows ? gload(p + (long)r * len) : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kRedBatch; ++j) sum += v[j];
  }
  red[w][lane] = sum;
  __syncthreads();
  if (w == 0 && e < len) {
    const int slot = gload(d->bwd.coef + e);
    if (slot < 0) return;
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < kRedWaves; ++i) tot += red[i][lane];
    const float v = scale * tot;
    gstore(out + slot, accumulate ? gload(out + slot) + v : v);
  }
}

}  // namespace

hipError_t launch_fwd_group_slab(const ff_plan_group* g, int T, const int* tokens, const void* const* X,
                                 int64_t ldx, const float* const* cs, float scale, float beta, void* const* Y,
                                 int64_t ldy, hipStream_t s) {
  const ff_plan* p = g->ref;
  hipEvent_t e0, e1;
  take_timing_events(&e0, &e1);
  const int S = Slab::S, nslab = (T + S - 1) / S, count = (int)g->count;
  if (nslab == 0) return hipSuccess;
  const FrameDev &fi = p->fin->dev, &fo = p->fout->dev;
  const SlabStream& st = p->slab.fwd;
  const size_t slab_bytes = call_bytes(fi, fo);
  const Split sp = split_call(1, nslab, g->slab_pool, slab_bytes);   // every adapter in its plan's own pool
  record(e0, s);
  for (int s0 = 0; s0 < nslab; s0 += sp.slabs) {
    const int ns = std::min(sp.slabs, nslab - s0);
    hipError_t e = launch_analysis({&fi, {nullptr, X}, ldx}, st, count, 0, T, s0, ns, nullptr, 0, nullptr, 0, s0 == 0,
                                   nullptr, cs, g->slab, tokens, 0, g->max_slab_fwd, s);
    if (e != hipSuccess) return e;
    SlabArgs a{};
    const Launch l = pass_args(a, fo, fi, st, T, s0, ns, 1, g->slab_nb_fwd, g->slab_groups_fwd);
    a.ws_adapter = (long)((size_t)sp.slabs * side_bytes(fi));
    a.Ys = Y;
    a.ldy = (long)ldy;
    a.scale = scale;
    a.beta = beta;
    a.group = g->slab;
    a.tokens = tokens;
    e = launch_pass(a, l, false, true, false, count, s);
    if (e != hipSuccess) return e;
  }
  record(e1, s);
  return hipGetLastError();
}

hipError_t launch_bwd_group_slab(const ff_plan_group* g, int T, const int* tokens, const void* const* X,
                                 int64_t ldx, const void* const* G, int64_t ldg, const float* const* cs, float scale,
                                 float beta_dx, void* const* dX, int64_t lddx, bool want_dx, int accumulate_dc,
                                 float* const* dCs, bool want_dc, hipStream_t s) {
  const ff_plan* p = g->ref;
  hipEvent_t e0, e1;
  take_timing_events(&e0, &e1);
  const int S = Slab::S, nslab = (T + S - 1) / S, count = (int)g->count;
  const FrameDev &fi = p->fin->dev, &fo = p->fout->dev;
  const SlabStream& st = p->slab.bwd;
  int sg = 1, nrows = 0;
  partial_rows(T, S, g->slab_rows, &sg, &nrows);
  const size_t slab_bytes = call_bytes(fo, fi);
  const Split sp = split_call(1, std::max(nslab, 1), g->slab_pool, slab_bytes);
  record(e0, s);
  for (int s0 = 0; s0 < nslab; s0 += sp.slabs) {
    const int ns = std::min(sp.slabs, nslab - s0);
    hipError_t e = launch_analysis({&fo, {nullptr, G}, ldg}, st, count, 0, T, s0, ns, nullptr, 0, nullptr, 0, s0 == 0,
                                   nullptr, want_dx ? cs : nullptr, g->slab, tokens, 1, g->max_slab_bwd, s);
    if (e != hipSuccess) return e;
    const long wd = (long)((size_t)sp.slabs * side_bytes(fo));   // in each adapter's pool
    if (want_dc && slab_ms_frame(fi)) {
      e = launch_analysis({&fi, {nullptr, X}, ldx}, st, count, 0, T, s0, ns, nullptr, wd, nullptr, 0, false, nullptr,
                          nullptr, g->slab, tokens, 1, 0, s);
      if (e != hipSuccess) return e;
    }
    SlabArgs a{};
    const Launch l = pass_args(a, fi, fo, st, T, s0, ns, sg, g->slab_nb_bwd, g->slab_groups_bwd);
    a.ws_adapter = wd;
    a.Xs = X;
    a.ldx = (long)ldx;
    a.Ys = dX;
    a.ldy = (long)lddx;
    a.scale = scale;
    a.beta = beta_dx;
    a.group = g->slab;
    a.tokens = tokens;
    e = launch_pass(a, l, true, want_dx, want_dc, count, s);
    if (e != hipSuccess) return e;
  }
  record(e1, s);
  if (want_dc) {
    const int nmain = (g->max_slab_bwd + 63) / 64;
    const int npadb = (g->max_gen_npad + 64 * kRedWaves - 1) / (64 * kRedWaves);
    hipLaunchKernelGGL(slab_reduce_group, dim3((unsigned)(nmain + npadb), (unsigned)count), dim3(64 * kRedWaves), 0, s,
                       g->slab, g->gen, tokens, T, S, sg, scale, accumulate_dc, dCs);
  }
  return hipGetLastError();
}

}  // namespace ff
