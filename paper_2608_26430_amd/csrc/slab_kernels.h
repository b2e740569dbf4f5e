// Slab kernels: forward and backward of the adapter in two passes through a coefficient-major
// workspace, for frames whose blocks are applied directly (up to 128 wide) or in one radix-4 stage.
//
// A slab is S = 64 consecutive tokens (bf16).  The workspace holds one side's coefficients
// as [slab][coefficient position][S tokens]: 128 bytes, one cache line, per coefficient and slab,
// plus one row of zeros per slab that padding entries read.  Position of block b's local
// coefficient: b W + a' W2 + 2 l + s for frequency a' + 4 l of a factored block, b W + c of a
// directly applied one.
//   slab_analysis   source side (x forward, g backward) -> workspace; streaming, no reuse
//   slab_fwd        per (group of output blocks, slab): v = C z gathered from the workspace into an
//                   LDS tile, then y = beta y + s P_out v from the tile
//   slab_bwd        per (group of input blocks, slab): z = P_in^T x into the tile, q = C^T u and the
//                   slab's dC sums from gathered u, q over z, then dX = beta dX + s P_in q
//
// Why two passes: the support is uniformly random, so every output coefficient may need any input
// one.  Keeping both sides of a token in LDS limits a workgroup to 4 (7B MLP) or 2 (70B) tokens, and
// each table row then serves so few tokens that instruction issue on the table walk is the bound
// (MLP up forward 114 us, 70B backward 1380 us).  Through the workspace only one group of blocks
// of the destination side sits in LDS, a table row serves 64 tokens with one full cache line per
// entry, and the price is one write and one read of the source side, which stays in the
// last-level cache (calls are split so that it does) and, a slab being worked on by one XCD at a
// time, mostly in that XCD's L2.
//
// The vector memory path takes one 64-byte access per clock and CU and merges only neighbouring
// lanes, while MFMA operands and results have neighbouring lanes in different rows (tokens or
// coefficients).  Reading and writing those directly cost 64 accesses an instruction and bound every
// phase; so token rows pass through an LDS stage, coefficients through the LDS tile, both moved
// with neighbouring lanes on neighbouring 16 bytes, and the walk gives each entry to four
// neighbouring lanes.
#pragma once

#include "gen_kernels.h"

namespace ff {
namespace slab {

using namespace gen;

struct Slab {
  static constexpr int ESZ = 2;
  static constexpr int S = kSlabTokens;   // tokens per slab
  static constexpr int TC = 16 / ESZ;     // tokens per 16 bytes
  static constexpr int NTG = S / 16;      // groups of 16 tokens (MFMA columns)
};

typedef short i16x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x4v __attribute__((ext_vector_type(4)));
typedef unsigned u32x4a __attribute__((ext_vector_type(4), aligned(4)));

// LDS tile: one 128-byte row per coefficient of the group, 144 bytes apart, so that the four
// consecutive rows of a transposed read and the 16 rows of a result fall on disjoint banks.
constexpr int kTileRow = kSlabRowBytes + 16;
__device__ __forceinline__ unsigned tile_at(int row, int byte) { return (unsigned)(row * kTileRow + byte); }

// Workgroup -> work item, contiguous runs of items per XCD (workgroups go to the eight XCDs in
// turn), so that the items of one slab share an L2.  The grid is padded to a multiple of 8.  The runs
// are dealt out one XCD further from adapter to adapter: in a group call the late slabs of most
// adapters are empty, and one XCD would get all the first ones (17 adapters of up to 418 tokens:
// 28.6 -> 22.5 us a call).
__device__ __forceinline__ int xcd_item(int id, int n, int adapter) {
  const int per = (n + 7) >> 3;
  const int w = ((id + adapter) & 7) * per + (id >> 3);
  return (id >> 3) < per ? w : n;
}

// LDS stage: token rows of a group's columns, `cb` 16-byte chunks each, at a stride of an odd
// number of chunks (so that 16 tokens' reads of one column fall on distinct banks).
__device__ __forceinline__ int stage_stride(int cb) { return (cb | 1) * 16; }

// The slab's token rows at `src` (row stride ld bytes) into the stage; rows nt .. S - 1 are zeros.
template <int S>
__device__ __forceinline__ void stage_load(const unsigned char* src, long ld, int nt, int cb, unsigned char* stage) {
  const int tid = phase_tid(), sb = stage_stride(cb), n = S * cb;
  const float inv = 1.f / (float)cb;
  constexpr int kU = 4;
  for (int i0 = tid; i0 < n; i0 += kU * kSlabThreads) {
    u32x4v v[kU];
    int at[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = min(i0 + u * kSlabThreads, n - 1), t = div_small(i, cb, inv), c = i - __mul24(t, cb);
      at[u] = __mul24(t, sb) + 16 * c;
      v[u] = gload(reinterpret_cast<const u32x4v*>(src + (long)min(t, nt - 1) * ld + 16 * c));
      if (nt < S && t >= nt) v[u] = u32x4v{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) *reinterpret_cast<u32x4v*>(stage + at[u]) = v[u];   // (past the end: the last again)
  }
}

// The stage's first nt rows to the token rows at dst.
__device__ __forceinline__ void stage_store(const unsigned char* stage, int nt, int cb, unsigned char* dst, long ld) {
  const int tid = phase_tid(), sb = stage_stride(cb), n = nt * cb;
  const float inv = 1.f / (float)cb;
  for (int i = tid; i < n; i += kSlabThreads) {
    const int t = div_small(i, cb, inv), c = i - __mul24(t, cb);
    gstore(reinterpret_cast<u32x4v*>(dst + (long)t * ld + 16 * c),
           *reinterpret_cast<const u32x4v*>(stage + __mul24(t, sb) + 16 * c));
  }
}

__device__ __forceinline__ u32x4v pack16(const float* x) {
  return u32x4v{pk_bf2(x[0], x[1]), pk_bf2(x[2], x[3]), pk_bf2(x[4], x[5]), pk_bf2(x[6], x[7])};
}

// A value at a wave-uniform address that nothing writes while the kernel runs, through the scalar
// cache: the descriptors at a kernel's start are then read together instead of one vector load
// after the other.
template <class T>
__device__ __forceinline__ T sload(const T* p) {
  return *(const __attribute__((address_space(4))) T*)p;
}

// Tokens of adapter bi in a group call.
__device__ __forceinline__ int adapter_tokens(const int* tokens, int T, int bi) {
  return tokens ? max(0, min(sload(tokens + bi), T)) : T;
}

// Work items (output tile mt, block, half of the token groups) of an MFMA phase: a contiguous run per
// wave in that order, so that a wave changes its fragments rarely.
struct Items {
  int i0, i1, nb;
  __device__ __forceinline__ Items(int MT, int nb_) : nb(nb_) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = MT * nb * 2;
    i0 = n * wave / kSlabWaves;
    i1 = n * (wave + 1) / kSlabWaves;
  }
  __device__ __forceinline__ void get(int it, int& mt, int& bl, int& th) const {
    mt = it / (2 * nb);
    const int r = it - mt * 2 * nb;
    bl = r >> 1;
    th = r & 1;
  }
};

// Most work items of a wave with factored blocks (whose matrices have at most KS KT rows).
constexpr int radix_items(int KT) {
  return (2 * (Mfma<true>::KS / 16) * KT + kSlabWaves - 1) / kSlabWaves;
}

template <class V, int KT>
__device__ __forceinline__ void load_frags(const void* frag, int mt, int lane, V (&fr)[KT]) {
#pragma unroll
  for (int ks = 0; ks < KT; ++ks) fr[ks] = gload(reinterpret_cast<const V*>(frag) + (mt * KT + ks) * 64 + lane);
}

// Four tokens (4 q .. + 3 of group tg) of one coefficient row into the tile.
__device__ __forceinline__ void put_tokens(unsigned char* tile, int row, int tg, int q, f32x4 v) {
  constexpr int ESZ = Slab::ESZ;
  unsigned char* p = tile + tile_at(row, (16 * tg + 4 * q) * ESZ);
  *reinterpret_cast<uint2*>(p) = Act<true>::pack4(v);
}

// Coefficients of the staged token rows into the tile: z = P^T x for nb blocks.  MFMA with swapped
// operands (D = X^T M^T), so that lane (q, L) ends with four tokens of output 16 mt + L.
// Contraction windows are clamped to the column (element min(KS ks + VL q, W2 - VL) + j, repeated
// elements having zero weights in `frag`), so that every read stays inside the block.
// Directly applied blocks: stage and tile are different LDS.
template <int KT>
__device__ __forceinline__ void analysis_direct(const FrameDev& f, const void* frag, int have,
                                                Mfma<true>::V (&fr)[KT], const unsigned char* stage, int cb,
                                                int nb, unsigned char* tile) {
  using M = Mfma<true>;
  using V = M::V;
  constexpr int ESZ = Slab::ESZ, NTH = Slab::NTG / 2;
  const int lane = phase_tid() & 63, q = lane >> 4, L = lane & 15, W = f.W, sb = stage_stride(cb);
  const Items items(f.MT, nb);
  for (int it = items.i0; it < items.i1; ++it) {
    int mt, bl, th;
    items.get(it, mt, bl, th);
    if (mt != have) load_frags<V, KT>(frag, mt, lane, fr);
    have = mt;
    f32x4 acc[NTH];
#pragma unroll
    for (int g = 0; g < NTH; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) {
      const int e = min(ks * M::KS + q * M::VL, W - M::VL);
#pragma unroll
      for (int g = 0; g < NTH; ++g)
        acc[g] = M::step(*reinterpret_cast<const V*>(stage + (16 * (NTH * th + g) + L) * sb + (bl * W + e) * ESZ), fr[ks],
                         acc[g]);
    }
    const int o = 16 * mt + L;
    if (o < W) {
#pragma unroll
      for (int g = 0; g < NTH; ++g) put_tokens(tile, bl * W + o, NTH * th + g, q, acc[g]);
    }
  }
}

// Factored blocks (one per group).  On the way into LDS the radix-4 stage
// Y_a'[c] = w^(-a' c) sum_a x[a k2 + c] (-i)^(a a') is formed in registers, in fp32, twiddles
// included; a token's column a' is nw windows of VL elements, 16 bytes each, the last clamped to end
// with the column.  A thread keeps one window, whose twiddles it loads once, of every `per`-th token.
__device__ __forceinline__ int radix_windows(int W2, int VL) { return (W2 + VL - 1) / VL; }
__device__ __forceinline__ int radix_stride(int nw) { return (4 * nw | 1) * 16; }

__device__ __forceinline__ void radix_load(const FrameDev& f, const unsigned char* src, long ld, int nt,
                                           unsigned char* lds) {
  using T = Slab;
  constexpr int VL = T::TC, NC = VL / 2, S = T::S, kU = 3;
  const int tid = phase_tid(), W2 = f.W2, nw = radix_windows(W2, VL), sb = radix_stride(nw);
  const float inv = 1.f / (float)nw;
  const int per = div_small(kSlabThreads, nw, inv), t0 = div_small(tid, nw, inv), w = tid - __mul24(t0, nw);
  if (t0 >= per) return;
  const int e0 = min(w * VL, W2 - VL);
  float2 tw[3][NC];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int k = 0; k < NC; ++k) tw[a][k] = gload(f.tw + a * f.k2 + e0 / 2 + k);
  src += e0 * T::ESZ;
  lds += 16 * w;
  for (int ts = t0; ts < S; ts += kU * per) {
    u32x4v x[kU][4];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int t = ts + u * per;
      const unsigned char* p = src + (long)min(t, nt - 1) * ld;
#pragma unroll
      for (int a = 0; a < 4; ++a) {   // (columns start at multiples of one complex coordinate)
        x[u][a] = u32x4v(*(const FF_GLOBAL u32x4a*)(p + a * W2 * T::ESZ));
        if (nt < S && t >= nt) x[u][a] = u32x4v{0u, 0u, 0u, 0u};
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int t = ts + u * per;
      if (t >= S) break;
      float y[4][VL];
#pragma unroll
      for (int k = 0; k < NC; ++k) {
        float2 v[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const unsigned word = x[u][a][k];
          v[a] = make_float2(__uint_as_float(word << 16), __uint_as_float(word & 0xffff0000u));
        }
        const float2 s02 = cadd(v[0], v[2]), d02 = csub(v[0], v[2]);
        const float2 s13 = cadd(v[1], v[3]), d13 = csub(v[1], v[3]);
        const float2 o[4] = {cadd(s02, s13), cmulc(make_float2(d02.x + d13.y, d02.y - d13.x), tw[0][k]),
                             cmulc(csub(s02, s13), tw[1][k]),
                             cmulc(make_float2(d02.x - d13.y, d02.y + d13.x), tw[2][k])};
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          y[a][2 * k] = o[a].x;
          y[a][2 * k + 1] = o[a].y;
        }
      }
#pragma unroll
      for (int a = 0; a < 4; ++a) *reinterpret_cast<u32x4v*>(lds + t * sb + 16 * a * nw) = pack16(y[a]);
    }
  }
}

// The DFTs of size k/4 of the four columns.  The tile takes the windows' LDS, so the results wait in
// registers until every wave has read its operands.
template <int KT>
__device__ __forceinline__ void analysis_radix(const FrameDev& f, const void* frag, unsigned char* lds) {
  using M = Mfma<true>;
  using V = M::V;
  constexpr int NTH = Slab::NTG / 2, NI = radix_items(KT);
  const int lane = phase_tid() & 63, q = lane >> 4, L = lane & 15, W2 = f.W2, nw = radix_windows(W2, M::VL),
            sb = radix_stride(nw);
  const Items items(f.MT, 1);
  V fr[KT];
  uint2 out[NI][NTH][4];
  int have = -1;
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int it = items.i0 + n;
    if (it >= items.i1) break;   // uniform
    int mt, bl, th;
    items.get(it, mt, bl, th);
    if (mt != have) load_frags<V, KT>(frag, mt, lane, fr);
    have = mt;
    f32x4 acc[NTH][4];
#pragma unroll
    for (int g = 0; g < NTH; ++g)
#pragma unroll
      for (int a = 0; a < 4; ++a) acc[g][a] = f32x4{0.f, 0.f, 0.f, 0.f};
    const unsigned char* row = lds + (16 * NTH * th + L) * sb;
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) {
      const unsigned char* p = row + 16 * min(4 * ks + q, nw - 1);
#pragma unroll
      for (int g = 0; g < NTH; ++g)
#pragma unroll
        for (int a = 0; a < 4; ++a)
          acc[g][a] = M::step(*reinterpret_cast<const V*>(p + 16 * g * sb + 16 * a * nw), fr[ks], acc[g][a]);
    }
#pragma unroll
    for (int g = 0; g < NTH; ++g)
#pragma unroll
      for (int a = 0; a < 4; ++a) {
        out[n][g][a] = Act<true>::pack4(acc[g][a]);
      }
    __builtin_amdgcn_sched_barrier(0);   // one item after the other (registers)
  }
  __syncthreads();
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int it = items.i0 + n;
    if (it >= items.i1) break;
    int mt, bl, th;
    items.get(it, mt, bl, th);
    const int o = 16 * mt + L;
    if (o >= W2) continue;
#pragma unroll
    for (int g = 0; g < NTH; ++g)
#pragma unroll
      for (int a = 0; a < 4; ++a)
        *reinterpret_cast<uint2*>(lds + tile_at(a * W2 + o, (16 * (NTH * th + g) + 4 * q) * Slab::ESZ)) = out[n][g][a];
  }
}

// Token rows of a group of blocks -> coefficients in the tile, with the barriers around them.  LDS:
// the tile first; directly applied blocks' stage after it.
template <int KT, bool RADIX>
__device__ __forceinline__ void group_analysis(const FrameDev& f, const void* frag, const unsigned char* rows, long ld,
                                               int nt, int nb, unsigned char* tile, unsigned char* stage) {
  if constexpr (RADIX) {
    radix_load(f, rows, ld, nt, stage);
    __syncthreads();
    analysis_radix<KT>(f, frag, stage);
  } else {
    const int cb = nb * f.W * Slab::ESZ / 16;
    // the wave's first fragments travel with the rows
    Mfma<true>::V fr[KT];
    const Items items(f.MT, nb);
    int mt = -1, bl, th;
    if (items.i0 < items.i1) {
      items.get(items.i0, mt, bl, th);
      load_frags<Mfma<true>::V, KT>(frag, mt, phase_tid() & 63, fr);
    }
    stage_load<Slab::S>(rows, ld, nt, cb, stage);
    __syncthreads();
    analysis_direct<KT>(f, frag, mt, fr, stage, cb, nb, tile);
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------------------------
// First pass: the source side into the workspace, and the destination stream's entries with this
// call's coefficients, (word, c) pairs in stream order.

struct AnaArgs {
  FrameDev f;
  const void* frag;      // analysis fragments over clamped windows
  int T, slab0, nslab;   // tokens of the call; slabs slab0 .. slab0 + nslab - 1 in this launch
  const void* X;
  const void* const* Xs;
  long ld;
  unsigned char* ws;     // [adapter][slab][P + 1][128 bytes]
  long ws_adapter;       // bytes between adapters (group calls: offset in each adapter's pool)
  int nb, ngroups;       // blocks per group (a workgroup stages a group at a time)
  int gpw, runs;         // groups per workgroup, workgroups per slab
  int stage_off;         // LDS offset of the stage (the tile is first)
  int nwork;             // workgroups of (slab, run) items; those after them copy entries
  // entries: ent[adapter][j] = (word[j], c_adapter[coef[j]]), j < nent (0: none in this launch)
  const unsigned* word;
  const int* coef;
  int nent;
  const float* c;        // NULL with cs == NULL: coefficients not needed (zeros)
  const float* const* cs;
  uint2* ent;
  long ent_adapter;
  const SlabDesc* group;
  const int* tokens;
  int bwd;               // group calls: which stream's entries
};

// Group calls: adapter bi's entries, stream and pool into `a`; returns the pool.
__device__ __forceinline__ unsigned char* group_entries(AnaArgs& a, int bi) {
  const SlabDesc* d = a.group + bi;
  const SlabStream* st = a.bwd ? &d->bwd : &d->fwd;
  a.word = sload(&st->word);
  a.coef = sload(&st->coef);
  if (a.nent) a.nent = 16 * (sload(&st->steps) + kSlabPadSteps);
  a.ent = sload(&d->ent) - (long)bi * a.ent_adapter;
  return sload(&d->ws);
}

// Entry j of adapter bi's stream with this call's coefficient.
__device__ __forceinline__ void copy_entry(const AnaArgs& a, int bi, int j) {
  if (j >= a.nent) return;
  const float* cv = a.cs ? sload(a.cs + bi) : a.c;
  const int k = gload(a.coef + j);
  uint2 e;
  e.x = gload(a.word + j);
  e.y = cv && k >= 0 ? __float_as_uint(gload(cv + k)) : 0u;
  gstore(a.ent + (long)bi * a.ent_adapter + j, e);
}

// Workgroups per CU that the widest blocks of a kernel leave LDS for (two also where factored blocks'
// results wait in fp32), which bounds its registers.
constexpr int slab_wgs(int KT, bool RADIX, bool BETA = false) { return RADIX && (KT >= 4 || BETA) ? 2 : 3; }

template <int KT, bool RADIX>
__global__ void __launch_bounds__(kSlabThreads, slab_wgs(KT, RADIX)) slab_analysis(AnaArgs a) {
  constexpr int S = Slab::S, ESZ = Slab::ESZ;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int bi = blockIdx.y;
  unsigned char* ws = a.ws + (long)bi * a.ws_adapter;
  int T = a.T;
  if (a.group) {
    ws = group_entries(a, bi) + a.ws_adapter;
    T = adapter_tokens(a.tokens, a.T, bi);
  }
  if ((int)blockIdx.x >= a.nwork) {
    copy_entry(a, bi, ((int)blockIdx.x - a.nwork) * kSlabThreads + (int)threadIdx.x);
    return;
  }
  const FrameDev& f = a.f;
  const int wi = xcd_item(blockIdx.x, a.nwork, bi);
  const int sl = wi / a.runs, run = wi - sl * a.runs;
  const long t0 = (long)(a.slab0 + sl) * S;
  const int nt = sl < a.nslab ? (int)min((long)S, (long)T - t0) : 0;
  if (nt <= 0) return;   // uniform
  const long P = (long)f.nblk * f.W;
  unsigned char* out = ws + (long)sl * (P + 1) * kSlabRowBytes;
  const unsigned char* X = reinterpret_cast<const unsigned char*>(a.Xs ? sload(a.Xs + bi) : a.X) + t0 * a.ld * ESZ;
  if (run == 0 && threadIdx.x < 8)
    gstore(reinterpret_cast<u32x4v*>(out + P * kSlabRowBytes) + threadIdx.x, u32x4v{0u, 0u, 0u, 0u});
  const int g1 = min(a.ngroups, (run + 1) * a.gpw);
  for (int g = run * a.gpw; g < g1; ++g) {
    const int blk0 = g * a.nb, nb = min(a.nb, f.nblk - blk0);
    if (g > run * a.gpw) __syncthreads();   // the previous group's tile is copied
    group_analysis<KT, RADIX>(f, a.frag, X + (long)blk0 * f.W * ESZ, a.ld * ESZ, nt, nb, smem,
                                    smem + (RADIX ? 0 : a.stage_off));
    unsigned char* o = out + (long)blk0 * f.W * kSlabRowBytes;
    for (int i = phase_tid(); i < nb * f.W * 8; i += kSlabThreads)
      gstore(reinterpret_cast<u32x4v*>(o) + i, *reinterpret_cast<const u32x4v*>(smem + tile_at(i >> 3, 16 * (i & 7))));
  }
}

// ---------------------------------------------------------------------------------------------
// Second pass.

// Quad lane i's value of x to the four lanes of the quad.
template <int I>
__device__ __forceinline__ unsigned quad_bcast(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, I * 0x55, 0xF, 0xF, true);
}
__device__ __forceinline__ void spread4(unsigned x, unsigned (&r)[4]) {
  r[0] = quad_bcast<0>(x);
  r[1] = quad_bcast<1>(x);
  r[2] = quad_bcast<2>(x);
  r[3] = quad_bcast<3>(x);
}
__device__ __forceinline__ float quad_sum(float x) {
  x += quad_swap<1>(x);
  return x + quad_swap<2>(x);
}

// The end of a bundle whose rows are spread over several entries (`last`: its last entry word): the sums of
// a row's entries, 2^level neighbouring quads, added up in all of them.
template <int N>
__device__ __forceinline__ void merge_quads(unsigned last, float (&acc)[N]) {
  const int end = 4 << ((last & kSlabLevelMask) >> kSlabLevelShift);
  for (int d = 4; d < end; d <<= 1)
#pragma unroll
    for (int t = 0; t < N; ++t) acc[t] += __shfl_xor(acc[t], d);
}

__device__ __forceinline__ void unpack16(u32x4v w, float (&x)[Slab::TC]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned v = w[i];
    x[2 * i] = __uint_as_float(v << 16);
    x[2 * i + 1] = __uint_as_float(v & 0xffff0000u);
  }
}

// sum += products of two 16-byte pieces of tokens (bf16 pairs exactly, fp32 accumulation).
__device__ __forceinline__ float dot16(u32x4v a, u32x4v b, float sum) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const unsigned x = a[i], y = b[i];
    sum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, x), __builtin_bit_cast(bf16x2_t, y), sum, false);
  }
  return sum;
}

// Walk of stream steps s0 .. s1 - 1 (multiples of four) by one wave.  A step is 16 entries, quad e of
// the lanes working on entry e: lane c of the quad takes bytes 16 c and 64 + 16 c of its row.  A
// bundle is a run of steps over the same 16 destination rows, whose last step is flagged.  DX: the
// entries' source rows times their coefficients are summed into the destination rows of the tile.
// DC: per entry, the sum over the slab's tokens of its source row times the tile row it points to
// (read at the bundle's start, before DX overwrites it).
// Batches of four steps, stored so that lane (e, c) of one load holds entry e of step c: entries two
// batches ahead, source rows one batch ahead.  Every batch is consumed whole on every path, so that
// the waits are counted exactly.
template <bool DX, bool DC>
__device__ __forceinline__ void slab_walk(const uint2* ent, int s0, int s1, const unsigned char* src,
                                          unsigned char* tile, float* part, bool add) {
  constexpr int TC = Slab::TC;
  if (s0 >= s1) return;
  const int lane = phase_tid() & 63, c = lane & 3;
  const uint2* ep = ent + lane;
  struct Batch {
    unsigned w[4], c[4];
    u32x4v g[4][2];
  };
  auto issue = [&](uint2 m, Batch& b) {
    spread4(m.x, b.w);
    if (DX) spread4(m.y, b.c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned off = (b.w[i] & kSlabSrcMask) * (unsigned)kSlabRowBytes + 16u * c;
      b.g[i][0] = gload(reinterpret_cast<const u32x4v*>(src + off));
      b.g[i][1] = gload(reinterpret_cast<const u32x4v*>(src + off + 64));
    }
  };
  float acc[2 * TC];
  u32x4v z[2] = {};
#pragma unroll
  for (int t = 0; t < 2 * TC; ++t) acc[t] = 0.f;
  bool start = true;
  auto consume = [&](int s, Batch& b) {
    float dcv = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = (int)((b.w[i] >> kSlabDstShift) & kSlabDstMask);
      if constexpr (DC) {
        if (start) {
          z[0] = *reinterpret_cast<const u32x4v*>(tile + tile_at(row, 16 * c));
          z[1] = *reinterpret_cast<const u32x4v*>(tile + tile_at(row, 64 + 16 * c));
        }
        start = false;
        const float d = quad_sum(dot16(b.g[i][1], z[1], dot16(b.g[i][0], z[0], 0.f)));
        dcv = c == i ? d : dcv;
      }
      if constexpr (DX) {
        float x[2][TC];
        unpack16(b.g[i][0], x[0]);
        unpack16(b.g[i][1], x[1]);
        const float cc = __uint_as_float(b.c[i]);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int t = 0; t < TC; ++t) acc[k * TC + t] = fmaf(cc, x[k][t], acc[k * TC + t]);
      }
      const int last = __builtin_amdgcn_readfirstlane((int)b.w[i]);
      if (last < 0) {   // the bundle's last step (uniform)
        if constexpr (DX) {
          if (last & kSlabLevelMask) merge_quads((unsigned)last, acc);
          *reinterpret_cast<u32x4v*>(tile + tile_at(row, 16 * c)) = pack16(acc);
          *reinterpret_cast<u32x4v*>(tile + tile_at(row, 64 + 16 * c)) = pack16(acc + TC);
#pragma unroll
          for (int t = 0; t < 2 * TC; ++t) acc[t] = 0.f;
        }
        start = true;
      }
    }
    if constexpr (DC) {
      float* p = part + (long)s * 16 + lane;
      gstore(p, add ? gload(p) + dcv : dcv);
    }
  };
  Batch ba, bb;
  uint2 m = gload(ep + (long)s0 * 16), mn = gload(ep + (long)(s0 + 4) * 16);
  issue(m, ba);
  for (int s = s0; s < s1; s += 8) {
    m = gload(ep + (long)(s + 8) * 16);
    issue(mn, bb);
    __builtin_amdgcn_sched_barrier(0);
    consume(s, ba);
    if (s + 4 >= s1) break;
    mn = gload(ep + (long)(s + 12) * 16);
    issue(m, ba);
    __builtin_amdgcn_sched_barrier(0);
    consume(s + 4, bb);
  }
}

// The rows of a group that no entry points to hold zeros (their coefficients are zero).
// (`first`: this thread's first row, loaded before the walk.)
__device__ __forceinline__ void zero_rows(unsigned char* tile, const unsigned short* rows, int n, int first) {
  const int tid = phase_tid();
  for (int i = tid >> 3, r = first; i < n;) {
    *reinterpret_cast<u32x4v*>(tile + tile_at(r, 16 * (tid & 7))) = u32x4v{0u, 0u, 0u, 0u};
    i += kSlabThreads / 8;
    if (i < n) r = (int)gload(rows + i);
  }
}

// The operand of 16 tokens tg of one column and contraction window (first row row0) from the tile:
// lane (q, L) gets token L at the VL elements of its window.
__device__ __forceinline__ Mfma<true>::V tile_operand(const unsigned char* tile, int row0, int tg, int L) {
  unsigned w[4];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const unsigned char* p = tile + tile_at(row0 + 4 * h + (L >> 2), 32 * tg + 8 * (L & 3));
    const raw2 r = __builtin_bit_cast(raw2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                (__attribute__((address_space(3))) i16x4v*)(const_cast<unsigned char*>(p))));
    w[2 * h] = r.x;
    w[2 * h + 1] = r.y;
  }
  return __builtin_bit_cast(bf16x8, raw4{w[0], w[1], w[2], w[3]});
}

// out = s P v (+ beta out) from the tile for one group of blocks of a slab, through the stage, where
// the old values wait when BETA, so that each output is rounded once.  Work items as above (token
// groups past the slab's tokens are left out).  Factored blocks: the DFT of size k/4 of the four
// columns leaves each lane with two complex coordinates of all four, which the radix-4 stage, twiddles
// included, combines in registers in fp32; their stage takes the tile's LDS, so the results wait in registers until
// every wave has read the tile.
template <int KT, bool RADIX, bool BETA>
__device__ __forceinline__ void group_synthesis(const FrameDev& f, const void* frag, unsigned char* tile,
                                                unsigned char* stage, int nb, int nt, unsigned char* dst, long ld,
                                                float s, float beta) {
  using M = Mfma<true>;
  using V = M::V;
  using A = Act<true>;
  constexpr int ESZ = Slab::ESZ, S = Slab::S, NTH = Slab::NTG / 2;
  const int lane = phase_tid() & 63, q = lane >> 4, L = lane & 15;
  const int W2 = f.W2, cb = nb * f.W * ESZ / 16, sb = stage_stride(cb);
  const Items items(f.MT, nb);
  int have = -1;
  if constexpr (!RADIX) {
    V fr[KT];
    if (BETA) {
      stage_load<S>(dst, ld, nt, cb, stage);
      __syncthreads();
    }
    for (int it = items.i0; it < items.i1; ++it) {
      int mt, bl, th;
      items.get(it, mt, bl, th);
      if (16 * NTH * th >= nt) continue;   // uniform
      if (mt != have) load_frags<V, KT>(frag, mt, lane, fr);
      have = mt;
      f32x4 acc[NTH];
#pragma unroll
      for (int g = 0; g < NTH; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KT; ++ks) {
        const int e = min(ks * M::KS + q * M::VL, W2 - M::VL);
#pragma unroll
        for (int g = 0; g < NTH; ++g)
          acc[g] = M::step(fr[ks], tile_operand(tile, bl * W2 + e, NTH * th + g, L), acc[g]);
      }
      const int o = 16 * mt + 4 * q;
      if (o < W2) {
#pragma unroll
        for (int g = 0; g < NTH; ++g) {
          auto* p = reinterpret_cast<A::E*>(stage + (16 * (NTH * th + g) + L) * sb) + bl * W2 + o;
          f32x4 v = acc[g] * s;
          if (BETA) v += beta * A::ld4(p);
          A::st4(p, v);
        }
      }
    }
  } else {
    constexpr int NI = radix_items(KT);
    V fr[KT];
    float2 tw[2][3];   // of the lane's two complex coordinates
    // results as stored, or in fp32 until the old values are added
    using O = typename std::conditional<!BETA, unsigned, float2>::type;
    O out[NI][NTH][2][4];   // [item][token group][complex coordinate][a]
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      const int it = items.i0 + n;
      if (it >= items.i1) break;   // uniform
      int mt, bl, th;
      items.get(it, mt, bl, th);
      if (16 * NTH * th >= nt) continue;   // uniform
      if (mt != have) {
        load_frags<V, KT>(frag, mt, lane, fr);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
          for (int a = 0; a < 3; ++a) tw[u][a] = gload(f.tw + a * f.k2 + min(8 * mt + 2 * q + u, f.k2 - 1));
      }
      have = mt;
#pragma unroll
      for (int g = 0; g < NTH; ++g) {
        if (16 * (NTH * th + g) >= nt) break;   // uniform
        f32x4 acc[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) acc[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KT; ++ks) {
          const int e = min(ks * M::KS + q * M::VL, W2 - M::VL);
#pragma unroll
          for (int a = 0; a < 4; ++a)
            acc[a] = M::step(fr[ks], tile_operand(tile, a * W2 + e, NTH * th + g, L), acc[a]);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          float2 y[4];
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            y[a] = make_float2(acc[a][2 * u], acc[a][2 * u + 1]);
            if (a > 0) y[a] = cmul(y[a], tw[u][a - 1]);
          }
          const float2 s02 = cadd(y[0], y[2]), d02 = csub(y[0], y[2]), s13 = cadd(y[1], y[3]), d13 = csub(y[1], y[3]);
          float2 x[4];
          x[0] = cadd(s02, s13);
          x[1] = make_float2(d02.x - d13.y, d02.y + d13.x);   // d02 + i d13
          x[2] = csub(s02, s13);
          x[3] = make_float2(d02.x + d13.y, d02.y - d13.x);   // d02 - i d13
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            if constexpr (!BETA)
              out[n][g][u][a] = pk_bf2(s * x[a].x, s * x[a].y);
            else
              out[n][g][u][a] = make_float2(s * x[a].x, s * x[a].y);
          }
        }
        // one token group after the other: the scheduler would interleave them past the registers
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();   // the tile is read
    if (BETA) {
      stage_load<S>(dst, ld, nt, cb, stage);
      __syncthreads();
    }
#pragma unroll
    for (int n = 0; n < NI; ++n) {
      const int it = items.i0 + n;
      if (it >= items.i1) break;
      int mt, bl, th;
      items.get(it, mt, bl, th);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int o = 16 * mt + 4 * q + 2 * u;
        if (o >= W2) continue;
#pragma unroll
        for (int g = 0; g < NTH; ++g) {
          if (16 * (NTH * th + g) >= nt) break;   // uniform
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            auto* p = reinterpret_cast<A::E*>(stage + (16 * (NTH * th + g) + L) * sb) + a * W2 + o;
            if constexpr (BETA) {
              const float2 old = ld2<true>(p), v = out[n][g][u][a];
              st2<true>(p, make_float2(fmaf(beta, old.x, v.x), fmaf(beta, old.y, v.y)));
            } else {
              *reinterpret_cast<O*>(p) = out[n][g][u][a];
            }
          }
        }
      }
    }
  }
  __syncthreads();
  stage_store(stage, nt, cb, dst, ld);
}

struct SlabArgs {
  FrameDev f;               // the destination side's frame
  const void* fa;           // its fragments over clamped windows: analysis (backward), synthesis
  const void* fs;
  int T, slab0, nslab;      // as in AnaArgs
  int sg;                   // slabs per dC partial row (rows counted from slab 0)
  int nb, ngroups;          // as in SlabStream, of the destination side (group calls: the adapter's own)
  int nruns;                // partial-row runs of this launch; work items: groups x runs
  int stage_off;            // LDS offset of the stage (the tile is first)
  long src_slab;            // bytes of a source slab
  const unsigned char* ws;
  long ws_adapter;          // bytes between adapters (group calls: offset of wd in each adapter's pool)
  unsigned char* wd;        // multi-stage frames: the destination slabs
  const uint2* ent;
  long ent_adapter;
  const int* wstep;         // [group][kSlabWaves + 1]
  const int* zptr;          // [group + 1]: rows without entries, in zrow
  const unsigned short* zrow;
  const void* X;            // backward: x (block-local analysis)
  const void* const* Xs;
  long ldx;
  void* Y;                  // y / dX
  void* const* Ys;
  long ldy;
  float scale, beta;
  float* partial;           // [adapter][row][pstride]
  long pstride, prows;
  const SlabDesc* group;
  const int* tokens;
};

template <int KT, bool RADIX, bool BWD, bool DX, bool DC, bool BETA>
__device__ __forceinline__ void slab_pass(SlabArgs& a) {
  constexpr int S = Slab::S, ESZ = Slab::ESZ;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int bi = blockIdx.y;
  const unsigned char* ws = a.ws + (long)bi * a.ws_adapter;
  const uint2* ent = a.ent + (long)bi * a.ent_adapter;
  float* part = DC ? a.partial + (long)bi * a.prows * a.pstride : nullptr;
  int T = a.T;
  if (a.group) {
    const SlabDesc* d = a.group + bi;
    const SlabStream* st = BWD ? &d->bwd : &d->fwd;
    ws = sload(&d->ws);
    ent = sload(&d->ent);
    a.wstep = sload(&st->wstep);
    a.zptr = sload(&st->zptr);
    a.zrow = sload(&st->zrow);
    a.nb = sload(&st->nb);
    a.ngroups = sload(&st->ngroups);
    if (DC) {
      part = sload(&d->partial);
      a.pstride = 16L * sload(&st->steps);
    }
    T = adapter_tokens(a.tokens, a.T, bi);
  }
  const int nwork = a.ngroups * a.nruns, wi = xcd_item(blockIdx.x, nwork, bi);
  if (wi >= nwork) return;
  const int run = wi / a.ngroups, grp = wi - run * a.ngroups;
  const FrameDev& f = a.f;
  const int blk0 = grp * a.nb, nb = min(a.nb, f.nblk - blk0);
  const int row = a.slab0 / a.sg + run;   // dC partial row
  const int sl0 = max(a.slab0, row * a.sg), sl1 = min(a.slab0 + a.nslab, (row + 1) * a.sg);
  if ((long)sl0 * S >= T) return;   // uniform
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s0 = sload(a.wstep + grp * (kSlabWaves + 1) + wave), s1 = sload(a.wstep + grp * (kSlabWaves + 1) + wave + 1);
  const int z0 = sload(a.zptr + grp), z1 = sload(a.zptr + grp + 1);
  const long col = (long)blk0 * f.W * ESZ;   // the group's first column in a token row (bytes)
  unsigned char* Y = (!BWD || DX) ? reinterpret_cast<unsigned char*>(a.Ys ? sload(a.Ys + bi) : a.Y) + col : nullptr;
  const unsigned char* X = DC ? reinterpret_cast<const unsigned char*>(a.Xs ? sload(a.Xs + bi) : a.X) + col : nullptr;
  unsigned char* stage = smem + (RADIX ? 0 : a.stage_off);
  for (int sl = sl0; sl < sl1; ++sl) {
    const long t0 = (long)sl * S;
    const int nt = (int)min((long)S, (long)T - t0);
    if (nt <= 0) break;   // uniform
    if (sl > sl0) __syncthreads();   // the previous slab's LDS reads are done
    if constexpr (DC)   // z of the group's blocks into the tile
      group_analysis<KT, RADIX>(f, a.fa, X + t0 * a.ldx * ESZ, a.ldx * ESZ, nt, nb, smem, stage);
    const unsigned char* src = ws + (long)(sl - a.slab0) * a.src_slab;
    int zfirst = 0;
    if ((!BWD || DX) && z0 + (int)(threadIdx.x >> 3) < z1) zfirst = (int)gload(a.zrow + z0 + (threadIdx.x >> 3));
    slab_walk<!BWD || DX, DC>(ent, s0, s1, src, smem, DC ? part + (long)row * a.pstride : nullptr, sl != row * a.sg);
    if constexpr (!BWD || DX) {
      zero_rows(smem, a.zrow + z0, z1 - z0, zfirst);
      __syncthreads();
      group_synthesis<KT, RADIX, BETA>(f, a.fs, smem, stage, nb, nt, Y + t0 * a.ldy * ESZ, a.ldy * ESZ, a.scale, a.beta);
    }
  }
}

template <int KT, bool RADIX, bool BETA>
__global__ void __launch_bounds__(kSlabThreads, slab_wgs(KT, RADIX, BETA)) slab_fwd(SlabArgs a) {
  slab_pass<KT, RADIX, false, true, false, BETA>(a);
}

template <int KT, bool RADIX, bool DX, bool DC, bool BETA>
__global__ void __launch_bounds__(kSlabThreads, slab_wgs(KT, RADIX, BETA)) slab_bwd(SlabArgs a) {
  slab_pass<KT, RADIX, true, DX, DC, BETA>(a);
}

// One frame kind (slab_inst.hip).
struct SlabLaunch {
  hipError_t (*analysis)(const AnaArgs&, dim3 grid, size_t lds, hipStream_t s);
  hipError_t (*fwd)(const SlabArgs&, dim3 grid, size_t lds, hipStream_t s);
  hipError_t (*bwd)(const SlabArgs&, bool dx, bool dc, dim3 grid, size_t lds, hipStream_t s);
  hipError_t (*configure)();
};
// Multi-stage frames (slab_ms.hip).
constexpr int kMsThreads = 512, kMsWaves = kMsThreads / 64;
constexpr int kMsTok = 16;   // tokens of a workgroup: one MFMA group
struct MsOutArgs {
  FrameDev f;
  int T, slab0, nslab, nwork;
  const unsigned char* ws;   // destination slabs
  long ws_adapter;           // as in SlabArgs
  void* Y;
  void* const* Ys;
  long ldy;
  float scale, beta;
  const SlabDesc* group;
  const int* tokens;
};
hipError_t launch_ms_analysis(const AnaArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_ms_synthesis(const MsOutArgs& a, dim3 grid, hipStream_t s);
hipError_t launch_ms_pass(const SlabArgs& a, bool bwd, bool dx, bool dc, dim3 grid, hipStream_t s);
hipError_t configure_ms();

const SlabLaunch& launch_direct();
const SlabLaunch& launch_radix();

}  // namespace slab
}  // namespace ff
