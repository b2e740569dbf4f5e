// Slab kernels of frames applied in several radix-4 stages (blocks 544 to 4096 wide, bf16): such a block
// is too wide for a group's tile, so the destination side goes through the workspace as well.
//   ms_analysis   token rows -> workspace, 16 tokens of one block per workgroup
//   ms_pass       per (group of destination rows, slab): v = C z (or q = C^T u and the dC sums)
//                 gathered from the source slab, row by row into the destination slab; the backward's q
//                 takes the place of z
//   ms_synthesis  destination slab -> token rows
//
// A workgroup's 16 tokens of a block are kept in LDS as 4^S regions, region j holding column j of the
// multi-stage transform (inputs b + k2 j; after the stages the sequence of the DFT of size k2): first
// [token][k2 complex], 16-byte windows at an odd stride, then (the DFT's result, in the same LDS, a
// region being one wave's work) [coefficient][16 tokens].  The radix-4 stages run in place: the four
// lanes of a quad hold the 4^S values of one (token, b), read and written at the same places.
// What bounded the kernels this replaces (whole tokens of both sides in LDS, 9 tokens a tile): their
// token rows were read and written in 4-byte words of neighbouring lanes 128 bytes apart, one cache
// access each (2048 per 4096-wide token and pass).  4096 -> 4096 wide, rho = 2, 4096 tokens: a
// training step 280 -> 163 us; 1024 wide: 74 -> 62 us.  Vector instructions bound what is left: the stages of
// 16 tokens 4096 wide are 4 x 640 of them per wave, 9 of an analysis's 25 us (27.5 with the rows loaded
// before the stages and 32-bit integer products, of a quarter of the rate, in the addresses).
#include "slab_kernels.h"

namespace ff {
namespace slab {
namespace {

__device__ __host__ inline int ms_token_stride(int k2) { return (((4 * k2 + 15) / 16) | 1) * 16; }
// (a region's 64 extra bytes put the four regions that a quad of lanes reads on different banks)
__device__ __host__ inline int ms_region(int k2) { return kMsTok * ms_token_stride(k2) + 64; }

// This workgroup's 16 tokens of one block: slab and quarter of a slab, block.
struct MsTile {
  int sl, quarter, blk;
  __device__ __forceinline__ MsTile(int wi, int nblk) {
    const int t = wi / nblk;   // the four quarters of a slab's block are neighbours in time on one XCD
    blk = wi - t * nblk;
    sl = t >> 2;
    quarter = t & 3;
  }
};

// Base twiddles of the stages in LDS after the regions: of stage T < S for a = 1..3 and bq < 4 k2, then of
// stage S for a = 1..3 and b < k2.  (From memory, the waits for them would be waits for the token rows
// in flight.)
template <int S>
__device__ __host__ constexpr int ms_twiddles(int k2) {
  return 3 * k2 * (4 * (S - 1) + 1);
}
template <int S>
struct Twiddles {
  static constexpr int kU = 2;   // (at most 960 factors)
  float2 w[kU];
  __device__ __forceinline__ void fetch(const FrameDev& f) {
    const int k2 = f.k2, n = ms_twiddles<S>(k2), per = 12 * k2;
    const float inv = 1.f / (float)k2;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int i = min(phase_tid() + u * kMsThreads, n - 1);
      const int T = (i >= per) + (S > 2 && i >= 2 * per), r = i - T * per;
      const int a = div_small(r, k2, inv) >> (T == S - 1 ? 0 : 2), m = T == S - 1 ? k2 : 4 * k2;
      w[u] = gload(f.twk + (a + 1) * (r - a * m) * (1 << (2 * T)));
    }
  }
  __device__ __forceinline__ void put(const FrameDev& f, float2* tw) const {
    const int n = ms_twiddles<S>(f.k2);
#pragma unroll
    for (int u = 0; u < kU; ++u) tw[min(phase_tid() + u * kMsThreads, n - 1)] = w[u];
  }
};

// The radix-4 stages of every b of nt tokens from t0 on, in place.
template <int S, bool INV, bool BETA>
__device__ __forceinline__ void ms_stages(const FrameDev& f, unsigned char* lds, const float2* tw, int t0, int nt, float s,
                                          float beta, const unsigned char* old, long ld) {
  constexpr int NL = 1 << (2 * S - 2);
  const int k2 = f.k2, TS = ms_token_stride(k2), R = ms_region(k2);
  const float inv = 1.f / (float)k2;
  const int n = 4 * nt * k2;   // whole quads
  for (int i = phase_tid(); i < n; i += kMsThreads) {
    const int q = i & 3, it = i >> 2, tl = div_small(it, k2, inv), t = t0 + tl, b = it - __mul24(tl, k2);
    const int bq = b + __mul24(k2, q);
    unsigned char* p = lds + __mul24(t, TS) + 4 * b;
    float2 v[NL], w1[3], w2[3], wl[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      w1[a] = tw[4 * k2 * a + bq];
      if constexpr (S >= 3) w2[a] = tw[4 * k2 * (3 + a) + bq];
      wl[a] = tw[12 * k2 * (S - 1) + k2 * a + b];
    }
    if constexpr (!INV) {
#pragma unroll
      for (int m = 0; m < NL; ++m) v[m] = ld2<true>(reinterpret_cast<const u16*>(p + __mul24(q, R) + 4 * m * R));
      msr_stage<S, 1, false>(v, w1, k2, f.twk);
      if constexpr (S >= 3) msr_stage<S, 2, false>(v, w2, k2, f.twk);
      quad_transpose(v, q);
      msr_last_stage<S, false>(v, wl);
#pragma unroll
      for (int g = 0; g < NL / 4; ++g)
#pragma unroll
        for (int a = 0; a < 4; ++a) st2<true>(reinterpret_cast<u16*>(p + __mul24(4 * q, R) + (16 * g + a) * R), v[4 * g + a]);
    } else {
#pragma unroll
      for (int g = 0; g < NL / 4; ++g)
#pragma unroll
        for (int a = 0; a < 4; ++a) v[4 * g + a] = ld2<true>(reinterpret_cast<const u16*>(p + __mul24(4 * q, R) + (16 * g + a) * R));
      msr_last_stage<S, true>(v, wl);
      quad_transpose(v, q);
      if constexpr (S >= 3) msr_stage<S, 2, true>(v, w2, k2, f.twk);
      msr_stage<S, 1, true>(v, w1, k2, f.twk);
#pragma unroll
      for (int m = 0; m < NL; ++m) {
        float2 o = make_float2(s * v[m].x, s * v[m].y);
        if constexpr (BETA) {
          const float2 y = gld2<true>(reinterpret_cast<const u16*>(old + (long)t * ld) + 2 * (bq + 4 * k2 * m));
          o.x = fmaf(beta, y.x, o.x);
          o.y = fmaf(beta, y.y, o.y);
        }
        st2<true>(reinterpret_cast<u16*>(p + __mul24(q, R) + 4 * m * R), o);
      }
    }
  }
}

// A workgroup's token rows are moved in kMsRuns runs of kMsRun tokens (whole cache lines), so that one run's
// transfer goes on during another's stages.
constexpr int kMsRuns = 4, kMsRun = kMsTok / kMsRuns;
// Two waves take a token of a run, neighbouring lanes neighbouring pieces.
template <int S>
struct MsRows {
  static constexpr int PT = S == 3 ? 4 : 2;   // 16-byte pieces of a thread: blocks up to 4096, 2048 wide
  bool whole;                                 // k2 a multiple of four: a piece lies in one column
  int t, c[PT];                               // token of the run; piece (past the row: its last again)
  int at[PT], k2, R, b[PT];                   // its place in the token's LDS, first b
  int run;                                    // LDS from run to run
  __device__ __forceinline__ explicit MsRows(const FrameDev& f)
      : whole(f.k2 % 4 == 0), t(__builtin_amdgcn_readfirstlane(threadIdx.x >> 7)), k2(f.k2), R(ms_region(f.k2)),
        run(kMsRun * ms_token_stride(f.k2)) {
    const int cb = f.W / 8;
    const float inv = 1.f / (float)k2;
#pragma unroll
    for (int u = 0; u < PT; ++u) {
      c[u] = min((phase_tid() & 127) + 128 * u, cb - 1);
      const int j = div_small(4 * c[u], k2, inv);
      b[u] = 4 * c[u] - __mul24(j, k2);
      at[u] = __mul24(j, R) + 4 * b[u] + t * ms_token_stride(k2);
    }
  }
  // piece u of run r
  __device__ __forceinline__ void put(unsigned char* lds, int r, int u, u32x4v v) const {
    unsigned char* p = lds + r * run + at[u];
    if (whole) {   // uniform
      *reinterpret_cast<u32x4v*>(p) = v;
      return;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)   // (a column's end: on to the next one's start)
      *reinterpret_cast<unsigned*>(p + 4 * e + (b[u] + e >= k2 ? R - 4 * k2 : 0)) = v[e];
  }
  __device__ __forceinline__ u32x4v get(const unsigned char* lds, int r, int u) const {
    const unsigned char* p = lds + r * run + at[u];
    if (whole) return *reinterpret_cast<const u32x4v*>(p);
    u32x4v v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const unsigned*>(p + 4 * e + (b[u] + e >= k2 ? R - 4 * k2 : 0));
    return v;
  }
};

template <int S, int MT, int KT>
__global__ void __launch_bounds__(kMsThreads, 2) ms_analysis(AnaArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int bi = blockIdx.y;
  unsigned char* ws = a.ws + (long)bi * a.ws_adapter;
  int T = a.T;
  if (a.group) {
    ws = group_entries(a, bi) + (long)a.ws_adapter;
    T = adapter_tokens(a.tokens, a.T, bi);
  }
  if ((int)blockIdx.x >= a.nwork) {
    copy_entry(a, bi, ((int)blockIdx.x - a.nwork) * kMsThreads + (int)threadIdx.x);
    return;
  }
  const FrameDev& f = a.f;
  const MsTile tile(xcd_item(blockIdx.x, a.nwork, bi), f.nblk);
  const long ts = (long)(a.slab0 + tile.sl) * Slab::S, t0 = ts + kMsTok * tile.quarter;
  if (tile.sl >= a.nslab || ts >= T) return;   // uniform
  const int nt = (int)max(0L, min((long)kMsTok, T - t0));
  const int k2 = f.k2, W2 = f.W2, TS = ms_token_stride(k2), R = ms_region(k2), ncol = 1 << (2 * S);
  const long P = (long)f.nblk * f.W;
  unsigned char* out = ws + (long)tile.sl * (P + 1) * kSlabRowBytes;
  if (tile.blk == 0 && tile.quarter == 0 && threadIdx.x < 8)
    gstore(reinterpret_cast<u32x4v*>(out + P * kSlabRowBytes) + threadIdx.x, u32x4v{0u, 0u, 0u, 0u});
  out += (long)tile.blk * f.W * kSlabRowBytes + 2 * kMsTok * tile.quarter;
  const int tid = phase_tid(), lane = tid & 63, q = lane >> 4, L = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (nt == 0) {   // a quarter past the tokens: zeros
    for (int i = tid; i < 2 * f.W; i += kMsThreads)
      gstore(reinterpret_cast<u32x4v*>(out + (long)(i >> 1) * kSlabRowBytes + 16 * (i & 1)), u32x4v{0u, 0u, 0u, 0u});
    return;
  }
  const unsigned char* X = reinterpret_cast<const unsigned char*>(a.Xs ? sload(a.Xs + bi) : a.X) +
                           (t0 * a.ld + (long)tile.blk * f.W) * 2;
  float2* tw = reinterpret_cast<float2*>(smem + ncol * R);
  Twiddles<S> twid;
  twid.fetch(f);
  // the wave's fragments, the same for all its columns
  bf16x8 fr[MT][KT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) fr[mt][ks] = gload(reinterpret_cast<const bf16x8*>(f.fa16) + (mt * KT + ks) * 64 + lane);
  // every piece in flight at once, with no branch among the loads: the waits are then for the run at hand
  // (tokens past the end: the last one's pieces, put down as zeros)
  const MsRows<S> rows(f);
  u32x4v v[kMsRuns][MsRows<S>::PT];
#pragma unroll
  for (int r = 0; r < kMsRuns; ++r)
#pragma unroll
    for (int u = 0; u < MsRows<S>::PT; ++u)
      v[r][u] = gload(reinterpret_cast<const u32x4v*>(X + (long)min(kMsRun * r + rows.t, nt - 1) * a.ld * 2 + 16 * rows.c[u]));
  __builtin_amdgcn_sched_barrier(0);
  twid.put(f, tw);
  if (k2 % 4 != 0) {   // the windows' padding
    const int pad = 4 - k2 % 4;
    for (int i = tid; i < ncol * kMsTok * pad; i += kMsThreads) {
      const int jt = i / pad, e = i - jt * pad;
      *reinterpret_cast<unsigned*>(smem + (jt >> 4) * R + (jt & 15) * TS + 4 * (k2 + e)) = 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kMsRuns; ++r) {
#pragma unroll
    for (int u = 0; u < MsRows<S>::PT; ++u)
      rows.put(smem, r, u, kMsRun * r + rows.t < nt ? v[r][u] : u32x4v{0u, 0u, 0u, 0u});
    __syncthreads();
    if (kMsRun * r < nt) ms_stages<S, false, false>(f, smem, tw, kMsRun * r, kMsRun, 0.f, 0.f, nullptr, 0);
  }
  __syncthreads();
  const int nw = (W2 + 7) / 8;
  for (int j = wave; j < ncol; j += kMsWaves) {
    unsigned char* reg = smem + j * R;
    bf16x8 op[KT];
#pragma unroll
    for (int ks = 0; ks < KT; ++ks)   // (windows past the column: the last again, with zero weights)
      op[ks] = *reinterpret_cast<const bf16x8*>(reg + L * TS + 16 * min(4 * ks + q, nw - 1));
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KT; ++ks)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = Mfma<true>::step(op[ks], fr[mt][ks], acc[mt]);
    // four tokens of output 16 mt + L; the region's reads are done (the results depend on them)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (16 * mt + L < W2) *reinterpret_cast<uint2*>(reg + (16 * mt + L) * 32 + 8 * q) = Act<true>::pack4(acc[mt]);
    __asm__ volatile("" ::: "memory");   // (a wave's LDS operations execute in order)
    for (int i = lane; i < 2 * W2; i += 64)
      gstore(reinterpret_cast<u32x4v*>(out + (long)(j * W2 + (i >> 1)) * kSlabRowBytes + 16 * (i & 1)),
             *reinterpret_cast<const u32x4v*>(reg + (i >> 1) * 32 + 16 * (i & 1)));
  }
}

template <int S, int MT, int KT, bool BETA>
__global__ void __launch_bounds__(kMsThreads, 2) ms_synthesis(MsOutArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int bi = blockIdx.y;
  const unsigned char* ws = a.ws + (long)bi * a.ws_adapter;
  int T = a.T;
  if (a.group) {
    ws = sload(&a.group[bi].ws) + a.ws_adapter;
    T = adapter_tokens(a.tokens, a.T, bi);
  }
  const FrameDev& f = a.f;
  const MsTile tile(xcd_item(blockIdx.x, a.nwork, bi), f.nblk);
  const long t0 = (long)(a.slab0 + tile.sl) * Slab::S + kMsTok * tile.quarter;
  if (tile.sl >= a.nslab || t0 >= T) return;   // uniform
  const int nt = (int)min((long)kMsTok, T - t0);
  const int k2 = f.k2, W2 = f.W2, TS = ms_token_stride(k2), R = ms_region(k2), ncol = 1 << (2 * S);
  const long P = (long)f.nblk * f.W;
  const unsigned char* in = ws + ((long)tile.sl * (P + 1) + (long)tile.blk * f.W) * kSlabRowBytes + 2 * kMsTok * tile.quarter;
  unsigned char* Y = reinterpret_cast<unsigned char*>(a.Ys ? sload(a.Ys + bi) : a.Y) + (t0 * a.ldy + (long)tile.blk * f.W) * 2;
  const int tid = phase_tid(), lane = tid & 63, q = lane >> 4, L = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  float2* tw = reinterpret_cast<float2*>(smem + ncol * R);
  Twiddles<S> twid;
  twid.fetch(f);
  bf16x8 fr[MT][KT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) fr[mt][ks] = gload(reinterpret_cast<const bf16x8*>(f.ws16) + (mt * KT + ks) * 64 + lane);
  // a column is one wave's: its coefficients to LDS, two columns in flight, transformed and back as
  // [token][k2 complex]
  constexpr int kPC = (MT + 1) / 2;   // 16-byte pieces of a lane: a column's rows are two each
  u32x4v cv[2][kPC];
  auto fetch = [&](int j, u32x4v (&v)[kPC]) {
#pragma unroll
    for (int u = 0; u < kPC; ++u) {
      const int i = min(lane + 64 * u, 2 * W2 - 1);
      v[u] = gload(reinterpret_cast<const u32x4v*>(in + (long)(j * W2 + (i >> 1)) * kSlabRowBytes + 16 * (i & 1)));
    }
  };
  auto column = [&](int j, u32x4v (&v)[kPC]) {
    unsigned char* reg = smem + j * R;
#pragma unroll
    for (int u = 0; u < kPC; ++u) {
      const int i = min(lane + 64 * u, 2 * W2 - 1);
      *reinterpret_cast<u32x4v*>(reg + (i >> 1) * 32 + 16 * (i & 1)) = v[u];
    }
    if (j + 2 * kMsWaves < ncol) fetch(j + 2 * kMsWaves, v);   // (uniform)
    __asm__ volatile("" ::: "memory");   // (a wave's LDS operations execute in order)
    bf16x8 op[KT];
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) {   // token L at the 8 coefficients of its clamped window, by transposed reads
      const int e = min(32 * ks + 8 * q, W2 - 8);
      unsigned w[4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        unsigned char* p = reg + (e + 4 * h + (L >> 2)) * 32 + 8 * (L & 3);
        const raw2 r = __builtin_bit_cast(raw2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) i16x4v*)p));
        w[2 * h] = r.x;
        w[2 * h + 1] = r.y;
      }
      op[ks] = __builtin_bit_cast(bf16x8, raw4{w[0], w[1], w[2], w[3]});
    }
    f32x4 acc[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) acc[mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KT; ++ks)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = Mfma<true>::step(fr[mt][ks], op[ks], acc[mt]);
    // outputs 16 mt + 4 q .. + 3 of token L (the padding of a window may be written too)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (16 * mt + 4 * q < W2) *reinterpret_cast<uint2*>(reg + L * TS + (16 * mt + 4 * q) * 2) = Act<true>::pack4(acc[mt]);
  };
  fetch(wave, cv[0]);
  fetch(wave + kMsWaves, cv[1]);
  __builtin_amdgcn_sched_barrier(0);
  twid.put(f, tw);
  for (int j = wave; j < ncol; j += 2 * kMsWaves) {   // (ncol: 16 or 64)
    column(j, cv[0]);
    column(j + kMsWaves, cv[1]);
  }
  __syncthreads();
  const MsRows<S> rows(f);
#pragma unroll 1
  for (int r = 0; kMsRun * r < nt; ++r) {
    ms_stages<S, true, BETA>(f, smem, tw, kMsRun * r, min(kMsRun, nt - kMsRun * r), a.scale, a.beta, Y, a.ldy * 2);
    __syncthreads();
    const int t = kMsRun * r + rows.t;
    if (t < nt) {   // (uniform)
#pragma unroll
      for (int u = 0; u < MsRows<S>::PT; ++u)
        gstore(reinterpret_cast<u32x4v*>(Y + (long)t * a.ldy * 2 + 16 * rows.c[u]), rows.get(smem, r, u));
    }
  }
}

// The walk (slab_walk) with the destination rows in memory: dst is the destination slab's row of the
// group's first row, `zero` its row of zeros (what lanes without a row read).  The z row of every entry
// is gathered with its source row.
template <bool DX, bool DC>
__device__ __forceinline__ void ms_walk(const uint2* ent, int s0, int s1, const unsigned char* src, unsigned char* dst,
                                        const unsigned char* zero, unsigned dump, float* part, bool add) {
  constexpr int TC = Slab::TC;
  if (s0 >= s1) return;
  const int lane = phase_tid() & 63, c = lane & 3;
  const uint2* ep = ent + lane;
  struct Batch {
    unsigned w[4], c[4];
    u32x4v g[4][2], z[4][2];
  };
  auto issue = [&](uint2 m, Batch& b) {
    spread4(m.x, b.w);
    if (DX) spread4(m.y, b.c);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned off = (b.w[i] & kSlabSrcMask) * (unsigned)kSlabRowBytes + 16u * c;
      b.g[i][0] = gload(reinterpret_cast<const u32x4v*>(src + off));
      b.g[i][1] = gload(reinterpret_cast<const u32x4v*>(src + off + 64));
      if constexpr (DC) {
        const unsigned row = (b.w[i] >> kSlabDstShift) & kSlabDstMask;
        const unsigned char* zp = (row == dump ? zero : dst + row * (unsigned)kSlabRowBytes) + 16u * c;
        b.z[i][0] = gload(reinterpret_cast<const u32x4v*>(zp));
        b.z[i][1] = gload(reinterpret_cast<const u32x4v*>(zp + 64));
      }
    }
  };
  float acc[2 * TC];
#pragma unroll
  for (int t = 0; t < 2 * TC; ++t) acc[t] = 0.f;
  auto consume = [&](int s, Batch& b) {
    float dcv = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (DC) {
        const float d = quad_sum(dot16(b.g[i][1], b.z[i][1], dot16(b.g[i][0], b.z[i][0], 0.f)));
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
        const int last = __builtin_amdgcn_readfirstlane((int)b.w[i]);
        if (last < 0) {   // the bundle's last step (uniform)
          if (last & kSlabLevelMask) merge_quads((unsigned)last, acc);
          const unsigned row = (b.w[i] >> kSlabDstShift) & kSlabDstMask;
          if (row != dump) {
            unsigned char* p = dst + row * (unsigned)kSlabRowBytes + 16u * c;
            gstore(reinterpret_cast<u32x4v*>(p), pack16(acc));
            gstore(reinterpret_cast<u32x4v*>(p + 64), pack16(acc + TC));
          }
#pragma unroll
          for (int t = 0; t < 2 * TC; ++t) acc[t] = 0.f;
        }
      }
    }
    if constexpr (DC) {
      float* p = part + (long)s * 16 + lane;
      gstore(p, add ? gload(p) + dcv : dcv);
    }
  };
  // (rows are written behind the next batch's reads, which never are of rows whose bundle has ended)
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

template <bool BWD, bool DX, bool DC>
__global__ void __launch_bounds__(kSlabThreads, DC ? 2 : 3) ms_pass(SlabArgs a) {
  constexpr int S = Slab::S;
  const int bi = blockIdx.y;
  const unsigned char* ws = a.ws + (long)bi * a.ws_adapter;
  unsigned char* wd = a.wd + (long)bi * a.ws_adapter;
  const uint2* ent = a.ent + (long)bi * a.ent_adapter;
  float* part = DC ? a.partial + (long)bi * a.prows * a.pstride : nullptr;
  int T = a.T;
  if (a.group) {
    const SlabDesc* d = a.group + bi;
    const SlabStream* st = BWD ? &d->bwd : &d->fwd;
    ws = sload(&d->ws);
    wd = sload(&d->ws) + a.ws_adapter;
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
  const int row = a.slab0 / a.sg + run;   // dC partial row
  const int sl0 = max(a.slab0, row * a.sg), sl1 = min(a.slab0 + a.nslab, (row + 1) * a.sg);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int s0 = sload(a.wstep + grp * (kSlabWaves + 1) + wave), s1 = sload(a.wstep + grp * (kSlabWaves + 1) + wave + 1);
  const int z0 = sload(a.zptr + grp), z1 = sload(a.zptr + grp + 1);
  const long P = (long)a.f.nblk * a.f.W;
  for (int sl = sl0; sl < sl1; ++sl) {
    if ((long)sl * S >= T) break;   // uniform
    const unsigned char* src = ws + (long)(sl - a.slab0) * a.src_slab;
    unsigned char* slab = wd + (long)(sl - a.slab0) * (P + 1) * kSlabRowBytes;
    unsigned char* dst = slab + (long)grp * a.nb * kSlabRowBytes;
    ms_walk<DX, DC>(ent, s0, s1, src, dst, slab + P * kSlabRowBytes, (unsigned)a.nb,
                    DC ? part + (long)row * a.pstride : nullptr, sl != row * a.sg);
    if constexpr (DX)   // the coefficients of rows without entries
      for (int i = 8 * z0 + (int)threadIdx.x; i < 8 * z1; i += kSlabThreads)
        gstore(reinterpret_cast<u32x4v*>(dst + (int)gload(a.zrow + (i >> 3)) * kSlabRowBytes + 16 * (i & 7)),
               u32x4v{0u, 0u, 0u, 0u});
  }
}

// Output tiles and contraction steps of the DFTs of size k2: 17 to 64 points in two stages, to 32 in three.
#define MS_SHAPES(X)                                    \
  switch (a.f.nst * 64 + a.f.MT * 8 + a.f.KT) {         \
    case 2 * 64 + 3 * 8 + 2: X(2, 3, 2); break;         \
    case 2 * 64 + 4 * 8 + 2: X(2, 4, 2); break;         \
    case 2 * 64 + 5 * 8 + 3: X(2, 5, 3); break;         \
    case 2 * 64 + 6 * 8 + 3: X(2, 6, 3); break;         \
    case 2 * 64 + 7 * 8 + 4: X(2, 7, 4); break;         \
    case 2 * 64 + 8 * 8 + 4: X(2, 8, 4); break;         \
    case 3 * 64 + 3 * 8 + 2: X(3, 3, 2); break;         \
    case 3 * 64 + 4 * 8 + 2: X(3, 4, 2); break;         \
    default: return hipErrorInvalidValue;               \
  }

size_t ms_lds(const FrameDev& f) {
  return (size_t)f.ncol * ms_region(f.k2) + (f.nst == 2 ? ms_twiddles<2>(f.k2) : ms_twiddles<3>(f.k2)) * sizeof(float2);
}

template <class K>
hipError_t allow_lds(K* k) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
}

}  // namespace

hipError_t launch_ms_analysis(const AnaArgs& a, dim3 grid, hipStream_t s) {
  const size_t lds = ms_lds(a.f);
#define X(S, mt, kt) hipLaunchKernelGGL((ms_analysis<S, mt, kt>), grid, dim3(kMsThreads), lds, s, a)
  MS_SHAPES(X)
#undef X
  return hipGetLastError();
}

hipError_t launch_ms_synthesis(const MsOutArgs& a, dim3 grid, hipStream_t s) {
  const size_t lds = ms_lds(a.f);
#define X(S, mt, kt)                                                                                  \
  if (a.beta != 0.f)                                                                                  \
    hipLaunchKernelGGL((ms_synthesis<S, mt, kt, true>), grid, dim3(kMsThreads), lds, s, a);            \
  else                                                                                                \
    hipLaunchKernelGGL((ms_synthesis<S, mt, kt, false>), grid, dim3(kMsThreads), lds, s, a)
  MS_SHAPES(X)
#undef X
  return hipGetLastError();
}

hipError_t launch_ms_pass(const SlabArgs& a, bool bwd, bool dx, bool dc, dim3 grid, hipStream_t s) {
  if (!bwd)
    hipLaunchKernelGGL((ms_pass<false, true, false>), grid, dim3(kSlabThreads), 0, s, a);
  else if (dx && dc)
    hipLaunchKernelGGL((ms_pass<true, true, true>), grid, dim3(kSlabThreads), 0, s, a);
  else if (dx)
    hipLaunchKernelGGL((ms_pass<true, true, false>), grid, dim3(kSlabThreads), 0, s, a);
  else
    hipLaunchKernelGGL((ms_pass<true, false, true>), grid, dim3(kSlabThreads), 0, s, a);
  return hipGetLastError();
}

hipError_t configure_ms() {
  hipError_t e = hipSuccess;
#define ONE(S, mt, kt)                                                                             \
  for (const hipError_t r : {allow_lds(&ms_analysis<S, mt, kt>), allow_lds(&ms_synthesis<S, mt, kt, false>), \
                             allow_lds(&ms_synthesis<S, mt, kt, true>)})                              \
    if (r != hipSuccess) e = r;
  ONE(2, 3, 2) ONE(2, 4, 2) ONE(2, 5, 3) ONE(2, 6, 3) ONE(2, 7, 4) ONE(2, 8, 4) ONE(3, 3, 2) ONE(3, 4, 2)
#undef ONE
  return e;
}

}  // namespace slab
}  // namespace ff
