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
// training step 280 -> 175 us; 1024 wide: 74 -> 68 us.
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

// The radix-4 stages of every (token, b) in place.
template <int S, bool INV, bool BETA>
__device__ __forceinline__ void ms_stages(const FrameDev& f, unsigned char* lds, int nt, float s, float beta,
                                          const unsigned char* old, long ld) {
  constexpr int NL = 1 << (2 * S - 2);
  const int k2 = f.k2, TS = ms_token_stride(k2), R = ms_region(k2);
  const float inv = 1.f / (float)k2;
  const int n = 4 * nt * k2;   // whole quads
  for (int i = phase_tid(); i < n; i += kMsThreads) {
    const int q = i & 3, it = i >> 2, t = div_small(it, k2, inv), b = it - t * k2, bq = b + k2 * q;
    unsigned char* p = lds + t * TS + 4 * b;
    float2 v[NL];
    if constexpr (!INV) {
#pragma unroll
      for (int m = 0; m < NL; ++m) v[m] = ld2<true>(reinterpret_cast<const u16*>(p + (4 * m + q) * R));
      msr_stage<S, 1, false>(v, bq, k2, f.twk);
      if constexpr (S >= 3) msr_stage<S, 2, false>(v, bq, k2, f.twk);
      quad_transpose(v, q);
      msr_last_stage<S, false>(v, b, f.twk);
#pragma unroll
      for (int g = 0; g < NL / 4; ++g)
#pragma unroll
        for (int a = 0; a < 4; ++a) st2<true>(reinterpret_cast<u16*>(p + (16 * g + 4 * q + a) * R), v[4 * g + a]);
    } else {
#pragma unroll
      for (int g = 0; g < NL / 4; ++g)
#pragma unroll
        for (int a = 0; a < 4; ++a) v[4 * g + a] = ld2<true>(reinterpret_cast<const u16*>(p + (16 * g + 4 * q + a) * R));
      msr_last_stage<S, true>(v, b, f.twk);
      quad_transpose(v, q);
      if constexpr (S >= 3) msr_stage<S, 2, true>(v, bq, k2, f.twk);
      msr_stage<S, 1, true>(v, bq, k2, f.twk);
#pragma unroll
      for (int m = 0; m < NL; ++m) {
        float2 o = make_float2(s * v[m].x, s * v[m].y);
        if constexpr (BETA) {
          const float2 y = gld2<true>(reinterpret_cast<const u16*>(old + (long)t * ld) + 2 * (bq + 4 * k2 * m));
          o.x = fmaf(beta, y.x, o.x);
          o.y = fmaf(beta, y.y, o.y);
        }
        st2<true>(reinterpret_cast<u16*>(p + (4 * m + q) * R), o);
      }
    }
  }
}

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
  const long ts = (long)(a.slab0 + tile.sl) * SlabT<true>::S, t0 = ts + kMsTok * tile.quarter;
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
  {   // token rows, 16 bytes per lane; the windows' padding and the tokens past the end are zero
    const unsigned char* X = reinterpret_cast<const unsigned char*>(a.Xs ? sload(a.Xs + bi) : a.X) +
                             (t0 * a.ld + (long)tile.blk * f.W) * 2;
    const int cb = f.W / 8;   // 16-byte chunks (4 complex coordinates) of a block's row
    const float inv_cb = 1.f / (float)cb, inv_k2 = 1.f / (float)k2;
    constexpr int kU = 4;
    for (int i0 = tid; i0 < kMsTok * cb; i0 += kU * kMsThreads) {
      u32x4v v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = min(i0 + u * kMsThreads, kMsTok * cb - 1), t = div_small(i, cb, inv_cb), c = i - t * cb;
        v[u] = gload(reinterpret_cast<const u32x4v*>(X + (long)min(t, nt - 1) * a.ld * 2 + 16 * c));
        if (t >= nt) v[u] = u32x4v{0u, 0u, 0u, 0u};
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = i0 + u * kMsThreads;
        if (i >= kMsTok * cb) break;
        const int t = div_small(i, cb, inv_cb), nn = 4 * (i - t * cb);
        int j = div_small(nn, k2, inv_k2), b = nn - j * k2;
        unsigned char* p = smem + t * TS;
        if (k2 % 4 == 0) {   // uniform: the chunk lies in one column
          *reinterpret_cast<u32x4v*>(p + j * R + 4 * b) = v[u];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            *reinterpret_cast<unsigned*>(p + j * R + 4 * b) = v[u][e];
            if (++b == k2) b = 0, ++j;
          }
        }
      }
    }
    if (k2 % 4 != 0) {
      const int pad = 4 - k2 % 4;
      for (int i = tid; i < ncol * kMsTok * pad; i += kMsThreads) {
        const int jt = i / pad, e = i - jt * pad;
        *reinterpret_cast<unsigned*>(smem + (jt >> 4) * R + (jt & 15) * TS + 4 * (k2 + e)) = 0u;
      }
    }
  }
  // the wave's fragments, the same for all its columns
  bf16x8 fr[MT][KT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) fr[mt][ks] = gload(reinterpret_cast<const bf16x8*>(f.fa16) + (mt * KT + ks) * 64 + lane);
  __syncthreads();
  ms_stages<S, false, false>(f, smem, kMsTok, 0.f, 0.f, nullptr, 0);
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
  const long t0 = (long)(a.slab0 + tile.sl) * SlabT<true>::S + kMsTok * tile.quarter;
  if (tile.sl >= a.nslab || t0 >= T) return;   // uniform
  const int nt = (int)min((long)kMsTok, T - t0);
  const int k2 = f.k2, W2 = f.W2, TS = ms_token_stride(k2), R = ms_region(k2), ncol = 1 << (2 * S);
  const long P = (long)f.nblk * f.W;
  const unsigned char* in = ws + ((long)tile.sl * (P + 1) + (long)tile.blk * f.W) * kSlabRowBytes + 2 * kMsTok * tile.quarter;
  unsigned char* Y = reinterpret_cast<unsigned char*>(a.Ys ? sload(a.Ys + bi) : a.Y) + (t0 * a.ldy + (long)tile.blk * f.W) * 2;
  const int tid = phase_tid(), lane = tid & 63, q = lane >> 4, L = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  {
    const float inv = 1.f / (float)W2;
    constexpr int kU = 4;
    const int n = 2 * f.W;
    for (int i0 = tid; i0 < n; i0 += kU * kMsThreads) {
      u32x4v v[kU];
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = min(i0 + u * kMsThreads, n - 1);
        v[u] = gload(reinterpret_cast<const u32x4v*>(in + (long)(i >> 1) * kSlabRowBytes + 16 * (i & 1)));
      }
#pragma unroll
      for (int u = 0; u < kU; ++u) {
        const int i = i0 + u * kMsThreads;
        if (i >= n) break;
        const int row = i >> 1, j = div_small(row, W2, inv);
        *reinterpret_cast<u32x4v*>(smem + j * R + (row - j * W2) * 32 + 16 * (i & 1)) = v[u];
      }
    }
  }
  bf16x8 fr[MT][KT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ks = 0; ks < KT; ++ks) fr[mt][ks] = gload(reinterpret_cast<const bf16x8*>(f.ws16) + (mt * KT + ks) * 64 + lane);
  __syncthreads();
  for (int j = wave; j < ncol; j += kMsWaves) {
    unsigned char* reg = smem + j * R;
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
  }
  __syncthreads();
  ms_stages<S, true, BETA>(f, smem, nt, a.scale, a.beta, Y, a.ldy * 2);
  __syncthreads();
  const int cb = f.W / 8;
  const float inv_cb = 1.f / (float)cb, inv_k2 = 1.f / (float)k2;
  for (int i = tid; i < nt * cb; i += kMsThreads) {
    const int t = div_small(i, cb, inv_cb), c = i - t * cb, nn = 4 * c;
    int j = div_small(nn, k2, inv_k2), b = nn - j * k2;
    const unsigned char* p = smem + t * TS;
    u32x4v v;
    if (k2 % 4 == 0) {
      v = *reinterpret_cast<const u32x4v*>(p + j * R + 4 * b);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] = *reinterpret_cast<const unsigned*>(p + j * R + 4 * b);
        if (++b == k2) b = 0, ++j;
      }
    }
    gstore(reinterpret_cast<u32x4v*>(Y + (long)t * a.ldy * 2 + 16 * c), v);
  }
}

// The walk (slab_walk) with the destination rows in memory: dst is the destination slab's row of the
// group's first row, `zero` its row of zeros (what lanes without a row read).  The z row of every entry
// is gathered with its source row.
template <bool DX, bool DC>
__device__ __forceinline__ void ms_walk(const uint2* ent, int s0, int s1, const unsigned char* src, unsigned char* dst,
                                        const unsigned char* zero, unsigned dump, float* part, bool add) {
  constexpr int TC = SlabT<true>::TC;
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
        const float d = quad_sum(dot16<true>(b.g[i][1], b.z[i][1], dot16<true>(b.g[i][0], b.z[i][0], 0.f)));
        dcv = c == i ? d : dcv;
      }
      if constexpr (DX) {
        float x[2][TC];
        unpack16<true>(b.g[i][0], x[0]);
        unpack16<true>(b.g[i][1], x[1]);
        const float cc = __uint_as_float(b.c[i]);
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
          for (int t = 0; t < TC; ++t) acc[k * TC + t] = fmaf(cc, x[k][t], acc[k * TC + t]);
        if (__builtin_amdgcn_readfirstlane((int)b.w[i]) < 0) {   // the bundle's last step (uniform)
          const unsigned row = (b.w[i] >> kSlabDstShift) & kSlabDstMask;
          if (row != dump) {
            unsigned char* p = dst + row * (unsigned)kSlabRowBytes + 16u * c;
            gstore(reinterpret_cast<u32x4v*>(p), pack16<true>(acc));
            gstore(reinterpret_cast<u32x4v*>(p + 64), pack16<true>(acc + TC));
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
  constexpr int S = SlabT<true>::S;
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

#define MS_SHAPES(S, X)                     \
  switch (a.f.MT * 8 + a.f.KT) {            \
    case 3 * 8 + 2: X(S, 3, 2); break;      \
    case 4 * 8 + 2: X(S, 4, 2); break;      \
    case 5 * 8 + 3: X(S, 5, 3); break;      \
    case 6 * 8 + 3: X(S, 6, 3); break;      \
    case 7 * 8 + 4: X(S, 7, 4); break;      \
    case 8 * 8 + 4: X(S, 8, 4); break;      \
    default: return hipErrorInvalidValue;   \
  }

size_t ms_lds(const FrameDev& f) { return (size_t)f.ncol * ms_region(f.k2); }

template <class K>
hipError_t allow_lds(K* k) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLdsBytes);
}

}  // namespace

hipError_t launch_ms_analysis(const AnaArgs& a, dim3 grid, hipStream_t s) {
  const size_t lds = ms_lds(a.f);
#define X(S, mt, kt) hipLaunchKernelGGL((ms_analysis<S, mt, kt>), grid, dim3(kMsThreads), lds, s, a)
  if (a.f.nst == 2) {
    MS_SHAPES(2, X)
  } else {
    MS_SHAPES(3, X)
  }
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
  if (a.f.nst == 2) {
    MS_SHAPES(2, X)
  } else {
    MS_SHAPES(3, X)
  }
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
#define ALL(S) ONE(S, 3, 2) ONE(S, 4, 2) ONE(S, 5, 3) ONE(S, 6, 3) ONE(S, 7, 4) ONE(S, 8, 4)
  ALL(2) ALL(3)
#undef ALL
#undef ONE
  return e;
}

}  // namespace slab
}  // namespace ff
