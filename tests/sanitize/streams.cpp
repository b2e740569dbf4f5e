// The slab kernels' entry streams, walked on the CPU against the stand-in of hip_host_stub.cpp: every
// entry of the support occurs once in each direction's stream with its own coefficient slot, the sums
// that the walk leaves in the destination rows are those of the support, and the padding is bounded.
// Exit status: the number of failed checks.
#include <cstdio>
#include <map>
#include <random>
#include <set>
#include <vector>

#include "ff_internal.h"
#include "frameft.h"

static int g_failed = 0;
#define CHECK(cond)                                                                                     \
  do {                                                                                                  \
    if (!(cond)) {                                                                                      \
      if (g_failed < 20) std::fprintf(stderr, "FAILED %s:%d: %s [%s]\n", __FILE__, __LINE__, #cond, g_name); \
      ++g_failed;                                                                                       \
    }                                                                                                   \
  } while (0)

namespace {

const char* g_name = "";

// src_of / dst_of: canonical index -> position, learnt from the first stream and the same in the second.
void walk(const ff_plan* p, const ff::SlabStream& st, const ff::FrameDev& dst, int64_t nsrc, const std::vector<int>& src_id,
          const std::vector<int>& dst_id, std::map<int, int>& src_of, std::map<int, int>& dst_of) {
  std::vector<int64_t> order((size_t)p->user_order.size());
  CHECK(ff_plan_order(p, order.data()) == FF_OK);
  const int64_t nnz = p->nnz;
  const int per = ff::slab_ms_frame(dst) ? st.nb : st.nb * dst.W, dump = per;
  std::vector<int> seen((size_t)nnz, 0);
  // integer values by position and coefficients by entry: the sums are exact
  auto x = [](int pos) { return (int64_t)(pos * 37 % 101 - 50); };
  auto c = [](int64_t e) { return (int64_t)(e * 53 % 97 - 48); };
  std::map<int, int64_t> got, want;
  int64_t end = 0;
  for (int g = 0; g < st.ngroups; ++g)
    for (int w = 0; w < ff::kSlabWaves; ++w) {
      const int s0 = st.wstep[g * (ff::kSlabWaves + 1) + w], s1 = st.wstep[g * (ff::kSlabWaves + 1) + w + 1];
      CHECK(s0 % 4 == 0 && s1 % 4 == 0 && s0 <= s1 && s0 == end);
      end = s1;
      int64_t acc[16] = {0};
      for (int s = s0; s < s1; ++s) {
        uint32_t word[16];
        for (int l = 0; l < 16; ++l) {
          const size_t j = (size_t)s / 4 * 64 + 4 * l + s % 4;
          word[l] = st.word[j];
          const int src = (int)(word[l] & ff::kSlabSrcMask), row = (int)(word[l] >> ff::kSlabDstShift & ff::kSlabDstMask);
          const int slot = st.coef[j];
          CHECK(src <= nsrc && row <= dump);
          if (slot < 0) {
            CHECK(src == nsrc);   // padding reads the row of zeros
            continue;
          }
          const int64_t e = order[(size_t)slot];
          CHECK(e >= 0 && e < nnz && row < per);
          if (e < 0 || e >= nnz) continue;
          ++seen[(size_t)e];
          const int pos = g * per + row;
          CHECK(src_of.emplace(src_id[e], src).first->second == src);
          CHECK(dst_of.emplace(dst_id[e], pos).first->second == pos);
          acc[l] += c(e) * x(src);
          want[pos] += c(e) * x(src);
        }
        if (word[0] & 0x80000000u) {
          const int level = (int)((word[0] & ff::kSlabLevelMask) >> ff::kSlabLevelShift);
          CHECK(level <= ff::kSlabMaxLevel);
          for (int d = 1; d < 1 << level; d <<= 1) {
            int64_t sum[16];
            for (int l = 0; l < 16; ++l) sum[l] = acc[l] + acc[l ^ d];
            for (int l = 0; l < 16; ++l) acc[l] = sum[l];
          }
          for (int l = 0; l < 16; ++l) {
            CHECK((word[l] & (0x80000000u | ff::kSlabLevelMask)) == (word[0] & (0x80000000u | ff::kSlabLevelMask)));
            const int row = (int)(word[l] >> ff::kSlabDstShift & ff::kSlabDstMask);
            if (row != dump) {
              const int pos = g * per + row;
              const auto it = got.find(pos);
              // (lanes of one row write the same sum)
              CHECK(it == got.end() || (level > 0 && it->second == acc[l]));
              got[pos] = acc[l];
            }
            acc[l] = 0;
          }
        }
      }
      for (int l = 0; l < 16; ++l) CHECK(acc[l] == 0);   // (steps after the last bundle are padding)
    }
  CHECK(end == st.steps && got == want);
  for (int64_t e = 0; e < nnz; ++e) CHECK(seen[(size_t)e] == 1);
  // the bounds that ff_adapter_bwd_noalloc's scratch rests on
  const int64_t words = 16L * st.steps;
  CHECK(words <= nnz + nnz / 2 + 448L * st.ngroups);
  std::printf("%s: %ld entries, %ld words in %d groups\n", g_name, (long)nnz, (long)words, st.ngroups);
}

void run(const char* name, const int64_t* fi, const int64_t* fo, const std::vector<int32_t>& rows,
         const std::vector<int32_t>& cols, int64_t tokens) {
  g_name = name;
  ff_frame *a = nullptr, *b = nullptr;
  CHECK(ff_framegen(fi[0], fi[1], fi[2], &a) == FF_OK && ff_framegen(fo[0], fo[1], fo[2], &b) == FF_OK);
  ff_plan* p = nullptr;
  CHECK(ff_plan_create(a, b, (int64_t)rows.size(), rows.data(), cols.data(), tokens, 1, &p) == FF_OK);
  if (p) {
    CHECK(p->slab.enabled);
    std::vector<int> r(rows.begin(), rows.end()), c(cols.begin(), cols.end());
    std::map<int, int> in, out;
    walk(p, p->slab.fwd, b->dev, fi[0], c, r, in, out);
    walk(p, p->slab.bwd, a->dev, fo[0], r, c, out, in);
    for (auto* m : {&in, &out}) {
      std::set<int> positions;
      for (const auto& kv : *m) CHECK(positions.insert(kv.second).second);
    }
  }
  ff_plan_destroy(p);
  ff_frame_destroy(a);
  ff_frame_destroy(b);
}

}  // namespace

int main() {
  // (d, k, rho): blocks applied directly, in one radix-4 stage, in two
  const int64_t direct[] = {1024, 16, 64}, wide[] = {2048, 64, 32}, factored[] = {688, 172, 4}, stages[] = {1024, 512, 2};
  const int64_t* frames[] = {direct, wide, factored, stages};
  const char* kinds[] = {"uniform", "dense_columns", "dense_rows", "one_dense_each", "long_tail"};
  std::mt19937_64 g(5);
  char name[96];
  for (const int64_t* fi : frames)
    for (const int64_t* fo : frames)
      for (int kind = 0; kind < 5; ++kind)
        for (int64_t tokens : {40, 40000}) {   // small and large groups
          if (fi == wide && fo == wide) continue;   // the fused kernels
          const int64_t n = fi[0], m = fo[0];
          std::set<std::pair<int32_t, int32_t>> sup;
          auto add = [&](int64_t r, int64_t c) { sup.emplace((int32_t)(r % m), (int32_t)(c % n)); };
          if (kind == 0)
            for (int i = 0; i < 3000; ++i) add((int64_t)(g() >> 1), (int64_t)(g() >> 1));
          if (kind == 1 || kind == 3)
            for (int64_t c = 0; c < n; c += kind == 1 ? 64 : n)
              for (int64_t r = 0; r < m; ++r) add(r, c + 5);
          if (kind == 2 || kind == 3)
            for (int64_t r = 0; r < m; r += kind == 2 ? 64 : m)
              for (int64_t c = 0; c < n; ++c) add(r + 3, c);
          if (kind == 4)   // row and column counts falling off like 1 / i
            for (int64_t i = 0; i < m; ++i)
              for (int64_t k = 0; k < n / (i + 1); ++k) add(i * 7, (int64_t)(g() >> 1) % (k + 1));
          std::vector<int32_t> rows, cols;
          for (const auto& rc : sup) rows.push_back(rc.first), cols.push_back(rc.second);
          std::snprintf(name, sizeof name, "%ld -> %ld %s, %ld tokens", (long)n, (long)m, kinds[kind], (long)tokens);
          run(name, fi, fo, rows, cols, tokens);
        }
  std::printf("streams: %d failed checks\n", g_failed);
  return g_failed != 0;
}
