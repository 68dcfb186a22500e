// Checks the pose-graph factorisation's schedule (PgoPlan tiers, groups, steps) on
// graphs of several shapes, built with the sanitizers: every column in exactly one
// step, its descendants in earlier steps of its group or in earlier tiers, steps
// within the workgroup's limits, and the step-order copies equal to the plan's lists.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "../../paper_2506_04359_amd/csrc/pgo_plan.hpp"

using namespace ba;

#define CHECK(x)                                                        \
  do {                                                                  \
    if (!(x)) {                                                         \
      std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #x);      \
      std::exit(1);                                                     \
    }                                                                   \
  } while (0)

static void check(const char* name, int n, const std::vector<int32_t>& ei, const std::vector<int32_t>& ej,
                  bool fix_first = true) {
  PgoPlan P;
  std::vector<uint8_t> fixed(n, 0);
  if (fix_first) fixed[0] = 1;
  CHECK(build_pgo_plan(n, (int)ei.size(), ei.data(), ej.data(), fixed.data(), P).empty());
  const int nt = P.n_tiers(), ng = (int)P.grp_ptr.size() - 1, ns = (int)P.steps.size() / 8;
  CHECK(nt >= 1 && P.tier_ptr[0] == 0 && P.tier_ptr[nt] == ng && P.tier_ptr[nt] - P.tier_ptr[nt - 1] == 1);
  CHECK(P.grp_ptr[0] == 0 && P.grp_ptr[ng] == ns);
  std::vector<int> tier(P.n_free, -1), grp(P.n_free, -1), step(P.n_free, -1);
  size_t nab = 0, nbc = 0, nblk = 0, ncol = 0;
  int n_big = 0;
  for (int t = 0; t < nt; ++t)
    for (int g = P.tier_ptr[t]; g < P.tier_ptr[t + 1]; ++g)
      for (int s = P.grp_ptr[g]; s < P.grp_ptr[g + 1]; ++s) {
        const int32_t* st = &P.steps[8 * (size_t)s];
        const bool big = st[1] < 0;
        CHECK((size_t)st[0] == nab && (size_t)st[2] == nbc && (size_t)st[4] == nblk && (size_t)st[6] == ncol);
        CHECK(st[7] >= 1 && st[7] <= kStepCols && st[1] <= kStepChunks && st[3] <= kStepFwd && st[5] <= kStepBlks);
        n_big += big;
        int lq = 0, lf = 0, lb = 0;
        for (int i = 0; i < st[7]; ++i) {
          const int32_t* col = &P.step_col[8 * (size_t)(st[6] + i)];
          const int c = col[0];
          CHECK(c >= 0 && c < P.n_free && step[c] < 0);
          tier[c] = t;
          grp[c] = g;
          step[c] = s;
          CHECK(col[1] == P.blk_ptr[c] && col[2] == P.blk_ptr[c + 1] - P.blk_ptr[c]);
          if (big) {
            CHECK(st[7] == 1);
            continue;
          }
          CHECK(col[3] == lb && col[4] == lf);
          for (int k = 0; k < col[2]; ++k, ++lb) {
            const int b = col[1] + k;
            const int32_t* r = &P.step_blk[4 * (size_t)(st[4] + lb)];
            CHECK(r[0] == b && r[1] == lq && r[3] == (k ? P.blk_row[b] : -1));
            for (int q = P.chunk_ptr[b]; q < P.chunk_ptr[b + 1]; ++q, ++lq)
              for (int x = 0; x < 2 * kPgoChunk; ++x)
                CHECK(P.step_ab[2 * kPgoChunk * (size_t)(st[0] + lq) + x] == P.chunk_ab[2 * kPgoChunk * (size_t)q + x]);
            CHECK(r[2] == lq);
          }
          for (int q = P.fchunk_ptr[c]; q < P.fchunk_ptr[c + 1]; ++q, ++lf)
            for (int x = 0; x < 2 * kPgoChunk; ++x)
              CHECK(P.step_bc[2 * kPgoChunk * (size_t)(st[2] + lf) + x] == P.fchunk_bc[2 * kPgoChunk * (size_t)q + x]);
          CHECK(col[5] == lf);
        }
        if (!big) CHECK(lq == st[1] && lf == st[3] && lb == st[5]);
        nab += big ? 0 : lq;
        nbc += lf;
        nblk += lb;
        ncol += st[7];
      }
  CHECK(ncol == (size_t)P.n_free && P.step_col.size() == 8 * ncol && P.step_blk.size() == 4 * nblk);
  CHECK(P.step_ab.size() == 2 * kPgoChunk * nab && P.step_bc.size() == 2 * kPgoChunk * nbc);
  // what a column reads is done: the columns of its updates and forward updates
  auto before = [&](int k, int c) {
    return tier[k] < tier[c] || (tier[k] == tier[c] && grp[k] == grp[c] && step[k] < step[c]);
  };
  for (int c = 0; c < P.n_free; ++c) {
    CHECK(step[c] >= 0);
    for (int f = P.fwd_ptr[c]; f < P.fwd_ptr[c + 1]; ++f) CHECK(before(P.fwd_col[f], c));
    for (int b = P.blk_ptr[c]; b < P.blk_ptr[c + 1]; ++b) {
      for (int u = P.upd_ptr[b]; u < P.upd_ptr[b + 1]; ++u)
        CHECK(before(P.blk_col[P.upd_a[u]], c) && before(P.blk_col[P.upd_b[u]], c));
      if (b > P.blk_ptr[c]) CHECK(before(c, P.blk_row[b]));   // back substitution goes the other way
    }
  }
  std::printf("%s: %d columns, %d tiers, %d groups, %d steps, %d large\n", name, P.n_free, nt, ng, ns, n_big);
}

int main() {
  std::mt19937 rng(5);
  auto chain = [](int n, std::vector<int32_t>& i, std::vector<int32_t>& j) {
    for (int k = 0; k + 1 < n; ++k) i.push_back(k), j.push_back(k + 1);
  };
  for (int n : {2, 3, 17, 33, 34, 100, 1500}) {
    std::vector<int32_t> i, j;
    chain(n, i, j);
    check("chain", n, i, j);
  }
  for (int per : {30, 200, 500}) {   // laps with closures to the lap before
    std::vector<int32_t> i, j;
    const int n = 3 * per;
    chain(n, i, j);
    for (int k = per; k < n; ++k)
      for (int o = -1; o <= 1; ++o)
        if (k - per + o >= 0 && (rng() & 1)) i.push_back(k - per + o), j.push_back(k);
    check("laps", n, i, j);
  }
  for (int n : {5, 80, 200}) {   // every pair: one chain of large columns
    std::vector<int32_t> i, j;
    for (int a = 0; a < n; ++a)
      for (int b = a + 1; b < n; ++b) i.push_back(a), j.push_back(b);
    check("complete", n, i, j);
  }
  {
    std::vector<int32_t> i, j;   // a hub with many leaves
    for (int k = 1; k < 600; ++k) i.push_back(0), j.push_back(k);
    check("star", 600, i, j, false);
  }
  {
    std::vector<int32_t> i, j;   // random
    for (int k = 1; k < 400; ++k) i.push_back((int)(rng() % k)), j.push_back(k);
    for (int k = 0; k < 300; ++k) {
      const int a = (int)(rng() % 400), b = (int)(rng() % 400);
      if (a != b) i.push_back(a), j.push_back(b);
    }
    check("random", 400, i, j);
  }
  {
    std::vector<int32_t> i, j;   // many components
    for (int k = 0; k < 300; k += 3) i.push_back(k), j.push_back(k + 1);
    check("pairs", 300, i, j);
  }
  return 0;
}
