// CPU run of quad_env (fossen_quad.h), which gives the lanes of the kernels with
// one env per quad their envs: over fleets with declared classes that have no
// envs, first, in the middle and last, at the edges of a block's 16 envs, every
// block of a launch and the surplus one that the paired reverse sweep forms when
// the number of blocks is odd.  Every lane's column exists, every env has exactly
// one quad, and a quad is active if and only if it has an env.  No kernel is
// launched.  Prints "N failures".
#include <cstdio>
#include <vector>

#include "fossen_quad.h"

using namespace mg;

namespace {

int failures = 0;
void check(bool ok, const char* what, const std::vector<int64_t>& count) {
  if (ok) return;
  ++failures;
  if (failures > 20) return;
  std::printf("FAIL %s, classes of", what);
  for (int64_t c : count) std::printf(" %lld", (long long)c);
  std::printf(" envs\n");
}

// the classes' segments as mg_create lays them out
void run(const std::vector<int64_t>& count) {
  ClassSegs segs{};
  segs.n = (int32_t)count.size();
  int64_t off = 0, blk = 0;
  for (size_t k = 0; k < count.size(); ++k) {
    segs.start[k] = off;
    segs.len[k] = count[k];
    off += (count[k] + kSegAlign - 1) / kSegAlign * kSegAlign;
    blk += (count[k] + kQuadEnvs - 1) / kQuadEnvs;
    segs.blk_end[k] = (int32_t)blk;
  }
  AdjArgs a{};
  a.Ep = off > kSegAlign ? off : kSegAlign;
  std::vector<int> quads(a.Ep, 0);
  for (int b = 0; b < (int)(blk + (blk & 1)); ++b) {
    for (int lane = 0; lane < kQuadBlock; ++lane) {
      const QuadEnv e = quad_env(a, segs, b, lane);
      check(e.cls >= 0 && e.cls < segs.n, "class", count);
      check((int64_t)e.j < a.Ep, "column", count);
      if (!e.active) continue;
      check(b < blk, "active in the surplus block", count);
      const int64_t local = (int64_t)e.j - segs.start[e.cls];
      check(local >= 0 && local < segs.len[e.cls], "env of its class", count);
      if ((int64_t)e.j < a.Ep) ++quads[e.j];
    }
  }
  for (int k = 0; k < segs.n; ++k)
    for (int64_t i = 0; i < segs.len[k]; ++i)
      check(quads[segs.start[k] + i] == 4, "four lanes to an env", count);
  int64_t lanes = 0;
  for (int q : quads) lanes += q;
  int64_t envs = 0;
  for (int64_t c : count) envs += c;
  check(lanes == 4 * envs, "no other quad", count);
}

}  // namespace

int main() {
  for (int64_t n : {1, 15, 16, 17, 48, 64, 65, 500, 4096, 4097, 4585, 5001, 5104, 8177, 8192}) {
    run({n});
    run({n, 0});
    run({0, n});
    run({n, 0, 0});
    run({0, n, 0});
    run({n, 0, 33});
    run({n, 1, 0, 16, 0});
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
