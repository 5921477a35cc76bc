// Prints what csrc/gemm_plan.h plans on 256 compute units (tests/test_gemm_plan.py): one line per request of
// mode M Nout K part_floats gemm_cfg gemm_parts gemm_ksplit on standard input, for every part of the plan
// rows:cfg:tiles:slices:reach:bm:bn (tile rows and columns), the few-rows kernels, which do not cut K, as
// rows:7:workgroups:1:reach:rg:ng:kw:s, all rows in a projection that normalises them with ":norm" behind it.  Reach: the byte
// offsets into a tile end below it (its rows of 2 K bytes), 0 where the kernel takes 64-bit addresses instead.  A mode with 16
// added has a LayerNorm without modulation in front.
// With the argument "norm": for every K that a projection normalises itself, "K first end missing", the elements of a
// row that the lanes of its wave read (first ... end - 1) and how many of the row none of them reads.
// With the argument "entropy": of every request of bytes rows images V, 1 where entropies and means are one launch, else 0.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <vector>

#include "entropy_core.h"
#include "gemm_plan.h"

size_t head_entropy_static_capacity() { return NOVA_HEAD_ENTROPY_STATIC_BYTES; }

static void norm_reads() {
  for (int K = 64; K <= kNormMaxK; K += 64) {
    std::vector<char> read(K, 0);
    int first = K, end = 0;
    for (int u = 0; u < (K + 511) / 512; ++u)
      for (int lane = 0; lane < 64; ++lane)
        for (int e = 0; e < 8; ++e) {
          const int at = norm_vector(u, lane, K) * 8 + e;
          first = std::min(first, at);
          end = std::max(end, at + 1);
          if (at >= 0 && at < K) read[at] = 1;
        }
    printf("%d %d %d %d\n", K, first, end, (int)std::count(read.begin(), read.end(), 0));
  }
}

static void entropy_launches() {
  int bytes, rows, batch, V;
  while (scanf("%d %d %d %d", &bytes, &rows, &batch, &V) == 4)
    printf("%d\n", bytes == 2 ? entropy_core::one_launch<bf16_t>(256, rows, batch, V) : entropy_core::one_launch<float>(256, rows, batch, V));
}

int main(int argc, char** argv) {
  if (argc > 1 && !strcmp(argv[1], "norm")) return norm_reads(), 0;
  if (argc > 1 && !strcmp(argv[1], "entropy")) return entropy_launches(), 0;
  long long part;
  int mode, M, Nout, K, cfg, parts, ksplit;
  while (scanf("%d %d %d %d %lld %d %d %d", &mode, &M, &Nout, &K, &part, &cfg, &parts, &ksplit) == 8) {
    nova_ctx c{};
    c.num_cus = 256;
    c.gemm_cfg = cfg;
    c.gemm_parts = parts;
    c.gemm_ksplit = ksplit;
    auto few_rows = [&](const RowsPlan& r, int rows, const char* norm) {
      printf("%d:7:%d:1:%lld:%d:%d:%d:%d%s ", rows, (rows + 8 * r.rg - 1) / (8 * r.rg) * (Nout / (8 * r.ng)),
             8LL * std::max(r.rg, r.ng) * 2 * K, r.rg, r.ng, r.kw, r.s, norm);
    };
    const bool norm = mode >= 16 && gemm_takes_norm(&c, mode & 15, M, Nout, K);
    mode &= 15;
    if (norm) {
      few_rows(gemm_norm_plan(256, mode, M, Nout, K), M, ":norm");
      printf("\n");
      continue;
    }
    const Plan p = plan_rows(&c, mode, M, Nout, K, part);
    for (int i = 0; i < p.n; ++i) {
      const int rows = p.m_end[i] - p.m_base[i];
      if (p.cfg[i] == kRowsCfg) {
        few_rows(gemm_rows_plan(256, mode, rows, Nout, K), rows, "");
        continue;
      }
      const bool low = low_launch(&c, p.cfg[i], mode, rows, Nout, K, part);
      const Candidate* t = &kCands[1];
      for (const Candidate& q : kCands)
        if (low ? low_tile(q) : q.cfg == p.cfg[i] && !low_tile(q)) t = &q;
      const int tiles = (rows + t->bm - 1) / t->bm * ((Nout + t->bn - 1) / t->bn);
      const int slices = cut_in_k(p.cfg[i], low) ? k_slices(256, mode, tiles, rows, Nout, K, part, ksplit) : 1;
      printf("%d:%d:%d:%d:%lld:%d:%d ", rows, p.cfg[i], tiles, slices, far_tile(K) ? 0 : 2LL * std::max(t->bm, t->bn) * K, t->bm,
             t->bn);
    }
    printf("\n");
  }
}
