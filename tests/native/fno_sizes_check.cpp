// Walks every surrogate shape that pf_fno_create accepts (host only) and checks
// that each block's partial sums and scalar sums lie inside the scratch allocated for them and
// apart from the others'.  Prints "ok <shapes>" or the first shape that fails.
#include <cstdio>

#include "../../paper_2609_36100_amd/csrc/pf_fno_sizes.hpp"

int main() {
  long long shapes = 0;
  for (int n = 8; n <= 256; n += 8)
    for (int w = 4; w <= 128; w += 4)
      for (int h = 8; h <= 128; h += 8)
        for (int ci = 1; ci <= 8; ++ci)
          for (int co = 1; co <= 8; ++co) {
            const long long P = (long long)n * n * n;
            const bool fuse = w <= 32;
            const long long cap = pf::part_elems(P, w, h, ci, co, fuse);
            bool ok = true;
            // one weight gradient: block b's set is [b, b + 1) (K + 1) N
            auto sets = [&](int K, int N) {
              const long long nb = pf::wgrad_blocks(P), set = (long long)(K + 1) * N;
              ok = ok && nb >= 1 && (nb - 1) * set + K * N + N <= cap;
            };
            sets(ci, w);
            sets(w, w);
            if (fuse) {
              const long long nb = pf::proj_blocks(P), s1 = (long long)(w + 1) * h, s2 = (long long)(h + 1) * co;
              const pf::ProjParts p = pf::proj_parts(P, w, h, co);
              ok = ok && nb >= 1 && (nb - 1) * s1 + w * h + h <= p.second && p.second + (nb - 1) * s2 + h * co + co <= cap;
            } else {
              sets(w, h);
              sets(h, co);
            }
            const long long sums = pf::dpart_elems(P, fuse);
            const bool dok = pf::pointwise_blocks(P) <= sums && (!fuse || pf::proj_blocks(P) <= sums);
            if (!ok || !dok) {
              std::printf("%s n %d w %d h %d cin %d cout %d\n", ok ? "sums" : "part", n, w, h, ci, co);
              return 1;
            }
            ++shapes;
          }
  std::printf("ok %lld\n", shapes);
  return 0;
}
