// Sizes of the surrogate's reduction scratch: what its kernels write per block,
// and so what is allocated.  Host code only.
#pragma once

#include <algorithm>

namespace pf {

constexpr int kWgradBlocks = 512;  // blocks of one weight-gradient reduction, at most
constexpr int kProjBlocks = 512;   // blocks of the fused projection, at most (two per CU, walking the points)

// A wave of either kernel takes 32 points at a time, a block has four.
inline int point_blocks(long long P, int most) { return (int)std::min<long long>(most, (P / 32 + 3) / 4); }
inline int wgrad_blocks(long long P) { return point_blocks(P, kWgradBlocks); }
inline int proj_blocks(long long P) { return point_blocks(P, kProjBlocks); }

// Partial sums of a K x N weight gradient over P points: per block K rows and
// the bias's.
inline long long wgrad_elems(long long P, int K, int N) { return (long long)wgrad_blocks(P) * (K + 1) * N; }

// Partial sums of the fused projection's backward pass: those of P1 (w x h) and
// c1 of every block, then, from `second` on, those of P2 (h x co) and c2.
struct ProjParts {
  long long second, elems;
};
inline ProjParts proj_parts(long long P, int w, int h, int co) {
  const long long nb = proj_blocks(P), second = nb * (w + 1) * h;
  return {second, second + nb * (h + 1) * co};
}

// Elements of the partial-sum buffer: those of its largest user.
inline long long part_elems(long long P, int w, int h, int ci, int co, bool fuse_proj) {
  const long long layers = std::max(wgrad_elems(P, ci, w), wgrad_elems(P, w, w));
  return std::max(layers, fuse_proj ? proj_parts(P, w, h, co).elems
                                    : std::max(wgrad_elems(P, w, h), wgrad_elems(P, h, co)));
}

// Blocks of the kernels with one point per thread.
inline int pointwise_blocks(long long P) { return (int)((P + 255) / 256); }

// Elements of the per-block FP64 sums: the squared error (k_loss, or the fused
// projection's blocks) and the mass of an advance (k_apply).
inline long long dpart_elems(long long P, bool fuse_proj) {
  return std::max(pointwise_blocks(P), fuse_proj ? proj_blocks(P) : 0);
}

}  // namespace pf
