// Plane passes of single grids (FP64, nx == ny).
#include "pf_plane.hpp"

#include <type_traits>

#include "pf_context.hpp"

namespace pf {

template <int N>
__global__ void __launch_bounds__(PlaneGeo<N>::THREADS)
k_plane_theta(const cx<double>* __restrict__ st, cx<double>* __restrict__ th, Geo g, const cx<double>* twN,
              const cx<double>* twM) {
  __shared__ cx<double> pl[PlaneGeo<N>::STRIDE];
  __shared__ cx<double> sN[N], sM[N / 2];
  for (int j = threadIdx.x; j < N; j += PlaneGeo<N>::THREADS) {
    sN[j] = twN[j];
    if (j < N / 2) sM[j] = twM[j];
  }
  __syncthreads();
  body_plane_theta<N>(st, th, g, sN, sM, blockIdx.x, blockIdx.y, threadIdx.x, pl);
}

template <int N>
__global__ void __launch_bounds__(3 * PlaneGeo<N>::THREADS)
k_plane_drive(const cx<double>* __restrict__ st, cx<double>* __restrict__ el, Geo g, ModelK m, const cx<double>* twN,
              const cx<double>* twM) {
  static_assert(PlaneGeo<N>::OK, "three planes per work-group");
  __shared__ cx<double> pl[3 * PlaneGeo<N>::STRIDE];
  __shared__ cx<double> sN[N], sM[N / 2];
  for (int j = threadIdx.x; j < N; j += 3 * PlaneGeo<N>::THREADS) {
    sN[j] = twN[j];
    if (j < N / 2) sM[j] = twM[j];
  }
  __syncthreads();
  body_plane_drive<N>(st, el, g, m, sN, sM, blockIdx.x, blockIdx.y, threadIdx.x, pl);
}

// The plane passes take every grid whose planes they are compiled for, with any
// number of planes: four ARK4 steps with the separate passes and with these took
// 1.165 and 1.163 ms on 64 x 64 x 8, 1.869 and 1.529 on 64^3, 7.93 and 7.87 on
// 64 x 64 x 512, 5.42 and 5.25 on 48 x 48 x 512, 2.93 and 2.30 on 32 x 32 x 512,
// 1.18 and 0.74 on 16^3, 1.48 and 1.21 on 8 x 8 x 512: slower on none.
template <class F>
static bool plane_dispatch(const Geo& g, F&& f) {
  if (g.nx != g.ny) return false;
  switch (g.nx) {
#define PF_CASE(N)                       \
  case N:                                \
    f(std::integral_constant<int, N>{}); \
    return true;
    PF_CASE(8) PF_CASE(16) PF_CASE(24) PF_CASE(32) PF_CASE(48) PF_CASE(64)
#undef PF_CASE
    default:
      return false;
  }
}

bool plane_supported(const Geo& g) {
  return plane_dispatch(g, [](auto) {});
}

bool launch_plane_theta(pf_ctx* c, const cx<double>* T1, cx<double>* T3) {
  return plane_dispatch(c->g, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    k_plane_theta<N><<<dim3(c->g.nz, 3), dim3(PlaneGeo<N>::THREADS), 0, c->stream>>>(T1, T3, c->g, c->tw64[3],
                                                                                     c->tw64[2]);
  });
}

bool launch_plane_drive(pf_ctx* c, const cx<double>* T1, cx<double>* T3) {
  return plane_dispatch(c->g, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    k_plane_drive<N><<<dim3(c->g.nz, 3), dim3(3 * PlaneGeo<N>::THREADS), 0, c->stream>>>(T1, T3, c->g, c->mk, c->tw64[3],
                                                                                     c->tw64[2]);
  });
}

}  // namespace pf
