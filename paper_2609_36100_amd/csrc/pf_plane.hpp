// Plane passes: the y and x transforms of one z plane in one kernel (FP64).
//
// On small grids a work-group holds one plane of one field in LDS from its
// inverse y transform to its forward y transform, so
//   k_plane_theta  inverse y, c2r, theta = h(eta), r2c, forward y
//   k_plane_drive  the same of c, e_v and eta_v to the driving force g_v
// replace six launches of a stage by two.  One work-group per (plane, variant):
// the composition is transformed once per variant, beside the other fields.
//
// The two real columns a row transform starts from and ends in, kx = 0 and
// nx / 2, share one complex column: their Hermitian parts along y (what the c2r
// keeps of them) are packed as real and imaginary part, so a plane is nx / 2
// columns.  Bound by latency: at 64^3 192 work-groups on 256 CUs, 32 us for the
// two passes where the six took about 45 and their gaps (an ARK4 step 0.47 ->
// 0.36 ms; at 32^3 0.29 -> 0.19 ms).  At 128 the
// plane (131 KB) leaves one work-group per CU, so nothing overlaps its loads,
// and the stage took 7 % longer than with the separate passes; at 40, 56 and
// from 80 on three planes exceed a work-group.
#pragma once

#include "pf_kernels.hpp"

namespace pf {

// Threads per plane: one column (or, past 1024 threads, two) each, in whole
// wavefronts.
constexpr int plane_threads(int n) {
  const int tl = line_threads(n), cols = n / 2;
  const int t = (cols * tl + 63) / 64 * 64;
  return t > 1024 ? ((cols + 1) / 2 * tl + 63) / 64 * 64 : t;
}

template <int N>
struct PlaneGeo {
  static constexpr int M = N / 2;
  static constexpr int RY = plan(N).r[0], TY = N / RY;  // columns: end radix, threads
  static constexpr int RX = plan(M).r[0], TX = M / RX;  // rows
  static constexpr int THREADS = plane_threads(N);
  static constexpr int CPP = THREADS / TY;              // columns side by side
  static constexpr int C = (M + CPP - 1) / CPP;         // columns per thread
  static constexpr int RPP = THREADS / TX;
  static constexpr int R = (N + RPP - 1) / RPP;         // rows per thread
  static constexpr int LDS = N * M;
  // LDS of a group: its plane and the Nyquist column, or its real pairs
  static constexpr int STRIDE = LDS + N > R * RX * THREADS ? LDS + N : R * RX * THREADS;
  // the driving-force pass holds three planes
  static constexpr bool OK = 3 * THREADS <= 1024 && (3 * STRIDE + N + M) * 16 <= 160 * 1024;
  // Place of (y, x): each block of eight x is permuted by its number, so that the
  // row exchanges (strides of the end radix) spread over the banks.
  __device__ static inline int at(int y, int x) { return y * M + (M % 8 == 0 ? x ^ ((x >> 3) & 7) : x); }
};

// line_fft for C lines per thread at once (a[c], exchanged through buf(c, pos)).
template <int N, int S, int C, int Q>
struct MultiMid {
  template <class Buf>
  __device__ static inline void run(int tid, const cx<double>* tw, Buf buf, const bool (&act)[C]) {
    constexpr Plan PL = plan(N);
    if constexpr (Q < PL.np - 1) {
      constexpr int r = PL.r[Q];
      constexpr int p = plan_prod(N, Q, 8);
      constexpr int TL = N / PL.r[0];
      constexpr int NB = N / r;
      constexpr int PER = (NB + TL - 1) / TL;
      cx<double> v[C][PER][r];
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
          const int b = tid + j * TL;
          if (act[c] && (PER * TL == NB || b < NB)) {
            const int k = b % p;
#pragma unroll
            for (int t = 0; t < r; ++t) v[c][j][t] = buf(c, b + t * NB);
            apply_twiddles<r, S>(v[c][j], tw, k * (N / (p * r)));
            dft<r, S>(v[c][j]);
          }
        }
      lds_barrier();
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int j = 0; j < PER; ++j) {
          const int b = tid + j * TL;
          if (act[c] && (PER * TL == NB || b < NB)) {
            const int k = b % p;
#pragma unroll
            for (int t = 0; t < r; ++t) buf(c, (b - k) * r + k + t * p) = v[c][j][t];
          }
        }
      lds_barrier();
      MultiMid<N, S, C, Q + 1>::run(tid, tw, buf, act);
    }
  }
};

template <int N, int S, int C, class Buf>
__device__ inline void multi_fft(cx<double> (&a)[C][plan(N).r[0]], int tid, const cx<double>* tw, Buf buf,
                                 const bool (&act)[C]) {
  constexpr Plan PL = plan(N);
  static_assert(PL.ok, "unsupported line length");
  constexpr int R0 = PL.r[0];
  constexpr int TL = N / R0;
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (act[c]) dft<R0, S>(a[c]);
  if constexpr (PL.np > 1) {
    lds_barrier();
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (act[c]) {
#pragma unroll
        for (int t = 0; t < R0; ++t) buf(c, tid * R0 + t) = a[c][t];
      }
    lds_barrier();
    MultiMid<N, S, C, 1>::run(tid, tw, buf, act);
#pragma unroll
    for (int c = 0; c < C; ++c)
      if (act[c]) {
#pragma unroll
        for (int t = 0; t < R0; ++t) a[c][t] = buf(c, tid + t * TL);
        apply_twiddles<R0, S>(a[c], tw, tid);
        dft<R0, S>(a[c]);
      }
  }
}

// A thread's places in a plane: its columns (y transforms) and rows.  Rebuilt
// for each phase from an opaque copy of the thread index, so that places and
// the addresses made from them are not held across the transforms.
template <int N>
struct PlaneItem {
  using PG = PlaneGeo<N>;
  int cb, col[PG::C], rb, row[PG::R];
  bool ca[PG::C], ra[PG::R];
  __device__ inline PlaneItem(int tid, bool on = true) {
    asm volatile("" : "+v"(tid));
    // columns: lane-contiguous in kx
    cb = tid / PG::CPP;
    const int c0 = tid % PG::CPP;
#pragma unroll
    for (int c = 0; c < PG::C; ++c) {
      col[c] = c0 + c * PG::CPP;
      ca[c] = on && cb < PG::TY && col[c] < PG::M;
    }
    rb = tid % PG::TX;
    const int r0 = tid / PG::TX;
#pragma unroll
    for (int r = 0; r < PG::R; ++r) {
      row[r] = r0 + r * PG::RPP;
      ra[r] = on && r0 < PG::RPP && row[r] < N;
    }
  }
};

// A thread's share of a plane as loaded: its columns, and the Nyquist column's
// values where it holds column 0.
template <int N>
struct PlaneLoad {
  using PG = PlaneGeo<N>;
  cx<double> b[PG::C][PG::RY], m[PG::RY];
  __device__ inline void load(const cx<double>* src, int P, int tid) {
    const PlaneItem<N> q(tid);
#pragma unroll
    for (int c = 0; c < PG::C; ++c)
      if (q.ca[c]) {
#pragma unroll
        for (int t = 0; t < PG::RY; ++t) b[c][t] = src[(q.cb + t * PG::TY) * P + q.col[c]];
      }
    if (q.ca[0] && q.col[0] == 0) {
#pragma unroll
      for (int t = 0; t < PG::RY; ++t) m[t] = src[(q.cb + t * PG::TY) * P + PG::M];
    }
  }
};

// A loaded plane of the half spectrum (after the inverse z transform) -> real
// pairs a[r][t] = (x_{2n}, x_{2n+1}), n = rb + t TX, of the thread's rows.
// pl: the plane's LDS, PlaneGeo::LDS values and N more for the Nyquist column.
template <int N>
__device__ inline void plane_inverse(PlaneLoad<N>& ld, int tid, cx<double>* pl, const cx<double>* twN,
                                     const cx<double>* twM, cx<double> (&a)[PlaneGeo<N>::R][PlaneGeo<N>::RX]) {
  using PG = PlaneGeo<N>;
  {
    const PlaneItem<N> q(tid);
    cx<double>(&b)[PG::C][PG::RY] = ld.b;
    auto buf = [&](int c, int pos) -> cx<double>& { return pl[PG::at(pos, q.col[c])]; };
    // Hermitian parts of columns 0 and M along y, packed as one column
    const bool edge = q.ca[0] && q.col[0] == 0;
    cx<double>* nyq = pl + PG::LDS;
    if (edge) {
#pragma unroll
      for (int t = 0; t < PG::RY; ++t) {
        buf(0, q.cb + t * PG::TY) = b[0][t];
        nyq[q.cb + t * PG::TY] = ld.m[t];
      }
    }
    lds_barrier();
    if (edge) {
#pragma unroll
      for (int t = 0; t < PG::RY; ++t) {
        const int ky = q.cb + t * PG::TY, kn = ky == 0 ? 0 : N - ky;
        const cx<double> x0 = b[0][t] + conj(buf(0, kn)), xm = ld.m[t] + conj(nyq[kn]);
        b[0][t] = 0.5 * (x0 + mul_si<1>(xm));
      }
    }
    if constexpr (plan(N).np == 1) lds_barrier();  // no exchange below
    multi_fft<N, +1, PG::C>(b, q.cb, twN, buf, q.ca);
#pragma unroll
    for (int c = 0; c < PG::C; ++c)
      if (q.ca[c]) {
#pragma unroll
        for (int t = 0; t < PG::RY; ++t) buf(c, q.cb + t * PG::TY) = b[c][t];
      }
  }
  lds_barrier();
  const PlaneItem<N> q(tid);
#pragma unroll
  for (int r = 0; r < PG::R; ++r)
    if (q.ra[r]) {
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) {
        const int k = q.rb + t * PG::TX;
        cx<double> xk = pl[PG::at(q.row[r], k)];
        cx<double> xmk = pl[PG::at(q.row[r], k == 0 ? 0 : PG::M - k)];
        if (k == 0) {
          xmk = mk(xk.im, 0.0);
          xk.im = 0.0;
        }
        a[r][t] = c2r_pre(xk, xmk, twN[k]);
      }
    }
  multi_fft<PG::M, +1, PG::R>(
      a, q.rb, twM, [&](int r, int pos) -> cx<double>& { return pl[PG::at(q.row[r], pos)]; }, q.ra);
}

// The plane's columns from LDS through their forward transform to dst.
template <int N>
__device__ inline void plane_columns_out(cx<double>* dst, int P, int tid, cx<double>* pl, const cx<double>* twN, bool on) {
  using PG = PlaneGeo<N>;
  const PlaneItem<N> q(tid, on);
  cx<double> b[PG::C][PG::RY];
  auto buf = [&](int c, int pos) -> cx<double>& { return pl[PG::at(pos, q.col[c])]; };
#pragma unroll
  for (int c = 0; c < PG::C; ++c)
    if (q.ca[c]) {
#pragma unroll
      for (int t = 0; t < PG::RY; ++t) b[c][t] = buf(c, q.cb + t * PG::TY);
    }
  multi_fft<N, -1, PG::C>(b, q.cb, twN, buf, q.ca);
  // split the packed column (its threads are in many wavefronts)
  if (q.col[0] == 0 && q.ca[0]) {
#pragma unroll
    for (int t = 0; t < PG::RY; ++t) buf(0, q.cb + t * PG::TY) = b[0][t];
  }
  lds_barrier();
#pragma unroll
  for (int c = 0; c < PG::C; ++c)
    if (q.ca[c]) {
      if (c == 0 && q.col[0] == 0) {
#pragma unroll
        for (int t = 0; t < PG::RY; ++t) {
          const int ky = q.cb + t * PG::TY, kn = ky == 0 ? 0 : N - ky;
          const cx<double> zc = conj(buf(0, kn)), d = b[0][t] - zc;
          dst[ky * P + PG::M] = mk(0.5 * d.im, -0.5 * d.re);
          b[0][t] = 0.5 * (b[0][t] + zc);
        }
      }
#pragma unroll
      for (int t = 0; t < PG::RY; ++t) dst[(q.cb + t * PG::TY) * P + q.col[c]] = b[c][t];
    }
}

// Real pairs of the thread's rows -> the plane's half spectrum after the
// forward y transform, at dst.
template <int N>
__device__ inline void plane_forward(cx<double> (&a)[PlaneGeo<N>::R][PlaneGeo<N>::RX], cx<double>* dst, int P,
                                     int tid, cx<double>* pl, const cx<double>* twN, const cx<double>* twM,
                                     bool on = true) {
  using PG = PlaneGeo<N>;
  const PlaneItem<N> q(tid, on);
  multi_fft<PG::M, -1, PG::R>(
      a, q.rb, twM, [&](int r, int pos) -> cx<double>& { return pl[PG::at(q.row[r], pos)]; }, q.ra);
  lds_barrier();
#pragma unroll
  for (int r = 0; r < PG::R; ++r)
    if (q.ra[r]) {
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) pl[PG::at(q.row[r], q.rb + t * PG::TX)] = a[r][t];
    }
  lds_barrier();
#pragma unroll
  for (int r = 0; r < PG::R; ++r)
    if (q.ra[r]) {
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) {
        const int k = q.rb + t * PG::TX;
        const cx<double> zk = a[r][t];
        a[r][t] = k == 0 ? mk(zk.re + zk.im, zk.re - zk.im)  // X_0 and X_M, both real, packed
                         : r2c_post(zk, pl[PG::at(q.row[r], PG::M - k)], twN[k]);
      }
    }
  lds_barrier();
#pragma unroll
  for (int r = 0; r < PG::R; ++r)
    if (q.ra[r]) {
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) pl[PG::at(q.row[r], q.rb + t * PG::TX)] = a[r][t];
    }
  lds_barrier();
  plane_columns_out<N>(dst, P, tid, pl, twN, on);
}

// theta_v = h(eta_v) of one plane: T1 (state after the inverse z transform) ->
// T3 (theta after its forward y transform).
template <int N>
__device__ inline void body_plane_theta(const cx<double>* st, cx<double>* th, const Geo& g, const cx<double>* twN,
                                        const cx<double>* twM, int z, int v, int tid, cx<double>* pl) {
  using PG = PlaneGeo<N>;
  const long long zo = (long long)z * g.ny * g.P;
  cx<double> a[PG::R][PG::RX];
  PlaneLoad<N> ld;
  ld.load(st + (1 + v) * g.fs + zo, g.P, tid);
  plane_inverse<N>(ld, tid, pl, twN, twM, a);
#pragma unroll
  for (int r = 0; r < PG::R; ++r)
#pragma unroll
    for (int t = 0; t < PG::RX; ++t) a[r][t] = mk(hfun(a[r][t].re), hfun(a[r][t].im));
  plane_forward<N>(a, th + v * g.fs + zo, g.P, tid, pl, twN, twM);
}

// g_v = h'(eta_v) (chi(c) + e_v) + 2 w eta_v (1 - eta_v)(1 - 2 eta_v) of one
// plane; el: e_v after the inverse z transform, g_v after the forward y one.
// Three thread groups (PlaneGeo::THREADS each, a plane's LDS each) take c, e_v
// and eta_v to real space side by side; the third forms g_v and transforms it
// back while the others only keep the barriers.  One group after another took
// 22.9 us at 64^3.
template <int N>
__device__ inline void body_plane_drive(const cx<double>* st, cx<double>* el, const Geo& g, const ModelK& m,
                                        const cx<double>* twN, const cx<double>* twM, int z, int v, int tid,
                                        cx<double>* pl) {
  using PG = PlaneGeo<N>;
  const int grp = tid / PG::THREADS;  // whole wavefronts
  tid %= PG::THREADS;
  const long long zo = (long long)z * g.ny * g.P;
  cx<double>* own = pl + grp * PG::STRIDE;
  cx<double> a[PG::R][PG::RX];
  {
    PlaneLoad<N> ld;
    ld.load((grp == 0 ? st : grp == 1 ? el + v * g.fs : st + (1 + v) * g.fs) + zo, g.P, tid);
    plane_inverse<N>(ld, tid, own, twN, twM, a);
  }
  lds_barrier();
  // c and e_v of this thread's pairs to the third group, through the planes
  if (grp < 2) {
#pragma unroll
    for (int r = 0; r < PG::R; ++r)
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) own[(r * PG::RX + t) * PG::THREADS + tid] = a[r][t];
  }
  lds_barrier();
  const double W = m.W, cm = m.cm, cp = m.cp, w2 = 2.0 * m.w;
  if (grp == 2) {
#pragma unroll
    for (int r = 0; r < PG::R; ++r)
#pragma unroll
      for (int t = 0; t < PG::RX; ++t) {
        const int i = (r * PG::RX + t) * PG::THREADS + tid;
        const cx<double> c = pl[i], e = pl[PG::STRIDE + i];
        const double chi0 = W * ((c.re - cp) * (c.re - cp) - (c.re - cm) * (c.re - cm));
        const double chi1 = W * ((c.im - cp) * (c.im - cp) - (c.im - cm) * (c.im - cm));
        const double e0 = a[r][t].re, e1 = a[r][t].im;
        a[r][t] = mk(dhfun(e0) * (chi0 + e.re) + w2 * e0 * (1.0 - e0) * (1.0 - 2.0 * e0),
                     dhfun(e1) * (chi1 + e.im) + w2 * e1 * (1.0 - e1) * (1.0 - 2.0 * e1));
      }
  }
  plane_forward<N>(a, el + v * g.fs + zo, g.P, tid, own, twN, twM, grp == 2);
}

}  // namespace pf
