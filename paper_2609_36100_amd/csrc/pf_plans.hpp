// Line lengths, tile plans and their compile-time dispatch, shared by the
// single-grid translation units.
#pragma once

#include <type_traits>

#include "pf_context.hpp"
#include "pf_kernels.hpp"

namespace pf {

// ---- supported line lengths --------------------------------------------
// Column passes (y, z) take N; row passes (x) take M = nx / 2.
#define PF_COL_SIZES(X)                                                                                  \
  X(8) X(16) X(24) X(32) X(40) X(48) X(56) X(64) X(80) X(96) X(128) X(160) X(168) X(192) X(256) X(320) X(336) \
  X(384) X(504) X(512)
#define PF_ROW_SIZES(X)                                                                                         \
  X(4) X(8) X(12) X(16) X(20) X(24) X(28) X(32) X(40) X(48) X(64) X(80) X(84) X(96) X(128) X(160) X(168) X(192) \
  X(252) X(256)

template <class F>
static bool col_dispatch(int n, F&& f) {
  switch (n) {
#define PF_CASE(N)                          \
  case N:                                   \
    f(std::integral_constant<int, N>{});    \
    return true;
    PF_COL_SIZES(PF_CASE)
#undef PF_CASE
    default:
      return false;
  }
}

template <class F>
static bool row_dispatch(int m, F&& f) {
  switch (m) {
#define PF_CASE(N)                          \
  case N:                                   \
    f(std::integral_constant<int, N>{});    \
    return true;
    PF_ROW_SIZES(PF_CASE)
#undef PF_CASE
    default:
      return false;
  }
}

static bool col_supported(int n) {
  return col_dispatch(n, [](auto) {});
}
static bool row_supported(int m) {
  return row_dispatch(m, [](auto) {});
}

// Column-pass tiles: TX consecutive kx columns per work-group, end radix RE.
// Two tile variants per kernel kind, chosen per context by the autotuner
// (pf_autotune): variant 0 gives each row segment `seg0` contiguous bytes,
// variant 1 twice that.  Small lines get wider tiles so a work-group has at
// least one full wavefront; lines shorter than 64 have only variant 0.
// Largest end radix of each kind's line plan (elem_bytes: 16 FP64, 8 FP32
// complex values).  The FP64 elastic pass holds three fields in registers, so
// it takes narrower tiles and its ends stay at radix 4 where 16 divides the
// line length (half the registers per field of radix 8; radix 8 gained
// nothing at 512^3); lines that 36 divides but 16 does not (504) take radix-6
// ends, since the radix-3 ends they would otherwise get cost the pass a
// quarter more time.  In FP32 the three fields fit at radix 8 (113 VGPRs at
// 512: 8-column tiles ran 1.03 ms against 1.43 ms for 4-column radix-4 ones).
constexpr int col_re(int kind, int elem_bytes = 16) {
  return kind != CK_ELASTIC ? 8 : elem_bytes == 8 ? 8 : 6;
}
constexpr int col_tx(int n, int kind, int elem_bytes, int v) {
  const int seg = (kind == CK_ELASTIC ? 32 : 64) << ((n >= 64) ? v : 0);
  int tx = seg / elem_bytes;
  if (tx < 1) tx = 1;
  while (tx * line_threads(n, col_re(kind, elem_bytes)) < 64 && tx < 16) tx *= 2;
  // long lines with small end radices (504 in the elastic pass: 168 threads
  // per line) stay within 1024 threads per work-group
  while (tx > 1 && tx * line_threads(n, col_re(kind, elem_bytes)) > 1024) tx /= 2;
  return tx;
}
// Whether the wave-specialised column FFT (variant 2 of "colfft") exists for
// lines of length n with elements of elem_bytes.
static bool ws_supported(int n, int elem_bytes) {
  bool ok = false;
  col_dispatch(n, [&](auto NC) {
    constexpr int N = decltype(NC)::value;
    ok = elem_bytes == 16 ? ws_ok<double, N, col_tx(N, CK_FFT, 16, 1)>()
                          : ws_ok<float, N, col_tx(N, CK_FFT, 8, 1)>();
  });
  return ok;
}
template <class F>
static void with_variant(int v, F&& f) {
  if (v)
    f(std::integral_constant<int, 1>{});
  else
    f(std::integral_constant<int, 0>{});
}
// Rows per row-pass work-group: about 256 threads.
constexpr int rb_of(int m) { return line_threads(m) >= 256 ? 1 : 256 / line_threads(m); }
// Rows per work-group of the stage cycle's theta and drive passes: 128
// threads where the line's thread count divides 128 (their drive pass ran
// 9-16 % faster so, their FP64 theta pass 3-8 %, at 512^3 and 256^3), else
// the general rule (lines of 42 or 84 threads would leave part-filled waves).
constexpr int rb_x(int m) {
  return line_threads(m) <= 128 && 128 % line_threads(m) == 0 ? 128 / line_threads(m) : rb_of(m);
}

template <typename T>
static const cx<T>* tw(const pf_ctx* c, int slot) {
  if constexpr (sizeof(T) == 8)
    return c->tw64[slot];
  else
    return c->tw32[slot];
}

}  // namespace pf
