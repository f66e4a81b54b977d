// Instantiations of the FFT-pass kernels for one precision (FFTH_REAL is
// float or double, set on the compiler command line) and every axis length
// in FFTH_SIZES, one kernel per translation unit (FFTH_PART: 0 z-pass, finish
// kernels and tile shapes, 1 x-forward, 2 x-inverse, 3 fused three-term CG
// pass, 4 y-pass).
#include "ffth_kernels.h"
#include "ffth_launch.h"

#if !defined(FFTH_REAL) || !defined(FFTH_PART)
#error "compile with -DFFTH_REAL=float|double and -DFFTH_PART=0..4"
#endif

namespace ffth {

using R = FFTH_REAL;

#if FFTH_PART == 0
template <typename T> int Launch<T>::x_rows(int n, int v) {
#define FFTH_CASE(N) if (n == N) return ffth::xf_rows_v<T>(N, v);
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return 0;
}
template <typename T> int Launch<T>::xi_rows(int n, int v) {
#define FFTH_CASE(N) if (n == N) return ffth::xi_rows_v<T>(N, v);
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return 0;
}
template <typename T> int Launch<T>::y_cols(int n, int v) {
#define FFTH_CASE(N) if (n == N) return ffth::y_cols_v<T>(N, v);
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return 0;
}
template <typename T> int Launch<T>::z_cols(int n, int v) {
#define FFTH_CASE(N) if (n == N) return ffth::z_cols_v<T>(N, v);
  FFTH_ZSIZES(FFTH_CASE)
#undef FFTH_CASE
  return 0;
}
#endif

// one launcher per (length, variant): the tile shape is a template argument
// Storage type of the spectrum: full precision, or binary16 (FP32 only)
template <typename T> using Full = C2<T>;

template <typename T, int N, int V, typename S = C2<T>>
static void xfwd_v(bool iso, dim3 grid, hipStream_t s, const Desc* d, int mode, long rows, long nvox) {
  constexpr int RW = ffth::xf_rows_v<T>(N, V), TB = ffth::x_threads_v<T>(N, V);
  constexpr int PL = ffth::plan_of(V);
  if (iso) hipLaunchKernelGGL((k_xfwd<T, N, true, RW, TB, S, PL>), grid, dim3(TB), 0, s, d, mode, rows, nvox, 1, 0);
  else hipLaunchKernelGGL((k_xfwd<T, N, false, RW, TB, S, PL>), grid, dim3(TB), 0, s, d, mode, rows, nvox, 1, 0);
}
template <typename T, int N, int V, typename S = C2<T>>
static void xinv_v(bool iso, dim3 grid, hipStream_t s, const Desc* d, int mode, long rows, long nvox) {
  constexpr int RW = ffth::xi_rows_v<T>(N, V), TB = ffth::xi_threads_v<T>(N, V);
  constexpr int PL = ffth::plan_of(V);
  if (iso) hipLaunchKernelGGL((k_xinv<T, N, true, RW, TB, PL>), grid, dim3(TB), 0, s, d, mode, rows, nvox, 1, 0);
  else hipLaunchKernelGGL((k_xinv<T, N, false, RW, TB, PL>), grid, dim3(TB), 0, s, d, mode, rows, nvox, 1, 0);
}
template <typename T, int N, int V, typename S = C2<T>>
static void xcg3_v(bool iso, dim3 grid, hipStream_t s, const Desc* d, long rows, long nvox) {
  constexpr int RW = ffth::xi_rows_v<T>(N, V), TB = ffth::xi_threads_v<T>(N, V);
  constexpr int PL = ffth::plan_of(V);
  if (iso) hipLaunchKernelGGL((k_xcg3<T, N, true, RW, TB, S, PL>), grid, dim3(TB), 0, s, d, rows, nvox, 1, 0);
  else hipLaunchKernelGGL((k_xcg3<T, N, false, RW, TB, S, PL>), grid, dim3(TB), 0, s, d, rows, nvox, 1, 0);
}
template <typename T, int N, int V, typename S = C2<T>>
static void ypass_v(dim3 grid, hipStream_t s, const Desc* d, int dir, int ncols, int ntiles) {
  constexpr int CW = ffth::y_cols_v<T>(N, V);
  constexpr int TB = ffth::y_threads_v<T>(N, V);
  hipLaunchKernelGGL((k_ypass<T, N, CW, TB, true, 1, S, ffth::plan_of(V)>), grid, dim3(TB), 0, s, d, dir, ncols,
                     ntiles);
}
template <typename T, int N, int V, typename S = C2<T>>
static void zpass_v(dim3 grid, hipStream_t s, const Desc* d, int op, int n1, int h, double scale, bool plane,
                    int fin, int nblk_f, int nblk_i) {
  constexpr int TK = ffth::z_cols_v<T>(N, V), TB = ffth::z_threads_v<T>(N, V);
  const int kc = kchunk(h), bpc = (int)(((long)n1 * kc + TK - 1) / TK);
  hipLaunchKernelGGL((k_zpass<T, N, TK, TB, S, ffth::plan_of(V)>), grid, dim3(TB), 0, s, d, op, n1, h,
                     FastDiv::of(bpc), FastDiv::of(kc), scale, plane ? 1 : 0, fin, nblk_f, nblk_i);
}

#define FFTH_VARIANTS_S(F, N, S, ...)        \
  switch (v) {                               \
    case 1: F<T, N, 1, S>(__VA_ARGS__); break; \
    case 2: F<T, N, 2, S>(__VA_ARGS__); break; \
    case 3: F<T, N, 3, S>(__VA_ARGS__); break; \
    case 4: F<T, N, 4, S>(__VA_ARGS__); break; \
    case 5: F<T, N, 5, S>(__VA_ARGS__); break; \
    default: F<T, N, 0, S>(__VA_ARGS__);     \
  }
#define FFTH_VARIANTS(F, N, ...) FFTH_VARIANTS_S(F, N, C2<T>, __VA_ARGS__)
// binary16 instantiations exist for FP32 only
#define FFTH_VARIANTS_H(F, N, ...)                                      \
  if constexpr (std::is_same<T, float>::value) {                        \
    if (h16) {                                                           \
      FFTH_VARIANTS_S(F, N, H2, __VA_ARGS__)                             \
    } else {                                                             \
      FFTH_VARIANTS_S(F, N, C2<T>, __VA_ARGS__)                          \
    }                                                                    \
  } else {                                                               \
    FFTH_VARIANTS_S(F, N, C2<T>, __VA_ARGS__)                            \
  }

#if FFTH_PART == 1
template <typename T> hipError_t Launch<T>::xfwd(int n2, bool iso, int v, bool h16, dim3 grid, hipStream_t s,
                                                const Desc* d, int mode, long rows, long nvox) {
#define FFTH_CASE(N)                                                          \
  if (n2 == N) {                                                              \
    FFTH_VARIANTS_H(xfwd_v, N, iso, grid, s, d, mode, rows, nvox)            \
    return hipGetLastError();                                                 \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
#endif

#if FFTH_PART == 2
template <typename T> hipError_t Launch<T>::xinv(int n2, bool iso, int v, dim3 grid, hipStream_t s, const Desc* d,
                                                int mode, long rows, long nvox) {
#define FFTH_CASE(N)                                                          \
  if (n2 == N) {                                                              \
    FFTH_VARIANTS(xinv_v, N, iso, grid, s, d, mode, rows, nvox)              \
    return hipGetLastError();                                                 \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
#endif

#if FFTH_PART == 3
template <typename T> hipError_t Launch<T>::xcg3(int n2, bool iso, int v, bool h16, dim3 grid, hipStream_t s,
                                                const Desc* d, long rows, long nvox) {
#define FFTH_CASE(N)                                                          \
  if (n2 == N) {                                                              \
    FFTH_VARIANTS_H(xcg3_v, N, iso, grid, s, d, rows, nvox)                  \
    return hipGetLastError();                                                 \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
#endif

#if FFTH_PART == 4
template <typename T> hipError_t Launch<T>::ypass(int n1, int v, bool h16, dim3 grid, hipStream_t s, const Desc* d,
                                                 int dir, int ncols, int ntiles) {
#define FFTH_CASE(N)                                                          \
  if (n1 == N) {                                                              \
    FFTH_VARIANTS_H(ypass_v, N, grid, s, d, dir, ncols, ntiles)              \
    return hipGetLastError();                                                 \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
#endif

#if FFTH_PART == 0
template <typename T> hipError_t Launch<T>::zpass(int n0, int v, bool h16, dim3 grid, hipStream_t s, const Desc* d,
                                                 int op, int n1, int h, double scale, bool plane,
                                                 int fin, int nblk_f, int nblk_i) {
#define FFTH_CASE(N)                                                          \
  if (n0 == N) {                                                              \
    FFTH_VARIANTS_H(zpass_v, N, grid, s, d, op, n1, h, scale, plane, fin, nblk_f, nblk_i)                \
    return hipGetLastError();                                                 \
  }
  FFTH_ZSIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}

// rows per block of the field passes
template <typename T> static dim3 field_grid(int n2, int nb, long rows) {
  int r = 0;
#define FFTH_CASE(N) if (n2 == N) r = ffth::x_rows<T>(N);
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return dim3(r > 0 ? (unsigned)((rows + r - 1) / r) : 0, nb);
}
template <typename T> hipError_t Launch<T>::field_fwd(int n2, int nb, hipStream_t s, const Desc* d, long rows, long nvox) {
#define FFTH_CASE(N)                                                                                                 \
  if (n2 == N) {                                                                                                     \
    hipLaunchKernelGGL((k_field_fwd<T, N, ffth::x_rows<T>(N), 1>), field_grid<T>(n2, nb, rows), dim3(NT), 0, s, d, rows, \
                       nvox, 1, 0);                                                                                  \
    return hipGetLastError();                                                                                        \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
template <typename T> hipError_t Launch<T>::field_fwd1(int n2, hipStream_t s, const Desc& d, const SolverState& st,
                                                      Desc* dd, long rows, long nvox) {
#define FFTH_CASE(N)                                                                                                 \
  if (n2 == N) {                                                                                                     \
    hipLaunchKernelGGL((k_field_fwd1<T, N, ffth::x_rows<T>(N), 1>), field_grid<T>(n2, 1, rows), dim3(NT), 0, s, d, st, \
                       dd, rows, nvox, 1, 0);                                                                        \
    return hipGetLastError();                                                                                        \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}
template <typename T> hipError_t Launch<T>::field_inv(int n2, int nb, hipStream_t s, const Desc* d, bool accum, long rows,
                                                     long nvox) {
#define FFTH_CASE(N)                                                                                                 \
  if (n2 == N) {                                                                                                     \
    hipLaunchKernelGGL((k_field_inv<T, N, ffth::x_rows<T>(N), 1>), field_grid<T>(n2, nb, rows), dim3(NT), 0, s, d, \
                       accum ? 1 : 0, rows, nvox, 1, 0);                                                             \
    return hipGetLastError();                                                                                        \
  }
  FFTH_SIZES(FFTH_CASE)
#undef FFTH_CASE
  return hipErrorInvalidValue;
}

template <typename T> hipError_t Launch<T>::bicg_finish(dim3 grid, hipStream_t s, const Desc* d, long n) {
  hipLaunchKernelGGL((k_bicg_finish<T>), grid, dim3(NT), 0, s, d, n);
  return hipGetLastError();
}

template <typename T> hipError_t Launch<T>::cg3_finish(dim3 grid, hipStream_t s, const Desc* d, long n) {
  hipLaunchKernelGGL((k_cg3_finish<T>), grid, dim3(NT), 0, s, d, n);
  return hipGetLastError();
}
#endif

template struct Launch<R>;

}  // namespace ffth
