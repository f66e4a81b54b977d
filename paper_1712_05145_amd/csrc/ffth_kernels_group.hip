// Instantiations of the grouped passes for one precision (FFTH_REAL) and one
// kernel (FFTH_PART: 0 z-pass, 1 x-forward, 2 x-inverse, 3 and 4 fused
// three-term CG pass of isotropic and of general phases).
#include "ffth_kernels.h"
#include "ffth_launch.h"

#if !defined(FFTH_REAL) || !defined(FFTH_PART)
#error "compile with -DFFTH_REAL=float|double and -DFFTH_PART=0..4"
#endif

namespace ffth {

using R = FFTH_REAL;
constexpr bool DBL = sizeof(R) == 8;

#if FFTH_PART == 0
template <int N, int R2> static bool gz_r(dim3 grid, bool h16, hipStream_t s, const Desc* d, int op, int n1,
                                          double scale, int kcs, int fin, int nblk_f, int nblk_i) {
  if constexpr (gz_used<R>(N, R2)) {
    if constexpr (!DBL) {
      if (h16) {
        hipLaunchKernelGGL((k_gz<R, N, R2, NT, H2>), grid, dim3(NT), 0, s, d, op, n1, scale, kcs, fin, nblk_f, nblk_i);
        return true;
      }
    }
    hipLaunchKernelGGL((k_gz<R, N, R2, NT, C2<R>>), grid, dim3(NT), 0, s, d, op, n1, scale, kcs, fin, nblk_f, nblk_i);
    return true;
  }
  return false;
}
template <> hipError_t GLaunch<R>::gz(int n0, const GroupShape& g, bool h16, int nb, hipStream_t s, const Desc* d,
                                      int op, int n1, double scale, int fin, int nblk_f, int nblk_i) {
  const dim3 grid(g.zblocks + (fin >= 0 ? 1 : 0), nb);
  bool ok = false;   // stays so where no kernel is compiled for (n0, R2)
  switch (n0) {
#define FFTH_CASE(N)                                                                                     \
  case N:                                                                                                \
    if (g.r2 == 4) ok = gz_r<N, 4>(grid, h16, s, d, op, n1, scale, g.kcs, fin, nblk_f, nblk_i);         \
    if (g.r2 == 8) ok = gz_r<N, 8>(grid, h16, s, d, op, n1, scale, g.kcs, fin, nblk_f, nblk_i);         \
    if (g.r2 == 16) ok = gz_r<N, 16>(grid, h16, s, d, op, n1, scale, g.kcs, fin, nblk_f, nblk_i);       \
    if constexpr (DBL) {                                                                                 \
      if (g.r2 == 2) ok = gz_r<N, 2>(grid, h16, s, d, op, n1, scale, g.kcs, fin, nblk_f, nblk_i);       \
    } else {                                                                                             \
      if (g.r2 == 6) ok = gz_r<N, 6>(grid, h16, s, d, op, n1, scale, g.kcs, fin, nblk_f, nblk_i);       \
    }                                                                                                    \
    break;
    FFTH_GROUP_N(FFTH_CASE)
#undef FFTH_CASE
  }
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

#ifdef FFTH_GROUP_RULE   // defined for one of the two precisions
template <typename T> static GroupShape shape_of(const int n[3]) {
  GroupShape g;
  g.r2 = group_pick<T>(n[0], n[1], n[2]);
  if (g.r2 == 0) return GroupShape{};
  g.on = true;
  g.r1 = n[1] / g.r2;
  const int grp = group_count(n[2], g.r1);
  g.kcs = group_kcs(g.r2, n[2] / 2);
  g.xblocks = (n[0] * g.r2 + grp - 1) / grp;
  g.zblocks = n[2] / 2 / gz_kc<T>(n[0], g.r2) * g.r1;
  return g;
}
GroupShape group_shape(const int n[3], bool dbl) { return dbl ? shape_of<double>(n) : shape_of<float>(n); }
#endif
#else
// kernel launch for (axis-2 length, R1): f(integral constants).  R1 = 3, 6, 12
// come up in FP64 (12, 24, 48 = 4 R1, 96 = 8 R1), R1 = 32 in FP32
template <int N> struct IC { static constexpr int v = N; };
template <int N, class F> static bool for_r1(int r1, F&& f) {
  switch (r1) {
#define FFTH_R1(K) case K: if constexpr (gx_used<R>(N, K)) { f(IC<N>(), IC<K>()); return true; } break;
#define FFTH_R1F(K) case K: if constexpr (!DBL && gx_used<R>(N, K)) { f(IC<N>(), IC<K>()); return true; } break;
#define FFTH_R1D(K) case K: if constexpr (DBL && gx_used<R>(N, K)) { f(IC<N>(), IC<K>()); return true; } break;
    FFTH_R1(2) FFTH_R1(4) FFTH_R1(8) FFTH_R1(16)
    FFTH_R1D(3) FFTH_R1D(6) FFTH_R1D(12) FFTH_R1F(32)
#undef FFTH_R1
#undef FFTH_R1F
#undef FFTH_R1D
  }
  return false;
}
template <class F> static hipError_t for_shape(int n2, int r1, F&& f) {
  bool ok = false;
  switch (n2) {
#define FFTH_CASE(N) case N: ok = for_r1<N>(r1, f); break;
    FFTH_GROUP_N(FFTH_CASE)
#undef FFTH_CASE
  }
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}
#endif

#if FFTH_PART == 1
template <> hipError_t GLaunch<R>::xfwd(int n2, const GroupShape& g, bool iso, bool h16, int nb, hipStream_t s,
                                        const Desc* d, int mode, long rows, long nvox) {
  const dim3 grid(g.xblocks, nb);
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v, RW = gx_rows<R>(N, K);
    if constexpr (!DBL) {
      if (h16) {
        if (iso) hipLaunchKernelGGL((k_xfwd<R, N, true, RW, NT, H2, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
        else hipLaunchKernelGGL((k_xfwd<R, N, false, RW, NT, H2, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
        return;
      }
    }
    if (iso) hipLaunchKernelGGL((k_xfwd<R, N, true, RW, NT, C2<R>, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
    else hipLaunchKernelGGL((k_xfwd<R, N, false, RW, NT, C2<R>, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
  });
}
#elif FFTH_PART == 2
template <> hipError_t GLaunch<R>::xinv(int n2, const GroupShape& g, bool iso, int nb, hipStream_t s, const Desc* d,
                                        int mode, long rows, long nvox) {
  const dim3 grid(g.xblocks, nb);
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v, RW = gx_rows<R>(N, K);
    if (iso) hipLaunchKernelGGL((k_xinv<R, N, true, RW, NT, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
    else hipLaunchKernelGGL((k_xinv<R, N, false, RW, NT, 0, K>), grid, dim3(NT), 0, s, d, mode, rows, nvox, g.r2, g.kcs);
  });
}

template <> hipError_t GLaunch<R>::field_fwd(int n2, const GroupShape& g, int nb, hipStream_t s, const Desc* d,
                                             long rows, long nvox) {
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v;
    hipLaunchKernelGGL((k_field_fwd<R, N, gx_rows<R>(N, K), K>), dim3(g.xblocks, nb), dim3(NT), 0, s, d, rows, nvox,
                       g.r2, g.kcs);
  });
}
template <> hipError_t GLaunch<R>::field_fwd1(int n2, const GroupShape& g, hipStream_t s, const Desc& d,
                                              const SolverState& st, Desc* dd, long rows, long nvox) {
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v;
    hipLaunchKernelGGL((k_field_fwd1<R, N, gx_rows<R>(N, K), K>), dim3(g.xblocks), dim3(NT), 0, s, d, st, dd, rows,
                       nvox, g.r2, g.kcs);
  });
}
template <> hipError_t GLaunch<R>::field_inv(int n2, const GroupShape& g, int nb, hipStream_t s, const Desc* d,
                                             bool accum, long rows, long nvox) {
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v;
    hipLaunchKernelGGL((k_field_inv<R, N, gx_rows<R>(N, K), K>), dim3(g.xblocks, nb), dim3(NT), 0, s, d, accum ? 1 : 0,
                       rows, nvox, g.r2, g.kcs);
  });
}
#elif FFTH_PART >= 3
// (one translation unit per material kind)
constexpr bool ISO = FFTH_PART == 3;
template <> template <> hipError_t GLaunch<R>::xcg3<ISO>(int n2, const GroupShape& g, bool h16, int nb, hipStream_t s,
                                                        const Desc* d, long rows, long nvox) {
  const dim3 grid(g.xblocks, nb);
  return for_shape(n2, g.r1, [&](auto n, auto r) {
    constexpr int N = decltype(n)::v, K = decltype(r)::v, RW = gx_rows<R>(N, K);
    if constexpr (!DBL) {
      if (h16) {
        hipLaunchKernelGGL((k_xcg3<R, N, ISO, RW, NT, H2, 0, K>), grid, dim3(NT), 0, s, d, rows, nvox, g.r2, g.kcs);
        return;
      }
    }
    hipLaunchKernelGGL((k_xcg3<R, N, ISO, RW, NT, C2<R>, 0, K>), grid, dim3(NT), 0, s, d, rows, nvox, g.r2, g.kcs);
  });
}
#endif

}  // namespace ffth
