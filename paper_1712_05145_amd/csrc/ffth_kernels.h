// HIP kernels of one iteration of the Moulinec-Suquet Basic Scheme / its CG
// form (Algorithm 1 and eq. (6) of arXiv:1712.05145), organised as five (the
// classical) or three (the grouped, below) passes over a half spectrum (k2 < n2/2, six interleaved
// components) stored k2-chunked as [k2 / KC][n0][n1][k2 % KC][6] complex,
// KC = kchunk(n2/2) (at most 16): every z-column then strides KC*6*n1
// complex values between rows instead of a whole plane:
//
//   x-pass (forward)   constitutive law / polarization tau (Algorithm 1, first
//                      step; eq. (2)) fused with the real-to-complex FFT along
//                      the contiguous axis (two real components per complex FFT)
//   y-pass             complex FFT along axis 1 (forward or inverse)
//   z-pass             forward FFT along axis 0, the spectral operator (Green
//                      operator below eq. (5) with eta_hat(0) = 0; theta of
//                      eq. (12); displacement recovery from eq. (1)), inverse FFT
//   y-pass (inverse)
//   x-pass (inverse)   complex-to-real FFT fused with the Basic Scheme / CG
//                      update and the residual reductions
//
// 2-D grids (n0 = 1) have no y-passes: the z-pass transforms axis 1.  Grouped
// passes split axis 1 between the x-passes and the z-pass (k_gz) and need no
// y-passes either.  The three-term CG joins the inverse x-pass of an iteration
// and the forward one of the next (k_xcg3); the field passes (k_field_*) serve
// operator calls without a solve.
//
// All FFTs run in LDS (mixed-radix Stockham, fft_device.h).  Block tile
// sizes are compile-time functions of the axis length and precision.
#pragma once
#include <type_traits>

#include "fft_device.h"
#include "ffth_finalize.h"
#include "ffth_types.h"

namespace ffth {

constexpr int NT = 256;   // threads per block of every FFT pass

constexpr int pow2_floor(int v) {
  int p = 1;
  while (p * 2 <= v) p *= 2;
  return p;
}
// Tile shapes and block sizes, chosen from a sweep of every pass at 256^3 on
// MI355X (rows per x-pass block, interleaved columns per y/z block, threads).
template <typename T> constexpr int x_rows(int n) {          // forward x-pass
  int r = 512 / n;
  return r < 1 ? 1 : pow2_floor(r);
}
template <typename T> constexpr int xi_rows(int n) {         // inverse x-pass
  int r = (sizeof(T) == 4 ? 256 : 512) / n;
  return r < 1 ? 1 : pow2_floor(r);
}
template <typename T> constexpr int y_cols(int n) {
  int c = (sizeof(T) == 4 ? 4096 : 2048) / n;
  int cap = sizeof(T) == 4 ? 16 : 8;
  c = c > cap ? cap : c;
  return c < 1 ? 1 : pow2_floor(c);
}
template <typename T> constexpr int y_threads(int n) { return sizeof(T) == 4 && n >= 128 ? 512 : 256; }
template <typename T> constexpr int z_cols(int n) {
  int c = 256 / n;
  c = c > 16 ? 16 : c;
  return c < 1 ? 1 : pow2_floor(c);
}
// Candidate shapes for the runtime autotuner: variant 0 is the measured
// default above, 1 and 2 halve / double the tile (or swap the block size of
// the y-pass), within 96 KB of LDS per block; 3 keeps the x tile of 0 with one
// wave per block (lengths whose Stockham stages have fewer butterflies than
// the default block has threads; for the inverse and fused x-passes, whose
// default is often one row, variant 1 is then two rows with 512 threads).
// The z-pass takes twice the columns (1),
// four times with 512 threads (2) or three times with 512 threads (3): rows
// of >= 144 contiguous bytes in FP32.  Variants 4 and 5 keep the default
// tile and change the radix plan of the transform (fft_device.h).
template <typename T> constexpr int lds_cap_rows(int n) {          // x-pass rows within 96 KB
  int r = 98304 / (3 * (n + n / 16) * (int)(2 * sizeof(T)));
  return r < 1 ? 1 : pow2_floor(r);
}
template <typename T> constexpr int var_rows(int r0, int n, int v) {
  int r = v == 1 ? (r0 > 1 ? r0 / 2 : 1) : v == 2 ? 2 * r0 : r0;   // v == 3: r0
  int c = lds_cap_rows<T>(n);
  return r > c ? c : r;
}
template <typename T> constexpr int xf_rows_v(int n, int v) { return var_rows<T>(x_rows<T>(n), n, v); }
// inverse / fused x-pass: variant 1 of a one-row tile (nothing to halve)
// doubles the rows with 512 threads instead
template <typename T> constexpr bool xi_wide_v(int n, int v) {
  return v == 1 && xi_rows<T>(n) == 1 && lds_cap_rows<T>(n) >= 2;
}
template <typename T> constexpr int xi_rows_v(int n, int v) {
  return xi_wide_v<T>(n, v) ? 2 : var_rows<T>(xi_rows<T>(n), n, v);
}
template <typename T> constexpr int y_cols_v(int n, int v) {
  int c = y_cols<T>(n);
  if (v == 2) c = c > 1 ? c / 2 : 1;
  return c;
}
template <typename T> constexpr int x_threads_v(int, int v) { return v == 3 ? 64 : NT; }
// (FP64 from 512 points on: 512 threads with the default shape as well; its
// one-column tile takes 48 KB or more, so few blocks share a CU.  One column,
// 256 -> 512 threads: 512^3 3.90 -> 3.60 ms, 1024x128x128 783 -> 753 us, planes
// of 512^2 12.9 -> 12.1 and, three fields, 1024^2 124 -> 113 us.  Variant 1 keeps
// 256 threads: two columns at 512 points, one at 1024)
template <typename T> constexpr int z_threads_v(int n, int v) {
  return v == 2 || v == 3 || (v != 1 && sizeof(T) == 8 && n >= 512) ? 512 : NT;
}
// variants 4 and 5: the default tile shape (variant 0) with radix plans 1 and 2
constexpr int plan_of(int v) { return v >= 4 ? v - 3 : 0; }
template <typename T> constexpr int xi_threads_v(int n, int v) { return xi_wide_v<T>(n, v) ? 512 : x_threads_v<T>(n, v); }
template <typename T> constexpr int y_threads_v(int n, int v) {
  return v == 1 ? (y_threads<T>(n) == 512 ? 256 : 512) : v == 2 ? 256 : y_threads<T>(n);
}
template <typename T> constexpr int z_cols_v(int n, int v) {
  int c = z_cols<T>(n);
  c = v == 1 ? 2 * c : v == 2 ? 4 * c : v == 3 ? 3 * c : c;
  const int cap = 98304 / (n * 6 * (int)(2 * sizeof(T)));
  c = c > cap ? (cap < 1 ? 1 : pow2_floor(cap)) : c;
  return c;
}

// k2 values per chunk of the half-spectrum layout: largest divisor of h up to 16
__host__ __device__ constexpr int kchunk(int h) {
  int c = h < 16 ? h : 16;
  while (h % c) --c;
  return c;
}
// index of (row = i0*n1 + i1, k2, component c) in the chunked half spectrum
__device__ __forceinline__ long spec_at(long row, int k2, int c, long rows, int kc) {
  return ((long)(k2 / kc) * rows + row) * (kc * 6) + (k2 % kc) * 6 + c;
}

// vector width of LDS / global accesses in the y and z passes (1: measured
// faster than 16-byte pairs, which halve the threads busy in each stage)
template <typename T> constexpr int vec_width() { return 1; }

// ---------------------------------------------------------------------------
// Constitutive law helpers.  Tensor-component vectors (11,22,33,23,13,12).
// Isotropic table row: (lam, mu, lam - lam0, mu - mu0).  Generic table row: the
// upper triangles of C and of C - C0, MAT_TRI values each.
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ const T* mat_of(const Desc& d);
template <> __device__ __forceinline__ const float* mat_of<float>(const Desc& d) { return d.mat32; }
template <> __device__ __forceinline__ const double* mat_of<double>(const Desc& d) { return d.mat64; }

// out = (C or C - C0)(phase) : e
template <typename T, bool ISO>
__device__ __forceinline__ void apply_mat(const T* mat, int ph, bool delta, const T (&e)[6], T (&out)[6]) {
  if constexpr (ISO) {
    const T lam = mat[ph * 4 + (delta ? 2 : 0)];
    const T mu2 = T(2) * mat[ph * 4 + (delta ? 3 : 1)];
    const T tr = e[0] + e[1] + e[2];
#pragma unroll
    for (int c = 0; c < 6; ++c) out[c] = mu2 * e[c] + (c < 3 ? lam * tr : T(0));
  } else {
    // upper triangle, padded to MAT_TRI values so that 16-byte loads fetch it:
    // the loads are gathers (neighbouring voxels differ in phase) and their
    // number bounds the pass, 11 (FP64) or 6 (FP32) here instead of 36
    // (48x24x96 BiCGSTAB solve, two loads: 7.76 -> 7.59 ms)
    constexpr int Q = 16 / (int)sizeof(T);
    struct alignas(16) Quad { T v[Q]; };
    const Quad* q = (const Quad*)(mat + ph * (2 * MAT_TRI) + (delta ? MAT_TRI : 0));
    T m[(21 + Q - 1) / Q * Q];
#pragma unroll
    for (int i = 0; i < (21 + Q - 1) / Q; ++i) {
      const Quad w = q[i];
#pragma unroll
      for (int j = 0; j < Q; ++j) m[i * Q + j] = w.v[j];
    }
    // engineering shear strains; factors of two are exact
    const T g[6] = {e[0], e[1], e[2], T(2) * e[3], T(2) * e[4], T(2) * e[5]};
#pragma unroll
    for (int a = 0; a < 6; ++a) {
      T s = 0;
#pragma unroll
      for (int b = 0; b < 6; ++b) {
        const int lo = a < b ? a : b, hi = a < b ? b : a;
        s += m[lo * (11 - lo) / 2 + hi] * g[b];
      }
      out[a] = s;
    }
  }
}

template <typename T> __device__ __forceinline__ T frob_w(const T (&a)[6], const T (&b)[6]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + T(2) * (a[3] * b[3] + a[4] * b[4] + a[5] * b[5]);
}
// a : b (off-diagonal tensor components counted twice) accumulated in FP64
template <typename T> __device__ __forceinline__ double frob_d(const T (&a)[6], const T (&b)[6]) {
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < 6; ++c) s += (c < 3 ? 1.0 : 2.0) * (double)a[c] * (double)b[c];
  return s;
}
// a : b for a block sum: FP32 operands are multiplied in FP64 (products of
// small residuals would underflow in FP32); FP64 keeps frob_w's order
template <typename T> __device__ __forceinline__ double frob_acc(const T (&a)[6], const T (&b)[6]) {
  if constexpr (sizeof(T) == 4) return frob_d(a, b);
  else return frob_w(a, b);
}
// C0 inner product density lam0 tr a tr b + 2 mu0 a:b
__device__ __forceinline__ double c0_ip(double lam0, double mu0, const double (&a)[6], const double (&b)[6]) {
  const double ta = a[0] + a[1] + a[2], tb = b[0] + b[1] + b[2];
  const double ab = a[0] * b[0] + a[1] * b[1] + a[2] * b[2] + 2.0 * (a[3] * b[3] + a[4] * b[4] + a[5] * b[5]);
  return lam0 * ta * tb + 2.0 * mu0 * ab;
}

// Residual slot of iteration k in the three-term CG: r_k sits in slot k mod 2
// (r_{k+1} overwrites r_{k-1}, which iteration k reads first).
__device__ __forceinline__ void* rslot(const Desc& d, int k) { return (k & 1) ? d.r1 : d.r; }

// ---------------------------------------------------------------------------
// x-pass, forward: polarization + real-to-complex FFT along axis 2.
// ---------------------------------------------------------------------------
// MI355X dispatches the blocks of a grid round-robin over its 8 XCDs (each
// with its own L2).  Renumbering so that each XCD walks a contiguous range of
// tiles keeps neighbouring tiles, which share cache lines at tile edges, in
// the same L2 at about the same time.
__device__ __forceinline__ int xcd_tile(int bid, int nblk) {
  constexpr int NX = 8;
  const int q = nblk / NX, r = nblk % NX;
  const int x = bid % NX, i = bid / NX;
  return x * q + (x < r ? x : r) + i;
}

// Rows of the x-passes sit in LDS as 3 complex sequences per row, each
// packing two real components (c = 2q, 2q + 1) as real and imaginary part,
// so that one complex FFT transforms two real rows.

// After a forward FFT: unpack the two real transforms of each sequence and
// store the half spectrum (k2 < N2/2) of the block's rows.
template <typename T, int N2, int ROWS, int NTB, typename S = C2<T>>
__device__ __forceinline__ void store_rows_r2c(S* spec, const C2<T>* z, long row0, long rows_total) {
  constexpr int RS = N2 + N2 / 16;
  constexpr int H = N2 / 2;
  for (int v = threadIdx.x; v < ROWS * H * 6; v += NTB) {
    const int rr = v / (H * 6), rem = v % (H * 6);
    const long row = row0 + rr;
    if (row >= rows_total) continue;
    const int k = rem / 6, c = rem % 6, q = c >> 1;
    const C2<T>* zr = z + (rr * 3 + q) * RS;
    const C2<T> z1 = zr[padx<true>(k)];
    const C2<T> z2 = conj(zr[padx<true>((N2 - k) % N2)]);
    C2<T> o;
    if ((c & 1) == 0) o = (z1 + z2) * T(0.5);
    else o = C2<T>{(z1.y - z2.y) * T(0.5), -(z1.x - z2.x) * T(0.5)};
    sstore<T>(spec + spec_at(row, k, c, rows_total, kchunk(H)), o);
  }
}

// Before an inverse FFT: load the half spectrum of the block's rows and
// rebuild the full Hermitian-packed sequences (Nyquist bin zero).
template <typename T, int N2, int ROWS, int NTB, typename S = C2<T>>
__device__ __forceinline__ void load_rows_c2r(const S* spec, C2<T>* z, long row0, long rows_total) {
  constexpr int RS = N2 + N2 / 16;
  constexpr int H = N2 / 2;
  // all of a thread's loads are issued before the first LDS write: inverse
  // field pass of 512^3 FP64 3.51 -> 2.63 ms, fused pass of 256^3 (three loads)
  // 1590 -> 1564 us FP32, (one) 1150 -> 1104 us FP64
  constexpr int NA = ROWS * H * 3, NL = (NA + NTB - 1) / NTB;
  C2<T> a[NL], b[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int u = threadIdx.x + i * NTB;
    const int v = NA % NTB == 0 || u < NA ? u : 0;
    const int rr = v / (H * 3), rem = v % (H * 3);
    const int k = rem / 3, q = rem % 3;
    // rows past the end are never used: they repeat the first
    const long row = row0 + rr < rows_total ? row0 + rr : row0;
    const S* s = spec + spec_at(row, k, 2 * q, rows_total, kchunk(H));
    a[i] = sload<T>(s);
    b[i] = sload<T>(s + 1);
  }
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int v = threadIdx.x + i * NTB;
    if (NA % NTB != 0 && v >= NA) continue;
    const int rr = v / (H * 3), rem = v % (H * 3);
    const int k = rem / 3, q = rem % 3;
    C2<T>* zr = z + (rr * 3 + q) * RS;
    if (k == 0) {
      zr[padx<true>(0)] = C2<T>{a[i].x, b[i].x};
      zr[padx<true>(H)] = C2<T>{0, 0};
    } else {
      zr[padx<true>(k)] = C2<T>{a[i].x - b[i].y, a[i].y + b[i].x};
      zr[padx<true>(N2 - k)] = C2<T>{a[i].x + b[i].y, b[i].x - a[i].y};
    }
  }
}

// ---------------------------------------------------------------------------
// Grouped x-passes (R1 > 1): axis 1 is transformed by two kernels.  With
// n1 = R1 R2, i1 = a R2 + b and k1 = q + R1 p,
//   sum_i1 x[i1] w_n1^(i1 k1) = sum_b w_R2^(b p) [ w_n1^(b q) sum_a w_R1^(a q) x[a R2 + b] ]:
// an x-pass block holds whole groups, the R1 rows (i0, a R2 + b) of fixed i0
// and b, and does the bracket in registers while it stores its half spectrum
// (value q in the place of row q R2 + b); the z-pass does the sum over b
// around its operator (k_gz).  The y-passes and their two trips through
// memory go; an application is three passes instead of five.
// ---------------------------------------------------------------------------

// Grid row of local row rr of a block (base: its first row, or first group).
template <int R1> __device__ __forceinline__ long tile_row(long base, int rr, long rows_total, int r2) {
  if constexpr (R1 == 1) {
    return base + rr;
  } else {
    const int gi = (int)base + rr / R1;
    const int i0 = gi / r2;
    return (long)gi * R1 < rows_total ? ((long)i0 * R1 + rr % R1) * r2 + (gi - i0 * r2) : rows_total;
  }
}

// tw1[g R1 + q] = exp(-2 pi i b q / n1) of the block's groups
// (every n1 with a grouped plan divides 768)
template <typename T, int R1, int G, int NTB>
__device__ __forceinline__ void build_group_twiddles(C2<T>* tw1, long g0, int r2) {
  const int step = 768 / (R1 * r2);
  for (int m = threadIdx.x; m < G * R1; m += NTB) {
    const int b = (int)(g0 + m / R1) % r2, q = m % R1;
    tw1[m] = tw_table<T, 768>.v[b * q * step];
  }
}

// store_rows_r2c for groups: the R1 rows of a (k2, component) are transformed
// along a in registers.  Chunks of 1 << kcs values of k2.  Binary16 storage
// divides by R1 so that the stored values stay in range.
template <typename T, int N2, int R1, int G, int NTB, typename S>
__device__ __forceinline__ void store_groups_r2c(S* spec, const C2<T>* z, const C2<T>* tw1, long g0, long rows_total,
                                                 int r2, int kcs) {
  constexpr int RS = N2 + N2 / 16;
  constexpr int H = N2 / 2;
  constexpr bool FULL = std::is_same<S, C2<T>>::value;
  for (int v = threadIdx.x; v < G * H * 6; v += NTB) {
    const int g = v / (H * 6), rem = v % (H * 6);
    const int gi = (int)g0 + g;
    if ((long)gi * R1 >= rows_total) continue;
    const int k = rem / 6, c = rem % 6, q = c >> 1;
    const C2<T>* zr = z + (g * R1 * 3 + q) * RS;
    const int kp = padx<true>(k), km = padx<true>((N2 - k) % N2);
    C2<T> o[R1];
#pragma unroll
    for (int a = 0; a < R1; ++a) {
      const C2<T> z1 = zr[a * 3 * RS + kp];
      const C2<T> z2 = conj(zr[a * 3 * RS + km]);
      if ((c & 1) == 0) o[a] = (z1 + z2) * T(0.5);
      else o[a] = C2<T>{(z1.y - z2.y) * T(0.5), -(z1.x - z2.x) * T(0.5)};
    }
    dft<R1, -1>(o);
    const int i0 = gi / r2, b = gi - i0 * r2;
    S* dst = spec + ((((long)(k >> kcs) * rows_total + (long)i0 * R1 * r2 + b) << kcs) + (k & ((1 << kcs) - 1))) * 6 + c;
    const int step = (r2 << kcs) * 6;
#pragma unroll
    for (int p = 0; p < R1; ++p) {
      C2<T> w = p ? cmul(o[p], tw1[g * R1 + p]) : o[p];
      if constexpr (!FULL) w = w * T(1.0 / R1);
      sstore<T>(dst + p * step, w);
    }
  }
}

// load_rows_c2r for groups: the inverse transform along q in registers first.
template <typename T, int N2, int R1, int G, int NTB>
__device__ __forceinline__ void load_groups_c2r(const C2<T>* spec, C2<T>* z, const C2<T>* tw1, long g0,
                                                long rows_total, int r2, int kcs) {
  constexpr int RS = N2 + N2 / 16;
  constexpr int H = N2 / 2;
  for (int v = threadIdx.x; v < G * H * 3; v += NTB) {
    const int g = v / (H * 3), rem = v % (H * 3);
    const int gi = (int)g0 + g;
    if ((long)gi * R1 >= rows_total) continue;   // rows past the end are never used
    const int k = rem / 3, q = rem % 3;
    const int i0 = gi / r2, b = gi - i0 * r2;
    const C2<T>* src =
        spec + ((((long)(k >> kcs) * rows_total + (long)i0 * R1 * r2 + b) << kcs) + (k & ((1 << kcs) - 1))) * 6 + 2 * q;
    const int step = (r2 << kcs) * 6;
    C2<T> a[R1], e[R1];
#pragma unroll
    for (int p = 0; p < R1; ++p) {
      C2<T> w[2];
      load_v<T, 2>(src + p * step, w);   // 2 q and the row offset are even: aligned to a pair
      a[p] = w[0];
      e[p] = w[1];
    }
#pragma unroll
    for (int p = 1; p < R1; ++p) {
      const C2<T> w = conj(tw1[g * R1 + p]);
      a[p] = cmul(a[p], w);
      e[p] = cmul(e[p], w);
    }
    dft<R1, 1>(a);
    dft<R1, 1>(e);
    C2<T>* zr = z + (g * R1 * 3 + q) * RS;
    if (k == 0) {
#pragma unroll
      for (int p = 0; p < R1; ++p) {
        zr[p * 3 * RS + padx<true>(0)] = C2<T>{a[p].x, e[p].x};
        zr[p * 3 * RS + padx<true>(H)] = C2<T>{0, 0};
      }
    } else {
      const int kp = padx<true>(k), km = padx<true>(N2 - k);
#pragma unroll
      for (int p = 0; p < R1; ++p) {
        zr[p * 3 * RS + kp] = C2<T>{a[p].x - e[p].y, a[p].y + e[p].x};
        zr[p * 3 * RS + km] = C2<T>{a[p].x + e[p].y, e[p].x - a[p].y};
      }
    }
  }
}

// groups per block of a grouped x-pass: at least 256 voxels
__host__ __device__ constexpr int group_count(int n2, int r1) { return 256 / (n2 * r1) > 1 ? 256 / (n2 * r1) : 1; }

template <typename T, int N2, bool ISO, int ROWS = x_rows<T>(N2), int NTB = NT, typename S = C2<T>, int PLAN = 0,
          int R1 = 1>
__global__ __launch_bounds__(NTB) void k_xfwd(const Desc* __restrict__ descs, int mode, long rows_total,
                                              long nvox, int r2, int kcs) {
  constexpr int RS = N2 + N2 / 16;
  __shared__ C2<T> z[ROWS * 3 * RS];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  const Desc& d = descs[blockIdx.y];
  if (!d.st->active) return;
  build_twiddles<T, N2, NTB>(tw);
  const int bid = R1 > 1 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const long row0 = (long)bid * (ROWS / R1);   // first row, or first group
  if constexpr (R1 > 1) build_group_twiddles<T, R1, ROWS / R1, NTB>(tw1, row0, r2);
  const T* mat = mat_of<T>(d);
  double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
  const T beta = (T)d.st->beta;
  const T ts = d.h16 ? (T)(d.tau_scale * d.st->idscale) : T(1);   // binary16 spectrum scale
  const bool first = d.st->first != 0;
  // correction fused into the FP64 residual pass (the three-term inner CG
  // leaves none after 0 iterations)
  const float* dl = (d.delta_gate && d.st2->iters == 0) ? nullptr : d.delta;

  for (int v = threadIdx.x; v < ROWS * N2; v += NTB) {
    const int rr = v / N2, i2 = v % N2;
    const long row = tile_row<R1>(row0, rr, rows_total, r2);
    T tau[6] = {0, 0, 0, 0, 0, 0};
    if (row < rows_total) {
      const long vox = row * N2 + i2;
      const int ph = d.phase[vox];
      if (mode == XF_LS) {
        T x[6] = {0, 0, 0, 0, 0, 0};
        T* xp = d.x_zero == X_ZERO ? nullptr : (T*)d.x;
        if (xp) {
          if (d.x_zero == X_READ) {
#pragma unroll
            for (int c = 0; c < 6; ++c) x[c] = xp[c * nvox + vox];
          }
          if (dl) {
#pragma unroll
            for (int c = 0; c < 6; ++c) {
              x[c] += (T)dl[c * nvox + vox];
              xp[c * nvox + vox] = x[c];
            }
          } else if (d.x_zero == X_INIT) {
#pragma unroll
            for (int c = 0; c < 6; ++c) xp[c * nvox + vox] = T(0);
          }
        }
        T pr[6];
        if (d.P) {
#pragma unroll
          for (int c = 0; c < 6; ++c) pr[c] = (T)d.P[c * nvox + vox];
        }
        if (!d.P) {
          T e[6];
#pragma unroll
          for (int c = 0; c < 6; ++c) e[c] = (T)d.E[c];
          apply_mat<T, ISO>(mat, ph, false, e, pr);
        }
        T dx[6];
        apply_mat<T, ISO>(mat, ph, true, x, dx);
#pragma unroll
        for (int c = 0; c < 6; ++c) tau[c] = pr[c] + dx[c];
        acc0 += frob_acc(pr, pr);
      } else if (mode == XF_MATVEC) {
        const T* vp = (const T*)d.x;
        T x[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) x[c] = vp[c * nvox + vox];
        apply_mat<T, ISO>(mat, ph, true, x, tau);
      } else if (mode == XF_CG) {
        const T* rp = (const T*)d.r;
        T* pp = (T*)d.p;
        T p[6], po[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          p[c] = rp[c * nvox + vox];
          po[c] = first ? T(0) : pp[c * nvox + vox];
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          if (!first) p[c] += beta * po[c];
          pp[c * nvox + vox] = p[c];
        }
        apply_mat<T, ISO>(mat, ph, true, p, tau);
        T cp[6];
        apply_mat<T, ISO>(mat, ph, false, p, cp);
        acc0 += frob_acc(p, cp);
      } else if (mode == XF_R3) {
        // start of the three-term CG: tau = (C - C0) r_0 and the sums
        // <r, r>_C0, <r, C r> (= <r, A r>_C0 on compatible r) and ||r||^2
        // (binary16 spectrum: tau carries the factor that keeps the transforms
        // in range, with the right-hand side's RMS divided out)
        const T* rp = (const T*)rslot(d, d.st->iters);
        T r[6], cr[6];
        double rd[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          r[c] = rp[c * nvox + vox];
          rd[c] = (double)r[c];
        }
        apply_mat<T, ISO>(mat, ph, true, r, tau);
        apply_mat<T, ISO>(mat, ph, false, r, cr);
        if (d.h16) {
#pragma unroll
          for (int c = 0; c < 6; ++c) tau[c] *= ts;
        }
        acc0 += c0_ip(d.lam0, d.mu0, rd, rd);
        acc1 += frob_acc(r, cr);
        acc2 += rd[0] * rd[0] + rd[1] * rd[1] + rd[2] * rd[2] + 2.0 * (rd[3] * rd[3] + rd[4] * rd[4] + rd[5] * rd[5]);
      } else if (mode == XF_BI1) {
        // BiCGSTAB, first pass of an iteration.  First iteration: p = r^ = r_0.
        // Later: the previous iteration's x += alpha p + omega s and r = s - omega t,
        // then p = r + beta (p - omega v).  tau = (C - C0) p.
        T* rp = (T*)d.r;
        T* pp = (T*)d.p;
        T p[6];
        if (first) {
          T* rh = (T*)d.rh;
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            const T rv = rp[c * nvox + vox];
            rh[c * nvox + vox] = rv;
            pp[c * nvox + vox] = rv;
            p[c] = rv;
          }
        } else {
          T* xp = (T*)d.x;
          const T* sp = (const T*)d.s;
          const T* tp = (const T*)d.t;
          const T* vp = (const T*)d.v;
          const T al = (T)d.st->alpha, om = (T)d.st->omega;
#pragma unroll
          for (int c = 0; c < 6; ++c) {
            const long i = c * nvox + vox;
            const T sv = sp[i], po = pp[i];
            xp[i] += al * po + om * sv;
            const T rv = sv - om * tp[i];
            rp[i] = rv;
            p[c] = rv + beta * (po - om * vp[i]);
            pp[i] = p[c];
          }
        }
        apply_mat<T, ISO>(mat, ph, true, p, tau);
      } else if (mode == XF_BI2) {
        // BiCGSTAB, second pass: s = r - alpha v, tau = (C - C0) s
        const T* rp = (const T*)d.r;
        const T* vp = (const T*)d.v;
        T* sp = (T*)d.s;
        const T al = (T)d.st->alpha;
        T sv[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          sv[c] = rp[c * nvox + vox] - al * vp[c * nvox + vox];
          sp[c * nvox + vox] = sv[c];
        }
        apply_mat<T, ISO>(mat, ph, true, sv, tau);
      } else {  // XF_C0
        // tau = C0 : r for the projection -Gamma0 * C0 r (r is the FP64 residual)
        const double* vp = (const double*)d.r;
        T v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = (T)vp[c * nvox + vox];
        const T tr = (T)d.lam0 * (v[0] + v[1] + v[2]);
#pragma unroll
        for (int c = 0; c < 6; ++c) tau[c] = T(2) * (T)d.mu0 * v[c] + (c < 3 ? tr : T(0));
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) z[(rr * 3 + q) * RS + padx<true>(i2)] = C2<T>{tau[2 * q], tau[2 * q + 1]};
  }
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NTB, 1, RS, false, true, -1, 1, PLAN>(z, tw);

  if constexpr (R1 > 1) store_groups_r2c<T, N2, R1, ROWS / R1, NTB, S>((S*)d.spec, z, tw1, row0, rows_total, r2, kcs);
  else store_rows_r2c<T, N2, ROWS, NTB, S>((S*)d.spec, z, row0, rows_total);
  double sums[3] = {acc0, acc1, acc2};
  block_sums<3, NTB>(sums, d.part_f + bid, gridDim.x);
}

// ---------------------------------------------------------------------------
// x-pass, inverse: complex-to-real FFT along axis 2 + update + reductions.
// ---------------------------------------------------------------------------
template <typename T, int N2, bool ISO, int ROWS = xi_rows<T>(N2), int NTB = NT, int PLAN = 0, int R1 = 1>
__global__ __launch_bounds__(NTB) void k_xinv(const Desc* __restrict__ descs, int mode, long rows_total, long nvox,
                                              int r2, int kcs) {
  constexpr int RS = N2 + N2 / 16;
  __shared__ C2<T> z[ROWS * 3 * RS];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  const Desc& d = descs[blockIdx.y];
  if (!d.st->active) return;
  build_twiddles<T, N2, NTB>(tw);
  const int bid = R1 > 1 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const long row0 = (long)bid * (ROWS / R1);   // first row, or first group
  if constexpr (R1 > 1) {
    build_group_twiddles<T, R1, ROWS / R1, NTB>(tw1, row0, r2);
    __syncthreads();
    load_groups_c2r<T, N2, R1, ROWS / R1, NTB>((const C2<T>*)d.spec, z, tw1, row0, rows_total, r2, kcs);
  } else {
    load_rows_c2r<T, N2, ROWS, NTB>((const C2<T>*)d.spec, z, row0, rows_total);
  }
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NTB, 1, RS, false, true, +1, 1, PLAN>(z, tw);

  const T alpha = (T)d.st->alpha;
  double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0, acc3 = 0.0, acc4 = 0.0;
  for (int v = threadIdx.x; v < ROWS * N2; v += NTB) {
    const int rr = v / N2, i2 = v % N2;
    const long row = tile_row<R1>(row0, rr, rows_total, r2);
    if (row >= rows_total) continue;
    const long vox = row * N2 + i2;
    T eta[6];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const C2<T> w = z[(rr * 3 + q) * RS + padx<true>(i2)];
      eta[2 * q] = w.x;
      eta[2 * q + 1] = w.y;
    }
    if (mode == XI_BS) {
      T* xp = (T*)d.x;
      T df[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) df[c] = eta[c] - (d.x_zero == X_ZERO ? T(0) : xp[c * nvox + vox]);
#pragma unroll
      for (int c = 0; c < 6; ++c) xp[c * nvox + vox] = eta[c];
      acc0 += frob_acc(df, df);
    } else if (mode == XI_RESID) {
      const T* xp = (const T*)d.x;
      double r[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) r[c] = (double)eta[c] - (d.x_zero == X_ZERO ? 0.0 : (double)xp[c * nvox + vox]);
      if (d.r_f32) {
        float* rp = (float*)d.r;
#pragma unroll
        for (int c = 0; c < 6; ++c) rp[c * nvox + vox] = (float)r[c];
      } else {
        T* rp = (T*)d.r;
#pragma unroll
        for (int c = 0; c < 6; ++c) rp[c * nvox + vox] = (T)r[c];
      }
      acc0 += r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + 2.0 * (r[3] * r[3] + r[4] * r[4] + r[5] * r[5]);
      acc1 += c0_ip(d.lam0, d.mu0, r, r);
    } else if (mode == XI_BS_INNER) {
      T* xp = (T*)d.x;
      const T* rp = (const T*)d.r;
      T df[6], nv[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        nv[c] = rp[c * nvox + vox] + eta[c];
        df[c] = nv[c] - xp[c * nvox + vox];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) xp[c * nvox + vox] = nv[c];
      acc0 += frob_acc(df, df);
    } else if (mode == XI_PROJ) {
      // eta = -P r.  Compatible part r_c = -eta goes to the FP32 inner right-hand
      // side; the rest, r - r_c = -(incompatible part of x), is applied to x.
      // x and r are FP64 in every instantiation (the projection itself may run
      // in FP32: it needs accuracy relative to r only).
      double* xp = (double*)d.x;
      const double* rp = (const double*)d.r;
      float* op = (float*)d.out;
      double rc[6], xv[6], rv[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        xv[c] = xp[c * nvox + vox];
        rv[c] = rp[c * nvox + vox];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        rc[c] = -(double)eta[c];
        xp[c * nvox + vox] = xv[c] + (rv[c] - rc[c]);
        op[c * nvox + vox] = (float)rc[c];
      }
      acc0 += rc[0] * rc[0] + rc[1] * rc[1] + rc[2] * rc[2] + 2.0 * (rc[3] * rc[3] + rc[4] * rc[4] + rc[5] * rc[5]);
      acc1 += c0_ip(d.lam0, d.mu0, rc, rc);
    } else if (mode == XI_BI1) {
      // BiCGSTAB: v = A p = p - eta; <r^, v>
      const T* pp = (const T*)d.p;
      const T* rh = (const T*)d.rh;
      T* vp = (T*)d.v;
      T v[6], h[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        v[c] = pp[c * nvox + vox] - eta[c];
        h[c] = rh[c * nvox + vox];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) vp[c * nvox + vox] = v[c];
      acc0 += frob_d(h, v);
    } else if (mode == XI_BI2) {
      // BiCGSTAB: t = A s = s - eta; <t,s>, <t,t>, <r^,s>, <r^,t>, <s,s>
      const T* sp = (const T*)d.s;
      const T* rh = (const T*)d.rh;
      T* tp = (T*)d.t;
      T sv[6], tv[6], h[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        sv[c] = sp[c * nvox + vox];
        h[c] = rh[c * nvox + vox];
        tv[c] = sv[c] - eta[c];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) tp[c * nvox + vox] = tv[c];
      acc0 += frob_d(tv, sv);
      acc1 += frob_d(tv, tv);
      acc2 += frob_d(h, sv);
      acc3 += frob_d(h, tv);
      acc4 += frob_d(sv, sv);
    } else {  // XI_CG: q = p - eta; x += alpha p; r -= alpha q
      T* xp = (T*)d.x;
      T* rp = (T*)d.r;
      const T* pp = (const T*)d.p;
      double r[6];
      T pv[6], xv[6], rv[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        pv[c] = pp[c * nvox + vox];
        xv[c] = xp[c * nvox + vox];
        rv[c] = rp[c * nvox + vox];
      }
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const T qv = pv[c] - eta[c];
        xp[c * nvox + vox] = xv[c] + alpha * pv[c];
        const T rn = rv[c] - alpha * qv;
        rp[c * nvox + vox] = rn;
        r[c] = (double)rn;
      }
      acc0 += c0_ip(d.lam0, d.mu0, r, r);
      acc1 += r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + 2.0 * (r[3] * r[3] + r[4] * r[4] + r[5] * r[5]);
    }
  }
  if (mode == XI_BI2) {
    double sums[5] = {acc0, acc1, acc2, acc3, acc4};
    block_sums<5, NTB>(sums, d.part_i + bid, gridDim.x);
  } else {
    double sums[2] = {acc0, acc1};
    block_sums<2, NTB>(sums, d.part_i + bid, gridDim.x);
  }
}

// ---------------------------------------------------------------------------
// Field x-passes: an FP64 field in (nc components, the others zero) and out
// (nc_out components, stored or accumulated), for the operator, displacement
// and theta transforms.  No constitutive law, no sums and no gating state: as
// modes of k_xfwd and k_xinv they had those passes' registers (112), a read of
// the phase ids and of the state before the first value.  Small calls are
// bound by the chain of launches, large ones by the memory rate.  With the
// descriptor in the launch arguments (no setup launch) an operator call takes,
// before -> now: 16^3 19.6 -> 15.6 us, 48x96x24 47.6 -> 41.0 us; the forward
// pass of 512^3 3.1 -> 2.4 ms (5.4 TB/s), the inverse 3.6 -> 2.6 (5.0 TB/s);
// the order-2 right-hand side of 64^3 725 -> 683 us.
// ---------------------------------------------------------------------------
template <typename T, int N2, int ROWS, int R1>
__device__ __forceinline__ void field_fwd_tile(const Desc& d, int bid, long rows_total, long nvox, int r2, int kcs,
                                               C2<T>* z, C2<T>* tw, C2<T>* tw1) {
  constexpr int RS = N2 + N2 / 16;
  const long row0 = (long)bid * (ROWS / R1);
  const double* ip = (const double*)d.io;
  const int nc = d.nc;
  for (int v = threadIdx.x; v < ROWS * N2; v += NT) {
    const int rr = v / N2, i2 = v % N2;
    const long row = tile_row<R1>(row0, rr, rows_total, r2);
    T t[6] = {0, 0, 0, 0, 0, 0};
    if (row < rows_total) {
#pragma unroll
      for (int c = 0; c < 6; ++c)
        if (c < nc) t[c] = (T)ip[c * nvox + row * N2 + i2];
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) z[(rr * 3 + q) * RS + padx<true>(i2)] = C2<T>{t[2 * q], t[2 * q + 1]};
  }
  build_twiddles<T, N2, NT>(tw);
  if constexpr (R1 > 1) build_group_twiddles<T, R1, ROWS / R1, NT>(tw1, row0, r2);
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NT, 1, RS, false, true, -1>(z, tw);
  if constexpr (R1 > 1) store_groups_r2c<T, N2, R1, ROWS / R1, NT, C2<T>>((C2<T>*)d.spec, z, tw1, row0, rows_total, r2, kcs);
  else store_rows_r2c<T, N2, ROWS, NT>((C2<T>*)d.spec, z, row0, rows_total);
}

template <typename T, int N2, int ROWS, int R1>
__global__ __launch_bounds__(NT) void k_field_fwd(const Desc* __restrict__ descs, long rows_total, long nvox, int r2,
                                                  int kcs) {
  __shared__ C2<T> z[ROWS * 3 * (N2 + N2 / 16)];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  field_fwd_tile<T, N2, ROWS, R1>(descs[blockIdx.y], xcd_tile(blockIdx.x, gridDim.x), rows_total, nvox, r2, kcs, z, tw,
                                  tw1);
}

// The same for one field whose descriptor comes with the launch; it leaves the
// descriptor and its gating state in memory for the passes that follow.
template <typename T, int N2, int ROWS, int R1>
__global__ __launch_bounds__(NT) void k_field_fwd1(Desc d, SolverState s, Desc* dd, long rows_total, long nvox, int r2,
                                                   int kcs) {
  __shared__ C2<T> z[ROWS * 3 * (N2 + N2 / 16)];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *dd = d;
    *d.st = s;
  }
  field_fwd_tile<T, N2, ROWS, R1>(d, xcd_tile(blockIdx.x, gridDim.x), rows_total, nvox, r2, kcs, z, tw, tw1);
}

template <typename T, int N2, int ROWS, int R1>
__global__ __launch_bounds__(NT) void k_field_inv(const Desc* __restrict__ descs, int accum, long rows_total, long nvox,
                                                  int r2, int kcs) {
  constexpr int RS = N2 + N2 / 16;
  __shared__ C2<T> z[ROWS * 3 * RS];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  const Desc& d = descs[blockIdx.y];
  const int bid = xcd_tile(blockIdx.x, gridDim.x);
  const long row0 = (long)bid * (ROWS / R1);
  build_twiddles<T, N2, NT>(tw);
  if constexpr (R1 > 1) {
    build_group_twiddles<T, R1, ROWS / R1, NT>(tw1, row0, r2);
    __syncthreads();
    load_groups_c2r<T, N2, R1, ROWS / R1, NT>((const C2<T>*)d.spec, z, tw1, row0, rows_total, r2, kcs);
  } else {
    load_rows_c2r<T, N2, ROWS, NT>((const C2<T>*)d.spec, z, row0, rows_total);
  }
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NT, 1, RS, false, true, +1>(z, tw);
  double* op = (double*)d.out;
  const int nco = d.nc_out ? d.nc_out : d.nc;
  for (int v = threadIdx.x; v < ROWS * N2; v += NT) {
    const int rr = v / N2, i2 = v % N2;
    const long row = tile_row<R1>(row0, rr, rows_total, r2);
    if (row >= rows_total) continue;
    const long vox = row * N2 + i2;
    double o[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) o[c] = accum && c < nco ? op[c * nvox + vox] : 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      const C2<T> w = z[(rr * 3 + c / 2) * RS + padx<true>(i2)];
      // streamed: 512^3 2635 -> 2567 us, 512^2 (three fields) 19.0 -> 16.5 us
      if (c < nco) __builtin_nontemporal_store(o[c] + (double)(c & 1 ? w.y : w.x), op + c * nvox + vox);
    }
  }
}

// ---------------------------------------------------------------------------
// Three-term CG iteration fused into one x-pass: inverse FFT of eta_k =
// -Gamma0 * (C - C0) r_k, the recurrences
//   w = A r_k = r_k - eta_k
//   r_{k+1} = omega_k (r_k - gamma_k w) + (1 - omega_k) r_{k-1}
//   x_{k+1} = omega_k (x_k + gamma_k r_k) + (1 - omega_k) x_{k-1}
// (gamma = <r,r>_C0 / <r,Ar>_C0, omega from the previous scalars; the first
// step has omega = 1; x_0 = 0 is never stored), the sums of r_{k+1} and the
// forward FFT of (C - C0) r_{k+1}, written back over the block's own spectrum
// rows.  r_k sits in slot k mod 2.  The x recurrence is applied two steps at a
// time: the odd iteration k forms x_k (from x_{k-1}, x_{k-2}, r_{k-1} and the
// previous scalars) and x_{k+1} from the same data plus r_k, the two residuals
// it reads anyway, so x is read and written on every other iteration only
// (the pair x_{k+1}, x_k overwrites x_{k-1}, x_{k-2} in slots x, x1).  A solve
// that stops after an even iteration forms its last x in k_cg3_finish.
// ---------------------------------------------------------------------------
// Row block b of nblk (its partial sums go to slot k at part_i + k nblk + b);
// z: ROWS * 3 * (N2 + N2/16) LDS elements, tw: tw_len(N2), tw1: ROWS (R1 > 1).
template <typename T, int N2, bool ISO, int ROWS, int NTB, typename S, int PLAN, int R1 = 1>
__device__ __forceinline__ void xcg3_tile(const Desc& d, int b, int nblk, long rows_total, long nvox, C2<T>* z,
                                          C2<T>* tw, C2<T>* tw1 = nullptr, int r2 = 1, int kcs = 0) {
  constexpr int RS = N2 + N2 / 16;
  build_twiddles<T, N2, NTB>(tw);
  const long row0 = (long)b * (ROWS / R1);   // first row, or first group
  // binary16 inner solve: eta comes from the FP32 copy, tau goes out in binary16
  constexpr bool FULL = std::is_same<S, C2<T>>::value;
  S* spec = (S*)d.spec;
  if constexpr (R1 > 1) {
    build_group_twiddles<T, R1, ROWS / R1, NTB>(tw1, row0, r2);
    __syncthreads();
    load_groups_c2r<T, N2, R1, ROWS / R1, NTB>((const C2<T>*)(FULL ? d.spec : d.spec2), z, tw1, row0, rows_total, r2,
                                               kcs);
  } else {
    load_rows_c2r<T, N2, ROWS, NTB>((const C2<T>*)(FULL ? d.spec : d.spec2), z, row0, rows_total);
  }
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NTB, 1, RS, false, true, +1, 1, PLAN>(z, tw);

  const int it = d.st->iters;
  const bool first = d.st->first != 0;
  const bool xstep = (it & 1) != 0;   // this iteration forms x_k and x_{k+1}
  const T gam = (T)d.st->alpha;
  const T om = first ? T(1) : (T)d.st->beta;
  const T gp = (T)d.st->alpha_prev;   // gamma_{k-1}
  const T op = (T)d.st->beta_prev;    // omega_{k-1} (1 at k = 1)
  const T* rc = (const T*)rslot(d, it);        // r_k
  const T* rpv = (const T*)rslot(d, it + 1);   // r_{k-1}, overwritten by r_{k+1}
  T* ro = (T*)rslot(d, it + 1);
  T* xn = (T*)d.x;    // x_{k-1} in, x_{k+1} out (odd k)
  T* xo = (T*)d.x1;   // x_{k-2} in, x_k out
  const T* mat = mat_of<T>(d);
  const T ts = d.h16 ? (T)(d.tau_scale * d.st->idscale) : T(1);   // binary16 spectrum scale
  double acc0 = 0.0, acc1 = 0.0, acc2 = 0.0;
  for (int v = threadIdx.x; v < ROWS * N2; v += NTB) {
    const int rr = v / N2, i2 = v % N2;
    const long row = tile_row<R1>(row0, rr, rows_total, r2);
    T tau[6] = {0, 0, 0, 0, 0, 0};
    if (row < rows_total) {
      const long vox = row * N2 + i2;
      const int ph = d.phase[vox];
      // every load of the voxel is issued before the first store (the output
      // slots may alias the inputs as far as the compiler knows)
      // (the iterates are streamed: each is read once per iteration, long after
      // it was written, so the accesses carry the non-temporal hint)
      T rk[6], rp[6], xa[6], xb[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        rk[c] = __builtin_nontemporal_load(rc + c * nvox + vox);
        rp[c] = first ? T(0) : __builtin_nontemporal_load(rpv + c * nvox + vox);
        // x_0 = 0 is never stored: the pair is read from the third iteration on
        xa[c] = (xstep && it > 1) ? __builtin_nontemporal_load(xn + c * nvox + vox) : T(0);
        xb[c] = (xstep && it > 1) ? __builtin_nontemporal_load(xo + c * nvox + vox) : T(0);
      }
      T rn[6];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const C2<T> e = z[(rr * 3 + q) * RS + padx<true>(i2)];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int c = 2 * q + h;
          const T eta = h ? e.y : e.x;
          const T r = rk[c];
          const T w = r - eta;
          const T rv = first ? r - gam * w : om * (r - gam * w) + (T(1) - om) * rp[c];
          __builtin_nontemporal_store(rv, ro + c * nvox + vox);
          if (xstep) {
            const T xk = op * (xa[c] + gp * rp[c]) + (T(1) - op) * xb[c];
            const T x1 = om * (xk + gam * r) + (T(1) - om) * xa[c];
            __builtin_nontemporal_store(x1, xn + c * nvox + vox);
            __builtin_nontemporal_store(xk, xo + c * nvox + vox);
          }
          rn[c] = rv;
        }
      }
      T cr[6];
      double rd[6];
#pragma unroll
      for (int c = 0; c < 6; ++c) rd[c] = (double)rn[c];
      apply_mat<T, ISO>(mat, ph, true, rn, tau);
      apply_mat<T, ISO>(mat, ph, false, rn, cr);
      acc0 += c0_ip(d.lam0, d.mu0, rd, rd);
      acc1 += frob_acc(rn, cr);
      acc2 += rd[0] * rd[0] + rd[1] * rd[1] + rd[2] * rd[2] + 2.0 * (rd[3] * rd[3] + rd[4] * rd[4] + rd[5] * rd[5]);
      if (d.h16) {
#pragma unroll
        for (int c = 0; c < 6; ++c) tau[c] *= ts;
      }
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) z[(rr * 3 + q) * RS + padx<true>(i2)] = C2<T>{tau[2 * q], tau[2 * q + 1]};
  }
  __syncthreads();
  lds_fft<T, N2, ROWS * 3, NTB, 1, RS, false, true, -1, 1, PLAN>(z, tw);
  if constexpr (R1 > 1) store_groups_r2c<T, N2, R1, ROWS / R1, NTB, S>(spec, z, tw1, row0, rows_total, r2, kcs);
  else store_rows_r2c<T, N2, ROWS, NTB, S>(spec, z, row0, rows_total);
  double sums[3] = {acc0, acc1, acc2};
  block_sums<3, NTB>(sums, d.part_i + b, nblk);
}

template <typename T, int N2, bool ISO, int ROWS = xi_rows<T>(N2), int NTB = NT, typename S = C2<T>, int PLAN = 0,
          int R1 = 1>
__global__ __launch_bounds__(NTB) void k_xcg3(const Desc* __restrict__ descs, long rows_total, long nvox, int r2,
                                              int kcs) {
  __shared__ C2<T> z[ROWS * 3 * (N2 + N2 / 16)];
  __shared__ C2<T> tw[tw_len(N2)];
  __shared__ C2<T> tw1[R1 > 1 ? ROWS : 1];
  const Desc& d = descs[blockIdx.y];
  if (!d.st->active) return;
  const int bid = R1 > 1 ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  xcg3_tile<T, N2, ISO, ROWS, NTB, S, PLAN, R1>(d, bid, (int)gridDim.x, rows_total, nvox, z, tw, tw1, r2, kcs);
}

// Three-term CG: the last x of loads whose solve stopped after an even
// iteration k (their state says so).  The odd iteration k - 1 left x_k and
// x_{k-1} in the slots x and x1; x_{k+1} = omega_k (x_k + gamma_k r_k) +
// (1 - omega_k) x_{k-1} goes to x (k = 0: x_1 = gamma_0 r_0); nothing reads
// x1 after a solve, so it is left as it is.  n = 6 x voxels.  Run once per
// stopped solve (the update is not idempotent).
template <typename T>
__global__ __launch_bounds__(NT) void k_cg3_finish(const Desc* __restrict__ descs, long n) {
  const Desc& d = descs[blockIdx.y];
  const SolverState* st = d.st;
  if (st->active || !st->xpend) return;
  const int k = st->iters - 1;
  const T gam = (T)st->alpha;
  const T om = k == 0 ? T(1) : (T)st->beta;
  const T* rk = (const T*)rslot(d, k);
  T* xn = (T*)d.x;
  const T* xo = (const T*)d.x1;
  for (long i = (long)blockIdx.x * NT + threadIdx.x; i < n; i += (long)gridDim.x * NT) {
    if (k == 0) {
      xn[i] = gam * rk[i];
    } else {
      const T xa = xn[i], xb = xo[i];
      xn[i] = om * (xa + gam * rk[i]) + (T(1) - om) * xb;
    }
  }
}

// BiCGSTAB: apply the last iteration's x += alpha p + omega s to loads that
// stopped (the next iteration's first pass would have done it).
template <typename T>
__global__ __launch_bounds__(NT) void k_bicg_finish(const Desc* __restrict__ descs, long n) {
  const Desc& d = descs[blockIdx.y];
  const SolverState* st = d.st;
  if (st->active || !st->pending) return;
  T* xp = (T*)d.x;
  const T* pp = (const T*)d.p;
  const T* sp = (const T*)d.s;
  const T al = (T)st->alpha, om = (T)st->omega;
  for (long i = (long)blockIdx.x * NT + threadIdx.x; i < n; i += (long)gridDim.x * NT) xp[i] += al * pp[i] + om * sp[i];
}

// ---------------------------------------------------------------------------
// y-pass: complex FFT along axis 1, in place.  Block = one i0 plane, CW
// consecutive columns of the [n1][n2/2 * 6] plane.
// ---------------------------------------------------------------------------
// ncols is a multiple of 6, so an access group of 2 columns is either all
// inside or all outside the plane (groups of 4 are used only when ncols is a
// multiple of 4).
// S = H2 (binary16 storage): the forward transform is divided by N1 so that
// the stored values stay in range.
// Binary16 tile transfers, G columns per access (ncols and c0 multiples of G,
// so a group is either all inside or all outside the plane).
// Tile loads of the y-pass: all of a thread's global loads are issued before
// its first LDS write, so their latencies overlap.  In FP32 places outside the
// plane load its first column instead of being skipped (their columns are not
// stored): around a skipped load the compiler waits for each binary16 value in
// turn (256^3, both directions, per load: 210 -> 193 us).  FP64 skips them, its
// loads then leave one by one: 512^3 2.53 ms a pass, else 3.59 ms.
template <typename T, int N1, int CW, int NTB, int G, typename S>
__device__ __forceinline__ void y_tile_load(const S* base, int ncols, int c0, C2<T>* buf) {
  constexpr int NA = N1 * CW / G, NL = (NA + NTB - 1) / NTB;
  C2<T> a[NL][G];
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int u = threadIdx.x + k * NTB;
    const int v = NA % NTB == 0 || u < NA ? u : 0;
    const int i1 = v / (CW / G), col = (v % (CW / G)) * G;
    const S* s = base + (long)i1 * ncols;
    if constexpr (sizeof(T) == 8) {
      a[k][0] = C2<T>{0, 0};
      if ((NA % NTB == 0 || u < NA) && c0 + col < ncols) a[k][0] = s[col];
    } else if constexpr (std::is_same<S, H2>::value) {
      hload_g<T, G>(s + (c0 + col < ncols ? col : 0), a[k]);
    } else {
      load_v<T, G>(s + (c0 + col < ncols ? col : 0), a[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int v = threadIdx.x + k * NTB;
    const int i1 = v / (CW / G), col = (v % (CW / G)) * G;
    if (NA % NTB == 0 || v < NA) {
#pragma unroll
      for (int q = 0; q < G; ++q) buf[i1 * CW + col + q] = a[k][q];
    }
  }
}
template <typename T, int N1, int CW, int NTB, int G>
__device__ __forceinline__ void y_h2_store(H2* base, int ncols, int c0, const C2<T>* buf, T scale) {
  for (int v = threadIdx.x; v < N1 * CW / G; v += NTB) {
    const int i1 = v / (CW / G), col = (v % (CW / G)) * G;
    if (c0 + col < ncols) {
      C2<T> a[G];
#pragma unroll
      for (int q = 0; q < G; ++q) a[q] = buf[i1 * CW + col + q] * scale;
      hstore_g<T, G>(base + (long)i1 * ncols + col, a);
    }
  }
}

template <typename T, int N1, int CW, int NTB, int DIR, int V, typename S, int PLAN>
__device__ __forceinline__ void ypass_body(S* base, int ncols, int c0, C2<T>* buf, const C2<T>* tw) {
  constexpr bool FULL = std::is_same<S, C2<T>>::value;
  static_assert(FULL || V == 1, "binary16 storage keeps one sequence per LDS slot");
  // binary16: up to 4 columns (16 bytes) per access when the plane width allows
  constexpr int G = CW % 4 == 0 ? 4 : CW % 2 == 0 ? 2 : 1;
  const bool wide = ncols % G == 0;
  // FP32: two columns (16 bytes) per access (ncols = 6 kc is even)
  constexpr int GF = (sizeof(T) == 4 && CW % 2 == 0) ? 2 : 1;
  if constexpr (FULL) {
    y_tile_load<T, N1, CW, NTB, GF>(base, ncols, c0, buf);
  } else {
    if (wide) y_tile_load<T, N1, CW, NTB, G>(base, ncols, c0, buf);
    else y_tile_load<T, N1, CW, NTB, 1>(base, ncols, c0, buf);
  }
  __syncthreads();
  lds_fft<T, N1, CW, NTB, CW, 1, true, false, DIR, V, PLAN>(buf, tw);
  if constexpr (FULL) {
    for (int v = threadIdx.x; v < N1 * CW / GF; v += NTB) {
      const int i1 = v / (CW / GF), col = (v % (CW / GF)) * GF;
      if (c0 + col < ncols) {
        C2<T> a[GF];
#pragma unroll
        for (int q = 0; q < GF; ++q) a[q] = buf[i1 * CW + col + q];
        store_v<T, GF>(base + (long)i1 * ncols + col, a);
      }
    }
  } else {
    // the forward transform is divided by N1 so that the stored values stay in range
    const T sc = DIR < 0 ? T(1) / T(N1) : T(1);
    if (wide) y_h2_store<T, N1, CW, NTB, G>(base, ncols, c0, buf, sc);
    else y_h2_store<T, N1, CW, NTB, 1>(base, ncols, c0, buf, sc);
  }
}

// Tile bid (plane i0 = bid / ntiles, columns from (bid % ntiles) CW) of one
// load; buf: N1 * CW LDS elements (16-byte aligned), tw: tw_len(N1).
template <typename T, int N1, int CW, int NTB, int V, typename S, int PLAN>
__device__ __forceinline__ void ypass_tile(const Desc& d, int bid, int dir, int ncols, int ntiles, C2<T>* buf,
                                           C2<T>* tw) {
  build_twiddles<T, N1, NTB>(tw);
  const long i0 = bid / ntiles;
  const int c0 = (bid % ntiles) * CW;
  // binary16 inner solve (spec2 set only in its descriptors): the inverse
  // y-transform runs in FP32 on the copy the spectral operator wrote
  const bool alt = std::is_same<S, C2<T>>::value && d.spec2 != nullptr && dir > 0;
  S* base = (S*)(alt ? d.spec2 : d.spec) + i0 * N1 * (long)ncols + c0;
  if (dir < 0) ypass_body<T, N1, CW, NTB, -1, V, S, PLAN>(base, ncols, c0, buf, tw);
  else ypass_body<T, N1, CW, NTB, +1, V, S, PLAN>(base, ncols, c0, buf, tw);
}

template <typename T, int N1, int CW = y_cols<T>(N1), int NTB = y_threads<T>(N1), bool REMAP = true,
          int V = vec_width<T>(), typename S = C2<T>, int PLAN = 0>
__global__ __launch_bounds__(NTB) void k_ypass(const Desc* __restrict__ descs, int dir, int ncols, int ntiles) {
  __shared__ __attribute__((aligned(16))) C2<T> buf[N1 * CW];
  __shared__ C2<T> tw[tw_len(N1)];
  const Desc& d = descs[blockIdx.y];
  if (!d.st->active) return;
  const int bid = REMAP ? xcd_tile(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  ypass_tile<T, N1, CW, NTB, V, S, PLAN>(d, bid, dir, ncols, ntiles, buf, tw);
}

// ---------------------------------------------------------------------------
// z-pass: forward FFT along axis 0, spectral operator, inverse FFT.
// Block = TK consecutive (i1, k2) columns x 6 components x all i0.
// ---------------------------------------------------------------------------
// 1 / x for a sum of squares of wave numbers (exact in T, >= 1).  FP32: the
// hardware estimate (1 ulp) and one Newton step
__device__ __forceinline__ float recip(float x) {
  const float r = __builtin_amdgcn_rcpf(x);
  return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}
__device__ __forceinline__ double recip(double x) { return 1.0 / x; }

// With integer wave vector k, |xi| = 2 pi |k|; every operator is a symmetric
// (or plain) product with w, which needs 1 / |k|^2 only and no square root.
// (gh, gr): the Green operator's constants of the entry.
template <typename T>
__device__ __forceinline__ void spectral_op(int op, T (&in)[6][2], T (&out)[6][2], T k0, T k1, T k2, T gh, T gr,
                                            T scale) {
  const T i2 = recip(k0 * k0 + k1 * k1 + k2 * k2);
  constexpr T I2PI = (T)(0.5 / 3.14159265358979323846);
  if (op == OP_GAMMA) {
    // eta_hat = -[ (n x v + v x n) / (2 mu0) - c2 (n.v) n x n ],  v = tau_hat n:
    // with u = gh tau_hat k / |k|^2 it is k x w + w x k, w = gr (k.u) k / |k|^2 - u.
    // No intermediate is larger than the result (before its scale) or smaller
    // by more than |k|, so FP32 fields and moduli of any magnitude pass; this
    // order also has the smallest error of those tried (relative L2 over
    // random modes, |k| to 128: FP64 2.0e-16, unit vectors 2.8e-16, constants
    // folded into 1 / |k|^2 and 1 / |k|^4 2.4e-16; FP32 0.99, 1.42, 1.18e-7)
    const T g0 = gh * (k0 * i2), g1 = gh * (k1 * i2), g2 = gh * (k2 * i2), b = gr * i2;
    const T f0 = scale * k0, f1 = scale * k1, f2 = scale * k2;
#pragma unroll
    for (int ri = 0; ri < 2; ++ri) {
      const T t0 = in[0][ri], t1 = in[1][ri], t2 = in[2][ri], t3 = in[3][ri], t4 = in[4][ri], t5 = in[5][ri];
      const T u0 = t0 * g0 + t5 * g1 + t4 * g2;
      const T u1 = t5 * g0 + t1 * g1 + t3 * g2;
      const T u2 = t4 * g0 + t3 * g1 + t2 * g2;
      const T s = (k0 * u0 + k1 * u1 + k2 * u2) * b;
      const T w0 = s * k0 - u0, w1 = s * k1 - u1, w2 = s * k2 - u2;
      out[0][ri] = T(2) * f0 * w0;
      out[1][ri] = T(2) * f1 * w1;
      out[2][ri] = T(2) * f2 * w2;
      out[3][ri] = f1 * w2 + f2 * w1;
      out[4][ri] = f0 * w2 + f2 * w0;
      out[5][ri] = f0 * w1 + f1 * w0;
    }
  } else if (op == OP_THETA) {
    // theta_hat_ij = (i/|xi|) [ n_i n_j (g.n) - (g_i n_j + n_i g_j) ] = i (k x w + w x k)_ij,
    // w = (-g + (g.k) k / (2 |k|^2)) / (2 pi |k|^2)
    const T f = scale * i2 * I2PI, h = T(0.5) * i2;
    T u[6][2];
#pragma unroll
    for (int ri = 0; ri < 2; ++ri) {
      const T g0 = in[0][ri], g1 = in[1][ri], g2 = in[2][ri];
      const T s = (g0 * k0 + g1 * k1 + g2 * k2) * h;
      const T w0 = f * (s * k0 - g0), w1 = f * (s * k1 - g1), w2 = f * (s * k2 - g2);
      u[0][ri] = T(2) * k0 * w0;
      u[1][ri] = T(2) * k1 * w1;
      u[2][ri] = T(2) * k2 * w2;
      u[3][ri] = k1 * w2 + k2 * w1;
      u[4][ri] = k0 * w2 + k2 * w0;
      u[5][ri] = k0 * w1 + k1 * w0;
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) {  // multiply by i
      out[c][0] = -u[c][1];
      out[c][1] = u[c][0];
    }
  } else {  // OP_DISP: u_hat = (-i/|xi|) [ 2 eps_hat n - n (n . eps_hat n) ], v = eps_hat k
    const T f = scale * i2 * I2PI;
    T w[3][2];
#pragma unroll
    for (int ri = 0; ri < 2; ++ri) {
      const T t0 = in[0][ri], t1 = in[1][ri], t2 = in[2][ri], t3 = in[3][ri], t4 = in[4][ri], t5 = in[5][ri];
      const T v0 = t0 * k0 + t5 * k1 + t4 * k2;
      const T v1 = t5 * k0 + t1 * k1 + t3 * k2;
      const T v2 = t4 * k0 + t3 * k1 + t2 * k2;
      const T s = (k0 * v0 + k1 * v1 + k2 * v2) * i2;
      w[0][ri] = T(2) * v0 - k0 * s;
      w[1][ri] = T(2) * v1 - k1 * s;
      w[2][ri] = T(2) * v2 - k2 * s;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {  // multiply by -i f
      out[c][0] = f * w[c][1];
      out[c][1] = -f * w[c][0];
    }
    out[3][0] = out[3][1] = out[4][0] = out[4][1] = out[5][0] = out[5][1] = T(0);
  }
}

// Tile bid (chunk bid / bpc, columns from (bid % bpc) TK) of one load; buf:
// N0 * 6 TK LDS elements, tw: tw_len(N0).
// plane: a 2-D grid (axis 0 of length 1).  N0 is then the length of axis 1 (n1
// is passed as 1), so this pass replaces both y-passes and the z-pass.
template <typename T, int N0, int TK, int NTB, typename S, int PLAN>
__device__ __forceinline__ void zpass_tile(const Desc& d, int bid, int op, int n1, int h, FastDiv bpc, FastDiv kcd,
                                           double scale, C2<T>* buf, C2<T>* tw, bool plane = false) {
  // (rows are not padded apart: a wave's FFT accesses cover several of them)
  constexpr int W = TK * 6;
  build_twiddles<T, N0, NTB>(tw);
  // columns (i1, k2 % kc) of one k2-chunk form a [N0][M][6] sub-array of bpc blocks
  const int kc = kcd.d, M = n1 * kc;
  int r;
  const int chunk = bpc.div(bid, r), m0 = r * TK;
  constexpr bool FULL = std::is_same<S, C2<T>>::value;
  // global accesses move GZ adjacent components (16 bytes in FP32, 8 in
  // binary16); W is even and so is every column's offset, so a group never
  // straddles a column
  constexpr int GZ = sizeof(T) == 4 ? 2 : 1;
  const int rs = M * 6;   // elements between rows i0
  const long base = (long)chunk * N0 * rs + m0 * 6;
  const S* src = (const S*)d.spec + base;
  // binary16 input; the output (after the spectral operator) goes to the FP32 copy
  C2<T>* dst = (C2<T>*)(FULL ? d.spec : d.spec2) + base;
  const int wlim = (M - m0) * 6;   // elements of a row inside the chunk (ragged last tile)
  // binary16 storage: the spectral operator also restores the scale of the
  // forward transforms (the descriptor's factor times the right-hand side's
  // RMS replaces 1/N)
  // (2-D: no forward y-pass divided by the axis length)
  const T sc = FULL ? (T)scale : (T)(d.op_scale * d.st->dscale * (plane ? 1.0 / N0 : 1.0));
  const T gh = (T)d.gam_h, gr = (T)d.gam_r;
  // all of a thread's loads are issued before the first LDS write, so their
  // latencies overlap (the tile's rows are far apart in memory).  Columns
  // outside the chunk load its first one in FP32: skipped instead, they made
  // the compiler wait for each binary16 value in turn (256^3, three loads: 569
  // -> 442 us).  FP64 skips them: its loads then leave one by one, and the
  // narrow rows of long axes (96 bytes) come faster (512^3 with 256 threads 3.9
  // ms, all at once about 6)
  constexpr int NA = N0 * W / GZ, NL = (NA + NTB - 1) / NTB;
  {
    C2<T> a[NL][GZ];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int u = threadIdx.x + k * NTB;
      const int v = NA % NTB == 0 || u < NA ? u : 0;
      const int i0 = v / (W / GZ), w = (v % (W / GZ)) * GZ;
      const S* s = src + (long)i0 * rs;
      if constexpr (sizeof(T) == 8) {
        a[k][0] = C2<T>{0, 0};
        if ((NA % NTB == 0 || u < NA) && w < wlim) a[k][0] = s[w];
      } else if constexpr (FULL) {
        load_v<T, GZ>(s + (w < wlim ? w : 0), a[k]);
      } else {
        hload_g<T, GZ>(s + (w < wlim ? w : 0), a[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int v = threadIdx.x + k * NTB;
      const int i0 = v / (W / GZ), w = (v % (W / GZ)) * GZ;
      if (NA % NTB == 0 || v < NA) {
#pragma unroll
        for (int q = 0; q < GZ; ++q) buf[i0 * W + w + q] = a[k][q];
      }
    }
  }
  __syncthreads();
  if constexpr (N0 > 1) lds_fft<T, N0, W, NTB, W, 1, true, false, -1, 1, PLAN>(buf, tw);
  const int k1b = kcd.div(m0, r), k2b = r;   // first column
  for (int v = threadIdx.x; v < N0 * TK; v += NTB) {
    const int k0 = v / TK, col = v % TK;
    if (m0 + col >= M) continue;
    int k1 = k1b, k2 = k2b + col;
    if (TK > 1) {
      for (; k2 >= kc; ++k1) k2 -= kc;
    }
    k2 += chunk * kc;
    const bool nyq = ((N0 % 2 == 0) && k0 == N0 / 2) || ((n1 % 2 == 0) && k1 == n1 / 2);
    const int k0s = k0 < (N0 + 1) / 2 ? k0 : k0 - N0;
    const int k1s = k1 < (n1 + 1) / 2 ? k1 : k1 - n1;
    C2<T>* e = buf + k0 * W + col * 6;
    T in[6][2], out[6][2];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      in[c][0] = e[c].x;
      in[c][1] = e[c].y;
    }
    if (nyq || (k0s == 0 && k1s == 0 && k2 == 0)) {
#pragma unroll
      for (int c = 0; c < 6; ++c) out[c][0] = out[c][1] = T(0);
    } else {
      spectral_op<T>(op, in, out, (T)(plane ? 0 : k0s), (T)(plane ? k0s : k1s), (T)k2, gh, gr, sc);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) e[c] = C2<T>{out[c][0], out[c][1]};
  }
  __syncthreads();
  if constexpr (N0 > 1) lds_fft<T, N0, W, NTB, W, 1, true, false, +1, 1, PLAN>(buf, tw);
#pragma unroll
  for (int k = 0; k < NL; ++k) {
    const int v = threadIdx.x + k * NTB;
    const int i0 = v / (W / GZ), w = (v % (W / GZ)) * GZ;
    if ((NA % NTB == 0 || v < NA) && w < wlim) {
      C2<T> a[GZ];
#pragma unroll
      for (int q = 0; q < GZ; ++q) a[q] = buf[i0 * W + w + q];
      if constexpr (FULL || TK % 4 != 0) {
        store_v<T, GZ>(dst + (long)i0 * rs + w, a);
      } else {
        // the FP32 copy after the operator goes to its own buffer: streamed
        // with the non-temporal hint, which pays only when every row segment
        // (48 TK bytes) covers whole 64-byte chunks
        static_assert(GZ == 2, "binary16 input implies FP32 pairs");
        typedef float f4 __attribute__((ext_vector_type(4)));
        const f4 o = {a[0].x, a[0].y, a[1].x, a[1].y};
        __builtin_nontemporal_store(o, (f4*)(dst + (long)i0 * rs + w));
      }
    }
  }
}

// fin >= 0 (z-passes of 2-D grids, grouped z-passes): the first block of every
// entry does that finalize instead of a tile.  The operator needs none of the
// scalars a finalize sets; blocks that still see a load active which it stops
// write a spectrum that nothing reads.  The flag can change while the launch
// runs, so each block reads it once for all of its waves (block_active): waves
// that read it by themselves could part ways ahead of the tile's barriers.
template <int NTB>
__device__ __forceinline__ bool carried_finalize(const Desc& d, int fin, int nblk_f, int nblk_i, int& bid, int& nblk) {
  bid = blockIdx.x;
  nblk = gridDim.x;
  if (fin < 0) return false;
  --nblk;
  if (bid-- > 0) return false;
  finalize_entry<256, true, NTB>(d, fin, nblk_f, nblk_i);
  return true;
}

__device__ __forceinline__ bool block_active(const Desc& d, int fin) {
  if (fin < 0) return d.st->active != 0;   // nothing writes the state in this launch
  __shared__ int act;
  if (threadIdx.x == 0) act = flag_read(d.st);
  __syncthreads();
  return act != 0;
}

template <typename T, int N0, int TK = z_cols<T>(N0), int NTB = NT, typename S = C2<T>, int PLAN = 0>
__global__ __launch_bounds__(NTB) void k_zpass(const Desc* __restrict__ descs, int op, int n1, int h, FastDiv bpc,
                                               FastDiv kcd, double scale, int plane, int fin, int nblk_f,
                                               int nblk_i) {
  __shared__ __attribute__((aligned(16))) C2<T> buf[N0 * TK * 6];
  __shared__ C2<T> tw[tw_len(N0)];
  const Desc& d = descs[blockIdx.y];
  int bid, nblk;
  if (carried_finalize<NTB>(d, fin, nblk_f, nblk_i, bid, nblk) || !block_active(d, fin)) return;
  bid = xcd_tile(bid, nblk);
  zpass_tile<T, N0, TK, NTB, S, PLAN>(d, bid, op, n1, h, bpc, kcd, scale, buf, tw, plane != 0);
}

// ---------------------------------------------------------------------------
// Grouped z-pass (after grouped x-passes, which did the radix-R1 part of axis
// 1): R2-point transforms along axis 1, forward FFT along axis 0, spectral
// operator at k1 = q + R1 p, and the inverses.  Block = KC values of k2, one
// q, every b and i0; a row of the tile, [b][k2][6], is contiguous.  Rows are
// an odd number of elements apart (WP): the passes along a column and the
// operator's threads then spread over the banks.
// Bound by vector instructions more than by memory: 128^3, six loads, binary16
// in, 151 MB read and 302 MB written in 150 us (3.0 TB/s; 77 us at the rate of
// an in-place stream), in which the SIMDs issue vector instructions for 101 us
// and LDS instructions for 29 us (bank conflicts 8 us).  FP32, launches of 2.9
// loads on average: 74 us, two y-passes and a z-pass before 139; the fused pass
// rose from 164 to 189.
// ---------------------------------------------------------------------------
template <typename T> __host__ __device__ constexpr int gz_kc(int n0, int r2) { return n0 * r2 * 6 * 2 * (int)sizeof(T) <= 16384 ? 2 : 1; }

// R2-point transforms along axis 1 of the tile, in place: each thread reads
// and writes the R2 values of its own (i0, k2, component).
template <typename T, int N0, int R2, int KC, int NTB, int DIR>
__device__ __forceinline__ void gz_axis1(C2<T>* buf) {
  constexpr int C = KC * 6, WP = R2 * C + 1;
  // lanes along i0: WP apart, every bank once
  for (int v = threadIdx.x; v < N0 * C; v += NTB) {
    C2<T>* e = buf + v % N0 * WP + v / N0;
    C2<T> x[R2];
#pragma unroll
    for (int b = 0; b < R2; ++b) x[b] = e[b * C];
    dft<R2, DIR>(x);
#pragma unroll
    for (int b = 0; b < R2; ++b) e[b * C] = x[b];
  }
}

template <typename T, int N0, int R2, int KC, int NTB, typename S>
__device__ __forceinline__ void gz_tile(const Desc& d, int bid, int op, int n1, double scale, int kcs, C2<T>* buf,
                                        C2<T>* tw) {
  constexpr int W = KC * R2 * 6, WP = W + 1;
  constexpr bool FULL = std::is_same<S, C2<T>>::value;
  constexpr int GZ = FULL && sizeof(T) == 8 ? 1 : 2;   // values per access: a segment of the tile holds 6 KC
  build_twiddles<T, N0, NTB>(tw);
  // blocks of one chunk and q, which share its lines, are neighbours
  const int r1 = n1 / R2, per = (1 << kcs) / KC;
  const int kk = bid % per * KC, cq = bid / per, chunk = cq / r1, q = cq - chunk * r1;
  const int k20 = (chunk << kcs) + kk;
  const int bs = 6 << kcs;                        // elements between values b
  const int rs = n1 * bs;                         // and between rows i0
  const long base = (long)chunk * N0 * rs + (long)q * R2 * bs + kk * 6;
  const S* src = (const S*)d.spec + base;
  C2<T>* dst = (C2<T>*)(FULL ? d.spec : d.spec2) + base;
  auto at = [&](int v) {   // offset of access v of the tile
    const int w = v % (W / GZ) * GZ;
    return (long)(v / (W / GZ)) * rs + w / (KC * 6) * bs + w % (KC * 6);
  };
  // binary16 storage: the operator restores the scale of the forward
  // transforms (the x-pass divided by R1 only)
  const T sc = FULL ? (T)scale : (T)(d.op_scale * d.st->dscale / R2);
  const T gh = (T)d.gam_h, gr = (T)d.gam_r;
  constexpr int NA = N0 * W / GZ, NL = (NA + NTB - 1) / NTB;
  {
    C2<T> a[NL][GZ];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int u = threadIdx.x + k * NTB;
      const S* s = src + at(NA % NTB == 0 || u < NA ? u : 0);
      if constexpr (FULL) load_v<T, GZ>(s, a[k]);
      else hload_g<T, GZ>(s, a[k]);
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int v = threadIdx.x + k * NTB;
      if (NA % NTB == 0 || v < NA) {
#pragma unroll
        for (int g = 0; g < GZ; ++g) buf[(v / (W / GZ)) * WP + (v % (W / GZ)) * GZ + g] = a[k][g];
      }
    }
  }
  __syncthreads();
  gz_axis1<T, N0, R2, KC, NTB, -1>(buf);
  __syncthreads();
  lds_fft<T, N0, W, NTB, WP, 1, true, false, -1>(buf, tw);
  for (int v = threadIdx.x; v < N0 * R2 * KC; v += NTB) {
    const int k0 = v % N0;
    int m = v / N0;   // one value per wave where N0 is a multiple of it
    if constexpr (N0 % 64 == 0) m = __builtin_amdgcn_readfirstlane(m);
    const int p = m / KC, k1 = q + r1 * p, k2 = k20 + m % KC;
    const bool nyq = (N0 % 2 == 0 && k0 == N0 / 2) || (n1 % 2 == 0 && k1 == n1 / 2);
    const int k0s = k0 < (N0 + 1) / 2 ? k0 : k0 - N0;
    const int k1s = k1 < (n1 + 1) / 2 ? k1 : k1 - n1;
    C2<T>* e = buf + k0 * WP + m * 6;
    T in[6][2], out[6][2];
#pragma unroll
    for (int c = 0; c < 6; ++c) {
      in[c][0] = e[c].x;
      in[c][1] = e[c].y;
    }
    if (nyq || (k0s == 0 && k1s == 0 && k2 == 0)) {
#pragma unroll
      for (int c = 0; c < 6; ++c) out[c][0] = out[c][1] = T(0);
    } else {
      spectral_op<T>(op, in, out, (T)k0s, (T)k1s, (T)k2, gh, gr, sc);
    }
#pragma unroll
    for (int c = 0; c < 6; ++c) e[c] = C2<T>{out[c][0], out[c][1]};
  }
  __syncthreads();
  lds_fft<T, N0, W, NTB, WP, 1, true, false, +1>(buf, tw);
  gz_axis1<T, N0, R2, KC, NTB, +1>(buf);
  __syncthreads();
  constexpr int GS = sizeof(T) == 4 ? 2 : 1;
  for (int v = threadIdx.x; v < N0 * W / GS; v += NTB) {
    const int i0 = v / (W / GS), w = (v % (W / GS)) * GS;
    C2<T> a[GS];
#pragma unroll
    for (int g = 0; g < GS; ++g) a[g] = buf[i0 * WP + w + g];
    store_v<T, GS>(dst + (long)i0 * rs + w / (KC * 6) * bs + w % (KC * 6), a);
  }
}

// LDS elements of the tile (tw besides: tw_len(N0))
template <typename T> constexpr int gz_elems(int n0, int r2) { return n0 * (gz_kc<T>(n0, r2) * r2 * 6 + 1); }

template <typename T, int N0, int R2, int NTB, typename S>
__global__ __launch_bounds__(NTB) void k_gz(const Desc* __restrict__ descs, int op, int n1, double scale, int kcs,
                                            int fin, int nblk_f, int nblk_i) {
  __shared__ __attribute__((aligned(16))) C2<T> buf[gz_elems<T>(N0, R2)];
  __shared__ C2<T> tw[tw_len(N0)];
  const Desc& d = descs[blockIdx.y];
  int bid, nblk;
  if (carried_finalize<NTB>(d, fin, nblk_f, nblk_i, bid, nblk) || !block_active(d, fin)) return;
  gz_tile<T, N0, R2, gz_kc<T>(N0, R2), NTB, S>(d, xcd_tile(bid, nblk), op, n1, scale, kcs, buf, tw);
}

// Which grids take the grouped passes: axis lengths whose kernels are compiled
// and whose tiles leave room for three blocks per CU (FP64: two).  R2 (0: not
// grouped) balances the two passes; measured, us per three-term iteration:
// FP64 six loads 64^3 R2 = 8 138, 4 144; 48^3 4 73, 8 78; 96^3 8 520 (five
// passes 595).  Axes of 256 (FP32 six loads, FP64 three; grouped against five
// passes): FP32 64x256x128 623, 730; 128x256x64 683, 746; 256x64x64 306, 356;
// 256x128x64 690, 772; 256x16x96 138, 192; FP64 48x256x64 250, 284; 256x16x64
// 93, 170; 64x128x64 161, 205.  At 256^3 no R2 has tiles that fit both passes.
template <typename T> constexpr int group_lds() { return sizeof(T) == 8 ? 80 * 1024 : 56 * 1024; }
// the preferred R2 of axis 1, and a second choice where its tile does not fit
template <typename T> __host__ __device__ constexpr int group_r2(int n1) {
  if (sizeof(T) == 8) return n1 == 64 || n1 == 96 || n1 == 128 ? 8 : n1 >= 8 && n1 <= 48 ? 4 : n1 == 256 ? 16 : 0;
  return n1 == 8 ? 4 : n1 == 16 || n1 == 32 || n1 == 64 || n1 == 128 ? 8
         : n1 == 12 || n1 == 24 || n1 == 48 || n1 == 96 ? 6 : n1 == 256 ? 16 : 0;
}
template <typename T> constexpr int group_r2b(int n1) {
  if (sizeof(T) == 8) return n1 == 64 ? 4 : n1 >= 8 && n1 <= 32 ? 2 : 0;
  return n1 == 256 ? 8 : n1 == 16 || n1 == 32 || n1 == 64 || n1 == 128 ? 4 : 0;
}
// With R1 >= 16 rows per group a block has few items in its spectrum transfers
// on short axes 2, and the fused pass loses more than the y-passes cost (five
// passes the second figure, FP32 six loads: 64x256x16 121, 111; 128x256x32 384,
// 354; 256x64x32 179, 193) unless the grid is small enough to be bound by its
// launches (64x128x16 70, 79; 16x256x8 33, 43)
constexpr bool group_pays(int r1, int n2, long nvox) {
  return r1 < 16 || n2 >= 2 * r1 || (r1 == 16 && nvox <= 1 << 17);
}
// log2 of the k2 values per chunk: the x-passes move segments of 6 << kcs
// values, the z-pass rows of 6 R2 values broken into segments of 6 kc.  Wider
// chunks speed up the one and slow down the other (128^3, six loads, kcs = 0,
// 1, 2: x 467, 442, 407 us, z 124, 137, 168; 96^3: 193, 185, 181 and 69, 69, 69).
__host__ __device__ constexpr int group_kcs(int r2, int h) { return r2 == 6 && h % 4 == 0 ? 2 : 1; }
template <typename T> constexpr int gx_rows(int n2, int r1) { return group_count(n2, r1) * r1; }
template <typename T> constexpr bool gx_fits(int n2, int r1) {
  return gx_rows<T>(n2, r1) * 3 * (n2 + n2 / 16) * 2 * (int)sizeof(T) <= group_lds<T>();
}
template <typename T> constexpr bool gz_fits(int n0, int r2) {
  return gz_elems<T>(n0, r2) * 2 * (int)sizeof(T) <= group_lds<T>();
}

// axis lengths of the grouped passes
#define FFTH_GROUP_N(X) X(8) X(12) X(16) X(24) X(32) X(48) X(64) X(96) X(128) X(256)
#define FFTH_GROUP_ITEM(N) N,
constexpr int GROUP_SIZES[] = {FFTH_GROUP_N(FFTH_GROUP_ITEM)};
#undef FFTH_GROUP_ITEM
constexpr bool group_size(int n) {
  for (int m : GROUP_SIZES)
    if (m == n) return true;
  return false;
}

// Lengths of the multi-size launches (below).
constexpr int MULTI_SIZES[] = {16, 24, 32, 48, 64, 96, 128};   // the lengths of FFTH_MULTI_SIZES
constexpr bool multi_size(int n) {
  for (int m : MULTI_SIZES)
    if (m == n) return true;
  return false;
}

// The rule: R2 of a grid's grouped passes, 0 where it runs the classical ones.
// (grids of the multi-size launches are grouped in FP32, whatever their axis 2)
template <typename T> constexpr int group_pick(int n0, int n1, int n2) {
  if (!group_size(n0) || !group_size(n1) || !group_size(n2)) return 0;
  const bool multi = sizeof(T) == 4 && multi_size(n0) && multi_size(n1) && multi_size(n2);
  for (int r2 : {group_r2<T>(n1), group_r2b<T>(n1)}) {
    if (r2 == 0 || !gx_fits<T>(n2, n1 / r2) || !gz_fits<T>(n0, r2)) continue;
    if (multi || group_pays(n1 / r2, n2, (long)n0 * n1 * n2)) return r2;
  }
  return 0;
}
// Whether a grid takes an x-pass of (n2, R1), a z-pass of (n0, R2): the others
// are not compiled.
template <typename T> constexpr bool gx_used(int n2, int r1) {
  for (int n0 : GROUP_SIZES)
    for (int n1 : GROUP_SIZES)
      if (n1 % r1 == 0 && group_pick<T>(n0, n1, n2) * r1 == n1) return true;
  return false;
}
template <typename T> constexpr bool gz_used(int n0, int r2) {
  for (int n1 : GROUP_SIZES)
    for (int n2 : GROUP_SIZES)
      if (group_pick<T>(n0, n1, n2) == r2) return true;
  return false;
}

// ---------------------------------------------------------------------------
// Multi-size launches of the FP32 inner iteration: one launch per grouped
// pass covers loads of grids of different sizes (axis lengths from
// FFTH_MULTI_SIZES, all grouped).  Each load's descriptor carries its grid
// (n); the launch's blocks are the tiles of all its loads, listed by a segment
// table (MultiSegs) of consecutive loads of one grid, each tile the code of
// the per-size kernel of its lengths (256 threads): the same arithmetic bit
// for bit.  LDS is sized by the launch for its largest tile.
// ---------------------------------------------------------------------------
#define FFTH_MULTI_SIZES(X) X(16) X(24) X(32) X(48) X(64) X(96) X(128)
constexpr int MULTI_NT = 256;
#define FFTH_MULTI_CHECK(N) static_assert(multi_size(N) && group_r2<float>(N) >= 6 && gz_fits<float>(N, 8) && gx_fits<float>(N, 16), "multi-size lengths are grouped");
FFTH_MULTI_SIZES(FFTH_MULTI_CHECK)
#undef FFTH_MULTI_CHECK
#define FFTH_MULTI_COUNT(N) +1
static_assert(0 FFTH_MULTI_SIZES(FFTH_MULTI_COUNT) == sizeof(MULTI_SIZES) / sizeof(int), "FFTH_MULTI_SIZES and MULTI_SIZES differ");
#undef FFTH_MULTI_COUNT
// blocks of one load of grid n in each multi-size pass, and its LDS bytes (host and device)
__host__ __device__ constexpr int multi_z_blocks(const int* n) {
  const int r2 = group_r2<float>(n[1]);
  return n[2] / 2 / gz_kc<float>(n[0], r2) * (n[1] / r2);
}
__host__ __device__ constexpr int multi_x_blocks(const int* n) {
  const int r2 = group_r2<float>(n[1]), g = group_count(n[2], n[1] / r2);
  return (n[0] * r2 + g - 1) / g;
}
constexpr int multi_z_lds(const int* n) { return (gz_elems<float>(n[0], group_r2<float>(n[1])) + n[0]) * 8; }
constexpr int multi_x_lds(const int* n) {
  const int rows = gx_rows<float>(n[2], n[1] / group_r2<float>(n[1]));
  return (rows * 3 * (n[2] + n[2] / 16) + n[2] + rows) * 8;
}

// Block of a multi-size launch: its load (descriptor index, -1 for padding)
// and that load's tile.  Each load of segment s owns bpd[s] blocks padded to
// a multiple of 8 (the XCDs; segments start at multiples of 8 too), so a
// block's XCD is its tile slot mod 8; the tiles of every load are renumbered
// XCD-aware as the per-size passes do (each XCD walks a contiguous run of
// each load's tiles).
__device__ __forceinline__ int multi_block(const MultiSegs& sg, int& tile) {
  const int b = blockIdx.x;
  int s = 0;
  while (s + 1 < sg.n && b >= sg.off[s + 1]) ++s;
  const int bpd = sg.bpd[s], slots = (bpd + 7) / 8 * 8;
  const int r = b - sg.off[s], load = r / slots, t = r % slots;
  if (t >= bpd) return -1;
  tile = xcd_tile(t, bpd);
  return sg.first[s] + load;
}

// fin >= 0: the blocks after the last segment finalize the launch's loads
template <typename S>
__global__ __launch_bounds__(MULTI_NT) void k_gz_multi(const Desc* __restrict__ descs, int op, MultiSegs sg, int fin) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  if ((int)blockIdx.x >= sg.off[sg.n]) {
    finalize_entry<MULTI_NT, true>(descs[sg.first[0] + blockIdx.x - sg.off[sg.n]], fin, 0, -1);
    return;
  }
  int bid;
  const int di = multi_block(sg, bid);
  if (di < 0) return;
  const Desc& d = descs[di];
  if (!block_active(d, fin)) return;
  const int n1 = d.n[1], kcs = group_kcs(group_r2<float>(n1), d.n[2] / 2);
  C2<float>* tw = (C2<float>*)lds;   // N0 values, then the tile
  switch (d.n[0]) {
#define FFTH_MULTI_Z(N)                                                                                               \
  case N:                                                                                                             \
    if (group_r2<float>(n1) == 8)                                                                                     \
      gz_tile<float, N, 8, gz_kc<float>(N, 8), MULTI_NT, S>(d, bid, op, n1, d.inv_nvox, kcs, tw + N, tw);                 \
    else                                                                                                              \
      gz_tile<float, N, 6, gz_kc<float>(N, 6), MULTI_NT, S>(d, bid, op, n1, d.inv_nvox, kcs, tw + N, tw);                 \
    break;
    FFTH_MULTI_SIZES(FFTH_MULTI_Z)
#undef FFTH_MULTI_Z
  }
}

// The tile of the fused pass is block b of its load, whose partial sums go to
// slot b of the load's array.
template <int N, bool ISO, typename S, int R1>
__device__ __forceinline__ void multi_x_tile(const Desc& d, int b, C2<float>* lds, int r2) {
  constexpr int ROWS = gx_rows<float>(N, R1);
  const int nb = (d.n[0] * r2 + ROWS / R1 - 1) / (ROWS / R1);
  const long rows = (long)d.n[0] * d.n[1];
  xcg3_tile<float, N, ISO, ROWS, MULTI_NT, S, 0, R1>(d, b, nb, rows, rows * N, lds + N + ROWS, lds, lds + N, r2,
                                                       group_kcs(r2, N / 2));
}
template <bool ISO, typename S>
__global__ __launch_bounds__(MULTI_NT) void k_xcg3_multi(const Desc* __restrict__ descs, MultiSegs sg) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  int b;
  const int di = multi_block(sg, b);
  if (di < 0) return;
  const Desc& d = descs[di];
  if (!d.st->active) return;
  const int r2 = group_r2<float>(d.n[1]);
  switch (d.n[2] * 32 + d.n[1] / r2) {
#define FFTH_MULTI_X(N)                                                                       \
  case N * 32 + 2: multi_x_tile<N, ISO, S, 2>(d, b, (C2<float>*)lds, r2); break;             \
  case N * 32 + 4: multi_x_tile<N, ISO, S, 4>(d, b, (C2<float>*)lds, r2); break;             \
  case N * 32 + 8: multi_x_tile<N, ISO, S, 8>(d, b, (C2<float>*)lds, r2); break;             \
  case N * 32 + 16: multi_x_tile<N, ISO, S, 16>(d, b, (C2<float>*)lds, r2); break;
    FFTH_MULTI_SIZES(FFTH_MULTI_X)
#undef FFTH_MULTI_X
  }
}

// ---------------------------------------------------------------------------
// Finalize: fixed-order sum of the block partials of one batch entry, then
// the scalar update of its iteration state.  One block per entry
// (ffth_finalize.h).
// ---------------------------------------------------------------------------
// Volume averages of sigma = P_rhs + C:x (or C:(E + x)): 6 sums per block.
template <bool ISO>
__global__ __launch_bounds__(NT) void k_mean_stress(const Desc* __restrict__ descs, long nvox);

// Order-1 pointwise right-hand side: P = C:sym(X1.G), g_i = sum_J c_J S^J_ij G_Jj.
template <bool ISO>
__global__ __launch_bounds__(NT) void k_order1_point(const Desc* __restrict__ descs, const double* __restrict__ eps0,
                                                     const double* __restrict__ x1, long nvox);

// out <- (double) x for FP32 x, n values.
__global__ void k_widen(const Desc* __restrict__ descs, long n);

// Largest phase id (validation of the problem input).
__global__ void k_phase_max(const uint16_t* __restrict__ phase, long n, int* out);

}  // namespace ffth
