// Fused angular stage of H*X for L <= 16 (gfx950): Legendre synthesis, phi
// synthesis, V_eff, phi analysis and Legendre quadrature of one radial node
// and 16 orbitals in one workgroup (eqs. G_lmr -> Ar_lm of Section 2.2.2 with
// V_eff between them).  Small bases are bound by launches and latency: three
// kernels of 3.4, 3.9 and 5.1 us become one of 9.1 (L = 9, 24 x 18 x 36, 11
// columns: H X 21.7 -> 16.1 us).  A group of at most 16 theta rows of g lives
// in LDS ([slot][row][16 columns]):
//   1. Legendre synthesis: g[s][row] = sum_l Pm[m][l][row] G[l, +-m], a wave
//      takes whole m (cos and sin share the table operand), m paired with L -
//      1 - m so that every wave has the same number of terms;
//   2. the phi operator, a wave per row.  With n' = 4 L points phi' = (p + 1/2)
//      2 pi / n' and V_eff resampled on them (exactly: only its Fourier sums up
//      to 2 (L - 1) couple the slots, and n' > 4 (L - 1) points integrate
//      them), the cosine and sine sums over even and odd m, ce co se so, of
//      the first quadrant give all four mirror points
//        f(phi) = ce + co + se + so        f(pi - phi) = ce - co - se + so
//        f(pi + phi) = ce - co + se - so   f(2 pi - phi) = ce + co - se - so
//      which are scaled by V_eff and folded back into the four analysis sums:
//      a quarter of the direct synthesis and analysis, on operand tables that
//      are the same for every row, where the Toeplitz + Hankel product of
//      larger L builds six tables per row.  The MFMA result registers of the
//      synthesis are the analysis's B operands as they stand (the k entries of
//      a step = the result rows of one register): nothing crosses lanes;
//   3. Legendre quadrature: A[l, +-m] += sum_rows w Pm[m][l][row] g[s][row],
//      kept in registers over all groups.
// Workgroups are n_r k / 16; for narrow blocks each takes half of the groups
// and the radial forward stage adds the two parts of A.
// Measured and not kept at 16 < L <= 32: this form (L = 25, k = 21, FP64: 45
// us against 44 for the three kernels; L = 31, k = 32, FP32: 55 against 52;
// 60 - 160 KB of LDS and up to 256 registers leave one or two workgroups per
// CU and a third of the chip idle), with the next operands prefetched (60 and
// 61 us: registers), and the quadrant phi operator as a kernel of its own on
// g (27 against 19.6 us; 28 against 23).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <type_traits>

#include "ces_internal.h"
#include "mfma.h"

namespace ces {
namespace {

constexpr int kFusedWaves = 8;

struct FusedDims {
  int L, LL, kp, n_theta, TH, ngrp, nsplit;
};

// T1 [class][t][lane], T2 [class][v][lane], PA [m][grp][t][lane], PC [m][grp]
// [t][lane]: MFMA A operands (fused_tables); V4 [row][image][16]; KC = ceil(L
// / 8) k-steps per class.
template <int KC>
constexpr int kQuadT1 = 4 * KC * 64;
constexpr int kQuadT2 = 16 * 64;

// The lane number, made opaque to the compiler: what is formed from it inside
// a loop (offsets, and table operands read from LDS) stays there instead of
// being kept in registers across the loop.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// A lane's operands of the phi operator: slots m = 2 (4 t + kk) [+ 1] of its
// column (slot stride ss; gr: the row, l16: the column); entries past a class
// read any slot and meet zeros of the table.
template <typename T, int KC>
__device__ __forceinline__ void quad_load(const T* gr, int ss, int L, int l16, int kk,
                                          T (&b)[4][KC]) {
#pragma unroll
  for (int t = 0; t < KC; ++t) {
    const int m = 2 * (4 * t + kk);
    b[0][t] = gr[unsigned(min(m, L - 1) * ss + l16)];
    b[1][t] = gr[unsigned(min(m + 1, L - 1) * ss + l16)];
    b[2][t] = gr[unsigned(min(L - 1 + m, 2 * L - 2) * ss + l16)];
    b[3][t] = gr[unsigned(min(L + m, 2 * L - 2) * ss + l16)];
  }
}
template <typename T>
__device__ __forceinline__ void quad_store(T* gr, int ss, int L, int ln,
                                           const typename MF<T>::acc (&h)[4]) {
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int m = 2 * MF<T>::row(ln, v);
    const unsigned o = unsigned(m * ss + (ln & 15));
    if (m < L) gr[o] = h[0][v];
    if (m + 1 < L) gr[o + ss] = h[1][v];
    if (m > 0 && m < L) gr[o + (L - 1) * ss] = h[2][v];
    if (m + 1 < L) gr[o + L * ss] = h[3][v];
  }
}
// h = the row's analysis sums, from its slots b and V_eff values v4
template <typename T, int KC>
__device__ __forceinline__ void quad_apply(const T (&b)[4][KC], const T* v4, const T* t1,
                                           const T* t2, int ln, typename MF<T>::acc (&h)[4]) {
  typedef typename MF<T>::acc acc_t;
  const int kk = ln >> 4;
  T y[4][4];      // V_eff at the four mirror points of this lane's result rows
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (sizeof(T) == 4) {
      load_vec<T, 4>(v4 + unsigned(i * 16 + 4 * kk), y[i]);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) y[i][v] = v4[unsigned(i * 16 + 4 * v + kk)];
    }
  }
  acc_t f[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) f[c] = h[c] = zero_acc<acc_t>();
#pragma unroll
  for (int t = 0; t < KC; ++t)
#pragma unroll
    for (int c = 0; c < 4; ++c) f[c] = MF<T>::mma(t1[(c * KC + t) * 64 + ln], b[c][t], f[c]);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const T ep = f[0][v] + f[1][v], em = f[0][v] - f[1][v];
    const T sp = f[2][v] + f[3][v], sm = f[2][v] - f[3][v];
    const T y0 = y[0][v] * (ep + sp), y1 = y[1][v] * (em - sm);
    const T y2 = y[2][v] * (em + sm), y3 = y[3][v] * (ep - sp);
    const T p03 = y0 + y3, m03 = y0 - y3, p12 = y1 + y2, m12 = y1 - y2;
    const T z[4] = {p03 + p12, p03 - p12, m03 - m12, m03 + m12};
#pragma unroll
    for (int c = 0; c < 4; ++c) h[c] = MF<T>::mma(t2[(c * 4 + v) * 64 + ln], z[c], h[c]);
  }
}

template <typename T, int KC>
__global__ __launch_bounds__(64 * kFusedWaves) void k_angular_fused(
    const T* __restrict__ G, T* __restrict__ A0, T* __restrict__ A1, const T* __restrict__ V4,
    const T* __restrict__ T12, const T* __restrict__ PA, const T* __restrict__ PC, FusedDims D) {
  typedef typename MF<T>::acc acc_t;
  constexpr int N1 = kQuadT1<KC>, N2 = kQuadT2;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* t1 = reinterpret_cast<T*>(smem_raw);
  T* t2 = t1 + N1;
  T* gs = t2 + N2;
  const int SS = 16 * D.TH + 8;                // slot stride: k groups of a read on other banks
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kk = lane >> 4;
  const int r = blockIdx.y, L = D.L;
  const int g0 = D.ngrp * blockIdx.z / D.nsplit, g1 = D.ngrp * (blockIdx.z + 1) / D.nsplit;
  copy_to_lds<64 * kFusedWaves>(T12, t1, N1 + N2);
  const T* Gr = G + static_cast<int64_t>(r) * D.LL * D.kp + blockIdx.x * 16 + l16;
  // this wave's pair of m: m1 < (L + 1) / 2 <= 8 and m2 = L - 1 - m1 (none
  // where they meet)
  const int m1 = wave, m2 = L - 1 - wave;
  const bool have1 = m1 <= m2, have2 = m1 < m2;
  acc_t a1[2], a2[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) a1[c] = a2[c] = zero_acc<acc_t>();
  // one m: KS steps of l = m + 4 t + kk (zero table entries past L)
  auto synth = [&](int m, int grp, auto ks_tag) __attribute__((always_inline)) {
    constexpr int KS = decltype(ks_tag)::value;
    const T* pa = PA + (static_cast<int64_t>(m) * D.ngrp + grp) * (2 * KC * 64) + lane;
    T a[KS], bc[KS], bs[KS];
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      const int l = min(m + 4 * t + kk, L - 1);
      a[t] = pa[t * 64];
      bc[t] = Gr[(l * l + l + m) * D.kp];
      bs[t] = Gr[(l * l + l - m) * D.kp];
    }
    acc_t c = zero_acc<acc_t>(), s = zero_acc<acc_t>();
#pragma unroll
    for (int t = 0; t < KS; ++t) {
      c = MF<T>::mma(a[t], bc[t], c);
      s = MF<T>::mma(a[t], bs[t], s);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = MF<T>::row(lane, v);
      if (row < D.TH) {
        gs[m * SS + row * 16 + l16] = c[v];
        if (m > 0) gs[(L - 1 + m) * SS + row * 16 + l16] = s[v];
      }
    }
  };
  // rows past TH hold nothing: they read the last one and meet zero weights
  auto analyse = [&](int m, int grp, acc_t (&a)[2]) __attribute__((always_inline)) {
    const T* pc = PC + (static_cast<int64_t>(m) * D.ngrp + grp) * (4 * 64) + lane;
    const T* gc = gs + m * SS + l16;
    const T* gsn = gs + (m > 0 ? L - 1 + m : 0) * SS + l16;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int row = min(4 * t + kk, D.TH - 1);
      const T w = pc[t * 64];
      a[0] = MF<T>::mma(w, gc[row * 16], a[0]);
      a[1] = MF<T>::mma(w, gsn[row * 16], a[1]);
    }
  };
  for (int grp = g0; grp < g1; ++grp) {
    if (have1) synth(m1, grp, std::integral_constant<int, 2 * KC>());
    if (have2) synth(m2, grp, std::integral_constant<int, KC>());
    __syncthreads();
    const int j0 = grp * D.TH, rows = min(D.TH, D.n_theta - j0);
    for (int row = wave; row < rows; row += kFusedWaves) {
      const int ln = opaque(lane);
      T* gr = gs + row * 16;
      T b[4][KC];
      quad_load<T, KC>(gr, SS, L, ln & 15, ln >> 4, b);
      acc_t h[4];
      quad_apply<T, KC>(b, V4 + (static_cast<int64_t>(r) * D.n_theta + j0 + row) * 64, t1, t2,
                           ln, h);
      quad_store<T>(gr, SS, L, ln, h);
    }
    __syncthreads();
    if (have1) analyse(m1, grp, a1);
    if (have2) analyse(m2, grp, a2);
    if (grp + 1 < g1) __syncthreads();
  }
  T* Ar = (blockIdx.z == 0 ? A0 : A1) + static_cast<int64_t>(r) * D.LL * D.kp + blockIdx.x * 16 +
          l16;
  auto put = [&](int m, const acc_t (&a)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int l = m + MF<T>::row(lane, v);
      if (l < L) {
        Ar[(l * l + l + m) * D.kp] = a[0][v];
        if (m > 0) Ar[(l * l + l - m) * D.kp] = a[1][v];
      }
    }
  };
  if (have1) put(m1, a1);
  if (have2) put(m2, a2);
}

// V_eff in the two forms the angular stage takes for L <= 16, each linear in a
// row's n_phi values, so one launch of a fixed n_phi x 128 matrix W per basis:
//   columns 0 .. 63   V4[row][image][p] = (2 pi / n') V_eff(phi'), by
//                     trigonometric interpolation up to degree 2 (L - 1)
//   column 64 + q     the phi stage's halved Fourier sums (q < S cosine, then
//                     sine; kernels.hip), scaled by `scale`
// A wave owns two rows, a lane one of 64 columns.  Replacing the potential is
// bound by launches: 10.4 us on a 24 x 18 x 36 grid, as with the sums alone (10.5;
// 13.8 with a launch for each form).
constexpr int kVeffCols = 128;
__global__ __launch_bounds__(256) void k_veff_forms(const double* __restrict__ V,
                                                    const double* __restrict__ W, int n_phi,
                                                    int S2, double scale, double* __restrict__ v64,
                                                    float* __restrict__ v32,
                                                    double* __restrict__ ab64,
                                                    float* __restrict__ ab32, int64_t n_rows) {
  const int q = blockIdx.y * 64 + (threadIdx.x & 63);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * 8 + 2 * wave;
  if (r0 >= n_rows || q >= 64 + S2) return;
  const double* va = V + r0 * n_phi;
  const double* vb = V + min(r0 + 1, n_rows - 1) * n_phi;
  const double* w = W + q;
  double a = 0.0, b = 0.0;
#pragma unroll 16
  for (int p = 0; p < n_phi; ++p) {
    const double t = w[p * kVeffCols];
    a = fma(va[p], t, a);
    b = fma(vb[p], t, b);
  }
  auto put = [&](int64_t row, double x) __attribute__((always_inline)) {
    if (q < 64) {
      v64[row * 64 + q] = x;
      v32[row * 64 + q] = static_cast<float>(x);
    } else {
      ab64[row * S2 + q - 64] = scale * x;
      ab32[row * S2 + q - 64] = static_cast<float>(scale * x);
    }
  };
  put(r0, a);
  if (r0 + 1 < n_rows) put(r0 + 1, b);
}

}  // namespace

FusedShape fused_shape(const Basis& b) {
  FusedShape f;
  f.kc = (b.L + 7) / 8;
  // as few groups as 16 rows allow, of equal size (18 rows as three groups of
  // 6, one round of the eight waves each, instead of two of 9: 16.1 -> 19.3 us)
  f.ngrp = (b.n_theta + 15) / 16;
  f.th = (b.n_theta + f.ngrp - 1) / f.ngrp;
  f.ngrp = (b.n_theta + f.th - 1) / f.th;
  return f;
}

// Operand tables in FP64 (layouts above); the row of D that a lane's register
// v holds differs between FP64 and FP32, so T2 does too (f32).
void fused_tables(const Basis& b, bool f32, std::vector<double>& t12, std::vector<double>& pa,
                  std::vector<double>& pc) {
  const FusedShape f = fused_shape(b);
  const int L = b.L, LP = L * (L + 1) / 2, n4 = 4 * L;
  // cos / sin(m (p + 1/2) 2 pi / n') = trig(m (2 p + 1) 2 pi / (2 n')), rounded
  // once (from long double: an argument of pi times a fraction rounded to FP64
  // is off by up to 4e-16 before the cosine)
  std::vector<double> cs[2];
  for (int u = 0; u < 2 * n4; ++u) {
    const long double x = acosl(-1.0L) * u / n4;
    cs[0].push_back(static_cast<double>(cosl(x)));
    cs[1].push_back(static_cast<double>(sinl(x)));
  }
  auto trig = [&](int sn, int m, int p2) { return cs[sn][m * p2 % (2 * n4)]; };
  auto entry = [&](int cls, int kap, int p) -> double {   // classes ce co se so
    const int m = 2 * kap + (cls & 1);
    if (m >= L || p >= L || (cls >= 2 && m == 0)) return 0.0;
    return trig(cls >= 2, m, 2 * p + 1);
  };
  // L <= 8: the analysis side of an FP32 product makes up for the rounding of
  // the synthesis side, c^2 / fl(c) instead of c: their few distinct values
  // otherwise scale whole slots alike, by up to 5.7e-8 (3.3e-8 so).  Error of
  // the mixed H X of the oscillator, N = 12, against 64 bits in units of the
  // three kernels' (relative 2-norm), c | c^2 / fl(c): L = 4 1.10 | 1.03, L = 8 1.06 |
  // 1.035; with wells 1.00 either way, from L = 9 0.98 to 1.00 with c.
  auto back = [&](double c) {
    return f32 && L <= 8 && c != 0.0 ? c * c / static_cast<double>(static_cast<float>(c)) : c;
  };
  const int n1 = 4 * f.kc * 64;
  t12.assign(n1 + kQuadT2, 0.0);
  pa.assign(size_t(L) * f.ngrp * 2 * f.kc * 64, 0.0);
  pc.assign(size_t(L) * f.ngrp * 4 * 64, 0.0);
  auto leg = [&](int m, int l, int j) {
    return b.legendre[size_t(j) * LP + l * (l + 1) / 2 + m] * (m > 0 ? std::sqrt(2.0) : 1.0);
  };
  for (int lane = 0; lane < 64; ++lane) {
    const int l16 = lane & 15, kk = lane >> 4;
    for (int c = 0; c < 4; ++c) {
      for (int t = 0; t < f.kc; ++t)
        t12[(c * f.kc + t) * 64 + lane] = entry(c, 4 * t + kk, l16);
      for (int v = 0; v < 4; ++v)
        t12[n1 + (c * 4 + v) * 64 + lane] = back(entry(c, l16, f32 ? 4 * kk + v : 4 * v + kk));
    }
    for (int m = 0; m < L; ++m)
      for (int g = 0; g < f.ngrp; ++g) {
        const size_t at = size_t(m) * f.ngrp + g;
        for (int t = 0; t < 2 * f.kc; ++t) {
          const int l = m + 4 * t + kk, j = g * f.th + l16;
          if (l < L && l16 < f.th && j < b.n_theta)
            pa[(at * 2 * f.kc + t) * 64 + lane] = leg(m, l, j);
        }
        for (int t = 0; t < 4; ++t) {
          const int l = m + l16, row = 4 * t + kk, j = g * f.th + row;
          if (l < L && row < f.th && j < b.n_theta)
            pc[(at * 4 + t) * 64 + lane] = b.wt[j] * leg(m, l, j);
        }
      }
  }
}

// W of k_veff_forms.  Columns 0 .. 63: V4 = (2 pi / n') (1 / n_phi) sum_p V_p
// [1 + 2 sum_{q <= 2L-2} cos q (phi' - phi_p)], the sum in closed form, sin((2L -
// 3/2) x) / sin(x / 2).  The differences are integer multiples x of pi / (n'
// n_phi), all of them multiples of gcd(n_phi, 2 n'), and each is evaluated once,
// in long double (first Hamiltonian of a basis, L = 16, n_phi = 64: 2.7 ms with
// every entry evaluated, for either precision, 0.8 so).
void veff_matrix(const Basis& b, std::vector<double>& dir) {
  const int L = b.L, n4 = 4 * L;
  const long double pi = acosl(-1.0L);
  dir.assign(size_t(b.n_phi) * kVeffCols, 0.0);
  const int64_t M = int64_t(n4) * b.n_phi, g = std::gcd(b.n_phi, 2 * n4);
  std::vector<double> known(size_t(2 * M / g), NAN);
  auto weight = [&](int64_t x) {      // 0 <= x < 2 M
    double& w = known[x / g];
    if (std::isnan(w)) {
      const int64_t c = 4 * L - 3;
      const long double num = sinl(pi * (long double)(c * x % (4 * M)) / (2 * M));
      const long double sum = x == 0 ? (long double)c : num / sinl(pi * (long double)x / (2 * M));
      w = static_cast<double>(2 * pi / n4 / b.n_phi * sum);
    }
    return w;
  };
  for (int img = 0; img < 4; ++img)
    for (int p = 0; p < L; ++p) {
      const int64_t up = (2 * p + 1) * int64_t(b.n_phi);
      const int64_t ph = img == 0 ? up : img == 1 ? M - up : img == 2 ? M + up : 2 * M - up;
      for (int q = 0; q < b.n_phi; ++q)
        dir[size_t(q) * kVeffCols + img * 16 + p] =
            weight(((ph - 2 * int64_t(n4) * q) % (2 * M) + 2 * M) % (2 * M));
    }
  const int S = 2 * L - 1;
  std::vector<double> cs[2];
  for (int u = 0; u < b.n_phi; ++u) {
    cs[0].push_back(std::cos(2.0 * M_PI * u / b.n_phi));
    cs[1].push_back(std::sin(2.0 * M_PI * u / b.n_phi));
  }
  for (int p = 0; p < b.n_phi; ++p)
    for (int q = 0; q < S; ++q) {
      const int u = static_cast<int>(int64_t(q) * p % b.n_phi);
      dir[size_t(p) * kVeffCols + 64 + q] = cs[0][u];
      dir[size_t(p) * kVeffCols + 64 + S + q] = cs[1][u];
    }
}

void launch_veff_forms(const Basis& b, const double* V, double* v64, float* v32, double* ab64,
                       float* ab32, hipStream_t s) {
  const int64_t rows = int64_t(b.n_r) * b.n_theta;
  k_veff_forms<<<dim3(static_cast<unsigned>((rows + 7) / 8), 2), 256, 0, s>>>(
      V, b.dev_dir, b.n_phi, 2 * (2 * b.L - 1), M_PI / b.n_phi, v64, v32, ab64, ab32, rows);
}

// Whether an H*X of kp columns takes the fused kernel (L <= kFusedL).  It
// saves two launches and g's three further crossings of memory, and pays with
// workgroups that run at their slowest wave: per 16 theta rows or fewer, eight
// waves take ceil(L / 2) pairs of m and the rows in rounds of eight, so few
// L and row counts fill them (L = 9: 5 of 8 waves, then 9 rows in two rounds).
// Narrow blocks (work = workgroups times rounds) are bound by launches: fused.
// Wide ones are fused where the waves are full enough, L = 6 .. 8 and from 11
// (FP64) or 12 (FP32), in FP32 from L = 5 to 8 always, and on grids with many
// more theta nodes than L needs where g no longer fits the last-level cache;
// with L <= 4 a workgroup's fixed steps soon outweigh it.  H X in us, three
// kernels | fused, FP64 and FP32: L = 9, 24 x 18 grid, k = 48 23.2 | 17.9, 24.3 |
// 19.1, k = 512 67 | 63, 51 | 48, k = 1500 143 | 157, 99 | 119; 45 x 18, k = 373 79 | 91,
// 60 | 72; L = 16, 36 x 32, k = 800 328 | 227, 180 | 166; L = 1, 90 x 2, k = 100 / 500, FP64
// 22.9 | 22.6 / 29 | 50, FP32 k = 500 26 | 31; L = 4, 90 x 8, k = 500 69 | 80.  For L >= 4, over
// 570 sizes a precision the rule costs 0.4 % (FP64) and 0.2 % (FP32) more than the
// faster form of each; always fused: 1.6 and 2.3 %, at worst 51 and 36 %.
bool fused_route(const Basis& b, int kp, size_t elem) {
  const FusedShape f = fused_shape(b);
  const bool f32 = elem == 4;
  const int64_t wgs = int64_t(b.n_r) * (kp / 16);
  const int64_t work = wgs * f.ngrp * ((f.th + kFusedWaves - 1) / kFusedWaves);
  const bool usual = 2 * b.n_theta <= 5 * b.L;      // theta nodes as L needs them
  const int narrow = f32 || b.L <= 8 ? 3072 : 2048;
  if (b.L <= 4) return work <= (512 + 64 * b.L * b.L) * (f32 ? 4 : 1);
  if (b.L <= 8) return f32 || work <= narrow || (usual && b.L >= 6);
  if (!usual) {
    const size_t g = size_t(b.n_r) * b.n_theta * (2 * b.L - 1) * kp * elem;
    return wgs <= 256 || (b.L >= 12 && g > size_t(180) * 1000 * 1000);
  }
  return work <= narrow || b.L >= (f32 ? 12 : 11);
}

// Parts of A the fused launch writes: two (each half of the theta groups)
// when the workgroups of one part fill at most half of the chip, `room`
// (elements available for the second part) holds it, and the radial forward
// stage loads its whole contraction at once (its streamed form takes one
// part).
int fused_parts(const Basis& b, int kp, size_t room) {
  const FusedShape f = fused_shape(b);
  const int64_t wgs = int64_t(b.n_r) * (kp / 16);
  const bool fits = size_t(b.n_r) * b.L * b.L * kp <= room;
  return f.ngrp > 1 && fits && b.n_r <= kOneChunkNodes && 2 * wgs <= 256 ? 2 : 1;
}

template <typename T>
void launch_angular_fused(const Basis& b, const FusedTables<T>& tb, const T* V4, const T* G, T* A0,
                          T* A1, int parts, int kp, hipStream_t s) {
  const FusedShape f = fused_shape(b);
  FusedDims D = {b.L, b.L * b.L, kp, b.n_theta, f.th, f.ngrp, parts};
  const dim3 grid(kp / 16, b.n_r, parts);
  auto go = [&](auto kc_tag) {
    constexpr int KC = decltype(kc_tag)::value;      // at most 80 KB: 31 slots, 16 rows, FP64
    const size_t lds =
        (kQuadT1<KC> + kQuadT2 + size_t(2 * b.L - 1) * (16 * f.th + 8)) * sizeof(T);
    if (lds > 65536)
      (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_angular_fused<T, KC>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
    k_angular_fused<T, KC><<<grid, 64 * kFusedWaves, lds, s>>>(G, A0, A1, V4, tb.T12, tb.PA, tb.PC,
                                                               D);
  };
  if (f.kc == 1)
    go(std::integral_constant<int, 1>());
  else
    go(std::integral_constant<int, 2>());
}

#define CES_INST(T)                                                                             \
  template void launch_angular_fused<T>(const Basis&, const FusedTables<T>&, const T*, const T*, \
                                        T*, T*, int, int, hipStream_t);
CES_INST(float)
CES_INST(double)
#undef CES_INST

}  // namespace ces
