// Phi transforms of grid functions, and the density, on MFMA (gfx950).
//
// The H*X product never forms orbitals on the grid; these kernels do, for the
// transforms between grid functions and coefficients (Section 2.2.2), the
// Kohn-Sham potential and the density (Section 2.2.5):
//   analysis   gh[row][s][i] = (2 pi / n) sum_p f_i[row][p] trig_s(phi_p)
//   synthesis  f_i[row][p]   = sum_s g[row][s][i] trig_s(phi_p)
//   density    rho[row][p]   = 2 sum_i occ_i psi_i[row][p]^2
// with n = n_phi, row = (r, theta_j) and trig_s = cos(m phi) (slot s = m < L)
// or sin(m phi) (slot L - 1 + m).  Since cos(m (2 pi - phi)) = cos(m phi) and
// sin(m (2 pi - phi)) = -sin(m phi), each contraction runs over the points
// p <= n / 2 alone: the analysis contracts f(p) + f(n - p) with the cosines
// and f(p) - f(n - p) with the sines, the synthesis forms the cosine sum C
// and the sine sum S and writes C + S at p and C - S at n - p.
//
// One wave takes one row and 16 columns i and holds every M tile (or every
// coefficient) of its contraction in registers, so the grid values cross the
// memory once, without LDS or barriers: an MFMA operand lane (column l16, k
// group kk) reads the points or slots it owns straight from global memory.
// The trig operands come from tables laid out in operand order (512 bytes per
// operand, L1 / L2 resident).  52 functions on the 90 x 62 x 124 grid (L = 31):
// analysis 912 -> 180 us, synthesis 653 -> 145 us against kernels that walked
// each sum in one thread with two LDS reads per term; the grid values and
// slots (463 MB) cross at 2.6 and 3.2 TB/s.  One function on 60 x 50 x 100 (L
// = 25): 20 -> 5.4 us and 9.8 -> 6.4 us (the latter now with the potential's
// pointwise terms), latency bound.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>
#include <utility>

#include "ces_internal.h"
#include "mfma.h"
#include "xc.h"

namespace ces {
namespace {

// Four consecutive doubles from an address aligned to 8 bytes only (a column
// of a grid block may start anywhere).
struct __attribute__((packed, aligned(8))) Quad {
  double v[4];
};
__device__ __forceinline__ void load_quad(const double* p, double (&x)[4]) {
  const Quad q = *reinterpret_cast<const Quad*>(p);
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = q.v[e];
}

// Analysis.  K runs over the pairs q (points 1 + q and n - 1 - q, q < n / 2;
// the last one is its own mirror when n is even and has half weight in the
// table), 16 pairs per step: lane group kk owns pairs 16 t + 4 kk + e, so a
// lane reads 32 consecutive bytes on either side.  Point 0 is one more MFMA.
// ta: [t][e][cos | sin][m tile][lane].  With DIFF the function is f - f2.
// SPLIT: the four waves of a workgroup share one (row, columns) task and take
// every fourth step each, their sums added through LDS in a fixed order.
template <int LT, bool DIFF, bool SPLIT>
__global__ __launch_bounds__(256) void k_phi_analysis(const double* __restrict__ f,
                                                      const double* __restrict__ f2, int64_t ldf,
                                                      int k, int kp, double* __restrict__ gh,
                                                      const double* __restrict__ ta, int L, int n,
                                                      double w, int64_t n_rows) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kk = lane >> 4;
  const int ncg = kp / 16;
  const int64_t task = SPLIT ? int64_t(blockIdx.x) : static_cast<int64_t>(blockIdx.x) * 4 + wave;
  const int64_t row = task / ncg;
  if (row >= n_rows) return;     // SPLIT: uniform over the workgroup
  const int i = static_cast<int>(task - row * ncg) * 16 + l16;
  const bool ok = i < k;
  const int64_t at = static_cast<int64_t>(min(i, k - 1)) * ldf + row * n;
  const double* fr = f + at;
  const double* fr2 = DIFF ? f2 + at : nullptr;
  const int npair = n / 2, nfull = npair / 16, nt = (npair + 15) / 16;
  const int t0 = SPLIT ? wave : 0;
  constexpr int ST = SPLIT ? 4 : 1;
  // step t's points; pairs past the last read the last (zero table entries)
  auto points = [&](int t, double (&x)[4], double (&y)[4]) __attribute__((always_inline)) {
    const int q = 16 * t + 4 * kk;
    if (t < nfull) {
      double yr[4];
      load_quad(fr + 1 + q, x);
      load_quad(fr + (n - 4 - q), yr);       // points n - 4 - q .. n - 1 - q
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = yr[3 - e];
      if constexpr (DIFF) {
        double x2[4];
        load_quad(fr2 + 1 + q, x2);
        load_quad(fr2 + (n - 4 - q), yr);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[e] -= x2[e];
          y[e] -= yr[3 - e];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int p = 1 + min(q + e, npair - 1);
        x[e] = fr[p];
        y[e] = fr[n - p];
        if constexpr (DIFF) {
          x[e] -= fr2[p];
          y[e] -= fr2[n - p];
        }
      }
    }
  };
  d4 ac[LT], as[LT];
  {
    double x0 = fr[0];
    if constexpr (DIFF) x0 -= fr2[0];
    const double b = ok && kk == 0 && t0 == 0 ? x0 : 0.0;
#pragma unroll
    for (int u = 0; u < LT; ++u) {
      const double a = kk == 0 && 16 * u + l16 < L ? w : 0.0;
      ac[u] = MF<double>::mma(a, b, zero_acc<d4>());
      as[u] = zero_acc<d4>();
    }
  }
  for (int t = t0; t < nt; t += ST) {
    double x[4], y[4];
    points(t, x, y);
    const double* tt = ta + static_cast<int64_t>(t) * (4 * 2 * LT * 64) + lane;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double xe = ok ? x[e] : 0.0, ye = ok ? y[e] : 0.0;
      const double u = xe + ye, v = xe - ye;
#pragma unroll
      for (int m = 0; m < LT; ++m) {
        ac[m] = MF<double>::mma(tt[((e * 2) * LT + m) * 64], u, ac[m]);
        as[m] = MF<double>::mma(tt[((e * 2 + 1) * LT + m) * 64], v, as[m]);
      }
    }
  }
  if constexpr (SPLIT) {
    // (0 + 2) + (1 + 3), two waves' sums at a time
    __shared__ double part[2][2 * LT * 4][64];
#pragma unroll
    for (int j = 2; j > 0; j >>= 1) {
      if (wave >= j && wave < 2 * j)
#pragma unroll
        for (int u = 0; u < LT; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            part[wave - j][8 * u + v][lane] = ac[u][v];
            part[wave - j][8 * u + 4 + v][lane] = as[u][v];
          }
      __syncthreads();
      if (wave < j)
#pragma unroll
        for (int u = 0; u < LT; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            ac[u][v] += part[wave][8 * u + v][lane];
            as[u][v] += part[wave][8 * u + 4 + v][lane];
          }
      __syncthreads();
    }
    if (wave > 0) return;
  }
  double* o = gh + row * (2 * L - 1) * kp + i;
#pragma unroll
  for (int u = 0; u < LT; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int m = 16 * u + MF<double>::row(lane, v);
      if (m < L) o[static_cast<int64_t>(m) * kp] = ac[u][v];
      if (m < L - 1) o[static_cast<int64_t>(L + m) * kp] = as[u][v];
    }
}

// This lane's coefficients of a row (columns i, slots 4 t + kk of the cosine
// and of the sine half), as MFMA operands; entries past a half repeat its
// last slot and meet zeros of the table.
template <typename T, int KT>
__device__ __forceinline__ void load_slots(const T* gr, int kp, int L, int kk, T (&c)[KT],
                                           T (&s)[KT]) {
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    c[t] = gr[static_cast<int64_t>(min(4 * t + kk, L - 1)) * kp];
    s[t] = gr[static_cast<int64_t>(min(L + 4 * t + kk, 2 * L - 2)) * kp];
  }
}

// Synthesis: the trig table is the B operand, so a result lane holds 4
// columns at 16 consecutive points and each store covers whole 128-byte runs
// of f.  tb: [p tile][t < KT][cos | sin][lane], KT = trig_kt(L) k-steps at
// compile time (a guard on each step would make its table load wait: density
// of the L = 25 basis 37 us guarded).  With KS the value written is the
// Kohn-Sham potential vext + f + V_x(rho) [+ v_c(rho)].
template <int KT, bool KS>
__global__ __launch_bounds__(256) void k_phi_synthesis(const double* __restrict__ g, int k,
                                                       int kp, double* __restrict__ f, int64_t ldf,
                                                       const double* __restrict__ tb, int L, int n,
                                                       int64_t n_rows, int ppw, int nsp,
                                                       const double* __restrict__ vext,
                                                       const double* __restrict__ rho, int corr) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kk = lane >> 4;
  const int ncg = kp / 16;
  const int64_t task = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  const int64_t rc = task / nsp;              // (row, column tile); then its span of p tiles
  const int p0 = static_cast<int>(task - rc * nsp) * ppw;
  const int64_t row = rc / ncg;
  if (row >= n_rows) return;
  const int i0 = static_cast<int>(rc - row * ncg) * 16;
  double c[KT], s[KT];
  load_slots<double, KT>(g + row * (2 * L - 1) * kp + i0 + l16, kp, L, kk, c, s);
  const int half = n / 2, npt = min(half / 16 + 1, p0 + ppw);
  for (int pt = p0; pt < npt; ++pt) {
    const double* tt = tb + pt * (KT * 2 * 64) + lane;
    d4 C = zero_acc<d4>(), S = zero_acc<d4>();
#pragma unroll
    for (int t = 0; t < KT; ++t) {
      C = MF<double>::mma(c[t], tt[(2 * t) * 64], C);
      S = MF<double>::mma(s[t], tt[(2 * t + 1) * 64], S);
    }
    const int p = 16 * pt + l16;
    const bool pok = p <= half, mok = pok && p > 0 && 2 * p != n;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int i = i0 + MF<double>::row(lane, v);
      if (i >= k) continue;
      const int64_t at = static_cast<int64_t>(i) * ldf + row * n;
      auto put = [&](int64_t e, double x) __attribute__((always_inline)) {
        if constexpr (KS) {
          const double r = rho[e];
          x = vext[e] + x + slater_vx(r);
          if (corr) {
            double eps, vc;
            pz81(r, eps, vc);
            x += vc;
          }
        }
        f[e] = x;
      };
      if (pok) put(at + p, C[v] + S[v]);
      if (mok) put(at + n - p, C[v] - S[v]);
    }
  }
}

// Density: the synthesis with each psi tile squared, weighted and summed over
// the columns in FP64.  A result lane holds 4 columns of one point pair, so
// the column sum is 4 terms in the lane and two cross-lane adds.  A wave takes
// whole rows, one column tile at a time with the next tile's coefficients in
// flight, and adds the tiles into its own LDS row of rho; with TL the trig
// table is copied to LDS once per workgroup, which walks many rows (from
// global memory each point tile waits for its operands).
template <typename T, int KT, bool TL>
__global__ __launch_bounds__(256) void k_density(const T* __restrict__ g,
                                                 const double* __restrict__ occ,
                                                 double* __restrict__ rho,
                                                 const T* __restrict__ tb, int k, int kp, int L,
                                                 int n, int64_t n_rows) {
  typedef typename MF<T>::acc acc_t;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kk = lane >> 4;
  double* racc = reinterpret_cast<double*>(smem_raw) + wave * n;   // [4][n]
  const int half = n / 2, npt = half / 16 + 1;
  const int64_t rstride = static_cast<int64_t>(2 * L - 1) * kp;
  int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + wave;
  const int64_t step = static_cast<int64_t>(gridDim.x) * 4;
  T c[KT], s[KT];
  if (row < n_rows) load_slots<T, KT>(g + row * rstride + l16, kp, L, kk, c, s);
  const T* tab = tb;
  if constexpr (TL) {
    T* tl = reinterpret_cast<T*>(reinterpret_cast<double*>(smem_raw) + 4 * n);   // 32-byte aligned
    copy_to_lds<256>(tb, tl, npt * KT * 2 * 64);
    __syncthreads();   // the only barrier
    tab = tl;
  }
  tab += lane;
  for (; row < n_rows; row += step) {
    for (int i0 = 0; i0 < kp; i0 += 16) {
      T nc[KT], ns[KT];
      const bool more = i0 + 16 < kp;
      const int64_t nrow = more ? row : row + step;
      if (nrow < n_rows)
        load_slots<T, KT>(g + nrow * rstride + (more ? i0 + 16 : 0) + l16, kp, L, kk, nc, ns);
      double wc[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = i0 + MF<T>::row(lane, v);
        wc[v] = i < k ? 2.0 * occ[min(i, k - 1)] : 0.0;
      }
      for (int pt = 0; pt < npt; ++pt) {
        const T* tt = tab + pt * (KT * 2 * 64);
        acc_t C = zero_acc<acc_t>(), S = zero_acc<acc_t>();
#pragma unroll
        for (int t = 0; t < KT; ++t) {
          C = MF<T>::mma(c[t], tt[(2 * t) * 64], C);
          S = MF<T>::mma(s[t], tt[(2 * t + 1) * 64], S);
        }
        double sp = 0.0, sm = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double x = static_cast<double>(C[v]), y = static_cast<double>(S[v]);
          const double a = x + y, b = x - y;
          sp = fma(wc[v] * a, a, sp);
          sm = fma(wc[v] * b, b, sm);
        }
#pragma unroll
        for (int off = 16; off < 64; off <<= 1) {
          sp += __shfl_xor(sp, off, 64);
          sm += __shfl_xor(sm, off, 64);
        }
        const int p = 16 * pt + l16;
        const bool pok = p <= half, mok = pok && p > 0 && 2 * p != n;
        if (kk == 0 && pok) racc[p] = i0 == 0 ? sp : racc[p] + sp;
        if (kk == 1 && mok) racc[n - p] = i0 == 0 ? sm : racc[n - p] + sm;
      }
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        c[t] = nc[t];
        s[t] = ns[t];
      }
    }
    for (int e = lane; e < n; e += 64) rho[row * n + e] = racc[e];
  }
}

// Density, a row per workgroup: where registers or the number of rows leave
// the kernel above too few waves (rule at launch_density_phi).  The points are
// the rows of D (M tiles dealt to the four waves), the slots go through LDS 32
// columns at a time with the next block in flight, the angle table cos | sin(2
// pi u / n) lies in LDS and is walked by (m p) mod n; each wave adds its
// tiles' column sums to an LDS row of rho.
constexpr int kDensityWorkgroups = 1024;
constexpr int kDensityNT = 2;
template <typename T, int LP>
__global__ __launch_bounds__(256) void k_density_rows(const T* __restrict__ g,
                                                      const double* __restrict__ occ,
                                                      double* __restrict__ rho,
                                                      const double* __restrict__ cs, int L, int kp,
                                                      int n_phi, int k, int64_t n_rows) {
  typedef typename MF<T>::acc acc_t;
  constexpr int GW = 16 * kDensityNT + 1;
  constexpr int K2 = 2 * LP, KPH = LP / 4;
  constexpr int GPT = K2 / 8;                   // g values per thread per tile
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int S = 2 * L - 1;
  double* racc = reinterpret_cast<double*>(smem_raw);            // [n_phi]
  T* ct = reinterpret_cast<T*>(racc + n_phi);                    // [2][n_phi] cos | sin
  T* gs = ct + 2 * n_phi;                                        // [K2][GW]
  const int tid = threadIdx.x;
  const int ii = tid & 31, kr = tid >> 5;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kk = lane >> 4;
  const int ncb = (kp + 16 * kDensityNT - 1) / (16 * kDensityNT);
  const int phalf = n_phi / 2;                  // points 0..phalf are formed
  const int nMT = (phalf + 1 + 15) / 16;
  for (int e = tid; e < 2 * n_phi; e += 256) ct[e] = static_cast<T>(cs[e]);
  // this thread's g rows (slot s < L -> K row s; slot L + j -> row LP + j)
  int sof[GPT];
  bool sok[GPT];
#pragma unroll
  for (int u = 0; u < GPT; ++u) {
    const int kx = kr + 8 * u;
    const bool sn = kx >= LP;
    const int kl = sn ? kx - LP : kx;
    sok[u] = sn ? kl < L - 1 : kl < L;
    sof[u] = sok[u] ? (sn ? L + kl : kl) * kp : 0;
  }
  const int64_t rstride = static_cast<int64_t>(S) * kp;
  const int64_t ntask = n_rows * ncb;
  T gp[GPT];
  auto fetch = [&](int64_t task) {
    const int64_t row = task / ncb;
    const int cb = static_cast<int>(task - row * ncb);
    const int col = min(cb * 16 * kDensityNT + ii, kp - 1);
    const T* gr = g + row * rstride + col;
#pragma unroll
    for (int u = 0; u < GPT; ++u) gp[u] = gr[sof[u]];
  };
  int64_t task = static_cast<int64_t>(blockIdx.x) * ncb;   // first column block of a row
  if (task < ntask) fetch(task);
  for (int64_t row = blockIdx.x; row < n_rows; row += gridDim.x) {
    for (int e = tid; e < n_phi; e += 256) racc[e] = 0.0;
    for (int cb = 0; cb < ncb; ++cb) {
      const int i0 = cb * 16 * kDensityNT;
      const bool ok_col = i0 + ii < kp;
#pragma unroll
      for (int u = 0; u < GPT; ++u) gs[(kr + 8 * u) * GW + ii] = sok[u] && ok_col ? gp[u] : T(0);
      __syncthreads();   // gs (and, at cb = 0, the zeroed racc and the tables) visible
      const int64_t next = cb + 1 < ncb ? row * ncb + cb + 1 : (row + gridDim.x) * ncb;
      if (next < ntask) fetch(next);                  // next tile, in flight
      // column weights 2 occ_i of this lane's columns (0 past k)
      double wcol[kDensityNT];
#pragma unroll
      for (int nt = 0; nt < kDensityNT; ++nt) {
        const int i = i0 + nt * 16 + l16;
        wcol[nt] = i < k ? 2.0 * occ[i] : 0.0;
      }
      for (int mt = wave; mt < nMT; mt += 4) {
        const int p = mt * 16 + l16;
        const int pc = p <= phalf ? p : 0;            // padded rows: any finite value
        const int d4 = (4 * pc) % n_phi;
        acc_t acc[2][kDensityNT];                          // [cos part, sin part]
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
          for (int nt = 0; nt < kDensityNT; ++nt) acc[half][nt] = zero_acc<acc_t>();
#pragma unroll
        for (int half = 0; half < 2; ++half) {
          // m = 4t + kk (cos half) or 4t + kk + 1 (sin half): u = (m p) mod n_phi
          int u = ((kk + half) * pc) % n_phi;
          const T* tb = ct + half * n_phi;
          const T* grow = gs + (half * LP + kk) * GW + l16;
#pragma unroll
          for (int t = 0; t < KPH; ++t) {
            const T a = tb[u];
#pragma unroll
            for (int nt = 0; nt < kDensityNT; ++nt)
              acc[half][nt] = MF<T>::mma(a, grow[4 * t * GW + nt * 16], acc[half][nt]);
            u += d4;
            u -= u >= n_phi ? n_phi : 0;
          }
        }
        // psi(p) = C + S and psi(n - p) = C - S: weighted squares summed over
        // this lane's columns, then over the 16 lanes of a row
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          double sp = 0.0, sm = 0.0;
#pragma unroll
          for (int nt = 0; nt < kDensityNT; ++nt) {
            const double c = static_cast<double>(acc[0][nt][v]);
            const double sn = static_cast<double>(acc[1][nt][v]);
            const double xp = c + sn, xm = c - sn;
            sp = fma(wcol[nt] * xp, xp, sp);
            sm = fma(wcol[nt] * xm, xm, sm);
          }
#pragma unroll
          for (int off = 1; off < 16; off <<= 1) {
            sp += __shfl_xor(sp, off, 64);
            sm += __shfl_xor(sm, off, 64);
          }
          const int pr = mt * 16 + MF<T>::row(lane, v);
          if (l16 == 0 && pr <= phalf) {
            racc[pr] += sp;
            if (pr > 0 && 2 * pr != n_phi) racc[n_phi - pr] += sm;
          }
        }
      }
      __syncthreads();   // gs is refilled next; racc complete after the last block
    }
    double* out = rho + row * n_phi;
    for (int e = tid; e < n_phi; e += 256) out[e] = racc[e];
    __syncthreads();   // racc is zeroed for the next row
  }
}

// ------------------------------------------- radial sums of one function

// One function's radial stages, columns = radial nodes.  A workgroup takes 64
// outputs (nodes r, or functions n) and MB values of m of one l; its four
// waves split the sum (each table entry is read once and used for all MB
// values, the other operand is wave-uniform) and add their parts through LDS
// in a fixed order.  The sums are short (40-225 terms): one batch of loads a
// wave, so the launch is bound by latency.
constexpr int kOneMB = 4;
template <typename F>
__device__ __forceinline__ void one_sum(int K, F&& step, double (&acc)[kOneMB]) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int per = (K + 3) / 4, k0 = wave * per, k1 = min(k0 + per, K);
#pragma unroll
  for (int u = 0; u < kOneMB; ++u) acc[u] = 0.0;
#pragma unroll 16
  for (int q = k0; q < k1; ++q) step(q, acc);
  __shared__ double part[3][kOneMB][64];
  const int lane = threadIdx.x & 63;
  if (wave > 0)
#pragma unroll
    for (int u = 0; u < kOneMB; ++u) part[wave - 1][u][lane] = acc[u];
  __syncthreads();
  if (wave == 0)
#pragma unroll
    for (int u = 0; u < kOneMB; ++u)
      acc[u] = ((acc[u] + part[0][u][lane]) + part[1][u][lane]) + part[2][u][lane];
}

// G[lm][r] (row pitch kp) = sum_n Ri[l][n][r] x[alpha(lm, n)]
__global__ __launch_bounds__(256) void k_radial_inverse_one(const double* __restrict__ RiT,
                                                            const double* __restrict__ x,
                                                            double* __restrict__ G,
                                                            const int* __restrict__ lay, int N4,
                                                            int R16, int kp) {
  const int l = blockIdx.y, m0 = blockIdx.x * kOneMB;
  if (m0 > 2 * l) return;
  const int r = blockIdx.z * 64 + (threadIdx.x & 63);
  const int Nl = lay[2 * l + 1];
  const double* T = RiT + static_cast<int64_t>(l) * N4 * R16 + min(r, R16 - 1);
  const double* xm[kOneMB];
#pragma unroll
  for (int u = 0; u < kOneMB; ++u)
    xm[u] = x + lay[2 * l] + static_cast<int64_t>(min(m0 + u, 2 * l)) * Nl;
  double acc[kOneMB];
  one_sum(Nl, [&](int n, double (&a)[kOneMB]) __attribute__((always_inline)) {
    const double t = T[static_cast<int64_t>(n) * R16];
#pragma unroll
    for (int u = 0; u < kOneMB; ++u) a[u] = fma(t, xm[u][n], a[u]);
  }, acc);
  if (threadIdx.x >= 64 || r >= kp) return;
#pragma unroll
  for (int u = 0; u < kOneMB; ++u)
    if (m0 + u <= 2 * l)
      G[static_cast<int64_t>(l * l + m0 + u) * kp + r] = r < R16 ? acc[u] : 0.0;
}

// z[alpha(lm, n)] = sum_r Rf[l][r][n] A[lm][r]
__global__ __launch_bounds__(256) void k_radial_forward_one(const double* __restrict__ RfT,
                                                            const double* __restrict__ A,
                                                            double* __restrict__ z,
                                                            const int* __restrict__ lay, int R4,
                                                            int N16, int n_r, int kp) {
  const int l = blockIdx.y, m0 = blockIdx.x * kOneMB;
  if (m0 > 2 * l) return;
  const int n = blockIdx.z * 64 + (threadIdx.x & 63);
  const int Nl = lay[2 * l + 1];
  const double* T = RfT + static_cast<int64_t>(l) * R4 * N16 + min(n, N16 - 1);
  const double* am[kOneMB];
#pragma unroll
  for (int u = 0; u < kOneMB; ++u)
    am[u] = A + static_cast<int64_t>(l * l + min(m0 + u, 2 * l)) * kp;
  double acc[kOneMB];
  one_sum(n_r, [&](int r, double (&a)[kOneMB]) __attribute__((always_inline)) {
    const double t = T[static_cast<int64_t>(r) * N16];
#pragma unroll
    for (int u = 0; u < kOneMB; ++u) a[u] = fma(t, am[u][r], a[u]);
  }, acc);
  if (threadIdx.x >= 64 || n >= Nl) return;
#pragma unroll
  for (int u = 0; u < kOneMB; ++u)
    if (m0 + u <= 2 * l) z[lay[2 * l] + static_cast<int64_t>(m0 + u) * Nl + n] = acc[u];
}

// f(std::integral_constant<int, L / 16 rounded up>()), L <= 96
template <typename F>
void with_ltiles(int L, F&& f) {
  switch ((L + 15) / 16) {
    case 1: f(std::integral_constant<int, 1>()); break;
    case 2: f(std::integral_constant<int, 2>()); break;
    case 3: f(std::integral_constant<int, 3>()); break;
    case 4: f(std::integral_constant<int, 4>()); break;
    case 5: f(std::integral_constant<int, 5>()); break;
    default: f(std::integral_constant<int, 6>()); break;
  }
}

// f(std::integral_constant<int, trig_kt(L)>()): an even count of k-steps, at
// most MOST
template <int MOST = 24, int KT = 2, typename F>
void with_kt(int L, F&& f) {
  if constexpr (KT < MOST) {
    if (trig_kt(L) > KT) return with_kt<MOST, KT + 2>(L, std::forward<F>(f));
  }
  f(std::integral_constant<int, KT>());
}

// One wave per (row, 16 columns), or the four waves of a workgroup on one
// when that alone gives less than two waves per SIMD.
void analysis_rows(const Basis& b, const double* f, const double* f2, int64_t ldf, int k, int kp,
                   double* gh, int64_t n_rows, hipStream_t s) {
  const int64_t rc = n_rows * (kp / 16);
  with_ltiles(b.L, [&](auto lt) {
    auto go = [&](auto diff, auto split) {
      constexpr bool SPLIT = decltype(split)::value;
      const unsigned nb = static_cast<unsigned>(SPLIT ? rc : (rc + 3) / 4);
      k_phi_analysis<decltype(lt)::value, decltype(diff)::value, SPLIT><<<nb, 256, 0, s>>>(
          f, f2, ldf, k, kp, gh, b.dev_trig_a, b.L, b.n_phi, 2.0 * M_PI / b.n_phi, n_rows);
    };
    if (rc >= 2048)
      f2 ? go(std::true_type(), std::false_type()) : go(std::false_type(), std::false_type());
    else
      f2 ? go(std::true_type(), std::true_type()) : go(std::false_type(), std::true_type());
  });
}

// A wave takes all p tiles of its row and columns (its coefficients are loaded
// once), unless that leaves fewer than two waves per SIMD: then one tile each
// (one function on the 60 x 50 x 100 grid: 200 waves of four tiles otherwise).
void synthesis_rows(const Basis& b, const double* g, int k, int kp, double* f, int64_t ldf,
                    int64_t n_rows, const double* vext, const double* rho, int corr,
                    hipStream_t s) {
  const int npt = b.n_phi / 2 / 16 + 1;
  const int64_t rc = n_rows * (kp / 16);
  const int ppw = rc < 2048 ? 1 : npt, nsp = (npt + ppw - 1) / ppw;
  const unsigned nb = static_cast<unsigned>((rc * nsp + 3) / 4);
  with_kt(b.L, [&](auto kt) {
    constexpr int KT = decltype(kt)::value;
    auto go = [&](auto ks) {
      k_phi_synthesis<KT, decltype(ks)::value><<<nb, 256, 0, s>>>(
          g, k, kp, f, ldf, b.dev_trig_s64, b.L, b.n_phi, n_rows, ppw, nsp, vext, rho, corr);
    };
    if (vext)
      go(std::true_type());
    else
      go(std::false_type());
  });
}

}  // namespace

void launch_phi_analysis_cols(const Basis& b, const double* f, int64_t ldf, int k, int kp,
                              double* gh, hipStream_t s) {
  analysis_rows(b, f, nullptr, ldf, k, kp, gh, int64_t(b.n_r) * b.n_theta, s);
}

void launch_phi_synthesis_cols(const Basis& b, const double* g, int k, int kp, double* f,
                               int64_t ldf, hipStream_t s) {
  synthesis_rows(b, g, k, kp, f, ldf, int64_t(b.n_r) * b.n_theta, nullptr, nullptr, 0, s);
}

// A wave per row, or a workgroup per row where a wave's coefficients of one
// tile and the next take so many registers that one or two waves are left per
// SIMD (FP64 from L = 57, FP32 from L = 89), and for several column tiles on
// few rows.  Density in us, a wave | a workgroup per row: k = 32, n_phi = 4 L,
// 60 nodes (L >= 88: 30), FP64 L = 55 195 | 242, 57 448 | 259, FP32 L = 88 300 |
// 307, 89 922 | 309; L = 9, FP64, 432 rows, n_phi = 72, k = 64 20.7 | 17.6,
// n_phi = 512, k = 64 51.5 | 37.9, k = 16 18.5 | 22.6; 1620 rows, n_phi = 512, k =
// 64 76.9 | 96.1; L = 16, 1152 rows, n_phi = 64, k = 64 33.4 | 33.8.
constexpr int64_t kDensityWaveRows = 1024;
template <typename T>
void launch_density_phi(const Basis& b, const T* gbuf, const double* occ, double* rho, int k,
                        int kp, hipStream_t s) {
  const int64_t n_rows = int64_t(b.n_r) * b.n_theta;
  constexpr int KTW = sizeof(T) == 8 ? 14 : 22;     // most k-steps of a half a wave takes
  if (trig_kt(b.L) > KTW || (kp > 16 && n_rows < kDensityWaveRows)) {
    const unsigned nb = static_cast<unsigned>(std::min<int64_t>(n_rows, kDensityWorkgroups));
    return with_ltiles(b.L, [&](auto lt) {
      constexpr int LP = 16 * decltype(lt)::value;
      const size_t lds = size_t(b.n_phi) * sizeof(double) + 2 * size_t(b.n_phi) * sizeof(T) +
                         size_t(2 * LP) * (16 * kDensityNT + 1) * sizeof(T);
      if (lds > 65536)      // n_phi <= 2048: at most 99 KB
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_density_rows<T, LP>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize,
                                  static_cast<int>(lds));
      k_density_rows<T, LP><<<nb, 256, lds, s>>>(gbuf, occ, rho, b.dev_cs, b.L, kp, b.n_phi, k,
                                                 n_rows);
    });
  }
  const T* tb = reinterpret_cast<const T*>(sizeof(T) == 8 ? (const void*)b.dev_trig_s64
                                                          : (const void*)b.dev_trig_s32);
  with_kt<KTW>(b.L, [&](auto kt) {
    constexpr int KT = decltype(kt)::value;
    const size_t acc = 4 * size_t(b.n_phi) * sizeof(double);
    const size_t tab = size_t(b.n_phi / 32 + 1) * KT * 2 * 64 * sizeof(T);
    const int64_t nb = (n_rows + 3) / 4;
    // the table in LDS while three workgroups of a CU hold it (registers
    // allow about that many), each then walking its share of the rows
    if (acc + tab <= 53248)
      k_density<T, KT, true><<<static_cast<unsigned>(std::min<int64_t>(nb, 768)), 256, acc + tab,
                               s>>>(gbuf, occ, rho, tb, k, kp, b.L, b.n_phi, n_rows);
    else
      k_density<T, KT, false><<<static_cast<unsigned>(nb), 256, acc, s>>>(gbuf, occ, rho, tb, k, kp,
                                                                          b.L, b.n_phi, n_rows);
  });
}
template void launch_density_phi<double>(const Basis&, const double*, const double*, double*, int,
                                         int, hipStream_t);
template void launch_density_phi<float>(const Basis&, const float*, const double*, double*, int,
                                        int, hipStream_t);

// One grid function: the radial nodes are the columns of the angular stages
// (kp = n_r rounded up to 16, one "radial node" of n_theta rows), so the
// 16-column MFMA tiles hold 16 nodes instead of one function and 15 zeros.
int one_kp(const Basis& b) { return static_cast<int>(round_up(b.n_r, kColPad)); }

void launch_forward_one(const Basis& b, const double* f, const double* f2, double* gh, double* A,
                        double* z, hipStream_t s) {
  const int kp = one_kp(b);
  analysis_rows(b, f, f2, int64_t(b.n_theta) * b.n_phi, b.n_r, kp, gh, b.n_theta, s);
  launch_legendre_analysis<double>(b, b.t64, gh, A, kp, s, 1);
  const int R4 = static_cast<int>(round_up(b.n_r, 4)), N16 = static_cast<int>(round_up(b.N, 16));
  const dim3 grid((2 * b.L - 1 + kOneMB - 1) / kOneMB, b.L, (b.N + 63) / 64);
  k_radial_forward_one<<<grid, 256, 0, s>>>(b.t64.RfT, A, z, b.dev_lay, R4, N16, b.n_r, kp);
}

void launch_inverse_one(const Basis& b, const double* RiT, const double* x, double* G, double* g,
                        double* f, const double* vext, const double* rho, int corr,
                        hipStream_t s) {
  const int kp = one_kp(b);
  const int N4 = static_cast<int>(round_up(b.N, 4)), R16 = static_cast<int>(round_up(b.n_r, 16));
  const dim3 grid((2 * b.L - 1 + kOneMB - 1) / kOneMB, b.L, (kp + 63) / 64);
  k_radial_inverse_one<<<grid, 256, 0, s>>>(RiT, x, G, b.dev_lay, N4, R16, kp);
  launch_legendre_synth<double>(b, b.t64, G, g, kp, s, 1);
  synthesis_rows(b, g, b.n_r, kp, f, int64_t(b.n_theta) * b.n_phi, b.n_theta, vext, rho, corr, s);
}

}  // namespace ces
