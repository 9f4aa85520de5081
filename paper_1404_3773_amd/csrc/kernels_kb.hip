// Kleinman-Bylander projector products of H*X (Section 2.3.2):
//   kb_gemm   C[q][i] = h_q sum_alpha P[q][alpha] Y[alpha][i]   (M = n_proj, N = k, K = d)
//   kb_apply  Z[alpha][i] = sum_q P[q][alpha] C[q][i]          (M = k, N = d, K = n_proj)
// Z is added in the radial forward kernel's epilogue.
//
// kb_gemm:
// Both operands run contiguously along the contraction index alpha (P is
// stored n_proj x d row-major, Y column-major): a workgroup stages a BM x BK
// tile of P and a BN x BK tile of Y per step in LDS, loaded as whole row
// segments (consecutive lanes on consecutive alpha), the next step's tiles
// in registers while the current one runs on 16x16x4 MFMA (2 x 2 waves, TM x
// TN fragments each).  K is split into chunks whose partial products go to a
// buffer; a second kernel sums them in a fixed order and applies h.
// Workgroup ids are dealt round-robin over the 8 XCDs.  With xcd_chunk set
// (a chunk count that is a multiple of 8) every workgroup of a chunk (all
// its M and N tiles) is placed on XCD chunk mod 8, in M-tile order, so the
// workgroups in flight on an XCD walk the same chunk's alpha steps together:
// its L2 serves the Y steps they share (all M tiles) and the P steps (all N
// tiles of an M tile), and each is fetched from HBM about once.  Otherwise
// the groups (chunk, M tile) of nN workgroups are dealt round-robin over the
// XCDs, which keeps all of them busy for any chunk count.  FP32 operands with
// 16-byte aligned rows are staged 64 alpha per step from 16-byte loads into
// one LDS buffer (309 atoms: 22.9 -> 20.8 ms against 32 alpha per step from
// 4-byte loads, double-buffered; 32 per step from 16-byte loads,
// double-buffered, 22.1 ms; 32 per step single-buffered at three waves per
// SIMD, 21.4 ms; wave tiles of 128 x 64 with 16 or 32 alpha per step, 22.7
// ms or slower).  FP64 operands with even leading dimensions and
// 16-byte aligned bases are staged from 16-byte loads (2 doubles; 309 atoms:
// 48.9 -> 45.4 ms), the Gram products of Cholesky-QR and Rayleigh-Ritz too.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "ces_internal.h"
#include "mfma.h"

namespace ces {
namespace {

template <typename T>
struct KbShape;
template <>
struct KbShape<float> {   // wave tile 64 x 64, workgroup 128 x 128, 32 alpha per step
  static constexpr int KB = 32, TM = 4, TN = 4;
};
template <>
struct KbShape<double> {  // wave tile 64 x 32, workgroup 128 x 64, 32 alpha per step
  static constexpr int KB = 32, TM = 4, TN = 2;
};
// C = P^T Y, FP32 with 16-byte aligned rows: the same 128 x 128 workgroup
// tiles, 64 alpha per step staged from 16-byte loads (each row's segment of
// a step is two whole 128-byte lines) into one LDS buffer (69.6 KB, two
// workgroups per CU).
struct KgVec {
  static constexpr int KB = 64, TM = 4, TN = 4;
};
// C = P^T Y, FP64, wide tiles (kb_wide64): wave tile 64 x 64, so an operand
// read from LDS serves four MFMAs instead of two or four; 16 alpha per step
// (one 128-byte line of a row) in two LDS buffers (73.7 KB, two workgroups per
// CU) and one barrier a step.  FP64 MFMA bound: 60 of 72.7 TFLOP/s at 309
// atoms, 1236 projectors, k = 250.
struct KgWide64 {
  static constexpr int KB = 16, TM = 4, TN = 4;
};
constexpr int kKbPerXcd = 64;      // resident workgroups per XCD (32 CUs, 2 each)
constexpr int kKbMaxPerXcd = kKbMaxChunks / 8;   // split-K chunks per XCD, at most

// LDS row pitch of the staged tiles: the MFMA operand reads take 16 rows x 4
// consecutive alpha (rows c16, columns kk); with pitch KB + 2 (FP32) the 64
// lanes of a read fall on distinct banks, where KB + 1 left them two-way
// (309-atom C = P^T Y: 25.4 -> 24.5 ms).  FP64 reads 8-byte words and keeps
// KB + 1 (its C was slower with KB + 2).
// Rows staged from 16-byte loads take an aligned pitch: FP32 (vw = 4) KB + 4,
// which spreads the operand reads the same way (64 alpha per step: rows c16
// start 4 c16 banks apart); FP64 (vw = 2) KB + 2, where the faster staging
// outweighs the slower reads.
template <typename T>
constexpr int kb_pitch(int kb, int vw = 1) {
  return kb + (sizeof(T) == 4 ? (vw > 1 ? 4 : 2) : (vw > 1 ? 2 : 1));
}

// With DB the P and Y tiles are double-buffered in (dynamic) LDS: a step
// computes from one buffer while the next step's tiles are written into the
// other, so it takes one barrier instead of two.
// S: KB alpha per step, TM x TN fragments per wave; VW: alpha per staging
// load (1, or 4 with 16-byte aligned rows: fewer row addresses to hold).
template <typename T, bool DB, typename S, int VW>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(VW == 4 ? 2 : 1, 8)))
void k_kb_gemm(const T* __restrict__ P, int64_t d, int64_t ldp, const T* __restrict__ Y,
               int64_t ldy, T* __restrict__ part, int n_proj, int k, int kp, int64_t kchunk,
               int nM, int nN, int nchunk, int xcd_chunk) {
  typedef typename MF<T>::acc acc_t;
  constexpr int KB = S::KB, TM = S::TM, TN = S::TN;
  constexpr int BM = 32 * TM, BN = 32 * TN;      // 2 x 2 waves
  constexpr int KW = kb_pitch<T>(KB, VW);        // padded LDS row
  static_assert(KW % VW == 0, "vector LDS writes need an aligned row pitch");
  constexpr int KV = KB / VW;                    // threads per tile row
  constexpr int RA = 256 / KV;                   // tile rows loaded per pass
  constexpr int LA = BM / RA, LB = BN / RA;      // passes for the P and Y tiles
  constexpr int STAGE = (BM + BN) * KW;          // one buffer: A tile then B tile
  extern __shared__ __align__(16) unsigned char kb_smem[];
  T* const lds = reinterpret_cast<T*>(kb_smem);
  // workgroup id -> (XCD x, position j on it) -> (t-th group of XCD x, N tile)
  // -> (chunk x + 8 (t / nM), M tile t % nM), or group x + 8 t = (chunk, M tile)
  const int id = blockIdx.x;
  const int x = id & 7, j = id >> 3;
  const int t = j / nN, ntb = j - t * nN;
  int chunk, mtb;
  if (xcd_chunk) {
    const int cx = t / nM;
    mtb = t - cx * nM;
    chunk = x + 8 * cx;
  } else {
    const int g = x + 8 * t;
    chunk = g / nM;
    mtb = g - chunk * nM;
  }
  if (chunk >= nchunk) return;
  const int64_t k0 = static_cast<int64_t>(chunk) * kchunk;
  const int64_t k1 = k0 + kchunk < d ? k0 + kchunk : d;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int c16 = lane & 15, kk = lane >> 4;
  // staging: thread -> (tile row r0 + RA p, alpha offset kc .. kc + VW - 1);
  // row addresses are formed per load (fewer registers held)
  const int kc = VW * (tid % KV), r0 = tid / KV;
  const int arow0 = mtb * BM + r0, bcol0 = ntb * BN + r0;
  // loads read clamped addresses and are masked when stored to LDS (a
  // select on a load makes the wave wait for it, which would serialise the
  // next step's loads); a vector past k1 is clamped to the last aligned one
  // (inside the rows, whose lengths are multiples of VW)
  T ra[LA][VW], rb[LB][VW];
  auto fetch = [&](int64_t kb) {
    const int64_t kx = kb + kc;
    const int64_t kcl = kx < k1 ? kx : (k1 - 1) / VW * VW;
#pragma unroll
    for (int p = 0; p < LA; ++p) {
      const int row = arow0 + RA * p;
      load_vec<T, VW>(P + static_cast<int64_t>(row < n_proj ? row : n_proj - 1) * ldp + kcl, ra[p]);
    }
#pragma unroll
    for (int p = 0; p < LB; ++p) {
      const int col = bcol0 + RA * p;
      load_vec<T, VW>(Y + static_cast<int64_t>(col < k ? col : k - 1) * ldy + kcl, rb[p]);
    }
  };
  acc_t acc[TM][TN];
#pragma unroll
  for (int u = 0; u < TM; ++u)
#pragma unroll
    for (int v = 0; v < TN; ++v) acc[u][v] = zero_acc<acc_t>();
  // the staged tiles of step kb into buffer `buf`
  auto stage = [&](int64_t kb, int buf) __attribute__((always_inline)) {
    T* As = lds + buf * STAGE;
    T* Bs = As + BM * KW;
#pragma unroll
    for (int p = 0; p < LA; ++p) {
      const bool okr = arow0 + RA * p < n_proj;
      T w[VW];
#pragma unroll
      for (int e = 0; e < VW; ++e) w[e] = okr && kb + kc + e < k1 ? ra[p][e] : T(0);
      if constexpr (VW == 1)
        As[(r0 + RA * p) * KW + kc] = w[0];
      else
        store_vec<T, VW, false>(As + (r0 + RA * p) * KW + kc, w);
    }
#pragma unroll
    for (int p = 0; p < LB; ++p) {
      const bool okr = bcol0 + RA * p < k;
      T w[VW];
#pragma unroll
      for (int e = 0; e < VW; ++e) w[e] = okr && kb + kc + e < k1 ? rb[p][e] : T(0);
      if constexpr (VW == 1)
        Bs[(r0 + RA * p) * KW + kc] = w[0];
      else
        store_vec<T, VW, false>(Bs + (r0 + RA * p) * KW + kc, w);
    }
  };
  // k-steps [s0, s1) of the staged tiles in buffer `buf`
  auto compute_steps = [&](int buf, int s0, int s1) __attribute__((always_inline)) {
    const T* Aw = lds + buf * STAGE + (wm * 16 * TM + c16) * KW + kk;
    const T* Bw = lds + buf * STAGE + BM * KW + (wn * 16 * TN + c16) * KW + kk;
#pragma unroll
    for (int st = s0; st < s1; ++st) {
      T a[TM], b[TN];
#pragma unroll
      for (int u = 0; u < TM; ++u) a[u] = Aw[16 * u * KW + 4 * st];
#pragma unroll
      for (int v = 0; v < TN; ++v) b[v] = Bw[16 * v * KW + 4 * st];
#pragma unroll
      for (int u = 0; u < TM; ++u)
#pragma unroll
        for (int v = 0; v < TN; ++v) acc[u][v] = MF<T>::mma(a[u], b[v], acc[u][v]);
    }
  };
  auto compute = [&](int buf) __attribute__((always_inline)) { compute_steps(buf, 0, KB / 4); };
  if (k0 < k1) fetch(k0);
  if constexpr (DB) {
    if (k0 < k1) {
      stage(k0, 0);
      if (k0 + KB < k1) fetch(k0 + KB);
    }
    __syncthreads();
    int buf = 0;
    for (int64_t kb = k0; kb < k1; kb += KB) {
      // the other buffer was last read in the previous step, before its
      // barrier: its LDS writes and the next global loads go out between the
      // two halves of this step's MFMAs
      const bool more = kb + KB < k1;
      compute_steps(buf, 0, KB / 8);
      if (more) stage(kb + KB, buf ^ 1);
      compute_steps(buf, KB / 8, KB / 4);
      if (more && kb + 2 * KB < k1) fetch(kb + 2 * KB);
      __syncthreads();
      buf ^= 1;
    }
  } else {
    for (int64_t kb = k0; kb < k1; kb += KB) {
      stage(kb, 0);
      __syncthreads();
      if (kb + KB < k1) fetch(kb + KB);          // next step's tiles, in flight
      compute(0);
      __syncthreads();
    }
  }
  T* pc = part + static_cast<int64_t>(chunk) * n_proj * kp;
#pragma unroll
  for (int u = 0; u < TM; ++u)
#pragma unroll
    for (int v = 0; v < TN; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = mtb * BM + wm * 16 * TM + 16 * u + MF<T>::row(lane, r);
        const int col = ntb * BN + wn * 16 * TN + 16 * v + c16;
        if (row < n_proj && col < k) pc[static_cast<int64_t>(row) * kp + col] = acc[u][v][r];
      }
}

// kb_apply: Z^T = C^T P on 16x16x4 MFMA, workgroup tile BM columns i x BN rows
// alpha, both operands staged per step of KB projectors in LDS (C rows run
// along i, P rows along alpha), the next step's tiles in registers.  The
// result lane holds 16 consecutive alpha of one column, so stores are
// coalesced.  Workgroups that read the same P tile (same alpha tile) share
// an XCD.  It serves the operands that the wide-tile kernel below cannot
// load as 16-byte vectors (FP64 projector rows of odd length d).  FP32 is held
// to four waves per SIMD (309 atoms, before the wide tiles: 23.1 -> 22.7 ms;
// three VGPRs spill, outside the K loop), FP64 to three (51.7 -> 46.7 ms, no
// spills).
template <typename T, bool DB, int KB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 3, 8)))
void k_kb_apply(const T* __restrict__ P, int64_t d,
                                                  int64_t ldp, const T* __restrict__ C,
                                                  int n_proj, int k, int kp, T* __restrict__ Z,
                                                  int nI, int nA) {
  typedef typename MF<T>::acc acc_t;
  constexpr int TM = KbShape<T>::TM, TN = KbShape<T>::TN;
  constexpr int BM = 32 * TN, BN = 32 * TM;      // i tile, alpha tile (2 x 2 waves)
  constexpr int KW = kb_pitch<T>(KB);
  constexpr int RC = 256 / BM, RP = 256 / BN;    // q rows per staging pass
  constexpr int LC = KB / RC, LP = KB / RP;
  constexpr int STAGE = (BM + BN) * KW;          // one buffer: Cs [i][q] then Ps [alpha][q]
  extern __shared__ __align__(16) unsigned char kb_smem[];
  T* const lds = reinterpret_cast<T*>(kb_smem);
  const int id = blockIdx.x;
  const int x = id & 7, j = id >> 3;
  const int ga = x + 8 * (j / nI), itb = j - (j / nI) * nI;
  if (ga >= nA) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int c16 = lane & 15, kk = lane >> 4;
  const int ci = tid % BM, cq = tid / BM;
  const int pa_ = tid % BN, pq = tid / BN;
  const int i_s = itb * BM + ci;
  const bool iok = i_s < kp;
  const int64_t a_s = static_cast<int64_t>(ga) * BN + pa_;
  const bool aok = a_s < d;
  const T* cbase = C + (iok ? i_s : 0);
  const T* pbase = P + (aok ? a_s : 0);
  T rc[LC], rp[LP];
  // clamped loads, masked when stored to LDS (see k_kb_gemm)
  auto fetch = [&](int q0) {
#pragma unroll
    for (int p = 0; p < LC; ++p) {
      const int q = q0 + cq + RC * p;
      rc[p] = cbase[static_cast<int64_t>(q < n_proj ? q : n_proj - 1) * kp];
    }
#pragma unroll
    for (int p = 0; p < LP; ++p) {
      const int q = q0 + pq + RP * p;
      rp[p] = pbase[static_cast<int64_t>(q < n_proj ? q : n_proj - 1) * ldp];
    }
  };
  acc_t acc[TN][TM];
#pragma unroll
  for (int u = 0; u < TN; ++u)
#pragma unroll
    for (int v = 0; v < TM; ++v) acc[u][v] = zero_acc<acc_t>();
  auto stage = [&](int q0, int buf) __attribute__((always_inline)) {
    T* Cs = lds + buf * STAGE;
    T* Ps = Cs + BM * KW;
#pragma unroll
    for (int p = 0; p < LC; ++p)
      Cs[ci * KW + cq + RC * p] = iok && q0 + cq + RC * p < n_proj ? rc[p] : T(0);
#pragma unroll
    for (int p = 0; p < LP; ++p)
      Ps[pa_ * KW + pq + RP * p] = aok && q0 + pq + RP * p < n_proj ? rp[p] : T(0);
  };
  // k-steps [s0, s1) of the staged tiles in buffer `buf`
  auto compute_steps = [&](int buf, int s0, int s1) __attribute__((always_inline)) {
    const T* Aw = lds + buf * STAGE + (wm * 16 * TN + c16) * KW + kk;
    const T* Bw = lds + buf * STAGE + BM * KW + (wn * 16 * TM + c16) * KW + kk;
#pragma unroll
    for (int st = s0; st < s1; ++st) {
      T a[TN], b[TM];
#pragma unroll
      for (int u = 0; u < TN; ++u) a[u] = Aw[16 * u * KW + 4 * st];
#pragma unroll
      for (int v = 0; v < TM; ++v) b[v] = Bw[16 * v * KW + 4 * st];
#pragma unroll
      for (int u = 0; u < TN; ++u)
#pragma unroll
        for (int v = 0; v < TM; ++v) acc[u][v] = MF<T>::mma(a[u], b[v], acc[u][v]);
    }
  };
  auto compute = [&](int buf) __attribute__((always_inline)) { compute_steps(buf, 0, KB / 4); };
  fetch(0);
  if constexpr (DB) {
    stage(0, 0);
    if (KB < n_proj) fetch(KB);
    __syncthreads();
    int buf = 0;
    for (int q0 = 0; q0 < n_proj; q0 += KB) {
      // the other buffer's LDS writes and the next global loads go out
      // between the two halves of this step's MFMAs (see k_kb_gemm)
      const bool more = q0 + KB < n_proj;
      compute_steps(buf, 0, KB / 8);
      if (more) stage(q0 + KB, buf ^ 1);
      compute_steps(buf, KB / 8, KB / 4);
      if (more && q0 + 2 * KB < n_proj) fetch(q0 + 2 * KB);
      __syncthreads();
      buf ^= 1;
    }
  } else {
    for (int q0 = 0; q0 < n_proj; q0 += KB) {
      stage(q0, 0);
      __syncthreads();
      if (q0 + KB < n_proj) fetch(q0 + KB);
      compute(0);
      __syncthreads();
    }
  }
#pragma unroll
  for (int u = 0; u < TN; ++u)
#pragma unroll
    for (int v = 0; v < TM; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = itb * BM + wm * 16 * TN + 16 * u + MF<T>::row(lane, r);
        const int64_t a = static_cast<int64_t>(ga) * BN + wn * 16 * TM + 16 * v + c16;
        if (i < k && a < d) Z[static_cast<int64_t>(i) * d + a] = acc[u][v][r];
      }
}

// kb_apply, wide tiles.  FP32: workgroup tile 128 columns i x 256 rows alpha,
// 2 x 2 waves of 64 x 128 (4 x 8 MFMA fragments, 128 accumulators per lane),
// so each staged operand value feeds twice the MFMAs of the 64 x 64 wave
// tile.  The projector steps (KA per step) are staged in LDS row-major by
// projector (C rows along i, P rows along alpha) from 16-byte loads and
// 16-byte LDS writes; the MFMA operand reads take 16 consecutive columns of 4
// projector rows whose starts lie 16 banks apart (row pitch = width + 16
// words).  Column loads are clamped into the arrays (rows are padded to a
// multiple of 4): a clamped column only feeds outputs of columns i >= kp or
// alpha >= ldp, which are not stored.  Projector rows past n_proj are
// clamped on load and zeroed in the C tile.  309 atoms (k = 1000, 1236
// projectors): 22.8 ms with the 64 x 64 wave tiles, 19.5 ms here (the same
// result bits: each accumulator takes the projectors in the same order);
// 8, 16 and 32 projectors per step (32 single-buffered) time alike, 32
// double-buffered (one workgroup per CU) 26.3 ms.  Measured and not kept:
// lanes owning 4 adjacent columns so that the operands come as 16-byte LDS
// reads (3 instead of 12 per 4 projectors: 19.5 ms as well), and a raised
// wave priority around the MFMA sections (19.4 -> 19.2 ms here, but C =
// P^T Y 20.6 -> 20.9 and both FP64 products slower).
// FP64 (operands with even rows): 2 x 2 waves of 64 x 64 (4 x 4 fragments),
// 128 x 128 workgroup tiles, 2 doubles per 16-byte access, row pitch width +
// 16 doubles (the 4 projector rows of an operand read start 128 bytes apart
// modulo 256); 309 atoms: 46.5 -> 39.2 ms, the same result bits.
template <typename T>
struct ApShape;
template <>
struct ApShape<float> {
  static constexpr int TI = 4, TA = 8, KA = 16;
};
template <>
struct ApShape<double> {
  static constexpr int TI = 4, TA = 4, KA = 16;
};
constexpr bool kApDB = true;   // double-buffered LDS

template <typename T>
constexpr size_t kb_apply_wide_lds() {
  typedef ApShape<T> S;
  return (kApDB ? 2 : 1) * size_t(S::KA) * (32 * S::TI + 16 + 32 * S::TA + 16) * sizeof(T);
}

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8)))
void k_kb_apply_wide(const T* __restrict__ P, int64_t d, int64_t ldp, const T* __restrict__ C,
                     int n_proj, int k, int kp, T* __restrict__ Z, int nI, int nA) {
  typedef typename MF<T>::acc acc_t;
  typedef ApShape<T> S;
  constexpr int TI = S::TI, TA = S::TA, KA = S::KA;
  constexpr bool DB = kApDB;
  constexpr int BI = 32 * TI, BA = 32 * TA;     // workgroup tile: i, alpha
  constexpr int PI = BI + 16, PA = BA + 16;     // LDS row pitch (elements)
  constexpr int VW = 16 / static_cast<int>(sizeof(T));   // elements per 16-byte access
  constexpr int STAGE = KA * (PI + PA);
  constexpr int CV = KA * BI / (VW * 256);      // 16-byte C loads per thread per step
  constexpr int PV = KA * BA / (VW * 256);      // 16-byte P loads per thread per step
  constexpr int CR = 256 / (BI / VW), PR = 256 / (BA / VW);   // rows per pass
  static_assert(CV >= 1 && PV >= 1, "step too short for the staging passes");
  extern __shared__ __align__(16) unsigned char kb_smem[];
  T* const lds = reinterpret_cast<T*>(kb_smem);
  const int id = blockIdx.x;
  const int x = id & 7, j = id >> 3;
  const int ga = x + 8 * (j / nI), itb = j - (j / nI) * nI;
  if (ga >= nA) return;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wi = wave >> 1, wa = wave & 1;
  const int c16 = lane & 15, kk = lane >> 4;
  const int cr = tid / (BI / VW), cc = VW * (tid % (BI / VW));
  const int pr = tid / (BA / VW), pc = VW * (tid % (BA / VW));
  const int ic = min(itb * BI + cc, kp - VW);
  const int64_t ac = min(static_cast<int64_t>(ga) * BA + pc, ldp - VW);
  const T* cbase = C + ic;
  const T* pbase = P + ac;
  T rc[CV][VW], rp[PV][VW];
  auto fetch = [&](int q0) {
#pragma unroll
    for (int p = 0; p < CV; ++p) {
      const int q = q0 + cr + CR * p;
      load_vec<T, VW>(cbase + static_cast<int64_t>(q < n_proj ? q : n_proj - 1) * kp, rc[p]);
    }
#pragma unroll
    for (int p = 0; p < PV; ++p) {
      const int q = q0 + pr + PR * p;
      load_vec<T, VW>(pbase + static_cast<int64_t>(q < n_proj ? q : n_proj - 1) * ldp, rp[p]);
    }
  };
  acc_t acc[TI][TA];
#pragma unroll
  for (int u = 0; u < TI; ++u)
#pragma unroll
    for (int v = 0; v < TA; ++v) acc[u][v] = zero_acc<acc_t>();
  auto stage = [&](int q0, int buf) __attribute__((always_inline)) {
    T* Cs = lds + buf * STAGE;
    T* Ps = Cs + KA * PI;
#pragma unroll
    for (int p = 0; p < CV; ++p) {
      const bool ok = q0 + cr + CR * p < n_proj;
      T w[VW];
#pragma unroll
      for (int e = 0; e < VW; ++e) w[e] = ok ? rc[p][e] : T(0);
      store_vec<T, VW, false>(Cs + (cr + CR * p) * PI + cc, w);
    }
#pragma unroll
    for (int p = 0; p < PV; ++p) store_vec<T, VW, false>(Ps + (pr + PR * p) * PA + pc, rp[p]);
  };
  auto compute_steps = [&](int buf, int s0, int s1) __attribute__((always_inline)) {
    const T* Aw = lds + buf * STAGE + kk * PI + wi * 16 * TI + c16;
    const T* Bw = lds + buf * STAGE + KA * PI + kk * PA + wa * 16 * TA + c16;
#pragma unroll
    for (int st = s0; st < s1; ++st) {
      T a[TI], b[TA];
#pragma unroll
      for (int u = 0; u < TI; ++u) a[u] = Aw[4 * st * PI + 16 * u];
#pragma unroll
      for (int v = 0; v < TA; ++v) b[v] = Bw[4 * st * PA + 16 * v];
#pragma unroll
      for (int u = 0; u < TI; ++u)
#pragma unroll
        for (int v = 0; v < TA; ++v) acc[u][v] = MF<T>::mma(a[u], b[v], acc[u][v]);
    }
  };
  fetch(0);
  if constexpr (DB) {
    stage(0, 0);
    if (KA < n_proj) fetch(KA);
    __syncthreads();
    int buf = 0;
    for (int q0 = 0; q0 < n_proj; q0 += KA) {
      const bool more = q0 + KA < n_proj;
      compute_steps(buf, 0, KA / 8);
      if (more) stage(q0 + KA, buf ^ 1);
      compute_steps(buf, KA / 8, KA / 4);
      if (more && q0 + 2 * KA < n_proj) fetch(q0 + 2 * KA);
      __syncthreads();
      buf ^= 1;
    }
  } else {
    for (int q0 = 0; q0 < n_proj; q0 += KA) {
      stage(q0, 0);
      __syncthreads();
      if (q0 + KA < n_proj) fetch(q0 + KA);
      compute_steps(0, 0, KA / 4);
      __syncthreads();
    }
  }
#pragma unroll
  for (int u = 0; u < TI; ++u)
#pragma unroll
    for (int v = 0; v < TA; ++v)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = itb * BI + wi * 16 * TI + 16 * u + MF<T>::row(lane, r);
        const int64_t a = static_cast<int64_t>(ga) * BA + wa * 16 * TA + 16 * v + c16;
        if (i < k && a < d) Z[static_cast<int64_t>(i) * d + a] = acc[u][v][r];
      }
}

// ------------------------------------------- FP32 products on bf16 MFMA
//
// An FP32 value of magnitude 2^-110 to 3.39e38 is the exact sum of three bf16
// values, x = h + m + l (each the rounding of what the former leave: 8
// significant bits each, 24 in all), so
// x y = hh' + (hm' + mh') + (hl' + mm' + lh') up to the dropped ml', lm' and
// ll' terms, which stay below 2^-24 |x y|: one FP32 rounding of the product.
// The six products run on bf16 MFMA with FP32 accumulators.  A 16x16x32 bf16
// MFMA takes as long as half a 16x16x4 FP32 one (2,416 against 144 TFLOP/s in
// register-only loops), so the six cost 0.37 of the FP32 MFMAs, and a K = 32
// step rounds each accumulator 6 times instead of 8.  Against 64 bits the
// results are no further off than the FP32 kernels' (H X of the 309-atom shape
// below, relative 2-norm: 6.6e-8 against 9.1e-8).  Below 2^-110 the last bits of
// x fall under bf16's smallest subnormal (2^-133; conversions and MFMA keep
// subnormals): at most 2^-134 of each value is lost, so a sum of n products with
// a y of magnitude one is off by up to n 2^-134 more (d = 16,000, 130 projectors
// whose term is the output's size, error of H X in units of its maximum: 1.4e-7
// for blocks of order 2^90 to 2^-110, 2.0e-7 at 2^-114, 2.7e-6 at 2^-118).  Values above
// the largest bf16 (3.39e38) round to infinity, and an infinite or NaN input
// makes the outputs of its row or column NaN; H X of a column with an infinity
// is NaN throughout in either form, the other columns are untouched.
//
// Workgroup: 256 x 256 outputs, 8 waves of 64 x 128 (128 accumulators per
// lane, two waves per SIMD), K in steps of 32 staged in one LDS buffer (98
// KB) as bf16 planes [operand][plane][row][32 k]; a row's four 16-byte pieces
// are rotated by its number so that the operand reads (16 rows of one piece)
// and the staging writes fall on distinct banks.  The next step's values are
// loaded into registers while the current one runs, and split on the way to
// LDS: 5.5 vector instructions per value, used for 256 outputs.
// 309 atoms (1236 projectors, k = 500), FP32 kernels -> split: C = P^T Y 11.0
// -> 5.9 ms, Z = P C 9.9 -> 6.2 ms; bf16 MFMA busy 0.60 of the time at about
// 2.1 GHz, the rest is the staging between the two barriers of a step.  Tiles
// of 128 x 256 double-buffered in 147 KB: 6.4 and 7.9 ms (half as much reuse
// of each staged value); leaving out the MFMA tiles past a narrow block by
// branches in this kernel: 219 registers spilled.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));
constexpr int kSplitM = 256, kSplitN = 256, kSplitK = 32;
constexpr size_t kSplitLds = size_t(3) * (kSplitM + kSplitN) * kSplitK * 2;

__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const f2 x = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
}
// The bf16 parts of two values, packed in pairs.
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&p)[3]) {
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    p[i] = pack_bf16(a, b);
    a -= __builtin_bit_cast(float, p[i] << 16);
    b -= __builtin_bit_cast(float, p[i] & 0xffff0000u);
  }
}

// D[m][n] = sum_k A(m, k) B(n, k) for one 256 x 256 tile and k in [k0, k1).
// KM: both operands run along k (element (row, k) at row ld + k, 16-byte
// aligned rows whose length is a multiple of 4); else along the rows (element
// at k ld + row).  Rows past nA / nB repeat the last one (their outputs are
// not stored); k past k1 counts as zero (only the last step can hold such
// k).  Addresses are a scalar base and one 32-bit lane offset per load (forming
// 64-bit lane addresses took as many vector instructions as the split:
// Z = P C 6.8 -> 6.2 ms).
template <bool KM>
__device__ __forceinline__ void split_tile(const float* __restrict__ A, int64_t lda, int64_t a0,
                                           int64_t nA, const float* __restrict__ B, int64_t ldb,
                                           int64_t b0, int64_t nB, int64_t k0, int64_t k1,
                                           uint4* lds, f4 (&acc)[4][8]) {
  constexpr int R = 256;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, kk = lane >> 4;
  const int mA = static_cast<int>(min(nA - a0, int64_t(R)));   // rows of this tile
  const int mB = static_cast<int>(min(nB - b0, int64_t(R)));
  // 16-byte piece c of (operand o, plane p, row r)
  auto at = [](int o, int p, int r, int c) {
    return ((o * 3 + p) * R + r) * 4 + (c ^ ((r >> 1) & 3));
  };
  // KM: 8 threads per row, 64 rows per pass q; else one row and 16 k per
  // thread, of either operand
  constexpr int NP = KM ? 4 : 1;
  const float* base[2][NP];
  unsigned off[2][NP];
#pragma unroll
  for (int o = 0; o < 2; ++o)
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int m = o ? mB : mA;
      const int g = KM ? 64 * q : 64 * (wave & 3);
      const int r = g + (KM ? tid >> 3 : lane);
      const int g0 = KM ? min(g, m - 1) : 0, rc = min(r, m - 1);
      const int64_t ld = o ? ldb : lda;
      base[o][q] = (o ? B : A) + (o ? b0 + g0 : a0 + g0) * (KM ? ld : 1);
      off[o][q] = KM ? static_cast<unsigned>((rc - g0) * ld) + 4 * (tid & 7) : unsigned(rc);
    }
  const int kw = KM ? 0 : 16 * (wave >> 2);
  float v[2][16];
  auto fetch = [&](int64_t kb) __attribute__((always_inline)) {
    // KM: a vector past the last aligned one of the chunk reads that one
    const int64_t rest = (k1 - 1 - kb) / 4 * 4;
    const int back = KM && 4 * (tid & 7) > rest ? static_cast<int>(4 * (tid & 7) - rest) : 0;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      if constexpr (KM) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float x[4];
          load_vec<float, 4>(base[o][q] + kb + (off[o][q] - back), x);
#pragma unroll
          for (int e = 0; e < 4; ++e) v[o][4 * q + e] = x[e];
        }
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int64_t k = kb + kw + j;
          v[o][j] = (base[o][0] + (k < k1 ? k : k1 - 1) * (o ? ldb : lda))[off[o][0]];
        }
      }
    }
  };
  auto stage = [&](int64_t kb) __attribute__((always_inline)) {
    if (kb + kSplitK > k1) {          // the last step of a chunk: k past k1
#pragma unroll
      for (int o = 0; o < 2; ++o)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (kb + (KM ? 4 * (tid & 7) + j % 4 : kw + j) >= k1) v[o][j] = 0.0f;
    }
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      if constexpr (KM) {
        uint2* l2 = reinterpret_cast<uint2*>(lds);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          unsigned p0[3], p1[3];
          split_pair(v[o][4 * q], v[o][4 * q + 1], p0);
          split_pair(v[o][4 * q + 2], v[o][4 * q + 3], p1);
#pragma unroll
          for (int p = 0; p < 3; ++p)
            l2[2 * at(o, p, (tid >> 3) + 64 * q, (tid & 7) >> 1) + (tid & 1)] =
                make_uint2(p0[p], p1[p]);
        }
      } else {
#pragma unroll
        for (int g = 0; g < 2; ++g) {     // 16-byte pieces
          unsigned w[4][3];
#pragma unroll
          for (int e = 0; e < 4; ++e) split_pair(v[o][8 * g + 2 * e], v[o][8 * g + 2 * e + 1], w[e]);
#pragma unroll
          for (int p = 0; p < 3; ++p)
            lds[at(o, p, tid & 255, kw / 8 + g)] = make_uint4(w[0][p], w[1][p], w[2][p], w[3][p]);
        }
      }
    }
  };
  const int ra = (wave >> 1) * 64 + l16, rb = (wave & 1) * 128 + l16;
  auto compute = [&]() __attribute__((always_inline)) {
    bf16x8 a[4][3];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int p = 0; p < 3; ++p)
        a[u][p] = __builtin_bit_cast(bf16x8, lds[at(0, p, ra + 16 * u, kk)]);
#pragma unroll
    for (int w = 0; w < 8; ++w) {
      bf16x8 b[3];
#pragma unroll
      for (int p = 0; p < 3; ++p)
        b[p] = __builtin_bit_cast(bf16x8, lds[at(1, p, rb + 16 * w, kk)]);
      // smallest terms first
#pragma unroll
      for (int t = 0; t < 6; ++t) {
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u)
          acc[u][w] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][PA[t]], b[PB[t]], acc[u][w], 0,
                                                              0, 0);
      }
    }
  };
  fetch(k0);
  for (int64_t kb = k0; kb < k1; kb += kSplitK) {
    stage(kb);
    __syncthreads();
    if (kb + kSplitK < k1) fetch(kb + kSplitK);     // next step's values, in flight
    compute();
    __syncthreads();
  }
}

// C = P^T Y: one split-K chunk's partial product; workgroups of a chunk share
// an XCD (chunk mod 8), so its L2 serves the rows they have in common.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_kb_gemm_split(const float* __restrict__ P, int64_t d, int64_t ldp,
                     const float* __restrict__ Y, int64_t ldy, float* __restrict__ part,
                     int n_proj, int k, int kp, int64_t kchunk, int nM, int nN, int nchunk) {
  extern __shared__ __align__(16) unsigned char kb_smem[];
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int per = nM * nN;
  const int chunk = x + 8 * (j / per);
  if (chunk >= nchunk) return;
  const int tile = j % per, mt = tile / nN, nt = tile - mt * nN;
  const int64_t k0 = static_cast<int64_t>(chunk) * kchunk;
  const int64_t k1 = k0 + kchunk < d ? k0 + kchunk : d;
  f4 acc[4][8];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 8; ++w) acc[u][w] = zero_acc<f4>();
  split_tile<true>(P, ldp, int64_t(mt) * kSplitM, n_proj, Y, ldy, int64_t(nt) * kSplitN, k,
                   k0, k1, reinterpret_cast<uint4*>(kb_smem), acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float* pc = part + static_cast<int64_t>(chunk) * n_proj * kp;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 8; ++w)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = mt * kSplitM + (wave >> 1) * 64 + 16 * u + MF<float>::row(lane, r);
        const int i = nt * kSplitN + (wave & 1) * 128 + 16 * w + (lane & 15);
        if (q < n_proj && i < k) pc[static_cast<int64_t>(q) * kp + i] = acc[u][w][r];
      }
}

// Z = P C: tile 256 columns i x 256 rows alpha; the workgroups of one alpha
// tile share an XCD.
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_kb_apply_split(const float* __restrict__ P, int64_t d, int64_t ldp,
                      const float* __restrict__ C, int n_proj, int k, int kp,
                      float* __restrict__ Z, int nI, int nA) {
  extern __shared__ __align__(16) unsigned char kb_smem[];
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  const int ga = x + 8 * (j / nI), it = j - (j / nI) * nI;
  if (ga >= nA) return;
  f4 acc[4][8];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int w = 0; w < 8; ++w) acc[u][w] = zero_acc<f4>();
  split_tile<false>(C, kp, int64_t(it) * kSplitM, k, P, ldp, int64_t(ga) * kSplitN, d, 0,
                    n_proj, reinterpret_cast<uint4*>(kb_smem), acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = it * kSplitM + (wave >> 1) * 64 + 16 * u + MF<float>::row(lane, r);
      if (i >= k) continue;
#pragma unroll
      for (int w = 0; w < 8; ++w) {
        const int64_t a = static_cast<int64_t>(ga) * kSplitN + (wave & 1) * 128 + 16 * w +
                          (lane & 15);
        if (a < d) Z[static_cast<int64_t>(i) * d + a] = acc[u][w][r];
      }
    }
}

// C[q][i] = h_q sum_c part[c][q][i] for i < k, 0 for k <= i < kp.  A workgroup
// takes 32 elements; 8 threads share an element's chunks (c mod 8) and their
// sums are added in order, so up to 512 chunks take 64 loads in a row instead
// of 512 (13 x 16 elements, 512 chunks: 140 us in one thread each).
template <typename T>
__global__ __launch_bounds__(256) void k_kb_reduce(const T* __restrict__ part, int nchunk,
                                                   const T* __restrict__ h, T* __restrict__ C,
                                                   int n_proj, int k, int kp) {
  __shared__ T sum[8][32];
  const int64_t n = static_cast<int64_t>(n_proj) * kp;
  const int el = threadIdx.x & 31, g = threadIdx.x >> 5;
  for (int64_t e0 = blockIdx.x * int64_t(32); e0 < n; e0 += gridDim.x * int64_t(32)) {
    const int64_t e = e0 + el;
    const int q = static_cast<int>(e / kp), i = static_cast<int>(e - static_cast<int64_t>(q) * kp);
    T s = T(0);
    if (e < n && i < k)
#pragma unroll 4
      for (int c = g; c < nchunk; c += 8) s += part[c * n + e];
    sum[g][el] = s;
    __syncthreads();
    if (g == 0 && e < n) {
#pragma unroll
      for (int j = 1; j < 8; ++j) s += sum[j][el];
      C[e] = h[q] * s;
    }
    __syncthreads();
  }
}

struct KbGrid {
  int nM, nN, nchunk;
  int64_t kchunk;
};

// Workgroups of a split-K grid with nchunk chunks: 8 XCDs x their largest
// group count x nN, with whole chunks per XCD (xcd_chunk) or groups dealt
// round-robin.
inline unsigned kb_workgroups(int nchunk, int nM, int nN, bool xcd_chunk) {
  const int per_xcd = xcd_chunk ? (nchunk + 7) / 8 * nM : (nchunk * nM + 7) / 8;
  return static_cast<unsigned>(8 * per_xcd * nN);
}

// Split-K grid of tiles BM x BN and KB alpha per step with 8 c chunks, c per
// XCD: the c that minimises rounds x (steps per chunk + 4), with rounds of
// `slots` resident workgroups per XCD and about 4 steps' time to start and
// end a chunk, plus the partial sums' traffic (an element written and read
// costs about 1 / 1.5 M of a step).  Few tiles (small blocks or few
// projectors) take many short chunks, so that every CU has work: 13
// projectors x 4 columns, d = 162,000: 32 chunks of 158 steps left 7/8 of the
// chip idle.  At most `room` chunks, what the partial sums' buffer holds.
KbGrid kb_grid_for(int BM, int BN, int KB, int slots, int n_proj, int k, int64_t d, int64_t room) {
  KbGrid gr;
  gr.nM = (n_proj + BM - 1) / BM;
  gr.nN = (k + BN - 1) / BN;
  const int64_t steps = (d + KB - 1) / KB;
  const double elems = double(n_proj) * gr.nN * BN;
  int c_best = 1;
  double best = 1e300;
  for (int c = 1; c <= kKbMaxPerXcd; ++c) {
    const int64_t per = (steps + 8 * c - 1) / (8 * c);   // steps per chunk
    if (c > 1 && (per < 4 || 8 * c > room)) break;
    const int64_t rounds = (int64_t(c) * gr.nM * gr.nN + slots - 1) / slots;
    const double cost = double(rounds) * double(per + 4) + 8.0 * c * elems / 1.5e6;
    if (cost < best) {
      best = cost;
      c_best = c;
    }
  }
  const int64_t want = std::max<int64_t>(1, std::min({int64_t(8) * c_best, steps, room}));
  gr.kchunk = round_up((d + want - 1) / want, KB);
  gr.nchunk = static_cast<int>((d + gr.kchunk - 1) / gr.kchunk);   // <= want
  return gr;
}
template <typename S>
KbGrid kb_grid(int n_proj, int k, int64_t d, int64_t room) {
  return kb_grid_for(32 * S::TM, 32 * S::TN, S::KB, kKbPerXcd, n_proj, k, d, room);
}
KbGrid kb_split_grid(int n_proj, int k, int64_t d, int64_t room) {
  // one workgroup per CU
  return kb_grid_for(kSplitM, kSplitN, kSplitK, 32, n_proj, k, d, room);
}

// Chunks the partial sums' own region is sized for: 8 c, c <= 4 such that an
// XCD's c nM nN workgroups fill whole rounds of kKbPerXcd as nearly as
// possible, of at least 16 steps.
template <typename S>
int64_t kb_region_chunks(int n_proj, int k, int64_t d) {
  constexpr int KB = S::KB;
  const int64_t nM = (n_proj + 32 * S::TM - 1) / (32 * S::TM);
  const int64_t nN = (k + 32 * S::TN - 1) / (32 * S::TN);
  const int64_t steps = (d + KB - 1) / KB;
  int c_best = 1;
  double waste_best = 2.0;
  for (int c = 1; c <= 4; ++c) {
    if (c > 1 && steps < int64_t(8 * c) * 16) break;
    const int64_t wg = c * nM * nN;
    const int64_t rounds = (wg + kKbPerXcd - 1) / kKbPerXcd;
    const double waste = double(rounds * kKbPerXcd - wg) / double(rounds * kKbPerXcd);
    if (waste < waste_best - 1e-9) {
      waste_best = waste;
      c_best = c;
    }
  }
  const int64_t want = std::max<int64_t>(1, std::min<int64_t>(8 * c_best, steps));
  const int64_t kchunk = round_up((d + want - 1) / want, KB);
  return (d + kchunk - 1) / kchunk;
}

// FP32 products with at least 96 projectors and more than 128 columns run on
// the split kernels when the contraction is long or the product large.  Below,
// their 256 x 256 tiles are mostly padding (d = 162,000, C and Z = P C in us,
// FP32 | split: 192 projectors, k = 128: 168, 97 | 166, 110; k = 200: 218, 150 |
// 168, 116; 64 projectors, k = 200: 160, 70 | 158, 54; 512, k = 512: 716, 706 |
// 411, 467) or too few: one workgroup per CU, d / 256 x k / 256 of them for Z
// (H X with k = 256 columns, time of the split kernels over the FP32 ones: 300
// projectors, d = 972 1.14, 8,000 1.23, 12,500 1.15, 19,220 1.00, 50,430 0.90; 1236
// projectors, d = 2,023 1.02, 8,000 1.00, 12,500 0.91, 50,430 0.69; over 600 sizes the
// rule costs 0.5 % more than the faster kernel of each, 15 % at most).
inline bool kb_split(int n_proj, int k, int64_t d) {
  return n_proj >= 96 && k > 128 && (d >= 15000 || double(d) * k * n_proj >= 1.5e9);
}

// FP64 C = P^T Y on 128 x 128 tiles (KgWide64) for long contractions whose
// columns fill them as well as 64-wide ones (an even number of 64-column
// tiles).  C in us, 128 x 64 | 128 x 128 tiles: d = 984,150, 1236 projectors,
// k = 250: 11,620 | 10,440; d = 162,000, k = 256: 192 projectors 382 | 372, 512
// 751 | 731; k = 400 (7 tiles against 4): 300 projectors 971 | 1132.  Below d =
// 100,000 the shorter chunks' starts outweigh it more often than not (d =
// 12,000, 256 projectors, k = 256: 46 | 52; whole H X on small grids, time of the wide tiles
// over the others: d = 33,620, k = 256, 96 projectors 1.03, 700 1.09, 1236 0.97; d =
// 57,132, 300 projectors, k = 128 1.21, k = 256 0.98, 1236, k = 500 0.99).  The
// 309-atom product fetches 74.8 GB with it against 65.0 (P and Y once: 17.6):
// its chunks share less in an XCD's L2, and it is bound by the matrix cores.
inline bool kb_wide64(int n_proj, int k, int64_t d) {
  return d >= 100000 && n_proj >= 96 && (k + 63) / 64 % 2 == 0;
}

}  // namespace

// The partial sums' own region of a product with up to k columns: the chunk
// count grows as the column count falls, so the largest need over every width
// <= k (a narrower call, e.g. a Lanczos vector or the last column chunk).  The
// grids above ask for up to 512 chunks (1130 MiB at 1236 projectors, k = 1000,
// against 270 MiB here); a product gets them in a buffer that is idle while it
// runs, and takes fewer where no buffer is larger than this region.
size_t kb_partial_bytes(int n_proj, int k, int64_t d) {
  if (n_proj <= 0) return 0;
  size_t most = 0;
  // the grids depend on kc through ceil(kc / 64) at most
  for (int kc = std::min(k, 64);; kc = std::min(kc + 64, k)) {
    const size_t kp = size_t(round_up(kc, kColPad));
    const size_t c32 = size_t(std::max(kb_region_chunks<KgVec>(n_proj, kc, d),
                                       kb_region_chunks<KbShape<float>>(n_proj, kc, d))) *
                       sizeof(float);
    const size_t c64 = size_t(kb_region_chunks<KbShape<double>>(n_proj, kc, d)) * sizeof(double);
    most = std::max(most, std::max(c32, c64) * size_t(n_proj) * kp);
    if (kc == k) break;
  }
  return most;
}

// LDS bytes of the projector kernels: one (A tile + B tile) stage, or two when
// double-buffered.  Measured on MI355X (309-atom shape, 32 alpha per step
// from 4-byte loads): double buffering took the FP32 C = P^T Y product from
// 28.3 to 25.4 ms and made P C slower
// (22.3 -> 24.3 ms), so only the former uses it (2 x 33.8 KB, two workgroups
// per CU still fit).
template <typename T>
constexpr size_t kb_lds_bytes(bool db, int kb = KbShape<T>::KB) {
  return (db ? 2 : 1) * size_t(32 * KbShape<T>::TM + 32 * KbShape<T>::TN) * kb_pitch<T>(kb) * sizeof(T);
}
template <typename T, typename S>
constexpr size_t kg_lds_bytes(bool db, int vw) {
  return (db ? 2 : 1) * size_t(32 * S::TM + 32 * S::TN) * kb_pitch<T>(S::KB, vw) * sizeof(T);
}

// Allow more than the default 64 KB of dynamic LDS for a kernel that needs it
// (set per kernel on each launch: no process-wide state).
template <typename K>
void allow_lds(K kern, size_t bytes) {
  if (bytes > 65536)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                              hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
}

template <typename T>
void launch_kb_gemm(const T* P, int64_t d, int64_t ldp, const T* Y, int64_t ldy, const T* h,
                    T* C, T* part, size_t part_elems, int n_proj, int k, int kp, hipStream_t s) {
  const int64_t room = static_cast<int64_t>(part_elems / (size_t(n_proj) * kp));
  int nchunk = 0;
  auto go = [&](auto shape, auto db, auto vw) {
    typedef decltype(shape) S;
    constexpr bool DB = decltype(db)::value;
    constexpr int VW = decltype(vw)::value;
    const KbGrid gr = kb_grid<S>(n_proj, k, d, room);
    const bool xc = gr.nchunk % 8 == 0;
    const unsigned nwg = kb_workgroups(gr.nchunk, gr.nM, gr.nN, xc);
    constexpr size_t lds = kg_lds_bytes<T, S>(DB, VW);
    allow_lds(&k_kb_gemm<T, DB, S, VW>, lds);
    k_kb_gemm<T, DB, S, VW><<<nwg, 256, lds, s>>>(P, d, ldp, Y, ldy, part, n_proj, k, kp,
                                                   gr.kchunk, gr.nM, gr.nN, gr.nchunk, xc ? 1 : 0);
    nchunk = gr.nchunk;
  };
  if constexpr (sizeof(T) == 4) {
    if (kb_split(n_proj, k, d) && ldp % 4 == 0 && ldy % 4 == 0 &&
        reinterpret_cast<uintptr_t>(P) % 16 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0) {
      const KbGrid gr = kb_split_grid(n_proj, k, d, room);
      allow_lds(&k_kb_gemm_split, kSplitLds);
      k_kb_gemm_split<<<8 * ((gr.nchunk + 7) / 8) * gr.nM * gr.nN, 512, kSplitLds, s>>>(
          P, d, ldp, Y, ldy, part, n_proj, k, kp, gr.kchunk, gr.nM, gr.nN, gr.nchunk);
      nchunk = gr.nchunk;
    } else if (ldp % 4 == 0 && ldy % 4 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0 &&
        reinterpret_cast<uintptr_t>(Y) % 16 == 0)
      go(KgVec{}, std::false_type{}, std::integral_constant<int, 4>{});
    else
      go(KbShape<float>{}, std::true_type{}, std::integral_constant<int, 1>{});
  } else {
    const bool vec = ldp % 2 == 0 && ldy % 2 == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(Y) % 16 == 0;
    if (vec && kb_wide64(n_proj, k, d))
      go(KgWide64{}, std::true_type{}, std::integral_constant<int, 2>{});
    else if (vec)
      go(KbShape<double>{}, std::false_type{}, std::integral_constant<int, 2>{});
    else
      go(KbShape<double>{}, std::false_type{}, std::integral_constant<int, 1>{});
  }
  const int64_t n = int64_t(n_proj) * kp;
  const unsigned rb = static_cast<unsigned>(std::min<int64_t>((n + 31) / 32, 8192));
  k_kb_reduce<T><<<rb, 256, 0, s>>>(part, nchunk, h, C, n_proj, k, kp);
}

int launch_atb_partial(const double* A, int64_t lda, const double* B, int64_t ldb, double* part,
                       int64_t part_cap, int64_t rows, int k, int kp, hipStream_t s) {
  // the projector product's split-K grid, with no more chunks than `part` holds
  const KbGrid gr =
      kb_grid<KbShape<double>>(k, k, rows, part_cap / (static_cast<int64_t>(k) * kp));
  const bool xc = gr.nchunk % 8 == 0;
  const unsigned nwg = kb_workgroups(gr.nchunk, gr.nM, gr.nN, xc);
  auto run = [&](auto vw) {
    constexpr int VW = decltype(vw)::value;
    k_kb_gemm<double, false, KbShape<double>, VW>
        <<<nwg, 256, kg_lds_bytes<double, KbShape<double>>(false, VW), s>>>(
            A, rows, lda, B, ldb, part, k, k, kp, gr.kchunk, gr.nM, gr.nN, gr.nchunk, xc ? 1 : 0);
  };
  if (lda % 2 == 0 && ldb % 2 == 0 && reinterpret_cast<uintptr_t>(A) % 16 == 0 &&
      reinterpret_cast<uintptr_t>(B) % 16 == 0)
    run(std::integral_constant<int, 2>{});
  else
    run(std::integral_constant<int, 1>{});
  return gr.nchunk;
}

template <typename T>
void launch_kb_apply(const T* P, int64_t d, int64_t ldp, const T* C, T* Z, int n_proj, int k,
                     int kp, hipStream_t s) {
  if constexpr (sizeof(T) == 4) {
    if (kb_split(n_proj, k, d)) {
      const int nI = (k + kSplitM - 1) / kSplitM;
      const int nA = static_cast<int>((d + kSplitN - 1) / kSplitN);
      allow_lds(&k_kb_apply_split, kSplitLds);
      k_kb_apply_split<<<8 * ((nA + 7) / 8) * nI, 512, kSplitLds, s>>>(P, d, ldp, C, n_proj, k, kp,
                                                                       Z, nI, nA);
      return;
    }
  }
  // wide tiles when the 16-byte column loads stay aligned
  constexpr int VW = 16 / static_cast<int>(sizeof(T));
  if (ldp % VW == 0 && kp % VW == 0 && reinterpret_cast<uintptr_t>(P) % 16 == 0 &&
      reinterpret_cast<uintptr_t>(C) % 16 == 0) {
    constexpr int BI = 32 * ApShape<T>::TI, BA = 32 * ApShape<T>::TA;
    const int nI = (k + BI - 1) / BI;
    const int nA = static_cast<int>((d + BA - 1) / BA);
    const unsigned nwg = static_cast<unsigned>(8 * ((nA + 7) / 8) * nI);
    constexpr size_t lds = kb_apply_wide_lds<T>();
    allow_lds(&k_kb_apply_wide<T>, lds);
    k_kb_apply_wide<T><<<nwg, 256, lds, s>>>(P, d, ldp, C, n_proj, k, kp, Z, nI, nA);
    return;
  }
  constexpr int BM = 32 * KbShape<T>::TN, BN = 32 * KbShape<T>::TM;
  const int nI = (k + BM - 1) / BM;
  const int nA = static_cast<int>((d + BN - 1) / BN);
  const unsigned nwg = static_cast<unsigned>(8 * ((nA + 7) / 8) * nI);
  constexpr int KBA = KbShape<T>::KB;   // projectors per staged step
  constexpr size_t lds = kb_lds_bytes<T>(false, KBA);
  allow_lds(&k_kb_apply<T, false, KBA>, lds);
  k_kb_apply<T, false, KBA><<<nwg, 256, lds, s>>>(P, d, ldp, C, n_proj, k, kp, Z, nI, nA);
}

template void launch_kb_apply<float>(const float*, int64_t, int64_t, const float*, float*, int,
                                     int, int, hipStream_t);
template void launch_kb_apply<double>(const double*, int64_t, int64_t, const double*, double*,
                                      int, int, int, hipStream_t);
template void launch_kb_gemm<float>(const float*, int64_t, int64_t, const float*, int64_t,
                                    const float*, float*, float*, size_t, int, int, int, hipStream_t);
template void launch_kb_gemm<double>(const double*, int64_t, int64_t, const double*, int64_t,
                                     const double*, double*, double*, size_t, int, int, int,
                                     hipStream_t);

}  // namespace ces
