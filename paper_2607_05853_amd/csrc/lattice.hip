// The TDA Hamiltonian over lattice vectors (FP64 plans with k-independent C^mu and real W(R)).
//
// With W(q) = sum_R W(R) exp(2 pi i q.R) on a short set of R and M^mu_ij(k, k') = psi_i(k)^H C^mu psi_j(k'), the
// sum over k' of the direct term separates:
//   D(k)_tt'   = sum_v'c' conj(psi_v'(k)_t) psi_c'(k)_t' X(k)_c'v'
//   D(R)       = sum_k exp(2 pi i k.R) D(k)
//   G^nu_ts    = sum_mu C^mu_ts W(R)_munu           per R, real W
//   U^nu_ts'   = sum_t' C^nu_s't' D(R)_tt'          per R
//   F(R)_ss'   = sum_nu,t G^nu_ts U^nu_ts'          per R
//   F(k)       = sum_R exp(-2 pi i k.R) F(R)
//   Y(k)_cv    = (E_c - E_v) X - (1/N_k) sum_ss' conj(psi_c(k)_s') psi_v(k)_s F(k)_ss'
// Its work grows with N_R n_b instead of N_k^2.  The exchange term is a change of F at R = 0,
//   t^nu = sum_tt' C^nu_tt' D(0)_tt' = sum_t U^nu_tt(0),   F(0)_ss' -= alpha sum_munu C^mu_s's Vbar_munu t^nu.
// Where they fit, the plan keeps the kernels
//   K(R)_ss',tt' = sum_munu C^mu_ts W(R)_munu C^nu_s't',   F(R) = K(R) D(R)
// instead (exchange in K(0)): 16 N_ao^4 bytes per R, of which Hermiticity and W(-R) = W(R)^T leave a quarter, read
// once per eight vectors, in place of 16 N_aux N_ao^3 n_b + 4 N_aux^2 N_ao^2 operations per R.  One application,
// pair route -> contractions -> kernels: 8x8x8, N_ao 64, N_aux 256, n_v 4, n_c 8, 125 R, 8 vectors (8.5 GB of
// kernels, 26 ms to make) 83.7 -> 23.3 -> 3.6 ms; N_ao 96, 4 vectors (no room for kernels) 102 -> 46 ms; 5x6x7, N_ao 30,
// N_aux 90, 27 R, 5 vectors (95 MB) 2.19 -> 0.111 ms; 4x4x4, N_ao 16, N_aux 64, 3 vectors (8 MB) 0.305 -> 0.034 ms.
// W(R) is contracted with C^mu again in every application (G, one vector's worth of work in a batched product) as G of
// all R takes as much memory as U.  The contractions remain for kernels beyond 16 GiB, or beyond a fifth of the free memory
// with their buffers, W_q that are not Hermitian, and where they are less work.  The pair route remains for every W_q that is
// no such sum to its rounding, and where neither form finds memory.
#include "bse_internal.h"
#include "fourier.h"
#include "mfma_common.h"

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <new>

namespace bse {

struct Lattice {
  FtArgs ax;                 // the active R on the dense mesh, unit weights
  int nR = 0, r0 = 0;        // r0: index of R = 0
  bool forced = false;       // taken for every block of vectors (BSE_LATTICE)
  double* Wr = nullptr;      // [nR][n_aux][n_aux], with kernels W(R), else W(R)^T
  // constants with padded rows: n_aux n_ao doubles is often a power of two, whose rows all start in one L2 channel
  long long ldc = 0;
  double* C1 = nullptr;      // [2][t'][ldc]: (nu, s') = C^nu_s't'
  double* C3 = nullptr;      // [2][s][ldc]:  (t, mu)  = C^mu_ts
  int nbc = 0, rc = 0;       // vectors and R per pass
  double* D = nullptr;       // c128 [Nk][n_ao][nbc][n_ao], later F(k) as [Nk][nbc][n_ao][n_ao]
  double* DR = nullptr;      // [nR][2][n_ao][nbc][n_ao]
  double* U = nullptr;       // [rc][n_ao][nbc][2][n_aux][n_ao]
  double* G = nullptr;       // [rc][2][s][ldc]: (nu, t) = G^nu_ts
  double* F = nullptr;       // [split][nR][nbc][2][n_ao][n_ao]
  long long f_doubles = 0;
  double* t = nullptr;       // c128 [n_aux][nbc]
  double* tab[2] = {};       // the axes' phases, sign +1 and -1 (ft_table_launch)
  // the Hermitian K(R) of one R of each pair (R, -R), R = 0 first: tiles (I, J), I <= J < S, at J (J + 1) / 2 + I, each
  // [re, im][16 columns][16 rows], the diagonal ones halved (half of a tile and its conjugate transpose are the tile); then
  // a tile of zeros
  double* K = nullptr;
  int nh = 0, S = 0;
  int2* pair = nullptr;      // [nh] places of R and -R in the list, the second -1 for R = 0
  double* part = nullptr;    // partial sums of lat_kx
};

namespace {

// ----------------------------------------------------------------------------
// FP64 GEMM on planar operands: C[m][n] = sum_k A[m][k] B[k][n], real, or complex with re and im planes
// ----------------------------------------------------------------------------
struct LatGemm {
  int M, N, K, Z;                       // Z batch entries
  const double* A;                      // row m at m lda, k contiguous
  long long lda, a_ps, a_z;
  const double* B;                      // row k at (k / kd) rs1 + (k % kd) rs0, column n at (n / nd) cs1 + n % nd
  int kd, nd;
  long long rs1, rs0, cs1, b_ps, b_z;
  double* C;                            // row m at m ldc, column n at (n / nd) cc1 + n % nd
  long long ldc, cc1, c_ps, c_z;
  int nsplit, klen;                     // split of K: part s covers [s klen, ..) and writes C + s c_split
  long long c_split;
  // TILED: C is one K(R) with S tiles per side.  Row m is (s, a) = rows[m], at s a_z + a lda of A; with column (b, s') it
  // is row (s, s') and column (a, b) of K(R) (swap: row (s, a), column (s', b)), times scale, on top if add
  // (rows with a >= s suffice then: the lower half of the diagonal tiles is filled in)
  const int2* rows;
  int S, swap, add;
  double scale;
};

// tiles in front of tile (I, J) of a Hermitian matrix
__device__ __forceinline__ long long lat_tile(int I, int J) { return (long long)J * (J + 1) / 2 + I; }

// 256 threads as 2 x 2 waves on a BM x BN tile, BK deep stages in two LDS buffers with the next stage's loads in
// flight during the products.  The 16x16x4 FP64 instruction takes 64 cycles and two 8-byte LDS reads feed it, so
// the tiles only have to keep the matrix cores busy: real 128 x 128 (64 x 64 per wave), complex 64 x 128 (32 x 64
// per wave and plane), both 128 accumulator registers and two blocks per CU.  LDS rows are padded so that a fragment's 64 lanes spread over the banks.
// VEC: 16-byte loads (even strides and sizes).
template <bool CPLX, int BM, int BN, int BK, bool VEC, bool TILED>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void lat_gemm(LatGemm g) {
  constexpr int NP = CPLX ? 2 : 1;
  constexpr int WM = BM / 2, WN = BN / 2, TM = WM / 16, TN = WN / 16;
  constexpr int SA = BK + 2, SB = BN + 16;
  constexpr int NA = BM * BK / 2 * NP / 256, NB = BK * BN / 2 * NP / 256;  // pairs per thread and stage
  constexpr int ASZ = NP * BM * SA, BSZ = NP * BK * SB;
  __shared__ double sm[2][ASZ + BSZ];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l4 = lane >> 4, l16 = lane & 15, wm = wave >> 1, wn = wave & 1;
  // block -> (group, m tile), a group being one n tile of one batch entry and K part: the m tiles of a group follow
  // each other on one XCD, which then reads the B panel once, and the groups go round the eight XCDs
  const int mt = (g.M + BM - 1) / BM, nt = (g.N + BN - 1) / BN;
  const unsigned id = blockIdx.x;
  const int m0 = (int)((id >> 3) % mt) * BM;
  const unsigned grp = (id >> 3) / mt * 8 + (id & 7);
  if (grp >= (unsigned)nt * g.Z * g.nsplit) return;
  const int n0 = (int)(grp % nt) * BN;
  const int z = (int)(grp / nt % g.Z), sp = (int)(grp / nt / g.Z);
  const int kbeg = sp * g.klen, kend = min(g.K, kbeg + g.klen);
  const double* A = g.A + z * g.a_z;
  const double* B = g.B + z * g.b_z;
  double* C = g.C + z * g.c_z + sp * g.c_split;

  // addresses of rows, columns or k outside the operands point at an element inside; lstore writes zeros there
  double2 ra[NA], rb[NB];
  long long ao[NA], bo[NB], bd[NB];
  int ak[NA], bk[NB], bkq[NB], bkr[NB];
  bool aok[NA], bok[NB], bok1[NB];
#pragma unroll
  for (int i = 0; i < NA; ++i) {
    const int t = tid + 256 * i, pl = t / (BM * BK / 2), u = t % (BM * BK / 2);
    const int row = m0 + u / (BK / 2);
    ak[i] = 2 * (u % (BK / 2));
    aok[i] = row < g.M;
    const int r = aok[i] ? row : 0;
    if constexpr (TILED)
      ao[i] = pl * g.a_ps + g.rows[r].x * g.a_z + g.rows[r].y * g.lda;
    else
      ao[i] = pl * g.a_ps + r * g.lda;
  }
#pragma unroll
  for (int i = 0; i < NB; ++i) {
    const int t = tid + 256 * i, pl = t / (BK * BN / 2), u = t % (BK * BN / 2);
    const int col = n0 + 2 * (u % (BN / 2));
    bk[i] = u / (BN / 2);
    bok[i] = col < g.N;
    bok1[i] = col + 1 < g.N;
    const int c = bok[i] ? col : 0, c1 = bok1[i] ? col + 1 : 0;
    bo[i] = pl * g.b_ps + (long long)(c / g.nd) * g.cs1 + c % g.nd;
    bd[i] = pl * g.b_ps + (long long)(c1 / g.nd) * g.cs1 + c1 % g.nd;
    bkq[i] = (kbeg + bk[i]) / g.kd;  // k = bkq kd + bkr, advanced by BK per stage
    bkr[i] = (kbeg + bk[i]) % g.kd;
  }
  auto gload = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int k = k0 + ak[i];
      if constexpr (VEC) {
        ra[i] = *reinterpret_cast<const double2*>(A + ao[i] + (k < kend ? k : kbeg));
      } else {
        ra[i].x = A[ao[i] + (k < kend ? k : kbeg)];
        ra[i].y = A[ao[i] + (k + 1 < kend ? k + 1 : kbeg)];
      }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const bool ok = k0 + bk[i] < kend;
      const long long ro = ok ? bkq[i] * g.rs1 + bkr[i] * g.rs0 : 0;
      if constexpr (VEC) {
        rb[i] = *reinterpret_cast<const double2*>(B + bo[i] + ro);
      } else {
        rb[i].x = B[bo[i] + ro];
        rb[i].y = B[bd[i] + ro];
      }
      bkr[i] += BK;
      while (bkr[i] >= g.kd) {
        bkr[i] -= g.kd;
        ++bkq[i];
      }
    }
  };
  const double2 zero2 = {0.0, 0.0};
  auto lstore = [&](double* s, int k0) {
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int t = tid + 256 * i, pl = t / (BM * BK / 2), u = t % (BM * BK / 2);
      const bool ok = aok[i] && k0 + ak[i] < kend;
      double2 v = ok ? ra[i] : zero2;
      if (!VEC && !(k0 + ak[i] + 1 < kend)) v.y = 0.0;
      *reinterpret_cast<double2*>(s + pl * BM * SA + (u / (BK / 2)) * SA + ak[i]) = v;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int t = tid + 256 * i, pl = t / (BK * BN / 2), u = t % (BK * BN / 2);
      const bool ok = k0 + bk[i] < kend;
      double2 v = ok && bok[i] ? rb[i] : zero2;
      if (!VEC && !bok1[i]) v.y = 0.0;
      *reinterpret_cast<double2*>(s + ASZ + pl * BK * SB + bk[i] * SB + 2 * (u % (BN / 2))) = v;
    }
  };

  d4v acc[NP][TM][TN];
#pragma unroll
  for (int p = 0; p < NP; ++p)
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[p][i][j] = d4v{0, 0, 0, 0};

  int cur = 0;
  if (kbeg < kend) gload(kbeg);
  if (kbeg < kend) lstore(sm[0], kbeg);
  __syncthreads();
  for (int k0 = kbeg; k0 < kend; k0 += BK) {
    const bool more = k0 + BK < kend;
    if (more) gload(k0 + BK);
    const double* sa = sm[cur] + (wm * WM + l16) * SA + l4;
    const double* sb = sm[cur] + ASZ + l4 * SB + wn * WN + l16;
#pragma unroll
    for (int kk = 0; kk < BK / 4; ++kk) {
      double av[NP][TM], bv[NP][TN];
#pragma unroll
      for (int p = 0; p < NP; ++p) {
#pragma unroll
        for (int i = 0; i < TM; ++i) av[p][i] = sa[p * BM * SA + i * 16 * SA + 4 * kk];
#pragma unroll
        for (int j = 0; j < TN; ++j) bv[p][j] = sb[p * BK * SB + 4 * kk * SB + j * 16];
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[0][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[0][i], bv[0][j], acc[0][i][j], 0, 0, 0);
          if constexpr (CPLX) {
            acc[1][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[0][i], bv[1][j], acc[1][i][j], 0, 0, 0);
            acc[0][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[1][i], bv[1][j], acc[0][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[1][i], bv[0][j], acc[1][i][j], 0, 0, 0);
          }
        }
    }
    if (more) lstore(sm[cur ^ 1], k0 + BK);
    cur ^= 1;
    __syncthreads();
  }
  // register q of a lane holds column l16 of tile row 4 q + l4
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int n = n0 + wn * WN + j * 16 + l16;
    if (n >= g.N) continue;
    if constexpr (TILED) {
      const int a = n % g.nd, b = n / g.nd;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int m = m0 + wm * WM + i * 16 + 4 * q + l4;
          if (m >= g.M) continue;
          const int2 r = g.rows[m];
          const int row = r.x * g.nd + (g.swap ? r.y : a), col = (g.swap ? a : r.y) * g.nd + b;
          if ((row >> 4) > (col >> 4)) continue;
          double* c = g.C + lat_tile(row >> 4, col >> 4) * 512 + (col & 15) * 16 + (row & 15);
          const bool diag = (row >> 4) == (col >> 4);
          const double f = diag ? 0.5 * g.scale : g.scale;
#pragma unroll
          for (int p = 0; p < NP; ++p) c[256 * p] = f * acc[p][i][j][q] + (g.add ? c[256 * p] : 0.0);
          if (!g.swap && r.x < r.y && diag) {  // its lower half
            c += (row & 15) * 16 + (col & 15) - ((col & 15) * 16 + (row & 15));
            c[0] = f * acc[0][i][j][q];
            c[256] = -f * acc[NP - 1][i][j][q];
          }
        }
      continue;
    }
    double* c = C + (long long)(n / g.nd) * g.cc1 + n % g.nd;
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = m0 + wm * WM + i * 16 + 4 * q + l4;
        if (m >= g.M) continue;
#pragma unroll
        for (int p = 0; p < NP; ++p) c[p * g.c_ps + m * g.ldc] = acc[p][i][j][q];
      }
  }
}

template <bool CPLX, int BM, int BN, int BK, bool TILED = false>
bse_status lat_gemm_go(const LatGemm& g, bool vec, hipStream_t st) {
  const int mt = (g.M + BM - 1) / BM, nt = (g.N + BN - 1) / BN;
  const long long groups = (long long)nt * g.Z * g.nsplit;
  const dim3 grid((unsigned)((groups + 7) / 8 * 8 * mt));
  if (vec)
    hipLaunchKernelGGL((lat_gemm<CPLX, BM, BN, BK, true, TILED>), grid, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL((lat_gemm<CPLX, BM, BN, BK, false, TILED>), grid, dim3(256), 0, st, g);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

long long tiles(const LatGemm& g, int bm, int bn) {
  return (long long)((g.M + bm - 1) / bm) * ((g.N + bn - 1) / bn) * g.Z * g.nsplit;
}

// Full-size tiles once there are enough of them to hide each other's loads (fewer if the sum is long), small shallow
// tiles (four to five blocks per CU) below and for operands of few rows: 5x6x7, N_ao 30, N_aux 90, 27 R, 5 vectors (1782
// full-size tiles of U, as many of F) 267 -> 245 us per application by contractions.  The real product, a tenth of the work, takes
// 96-row tiles where these leave less empty than 128 (245 us against 250 with 128 or 64 rows), 64 x 64 for few rows or
// tiles (8x8x8: 22.9 ms with 128 x 128, 23.1 with 64 x 64).
template <bool CPLX, bool TILED = false>
bse_status lat_gemm_run(const LatGemm& g, hipStream_t st) {
  auto even = [](long long x) { return (x & 1) == 0; };
  const bool vec = even(g.lda) && even(g.a_ps) && even(g.a_z) && even(g.K) && even(g.klen) && even(g.N) && even(g.nd) &&
                   even(g.rs0) && even(g.rs1) && even(g.cs1) && even(g.b_ps) && even(g.b_z);
  if constexpr (TILED) {
    if (tiles(g, 64, 128) >= 512) return lat_gemm_go<true, 64, 128, 8, true>(g, vec, st);
    return lat_gemm_go<true, 32, 64, 8, true>(g, vec, st);
  } else if constexpr (CPLX) {
    const long long full = tiles(g, 64, 128);
    if (g.M > 32 && (full >= 2048 || (full >= 384 && g.klen >= 1024))) return lat_gemm_go<true, 64, 128, 8>(g, vec, st);
    return lat_gemm_go<true, 32, 64, 8>(g, vec, st);
  } else {
    auto rows = [&](int bm) { return (g.M + bm - 1) / bm * bm; };
    if (g.M > 64 && tiles(g, 128, 128) >= 384) {
      if (rows(96) < rows(128)) return lat_gemm_go<false, 96, 128, 16>(g, vec, st);
      return lat_gemm_go<false, 128, 128, 16>(g, vec, st);
    }
    return lat_gemm_go<false, 64, 64, 16>(g, vec, st);
  }
}

// ----------------------------------------------------------------------------
// D(k) and Y(k): one block per (k, vector)
// ----------------------------------------------------------------------------
__device__ __forceinline__ double2 cmadd(double2 a, double2 x, double2 y) {  // a + x y
  return double2{fma(x.x, y.x, fma(-x.y, y.y, a.x)), fma(x.x, y.y, fma(x.y, y.x, a.y))};
}
__device__ __forceinline__ double2 cmaddc(double2 a, double2 x, double2 y) {  // a + conj(x) y
  return double2{fma(x.x, y.x, fma(x.y, y.y, a.x)), fma(x.x, y.y, fma(-x.y, y.x, a.y))};
}

// D[k][t][b][t'] = sum_v conj(psi_v(k)_t) Z_v t', Z_v t' = sum_c psi_c(k)_t' X(k)_cv (kept in LDS); bound by
// writing D
__global__ __launch_bounds__(256) void lat_outer(int nv, int nc, int no, int nb, int b0, int nbc,
                                                 const double* __restrict__ psi, const double* __restrict__ X,
                                                 double* __restrict__ D) {
  extern __shared__ double2 lsm[];
  const int k = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, nt = nv * nc;
  double2* const Zs = lsm;            // [nv][no]
  double2* const Xs = Zs + nv * no;   // [nc][nv]
  const double2* pk = reinterpret_cast<const double2*>(psi) + (long long)k * (nv + nc) * no;
  for (int i = tid; i < nt; i += 256) {
    const double* x = X + 2 * (((long long)k * nt + i) * nb + b0 + b);
    Xs[i] = double2{x[0], x[1]};
  }
  __syncthreads();
  for (int i = tid; i < nv * no; i += 256) {
    const int v = i / no, t = i % no;
    double2 s = {0.0, 0.0};
    for (int c = 0; c < nc; ++c) s = cmadd(s, pk[(nv + c) * no + t], Xs[c * nv + v]);
    Zs[i] = s;
  }
  __syncthreads();
  double2* Dk = reinterpret_cast<double2*>(D) + ((long long)k * no * nbc + b) * no;
  for (int i = tid; i < no * no; i += 256) {
    const int t = i / no, tp = i % no;
    double2 s = {0.0, 0.0};
    for (int v = 0; v < nv; ++v) s = cmaddc(s, pk[v * no + t], Zs[v * no + tp]);
    Dk[(long long)t * nbc * no + tp] = s;
  }
}

// Y[k][c][v][b] = (E_c - E_v) X - (1/N_k) sum_ss' conj(psi_c s') psi_v s F[k][b][s][s']: H_v s' = sum_s psi_v s F
// by 256 / n_ao groups of s, then one wave per (c, v); bound by reading F
__global__ __launch_bounds__(256) void lat_project(int nv, int nc, int no, int nb, int b0, int nbc, int groups,
                                                   double scale, const double* __restrict__ eps,
                                                   const double* __restrict__ psi, const double* __restrict__ F,
                                                   const double* __restrict__ X, double* __restrict__ Y) {
  extern __shared__ double2 lsm[];
  const int k = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, nt = nv * nc;
  double2* const H = lsm;  // [groups][nv][no]
  const double2* pk = reinterpret_cast<const double2*>(psi) + (long long)k * (nv + nc) * no;
  const double2* Fk = reinterpret_cast<const double2*>(F) + ((long long)k * nbc + b) * no * no;
  const int gr = tid / no;
  if (groups > 1 ? gr < groups : true) {
    for (int sp = groups > 1 ? tid % no : tid; sp < no; sp += 256) {
      const int s0 = groups > 1 ? gr : 0;
      for (int v0 = 0; v0 < nv; v0 += 4) {
        double2 h[4] = {};
        for (int s = s0; s < no; s += groups) {
          const double2 f = Fk[(long long)s * no + sp];
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (v0 + v < nv) h[v] = cmadd(h[v], pk[(v0 + v) * no + s], f);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (v0 + v < nv) H[(s0 * nv + v0 + v) * no + sp] = h[v];
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < nv * no; i += 256) {
    double2 s = H[i];
    for (int q = 1; q < groups; ++q) {
      const double2 h = H[q * nv * no + i];
      s.x += h.x;
      s.y += h.y;
    }
    H[i] = s;
  }
  __syncthreads();
  const int lane = tid & 63;
  for (int o = tid >> 6; o < nt; o += 4) {
    const int c = o / nv, v = o % nv;
    double2 s = {0.0, 0.0};
    for (int sp = lane; sp < no; sp += 64) s = cmaddc(s, pk[(nv + c) * no + sp], H[v * no + sp]);
    for (int w = 32; w > 0; w >>= 1) {
      s.x += __shfl_down(s.x, w);
      s.y += __shfl_down(s.y, w);
    }
    if (lane == 0) {
      const long long i = 2 * (((long long)k * nt + o) * nb + b0 + b);
      const double d = eps[(long long)k * (nv + nc) + nv + c] - eps[(long long)k * (nv + nc) + v];
      Y[i] = d * X[i] - scale * s.x;
      Y[i + 1] = d * X[i + 1] - scale * s.y;
    }
  }
}

// ----------------------------------------------------------------------------
// F(R) = K(R) D(R) and F(-R) = K(-R) D(-R) from one reading of half of K(R)
// ----------------------------------------------------------------------------
// With Hermitian C^mu and Vbar, K(R) is Hermitian, and W(-R) = W(R)^T makes K(-R)_ab,cd = K(R)_dc,ba: with
// E_dc = conj(D(-R)_cd), G = K(R) E is G_ba = conj(F(-R)_ab).  So a pair (R, -R) and nb vectors are one Hermitian
// matrix times 2 nb vectors.
struct LatKx {
  int no, w, b0, nb;       // D(R) is [2][no][w][no]; vectors b0 .. b0 + nb - 1 of w
  int S, nh, RS, panels, cl;  // tiles per side, pairs of R, row tiles per panel, panels, column tiles per block
  int blocks;              // per pair
  long long E;             // no no w
  const double* K;
  const double* zero;      // a tile of zeros, for the places of a panel below the diagonal or past the last row
  const double* DR;
  const int2* pair;
  double* PF;              // [block of the panel][nh][16 S][16 NT]: upper tiles, columns 8 re then 8 im of eight vectors
  double* PT;              // [panel][nh][16 S][16 NT]: their conjugate transposes
};

// One block per RS row tiles of a K(R) and cl of its column tiles, one column tile per wave at a time.  A wave reads
// each 16 x 16 complex tile once, a tile ahead, multiplies it with the columns' vectors and its conjugate transpose,
// turned in LDS, with the rows' vectors (in LDS); the sums of its rows stay in registers over all its column tiles,
// those of its columns over its row tiles.  Eight vectors fill the 16 columns of the FP64 instruction with real and
// imaginary parts, so a tile of 4 KiB is 16 NT instructions of 64 cycles: a CU that runs them back to back takes
// 16 / NT bytes per cycle, where its share of the memory's rate is 8 to 9.  8x8x8 workload, 8 vectors (NT = 2): 8.5 GB
// of kernels, 1.3 GB of sums and 0.135 TFLOP in 3.1 ms; matrix cores busy 66 % of it, the rest being the turn through
// LDS, the columns' vectors and the block's start and end (1.1 ms with all loads from a cache).
template <int RS, int NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void lat_kx(LatKx g) {
  constexpr int N = 16 * NT, TS = 18;
  __shared__ double dt[RS * 16 * N];
  __shared__ double turn[4][2][16 * TS];
  const int tid = threadIdx.x, lane = tid & 63, l4 = lane >> 4, l16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // each XCD takes an eighth of the blocks, in order: D(R) then stays in its L2 while it works on that R
  const unsigned all = (unsigned)g.nh * g.blocks, per = (all + 7) / 8, id = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (id >= all) return;
  const int h = (int)(id / g.blocks), no2 = g.no * g.no;
  int panel = 0, c = (int)(id % g.blocks);  // block c of the panel
  for (int n; c >= (n = (g.S - panel * RS + g.cl - 1) / g.cl); ++panel) c -= n;
  const int i0 = panel * RS, ns = min(RS, g.S - i0);
  const int c1 = min(g.S, i0 + (c + 1) * g.cl);
  const int2 pr = g.pair[h];
  const double* K = g.K + (long long)h * (g.S * (long long)(g.S + 1) / 2) * 512;
  double tr[2][4], ti[2][4];
  auto load = [&](int slot, int ct, int s) {
    const double* p = s < ns && i0 + s <= ct ? K + lat_tile(i0 + s, ct) * 512 : g.zero;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      tr[slot][q] = p[q * 64 + lane];
      ti[slot][q] = p[256 + q * 64 + lane];
    }
  };
  int ct = i0 + c * g.cl + wave;
  if (ct < c1) load(0, ct, 0);
  // element e = (a, b) of vector v (D(R), then E) is D[e / no * s1 + e % no * s2], im g.E behind
  auto vec = [&](int v, int* s1, int* s2) {
    const bool plus = v < g.nb;
    *s1 = plus ? g.w * g.no : 1;
    *s2 = plus ? 1 : g.w * g.no;
    return g.DR + 2 * g.E * (plus ? pr.x : max(pr.y, 0)) + (g.b0 + (plus ? v : v - g.nb)) * g.no;
  };
  const int nvec = pr.y >= 0 ? 2 * g.nb : g.nb;
  {
    const int n = tid % N, v = (n >> 4) * 8 + (n & 7);
    int s1, s2;
    const double* d = vec(min(v, nvec - 1), &s1, &s2) + (n & 8 ? g.E : 0);
    const double f = (n & 8) && v >= g.nb ? -1.0 : 1.0;
    double x[4];
    static_assert(RS * N % 64 == 0, "four elements per thread at a time");
    for (int i = 0; i < RS * 16 * N; i += 4 * 256) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = i0 * 16 + (i + k * 256 + tid) / N;
        x[k] = d[e < no2 ? e / g.no * s1 + e % g.no * s2 : 0];
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int e = i0 * 16 + (i + k * 256 + tid) / N;
        dt[i + k * 256 + tid] = e < no2 && v < nvec ? f * x[k] : 0.0;
      }
    }
  }
  __syncthreads();
  d4v acc[RS][NT];
#pragma unroll
  for (int s = 0; s < RS; ++s)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[s][t] = d4v{0, 0, 0, 0};
  double* const tu = turn[wave][0];
  const double sign = l16 < 8 ? 1.0 : -1.0;
  for (; ct < c1; ct += 4) {
    const int next = ct + 4 < c1 ? ct + 4 : ct;
    double b1[NT][4], b2[NT][4];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const int v = 8 * j + (l16 & 7);
      int s1, s2;
      const double* d = vec(min(v, nvec - 1), &s1, &s2);
      const double im = v < g.nb ? 1.0 : -1.0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = ct * 16 + 4 * q + l4;
        const bool ok = e < no2 && v < nvec;
        const int o = ok ? e / g.no * s1 + e % g.no * s2 : 0;
        const double x = d[o], y = im * d[g.E + o];
        b1[j][q] = ok ? (l16 < 8 ? x : y) : 0.0;
        b2[j][q] = ok ? (l16 < 8 ? -y : x) : 0.0;
      }
    }
    d4v at[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) at[j] = d4v{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < RS; ++s) {
      const int sl = s & 1;
      if (s + 1 < RS)
        load(sl ^ 1, ct, s + 1);
      else
        load(sl ^ 1, next, 0);
      // turned: the buffer is the wave's own, whose LDS accesses run in order; the fences only hold the compiler
      double ar[4], ai[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        tu[(4 * q + l4) * TS + l16] = tr[sl][q];
        tu[16 * TS + (4 * q + l4) * TS + l16] = ti[sl][q];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        ar[q] = tu[l16 * TS + 4 * q + l4];
        ai[q] = tu[16 * TS + l16 * TS + 4 * q + l4];
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          acc[s][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(tr[sl][q], b1[j][q], acc[s][j], 0, 0, 0);
          acc[s][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ti[sl][q], b2[j][q], acc[s][j], 0, 0, 0);
        }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double* d = dt + (s * 16 + 4 * q + l4) * N;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
          at[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[q], d[16 * j + l16], at[j], 0, 0, 0);
          at[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(ai[q], sign * d[16 * j + (l16 ^ 8)], at[j], 0, 0, 0);
        }
      }
    }
    double* o = g.PT + (((long long)panel * g.nh + h) * g.S + ct) * 16 * N;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int j = 0; j < NT; ++j) o[(4 * q + l4) * N + 16 * j + l16] = at[j][q];
  }
  // the four waves' rows added in order
  for (int v = 0; v < 4; ++v) {
    __syncthreads();
    if (wave == v) {
#pragma unroll
      for (int s = 0; s < RS; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
          for (int j = 0; j < NT; ++j) {
            const int i = (s * 16 + 4 * q + l4) * N + 16 * j + l16;
            dt[i] = v ? dt[i] + acc[s][j][q] : acc[s][j][q];
          }
    }
  }
  __syncthreads();
  double* o = g.PF + (((long long)c * g.nh + h) * g.S + i0) * 16 * N;
  for (int i = tid; i < ns * 16 * N; i += 256) o[i] = dt[i];
}

// F from the partial sums, F(R)_ab at row (a, b) and conj F(-R)_ab at row (b, a): block (16 b of an a; pair and sign;
// eight vectors) of 16 rows x 16 columns, turned in LDS so that F [R][vector][2][a][b] is written in runs of b
__global__ __launch_bounds__(256) void lat_kx_sum(LatKx g, int N, double* __restrict__ F) {
  __shared__ double x[16][17];
  const int bl = (g.no + 15) / 16;
  const int a = blockIdx.x / bl, b = blockIdx.x % bl * 16 + (threadIdx.x >> 4);
  const int h = blockIdx.y >> 1, minus = blockIdx.y & 1, n = threadIdx.x & 15;
  const int2 pr = g.pair[h];
  const int R = minus ? pr.y : pr.x, v0 = blockIdx.z * 8 - (minus ? g.nb : 0);  // vector of column 0
  if (R < 0 || v0 + 7 < 0 || v0 >= g.nb) return;
  const long long rows = 16ll * g.S, step = (long long)g.nh * rows * N;
  double s = 0.0;
  if (b < g.no && (unsigned)(v0 + (n & 7)) < (unsigned)g.nb) {
    const int e = minus ? b * g.no + a : a * g.no + b, panel = (e >> 4) / g.RS;
    const long long o = (h * rows + e) * N + blockIdx.z * 16 + n;
    const int nf = (g.S - panel * g.RS + g.cl - 1) / g.cl;
#pragma unroll 4
    for (int i = 0; i < nf; ++i) s += g.PF[o + i * step];
#pragma unroll 4
    for (int i = 0; i <= panel; ++i) s += g.PT[o + i * step];
  }
  x[n][threadIdx.x >> 4] = minus && (n & 8) ? -s : s;
  __syncthreads();
  const int m = threadIdx.x >> 4, v = v0 + (m & 7), bo = blockIdx.x % bl * 16 + (threadIdx.x & 15);
  if ((unsigned)v < (unsigned)g.nb && bo < g.no)
    F[2 * g.E * R + ((long long)(g.b0 + v) * 2 + (m >> 3)) * g.no * g.no + a * g.no + bo] = x[m][threadIdx.x & 15];
}

// ----------------------------------------------------------------------------
// exchange term
// ----------------------------------------------------------------------------
__device__ __forceinline__ void wave_sum(double2& s) {
  for (int w = 32; w > 0; w >>= 1) {
    s.x += __shfl_down(s.x, w);
    s.y += __shfl_down(s.y, w);
  }
}

// t^nu = sum_t U^nu_tt(0), block (nu, b) of one wave
__global__ __launch_bounds__(64) void lat_ex_t(int na, int no, int nbc, const double* __restrict__ U0,
                                               double* __restrict__ t) {
  const int nu = blockIdx.x, b = blockIdx.y;
  const long long pl = (long long)na * no;
  double2 s = {0.0, 0.0};
  for (int a = threadIdx.x; a < no; a += 64) {
    const double* u = U0 + ((long long)a * nbc + b) * 2 * pl + (long long)nu * no + a;
    s.x += u[0];
    s.y += u[pl];
  }
  wave_sum(s);
  if (threadIdx.x == 0) {
    t[2 * (nu * nbc + b)] = s.x;
    t[2 * (nu * nbc + b) + 1] = s.y;
  }
}

// u^mu = alpha sum_nu Vbar_munu t^nu, block (mu, b) of one wave
__global__ __launch_bounds__(64) void lat_ex_u(int na, int nbc, double alpha, const double* __restrict__ vbar,
                                               const double* __restrict__ t, double* __restrict__ u) {
  const int mu = blockIdx.x, b = blockIdx.y;
  double2 s = {0.0, 0.0};
  for (int nu = threadIdx.x; nu < na; nu += 64) {
    const double* v = vbar + 2 * ((long long)mu * na + nu);
    s = cmadd(s, double2{v[0], v[1]}, double2{t[2 * (nu * nbc + b)], t[2 * (nu * nbc + b) + 1]});
  }
  wave_sum(s);
  if (threadIdx.x == 0) {
    u[2 * (b * na + mu)] = alpha * s.x;
    u[2 * (b * na + mu) + 1] = alpha * s.y;
  }
}

// F(0)_ss' -= sum_mu C^mu_s's u^mu, block (64 s', s, b): four waves share the mu
__global__ __launch_bounds__(256) void lat_ex_f(int na, int no, long long ldc, const double* __restrict__ C1,
                                                const double* __restrict__ u, double* __restrict__ F0) {
  __shared__ double2 red[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, s = blockIdx.y, b = blockIdx.z;
  const int sp = blockIdx.x * 64 + lane;
  double2 x = {0.0, 0.0};
  if (sp < no) {
    const double* c = C1 + s * ldc + sp;
    for (int mu = wave; mu < na; mu += 4)
      x = cmadd(x, double2{c[(long long)mu * no], c[no * ldc + (long long)mu * no]},
                double2{u[2 * (b * na + mu)], u[2 * (b * na + mu) + 1]});
  }
  red[wave][lane] = x;
  __syncthreads();
  if (wave || sp >= no) return;
  double* f = F0 + ((long long)b * 2 * no + s) * no + sp;
  f[0] -= red[0][lane].x + red[1][lane].x + red[2][lane].x + red[3][lane].x;
  f[(long long)no * no] -= red[0][lane].y + red[1][lane].y + red[2][lane].y + red[3][lane].y;
}

// ----------------------------------------------------------------------------
// plan construction
// ----------------------------------------------------------------------------
// max |re| and max |im| of each matrix of Wb [nbox][n] c128, as bits of non-negative doubles
__global__ void lat_absmax(long long n, const double* __restrict__ W, unsigned long long* __restrict__ out) {
  const double2* w = reinterpret_cast<const double2*>(W) + blockIdx.y * n;
  double mr = 0.0, mi = 0.0;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const double2 v = w[i];
    mr = max_or_nan(mr, fabs(v.x));
    mi = max_or_nan(mi, fabs(v.y));
  }
  for (int o = 32; o > 0; o >>= 1) {
    mr = max_or_nan(mr, __shfl_down(mr, o));
    mi = max_or_nan(mi, __shfl_down(mi, o));
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMax(&out[2 * blockIdx.y], (unsigned long long)__double_as_longlong(mr));
    atomicMax(&out[2 * blockIdx.y + 1], (unsigned long long)__double_as_longlong(mi));
  }
}

// Wr[j] = Re W[idx[j]] and the same with a zero imaginary part in place (for the check)
__global__ void lat_take_real(long long n, const int* __restrict__ idx, const double* __restrict__ W,
                              double* __restrict__ Wr, double* __restrict__ Wc) {
  const int j = blockIdx.y;
  const double2* w = reinterpret_cast<const double2*>(W) + idx[j] * n;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    const double v = w[i].x;
    Wr[j * n + i] = v;
    reinterpret_cast<double2*>(Wc)[j * n + i] = double2{v, 0.0};
  }
}

// largest |W(R)_ij - W(-R)_ji| of the pairs (R = 0 with itself), as bits; 16 x 16 elements per block
__global__ __launch_bounds__(256) void lat_asym(int na, const int2* __restrict__ pair, int r0,
                                                const double* __restrict__ Wr, unsigned long long* __restrict__ out) {
  __shared__ double x[16][17];
  const int2 pr = pair[blockIdx.z];
  const double* w = Wr + (long long)pr.x * na * na;
  const double* v = Wr + (long long)(pr.y < 0 ? r0 : pr.y) * na * na;
  const int a = threadIdx.x >> 4, b = threadIdx.x & 15, i0 = blockIdx.x * 16, j0 = blockIdx.y * 16;
  x[a][b] = j0 + a < na && i0 + b < na ? v[(long long)(j0 + a) * na + i0 + b] : 0.0;
  __syncthreads();
  double m = i0 + a < na && j0 + b < na ? fabs(w[(long long)(i0 + a) * na + j0 + b] - x[b][a]) : 0.0;
  for (int o = 32; o > 0; o >>= 1) m = max_or_nan(m, __shfl_down(m, o));
  const unsigned long long bits = (unsigned long long)__double_as_longlong(m);
  if ((threadIdx.x & 63) == 0 && bits > *(volatile unsigned long long*)out) atomicMax(out, bits);
}

// each [na][na] matrix transposed in place, a pair of 16 x 16 tiles per block
__global__ __launch_bounds__(256) void lat_transpose(int na, double* __restrict__ W) {
  if (blockIdx.x > blockIdx.y) return;
  __shared__ double x[16][17], y[16][17];
  double* w = W + (long long)blockIdx.z * na * na;
  const int a = threadIdx.x >> 4, b = threadIdx.x & 15, i = blockIdx.x * 16, j = blockIdx.y * 16;
  const bool u = i + a < na && j + b < na, l = j + a < na && i + b < na;
  if (u) x[a][b] = w[(long long)(i + a) * na + j + b];
  if (l) y[a][b] = w[(long long)(j + a) * na + i + b];
  __syncthreads();
  if (u) w[(long long)(i + a) * na + j + b] = y[b][a];
  if (l) w[(long long)(j + a) * na + i + b] = x[b][a];
}

// planes of re and im
__global__ void lat_planes(long long n, const double* __restrict__ A, double* __restrict__ P) {
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    P[i] = A[2 * i];
    P[n + i] = A[2 * i + 1];
  }
}

__global__ void lat_pack_C(int na, int no, long long ldc, const double* __restrict__ C, double* __restrict__ C1,
                           double* __restrict__ C3) {
  const long long n = (long long)na * no * no;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (long long)gridDim.x * blockDim.x) {
    // C[mu][s][t]; C1[t'][nu][s'] = C^nu_s't', C3[s][t][mu] = C^mu_ts
    const int t = (int)(i % no), s = (int)((i / no) % no), mu = (int)(i / ((long long)no * no));
    const long long i1 = t * ldc + (long long)mu * no + s, i3 = t * ldc + (long long)s * na + mu;
    const double re = C[2 * i], im = C[2 * i + 1];
    C1[i1] = re;
    C1[no * ldc + i1] = im;
    C3[i3] = re;
    C3[no * ldc + i3] = im;
  }
}

size_t lds_outer(const Plan* p) { return 16 * ((size_t)p->d.nv * p->d.n_ao + (size_t)p->nt); }
int project_groups(const Plan* p) { return p->d.n_ao <= 256 ? 256 / p->d.n_ao : 1; }
size_t lds_project(const Plan* p) { return 16 * (size_t)project_groups(p) * p->d.nv * p->d.n_ao; }

struct Tmp {
  void* p = nullptr;
  ~Tmp() { dfree(p); }
};

// seconds of the matrix work of one application over pairs of k, over nR lattice vectors by contractions, and over
// kernels K(R); the rates are those of the 8x8x8 workload (N_ao 64, N_aux 256, n_v 4, n_c 8, 125 R, 8 vectors), whose
// pair route has GEMMs of a few rows per pair
double secs_pairs(const Plan* p) {
  const double na = p->d.n_aux, no = p->d.n_ao, nv = p->d.nv, nc = p->d.nc;
  return 8.0 * p->Nk * p->nhalf * (na * no * (nv * nv + nc * nc) + na * na * nv * nv + na * nv * nv * nc * nc) / 37e12;
}
double secs_gemm(const Plan* p, int nR, int nb) {
  const double na = p->d.n_aux, no = p->d.n_ao;
  return nR * (nb * 16.0 * na * no * no * no + 4.0 * na * na * no * no) / 56e12;
}
int kx_tiles(const Plan* p) { return (p->d.n_ao * p->d.n_ao + 15) / 16; }
size_t kx_bytes(const Plan* p, int nh) { return (size_t)kx_tiles(p) * (kx_tiles(p) + 1) / 2 * 4096 * nh; }
double secs_kernel(const Plan* p, int nR, int nb) {
  const double b = (double)kx_bytes(p, (nR + 1) / 2);
  return (nb / 8 + (nb % 8 > 4)) * b / 3.2e12 + (nb % 8 && nb % 8 <= 4 ? b / 4e12 : 0.0);
}

struct KxShape {
  int RS, NT, panels, cl, blocks, most;
  size_t doubles(int nh, int S) const { return (size_t)(most + panels) * nh * S * 256 * NT; }
};
// NT: 2 nb vectors in groups of eight.  Rows per block: 16 NT = 1 or 8 NT = 2 tiles (the same registers; the sums of the
// columns go through memory once per panel), 4 where that leaves CUs idle.  Columns per block: about 2 MiB of tiles,
// less until there are 1024 blocks.
KxShape kx_shape(int nh, int S, int nb) {
  KxShape x;
  x.NT = nb > 4 ? 2 : 1;
  x.RS = 16 / x.NT;
  auto count = [&] {
    x.panels = (S + x.RS - 1) / x.RS;
    x.blocks = 0;
    for (int i = 0; i < x.panels; ++i) x.blocks += (S - i * x.RS + x.cl - 1) / x.cl;
    x.most = (S + x.cl - 1) / x.cl;
  };
  x.cl = 4;
  count();
  if ((long long)nh * x.blocks < 2048) x.RS = 4;
  for (x.cl = 512 / x.RS, count(); x.cl > 4 && (long long)nh * x.blocks < 768; count()) x.cl /= 2;
  return x;
}

// doubles of the partial sums for up to nb vectors
size_t kx_part(int nh, int S, int nb) {
  const size_t one = kx_shape(nh, S, 1).doubles(nh, S);
  return nb > 4 ? std::max(one, kx_shape(nh, S, 8).doubles(nh, S)) : one;
}

bse_status kx_go(const LatKx& g, const KxShape& x, hipStream_t st) {
  const dim3 grid((unsigned)(g.nh * x.blocks + 7) / 8 * 8);
  if (x.NT == 1 && x.RS == 16)
    hipLaunchKernelGGL((lat_kx<16, 1>), grid, dim3(256), 0, st, g);
  else if (x.NT == 1)
    hipLaunchKernelGGL((lat_kx<4, 1>), grid, dim3(256), 0, st, g);
  else if (x.RS == 8)
    hipLaunchKernelGGL((lat_kx<8, 2>), grid, dim3(256), 0, st, g);
  else
    hipLaunchKernelGGL((lat_kx<4, 2>), grid, dim3(256), 0, st, g);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

}  // namespace

void lattice_free(Plan* p) {
  delete p->lat;
  p->lat = nullptr;
}

// Whether an application to nb vectors goes over R: by the matrix work of the two routes at the rates above (the launches
// are not counted: six to ten here, ten and more per batch of q there)
bool lattice_applies(const Plan* p, int nb) {
  if (!p->lat) return false;
  if (p->lat->forced) return true;
  const int nR = p->lat->nR;
  return (p->lat->K ? secs_kernel(p, nR, nb) : secs_gemm(p, nR, nb)) < secs_pairs(p);
}

namespace {

// K(R)_ss',tt' = sum_munu C^mu_ts W(R)_munu C^nu_s't' of one R of each pair; the exchange term, the same at all R = 0,
// is K(0)_ss',tt' -= alpha sum_munu C^mu_s's Vbar_munu C^nu_tt'
bse_status kernels_build(Plan* p, const std::vector<int2>& pair, hipStream_t st) {
  Lattice* L = p->lat;
  const int na = p->d.n_aux, no = p->d.n_ao;
  const long long no2 = (long long)no * no, n2 = (long long)na * na, hp = no2 * na;
  L->nh = (int)pair.size();
  L->S = kx_tiles(p);
  BSE_TRY(plan_alloc(p, (void**)&L->pair, sizeof(int2) * pair.size()));
  BSE_HIP(hipMemcpyAsync(L->pair, pair.data(), sizeof(int2) * pair.size(), hipMemcpyHostToDevice, st));
  const size_t kb = kx_bytes(p, L->nh);
  BSE_TRY(plan_alloc(p, (void**)&L->K, kb + 4096));
  if (no2 % 16)
    BSE_TRY(zero_fill(L->K, kb + 4096, st));
  else
    BSE_TRY(zero_fill((char*)L->K + kb, 4096, st));
  Tmp H, vp, rows;
  BSE_TRY(dmalloc(&H.p, 16 * (size_t)hp));
  std::vector<int2> list;  // (s, t) with t >= s, then all
  for (int s = 0; s < no; ++s)
    for (int t = s; t < no; ++t) list.push_back(int2{s, t});
  const int tri = (int)list.size();
  for (int i = 0; i < (int)no2; ++i) list.push_back(int2{i / no, i % no});
  BSE_TRY(dmalloc(&rows.p, sizeof(int2) * list.size()));
  BSE_HIP(hipMemcpyAsync(rows.p, list.data(), sizeof(int2) * list.size(), hipMemcpyHostToDevice, st));
  LatGemm k{};  // rows (s, t), columns (t', s')
  k.M = tri;
  k.N = (int)no2;
  k.K = na;
  k.Z = 1;
  k.rows = (const int2*)rows.p;
  k.A = L->C3;
  k.lda = na;
  k.a_ps = no * L->ldc;
  k.a_z = L->ldc;
  k.B = (const double*)H.p;
  k.kd = na;
  k.rs0 = no;
  k.nd = no;
  k.cs1 = (long long)na * no;
  k.b_ps = hp;
  k.nsplit = 1;
  k.klen = na;
  k.S = L->S;
  LatGemm h{};  // H^mu_s't' = sum_nu W(R)_munu C^nu_s't', [2][t'][mu][s']
  h.M = na;
  h.K = na;
  h.Z = 1;
  h.lda = na;
  h.B = L->C1;
  h.kd = na;
  h.rs0 = no;
  h.nd = no;
  h.cs1 = L->ldc;
  h.C = (double*)H.p;
  h.ldc = no;
  h.cc1 = (long long)na * no;
  h.nsplit = 1;
  h.klen = na;
  for (int i = 0; i < L->nh; ++i) {
    h.N = 2 * (int)no2;
    h.A = L->Wr + pair[i].x * n2;
    BSE_TRY(lat_gemm_run<false>(h, st));
    k.C = L->K + (long long)i * (L->S * (long long)(L->S + 1) / 2) * 512;
    k.scale = 1.0;
    BSE_TRY((lat_gemm_run<true, true>(k, st)));
    if (i == 0 && p->d.alpha != 0.0) {
      BSE_TRY(dmalloc(&vp.p, 16 * (size_t)n2));
      hipLaunchKernelGGL(lat_planes, dim3(256), dim3(256), 0, st, n2, p->vbar, (double*)vp.p);
      BSE_CHECK_LAUNCH();
      h.N = (int)no2;
      h.A = (const double*)vp.p;
      h.a_ps = n2;
      h.b_ps = no * L->ldc;
      h.c_ps = hp;
      BSE_TRY(lat_gemm_run<true>(h, st));
      k.swap = k.add = 1;
      k.scale = -p->d.alpha;
      k.M = (int)no2;
      k.rows += tri;
      BSE_TRY((lat_gemm_run<true, true>(k, st)));
      k.swap = k.add = 0;
      k.M = tri;
      k.rows -= tri;
    }
  }
  BSE_TRY(plan_alloc(p, (void**)&L->part, 8 * kx_part(L->nh, L->S, L->nbc)));
  BSE_HIP(hipStreamSynchronize(st));
  return BSE_OK;
}

}  // namespace

namespace {

// The rounding of a W_q that is a sum over R, as a part of its largest element: such sums, by this library or as a matrix
// product, on 4x4x4 to 16x16x16 meshes and up to 125 R come back to 2e-15, and W(R) - W(-R)^T is below 6e-16 of the
// largest W(R).
constexpr double W_ROUNDING = 4e-15;

// Finds the R set of W_q: W(R) on a box of at most 7 x 7 x 7 around R = 0 by the inverse sum, the R whose matrix is
// not rounding noise, and a check that their real parts give W_q back to its rounding (a W_q that is no such sum keeps the
// pair route, which takes it as it is).  p->lat stays empty, or is left incomplete, where the plan does not take it.
bse_status lattice_try(Plan* p, const void* C, const void* W_q, hipStream_t st, bool* taken) {
  const bse_dims& d = p->d;
  const int Nk = p->Nk, na = d.n_aux, no = d.n_ao;
  const long long n2 = (long long)na * na, nc1 = (long long)na * no * no;
  // BSE_LATTICE in the environment at plan creation: 0 keeps the pair route, contract takes the contractions whatever
  // they cost (to time and compare)
  const char* const form = std::getenv("BSE_LATTICE");
  if (form && form[0] == '0') return BSE_OK;
  const bool forced = form && form[0] == 'c';
  if (lds_outer(p) > 64 * 1024 || lds_project(p) > 64 * 1024 || na > 3000) return BSE_OK;
  std::vector<int32_t> R;
  int lo[3], hi[3];
  for (int x = 0; x < 3; ++x) {
    const int n = d.nk[x];
    if (n > FT_MAXQ) return BSE_OK;
    lo[x] = n >= 7 ? -3 : -(n - 1) / 2;
    hi[x] = n >= 7 ? 3 : n / 2;
  }
  for (int a = lo[0]; a <= hi[0]; ++a)
    for (int b = lo[1]; b <= hi[1]; ++b)
      for (int c = lo[2]; c <= hi[2]; ++c) {
        R.push_back(a);
        R.push_back(b);
        R.push_back(c);
      }
  const int nbox = (int)R.size() / 3;
  // worth looking at only if a small set would win for one vector
  {
    const int few = std::min(nbox, 7);
    if (!forced && std::min(secs_gemm(p, few, 1), secs_kernel(p, few, 1)) > secs_pairs(p)) return BSE_OK;
  }
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    (void)hipGetLastError();
    return BSE_OK;
  }
  const size_t most = (size_t)16 << 30, fifth = free_b / 5;
  if (32 * (size_t)nbox * n2 > std::min(most, fifth)) return BSE_OK;

  std::vector<double> q = plan_kfrac(p);
  // the inverse sum over the whole box (the kernels' R list is limited to FT_MAXNR: as many R1 at a time as fit)
  Tmp box, red, idx, chk;
  BSE_TRY(dmalloc(&box.p, 16 * (size_t)nbox * n2));
  BSE_TRY(dmalloc(&red.p, 8 * (2 * (size_t)nbox + 1)));
  BSE_TRY(zero_fill(red.p, 8 * (2 * (size_t)nbox + 1), st));
  const int slab = nbox / (hi[0] - lo[0] + 1), per = FT_MAXNR / slab * slab;
  const std::vector<double> w(nbox, 1.0 / Nk);
  for (int i = 0; i < nbox; i += per) {
    FtArgs ax;
    if (!ft_axes(&ax, Nk, q.data(), std::min(per, nbox - i), R.data() + 3 * (size_t)i, w.data())) return BSE_OK;
    BSE_TRY(ft_gather_launch(ax, -1.0, (const double*)W_q, n2, 0, (double*)box.p + 2 * (size_t)i * n2, st));
  }
  hipLaunchKernelGGL(lat_absmax, dim3(8, nbox), dim3(256), 0, st, n2, (const double*)box.p, (unsigned long long*)red.p);
  BSE_CHECK_LAUNCH();
  std::vector<double> mx(2 * (size_t)nbox);
  BSE_HIP(hipMemcpyAsync(mx.data(), red.p, 16 * (size_t)nbox, hipMemcpyDeviceToHost, st));
  BSE_HIP(hipStreamSynchronize(st));
  double top = 0.0;
  for (double v : mx) {
    if (!std::isfinite(v)) return BSE_OK;
    top = std::max(top, v);
  }
  if (!(top > 0.0)) return BSE_OK;
  std::vector<int32_t> act, ids;
  for (int r = 0; r < nbox; ++r) {
    const bool zero = R[3 * r] == 0 && R[3 * r + 1] == 0 && R[3 * r + 2] == 0;
    if (!(mx[2 * r] > 2e-15 * top || mx[2 * r + 1] > 2e-15 * top) && !zero) continue;
    ids.push_back(r);
    act.insert(act.end(), {R[3 * r], R[3 * r + 1], R[3 * r + 2]});
  }
  const int nR = (int)ids.size();
  FtArgs ax;
  if (!ft_axes(&ax, Nk, q.data(), nR, act.data(), nullptr)) return BSE_OK;
  Lattice* L = new (std::nothrow) Lattice();
  if (!L) return BSE_ENOMEM;
  p->lat = L;
  L->ax = ax;
  L->nR = nR;
  L->forced = forced;
  for (int r = 0; r < nR; ++r)
    if (act[3 * r] == 0 && act[3 * r + 1] == 0 && act[3 * r + 2] == 0) L->r0 = r;
  // the R in pairs, R = 0 first
  std::vector<int2> pair{int2{L->r0, -1}};
  for (int r = 0; r < nR; ++r)
    for (int s = r + 1; s < nR; ++s)
      if (act[3 * r] == -act[3 * s] && act[3 * r + 1] == -act[3 * s + 1] && act[3 * r + 2] == -act[3 * s + 2])
        pair.push_back(int2{r, s});
  // All that either form allocates besides its copies of the inputs stays below a fifth of the free memory and
  // BSE_WORKSPACE_GB (below that only at the least the contractions need, one vector and one R at a time); the kernels
  // alone below 16 GiB, the contractions' buffers too
  size_t limit = fifth;
  if (const char* e = std::getenv("BSE_WORKSPACE_GB"))
    limit = (size_t)std::min((double)limit, std::max(0.0, std::atof(e) * (double)(1ull << 30)));
  const size_t no2 = (size_t)no * no;
  const int nh = (int)pair.size();
  auto kernel_bytes = [&](int b) {  // for b vectors at a time
    return kx_bytes(p, nh) + 8 * kx_part(nh, kx_tiles(p), b) + 16 * no2 * b * ((size_t)Nk + 2 * (size_t)nR);
  };
  bool kernels = !forced && 2 * nh - 1 == nR && kx_bytes(p, nh) <= most && kernel_bytes(std::min(8, p->max_nb)) <= limit &&
                 secs_kernel(p, nR, p->max_nb) < secs_gemm(p, nR, p->max_nb);
  if (!forced && !((kernels ? secs_kernel(p, nR, 1) : secs_gemm(p, nR, 1)) < secs_pairs(p))) return BSE_OK;
  BSE_TRY(plan_alloc(p, (void**)&L->Wr, 8 * (size_t)nR * n2));
  BSE_TRY(dmalloc(&idx.p, 4 * (size_t)nR));
  BSE_TRY(dmalloc(&chk.p, 16 * (size_t)nR * n2));
  BSE_HIP(hipMemcpyAsync(idx.p, ids.data(), 4 * (size_t)nR, hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(lat_take_real, dim3(64, nR), dim3(256), 0, st, n2, (const int*)idx.p, (const double*)box.p, L->Wr,
                     (double*)chk.p);
  BSE_CHECK_LAUNCH();
  double* const dmax = (double*)red.p + 2 * (size_t)nbox;
  BSE_TRY(ft_spread_launch(ax, 1.0, (const double*)chk.p, n2, 0, 1, 1, 0, 2, dmax, (const double*)W_q, st));
  double off = 0.0;
  BSE_HIP(hipMemcpyAsync(&off, dmax, 8, hipMemcpyDeviceToHost, st));
  BSE_HIP(hipStreamSynchronize(st));
  if (!(off <= W_ROUNDING * p->w_max)) return BSE_OK;
  if (kernels) {  // W(-R) = W(R)^T as of a Hermitian W_q
    double asym = 0.0;
    Tmp pr;
    BSE_TRY(dmalloc(&pr.p, sizeof(int2) * pair.size()));
    BSE_HIP(hipMemcpyAsync(pr.p, pair.data(), sizeof(int2) * pair.size(), hipMemcpyHostToDevice, st));
    BSE_TRY(zero_fill(dmax, 8, st));
    hipLaunchKernelGGL(lat_asym, dim3((na + 15) / 16, (na + 15) / 16, (unsigned)pair.size()), dim3(256), 0, st, na,
                       (const int2*)pr.p, L->r0, L->Wr, (unsigned long long*)dmax);
    BSE_CHECK_LAUNCH();
    BSE_HIP(hipMemcpyAsync(&asym, dmax, 8, hipMemcpyDeviceToHost, st));
    BSE_HIP(hipStreamSynchronize(st));
    kernels = asym <= W_ROUNDING * top;
    if (!kernels && !(secs_gemm(p, nR, 1) < secs_pairs(p))) return BSE_OK;
  }
  L->ldc = ((long long)na * no + 15) / 16 * 16 + 16;
  BSE_TRY(plan_alloc(p, (void**)&L->C1, 16 * (size_t)(no * L->ldc)));
  BSE_TRY(plan_alloc(p, (void**)&L->C3, 16 * (size_t)(no * L->ldc)));
  hipLaunchKernelGGL(lat_pack_C, dim3(2048), dim3(256), 0, st, na, no, L->ldc, (const double*)C, L->C1, L->C3);
  BSE_CHECK_LAUNCH();
  // workspaces: all max_nb vectors at once, and for the contractions R in passes of about 4 GiB of U and G, fewer where
  // they would not fit; 8 partial F(R) for the split of the last contraction, 32 of small ones
  int nbc = p->max_nb;
  const size_t room = std::min(most, limit), u1 = 16 * (size_t)nc1, g_r = 16 * (size_t)(no * L->ldc);
  if (kernels)
    while (nbc > 8 && kernel_bytes(nbc) > limit) nbc = (nbc + 1) / 2;
  else
    while (nbc > 1 && 16 * no2 * nbc * ((size_t)Nk + 10 * (size_t)nR) > room / 2) nbc = (nbc + 1) / 2;
  const size_t d_bytes = 16 * no2 * nbc * (size_t)(Nk + nR), f1 = 16 * no2 * nbc * (size_t)nR;
  const size_t f_room = room / 2 > d_bytes ? (room / 2 - d_bytes) / f1 : 0;
  const size_t copies = std::max<size_t>(1, std::min<size_t>(f_room, f1 > ((size_t)32 << 20) ? 8 : 32));
  L->rc = (int)std::max<size_t>(1, std::min<size_t>(nR, std::min<size_t>((size_t)4 << 30, room / 2) / (u1 * nbc + g_r)));
  if (!kernels && d_bytes + copies * f1 + (u1 * nbc + g_r) * L->rc > fifth) return BSE_OK;
  L->nbc = nbc;
  BSE_TRY(plan_alloc(p, (void**)&L->D, 16 * no2 * nbc * (size_t)Nk));
  BSE_TRY(plan_alloc(p, (void**)&L->DR, 16 * no2 * nbc * (size_t)nR));
  for (int s = 0; s < 2; ++s) {
    BSE_TRY(plan_alloc(p, (void**)&L->tab[s], ft_table_bytes(ax)));
    BSE_TRY(ft_table_launch(ax, s == 0 ? 1.0 : -1.0, L->tab[s], st));
  }
  if (kernels) {
    BSE_TRY(plan_alloc(p, (void**)&L->F, 16 * no2 * nbc * (size_t)nR));
    BSE_TRY(kernels_build(p, pair, st));
    *taken = true;
    return BSE_OK;
  }
  L->f_doubles = (long long)(copies * f1 / 8);
  BSE_TRY(plan_alloc(p, (void**)&L->U, u1 * nbc * L->rc));
  BSE_TRY(plan_alloc(p, (void**)&L->G, g_r * L->rc));
  BSE_TRY(plan_alloc(p, (void**)&L->F, 8 * (size_t)L->f_doubles));
  BSE_TRY(plan_alloc(p, (void**)&L->t, 32 * (size_t)na * nbc));
  hipLaunchKernelGGL(lat_transpose, dim3((na + 15) / 16, (na + 15) / 16, nR), dim3(256), 0, st, na, L->Wr);
  BSE_CHECK_LAUNCH();
  *taken = true;
  return BSE_OK;
}

}  // namespace

// Called for FP64 plans whose W_q has the pair symmetry, i.e. real W(R).
bse_status lattice_build(Plan* p, const void* C, const void* W_q, hipStream_t st) {
  const size_t held = p->owned.size();
  bool taken = false;
  const bse_status s = lattice_try(p, C, W_q, st, &taken);
  if (s == BSE_OK && taken) return BSE_OK;
  // the plan keeps the pair route, and nothing of this
  lattice_free(p);
  plan_release(p, held);
  if (s != BSE_ENOMEM) return s;
  set_error("");  // too little memory for it
  return BSE_OK;
}

int lattice_size(const Plan* p, int nb) { return lattice_applies(p, nb) ? p->lat->nR : 0; }

bse_status lattice_apply(Plan* p, const double* X, double* Y, int nb, hipStream_t st) {
  const bse_dims& d = p->d;
  Lattice* L = p->lat;
  const int Nk = p->Nk, na = d.n_aux, no = d.n_ao, nR = L->nR;
  const long long no2 = (long long)no * no, nu = (long long)na * no;
  for (int b0 = 0; b0 < nb; b0 += L->nbc) {
    const int w = std::min(L->nbc, nb - b0);
    const long long E = no2 * w;
    auto project = [&](int nsplit) -> bse_status {
      BSE_TRY(ft_spread_launch(L->ax, -1.0, L->F, E, 1, no2, nsplit, 2 * E * nR, 0, L->D, nullptr, st, L->tab[1]));
      hipLaunchKernelGGL(lat_project, dim3(Nk, w), dim3(256), lds_project(p), st, d.nv, d.nc, no, nb, b0, w,
                         project_groups(p), 1.0 / (double)Nk, p->eps, p->psi64, L->D, X, Y);
      BSE_CHECK_LAUNCH();
      return BSE_OK;
    };
    {
      StageMark sm_(p, BSE_STAGE_PAIRDENS_V, st);
      hipLaunchKernelGGL(lat_outer, dim3(Nk, w), dim3(256), lds_outer(p), st, d.nv, d.nc, no, nb, b0, w, p->psi64, X,
                         L->D);
      BSE_CHECK_LAUNCH();
      BSE_TRY(ft_gather_launch(L->ax, 1.0, L->D, E, 1, L->DR, st, L->tab[0]));
    }
    if (L->K) {
      for (int g0 = 0; g0 < w; g0 += 8) {
        const int n = std::min(8, w - g0);
        const KxShape x = kx_shape(L->nh, L->S, n);
        LatKx g{no, w, g0, n, L->S, L->nh, x.RS, x.panels, x.cl, x.blocks, E, L->K, L->K + kx_bytes(p, L->nh) / 8, L->DR, L->pair, L->part, nullptr};
        g.PT = L->part + (size_t)x.most * L->nh * L->S * 256 * x.NT;
        StageMark sm_(p, BSE_STAGE_DBLOCK, st);
        BSE_TRY(kx_go(g, x, st));
        hipLaunchKernelGGL(lat_kx_sum, dim3(no * ((no + 15) / 16), 2 * L->nh, x.NT), dim3(256), 0, st, g, 16 * x.NT,
                           L->F);
        BSE_CHECK_LAUNCH();
      }
      StageMark sm_(p, BSE_STAGE_TX, st);
      BSE_TRY(project(1));
      continue;
    }
    // split of the last contraction's (nu, t) sum: enough parts for 1024 blocks of its tiles, at least 64 deep
    const int rc = std::min(L->rc, nR);
    const long long t3 = (long long)((no + 63) / 64) * ((no * w + 127) / 128) * rc;
    const long long cap = std::min<long long>(L->f_doubles / (2 * E * nR), std::max<long long>(1, (long long)no * na / 64));
    const int nsplit = (int)std::max<long long>(1, std::min<long long>(cap, (1024 + t3 - 1) / t3));
    for (int r = 0; r < nR; r += rc) {
      const int n = std::min(rc, nR - r);
      LatGemm g{};
      {
        StageMark sm_(p, BSE_STAGE_PAIRDENS_C, st);
        g.M = no * w;
        g.N = na * no;
        g.K = no;
        g.Z = n;
        g.A = L->DR + 2 * E * r;
        g.lda = no;
        g.a_ps = E;
        g.a_z = 2 * E;
        g.B = L->C1;
        g.kd = no;
        g.rs0 = L->ldc;
        g.nd = na * no;
        g.b_ps = no * L->ldc;
        g.C = L->U;
        g.ldc = 2 * nu;
        g.c_ps = nu;
        g.c_z = 2 * nu * no * w;
        g.nsplit = 1;
        g.klen = no;
        BSE_TRY(lat_gemm_run<true>(g, st));
      }
      g = LatGemm{};
      {
        StageMark sm_(p, BSE_STAGE_WSTEP, st);
        g.M = na;
        g.N = 2 * (int)no2;
        g.K = na;
        g.Z = n;
        g.A = L->Wr + (long long)r * na * na;
        g.lda = na;
        g.a_z = (long long)na * na;
        g.B = L->C1;
        g.kd = na;
        g.rs0 = no;
        g.nd = no;
        g.cs1 = L->ldc;
        g.C = L->G;
        g.ldc = no;
        g.cc1 = L->ldc;
        g.c_z = 2 * no * L->ldc;
        g.nsplit = 1;
        g.klen = na;
        BSE_TRY(lat_gemm_run<false>(g, st));
      }
      g = LatGemm{};
      {
        StageMark sm_(p, BSE_STAGE_DBLOCK, st);
        g.M = no;
        g.N = w * no;
        g.K = no * na;
        g.Z = n;
        g.A = L->G;
        g.lda = L->ldc;
        g.a_ps = no * L->ldc;
        g.a_z = 2 * no * L->ldc;
        g.B = L->U;
        g.kd = no;
        g.rs0 = 2 * nu * w;
        g.rs1 = no;
        g.nd = no;
        g.cs1 = 2 * nu;
        g.b_ps = nu;
        g.b_z = 2 * nu * no * w;
        g.C = L->F + 2 * E * r;
        g.ldc = no;
        g.cc1 = 2 * no2;
        g.c_ps = no2;
        g.c_z = 2 * E;
        g.nsplit = nsplit;
        g.klen = ((no * na + nsplit - 1) / nsplit + 15) / 16 * 16;
        g.c_split = 2 * E * nR;
        BSE_TRY(lat_gemm_run<true>(g, st));
      }
      if (d.alpha != 0.0 && r <= L->r0 && L->r0 < r + n) {
        StageMark sm_(p, BSE_STAGE_EXCHANGE, st);
        double* const u = L->t + 2 * (size_t)na * L->nbc;
        hipLaunchKernelGGL(lat_ex_t, dim3(na, w), dim3(64), 0, st, na, no, w, L->U + 2 * nu * no * w * (L->r0 - r), L->t);
        hipLaunchKernelGGL(lat_ex_u, dim3(na, w), dim3(64), 0, st, na, w, d.alpha, p->vbar, L->t, u);
        hipLaunchKernelGGL(lat_ex_f, dim3((no + 63) / 64, no, w), dim3(256), 0, st, na, no, L->ldc, L->C1, u,
                           L->F + 2 * E * L->r0);
        BSE_CHECK_LAUNCH();
      }
    }
    StageMark sm_(p, BSE_STAGE_TX, st);
    BSE_TRY(project(nsplit));
  }
  return BSE_OK;
}

}  // namespace bse
