// Haydock recurrence for the absorption spectrum: nb independent Lanczos chains
// share one block apply per step; the recurrence, the full re-orthogonalisation
// (classical Gram-Schmidt twice) and the continued fraction run in FP64 on the
// device.  Breakdown is masked per chain on the device, so the host loop never
// synchronises until the end.
#include <algorithm>
#include <cmath>

#include "bse_internal.h"

namespace bse {
namespace {

constexpr int RB = 256;  // threads per reduction block

__device__ __forceinline__ void block_sum2(double& a, double& b) {
  __shared__ double sa[RB], sb[RB];
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int s = RB / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) {
      sa[threadIdx.x] += sa[threadIdx.x + s];
      sb[threadIdx.x] += sb[threadIdx.x + s];
    }
    __syncthreads();
  }
  a = sa[0];
  b = sb[0];
}

// part[bi][blk] = sum over the block's slice of conj(x[bi][I]) y[bi][I]
__global__ void dotc_partial(long long N, const double* __restrict__ x, long long xs, const double* __restrict__ y,
                             long long ys, double* __restrict__ part) {
  const int bi = blockIdx.y, nblk = gridDim.x;
  const double* xb = x + 2 * bi * xs;
  const double* yb = y + 2 * bi * ys;
  double sr = 0, si = 0;
  for (long long I = (long long)blockIdx.x * RB + threadIdx.x; I < N; I += (long long)nblk * RB) {
    const double ar = xb[2 * I], ai = -xb[2 * I + 1], br = yb[2 * I], bi_ = yb[2 * I + 1];
    sr += ar * br - ai * bi_;
    si += ar * bi_ + ai * br;
  }
  block_sum2(sr, si);
  if (threadIdx.x == 0) {
    part[2 * ((long long)bi * nblk + blockIdx.x)] = sr;
    part[2 * ((long long)bi * nblk + blockIdx.x) + 1] = si;
  }
}

// mode 0: out[bi*ostride] = Re(sum)      mode 1: out = sqrt(Re(sum))
__global__ void dot_finalize(int nblk, const double* __restrict__ part, double* __restrict__ out, long long ostride,
                             int mode) {
  const int bi = blockIdx.x;
  double sr = 0, si = 0;
  for (int i = threadIdx.x; i < nblk; i += RB) {
    sr += part[2 * ((long long)bi * nblk + i)];
    si += part[2 * ((long long)bi * nblk + i) + 1];
  }
  block_sum2(sr, si);
  if (threadIdx.x == 0) out[bi * ostride] = mode == 1 ? sqrt(fmax(sr, 0.0)) : sr;
}

// start: q_1 = p / b_0 into the basis row 0 and the apply block
__global__ void lz_init(long long N, int nb, int m, const double* __restrict__ P, const double* __restrict__ b,
                        double* __restrict__ basis, double* __restrict__ Qcur, int* __restrict__ active,
                        int* __restrict__ steps) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < nb) {
    active[t] = b[t * (m + 1)] > 0.0 ? 1 : 0;
    steps[t] = b[t * (m + 1)] > 0.0 ? m : 0;
  }
  if (t >= N * nb) return;
  const long long I = t / nb;
  const int bi = (int)(t % nb);
  const double b0 = b[(long long)bi * (m + 1)];
  const double s = b0 > 0.0 ? 1.0 / b0 : 0.0;
  const double vr = P[2 * t] * s, vi = P[2 * t + 1] * s;
  Qcur[2 * t] = vr;
  Qcur[2 * t + 1] = vi;
  double* row = basis + 2 * ((long long)bi * m * N + I);
  row[0] = vr;
  row[1] = vi;
}

// w[bi][I] = Wblk[I][bi] (transpose the apply result into per-chain rows)
__global__ void lz_gather(long long N, int nb, const double* __restrict__ Wblk, double* __restrict__ w) {
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= N * nb) return;
  const long long I = t / nb;
  const int bi = (int)(t % nb);
  w[2 * (bi * N + I)] = Wblk[2 * t];
  w[2 * (bi * N + I) + 1] = Wblk[2 * t + 1];
}

// h[bi][i] = q_i^H w for i < j (grid: j x nb blocks); element I of chain bi of w at bi sb + I si.  With a, the last
// block also gives a_j = Re q_j^H w.
__global__ __launch_bounds__(RB) void lz_project(long long N, int m, int j, const double* __restrict__ basis,
                                                 const double* __restrict__ w, long long sb, long long si,
                                                 double* __restrict__ h, double* __restrict__ a) {
  const int i = blockIdx.x, bi = blockIdx.y;
  const double2* q = reinterpret_cast<const double2*>(basis) + ((long long)bi * m * N + (long long)i * N);
  const double2* wb = reinterpret_cast<const double2*>(w) + bi * sb;
  double sr = 0, sim = 0;
#pragma unroll 4
  for (long long I = threadIdx.x; I < N; I += RB) {
    const double2 x = q[I], y = wb[I * si];
    sr += x.x * y.x + x.y * y.y;
    sim += x.x * y.y - x.y * y.x;
  }
  block_sum2(sr, sim);
  if (threadIdx.x == 0) {
    h[2 * ((long long)bi * m + i)] = sr;
    h[2 * ((long long)bi * m + i) + 1] = sim;
    if (a && i == j - 1) a[(long long)bi * m + i] = sr;
  }
}

// out = w - sum_{i<j} q_i h_i (grid: blocks of RB / G elements x nb), w as in lz_project, out [nb][N]; the G groups of a
// block share the sum over i.  With part also each block's share of |out|^2.
template <int G>
__global__ __launch_bounds__(RB) void lz_subtract(long long N, int m, int j, const double* __restrict__ basis,
                                                  const double* __restrict__ h, const double* w, long long sb,
                                                  long long si, double* out, double* __restrict__ part) {
  constexpr int E = RB / G;
  extern __shared__ double hs[];
  __shared__ double2 gs[G][E];
  const int bi = blockIdx.y, el = threadIdx.x % E, gr = threadIdx.x / E;
  for (int i = threadIdx.x; i < 2 * j; i += RB) hs[i] = h[2 * (long long)bi * m + i];
  __syncthreads();
  const long long I = (long long)blockIdx.x * E + el;
  double sr = 0, sim = 0;
  if (I < N) {
    const double2* q = reinterpret_cast<const double2*>(basis) + ((long long)bi * m * N + I);
#pragma unroll 8
    for (int i = gr; i < j; i += G) {
      const double2 x = q[(long long)i * N];
      const double hr = hs[2 * i], hi = hs[2 * i + 1];
      sr += x.x * hr - x.y * hi;
      sim += x.x * hi + x.y * hr;
    }
  }
  if (G > 1) {
    gs[gr][el] = double2{sr, sim};
    __syncthreads();
    if (gr == 0)
      for (int s = 1; s < G; ++s) {
        sr += gs[s][el].x;
        sim += gs[s][el].y;
      }
  }
  double vr = 0, vi = 0;
  if (gr == 0 && I < N) {
    const double2 y = reinterpret_cast<const double2*>(w)[bi * sb + I * si];
    vr = y.x - sr;
    vi = y.y - sim;
    reinterpret_cast<double2*>(out)[(long long)bi * N + I] = double2{vr, vi};
  }
  if (part) {
    double s = vr * vr + vi * vi, z = 0;
    block_sum2(s, z);
    if (threadIdx.x == 0) part[(long long)bi * gridDim.x + blockIdx.x] = s;
  }
}

// npart partial sums of each chain to one (grid nb)
__global__ __launch_bounds__(RB) void lz_norm(int npart, const double* __restrict__ part, double* __restrict__ out) {
  double s = 0, z = 0;
  for (int i = threadIdx.x; i < npart; i += RB) s += part[(long long)blockIdx.x * npart + i];
  block_sum2(s, z);
  if (threadIdx.x == 0) out[blockIdx.x] = s;
}

// End of step j: b_j = |w| from its partial sums; breakdown test per chain, b_j <= tol * s_j with s_j = max(|a_1|, ..,
// |a_j|, b_1, .., b_{j-1}), the largest recurrence coefficient of the chain so far; q_{j+1} = w / b_j on the chains
// still active (zero on the others) into the basis and the apply block.  b_j is in the units of A (the q_j are unit
// vectors); b_0 = |p| is the start vector's size and does not enter, so the test does not depend on how p is scaled.
// Every block works the few chain scalars out for itself; scale and active are kept per step (rows of nb), so that
// the first block's new row does not race with the others' reading of the old one.
__global__ __launch_bounds__(RB) void lz_next(long long N, int nb, int m, int j, double tol, int npart,
                                              const double* __restrict__ part, const double* __restrict__ a,
                                              double* __restrict__ b, double* __restrict__ scale,
                                              int* __restrict__ active, int* __restrict__ steps,
                                              const double* __restrict__ w, double* __restrict__ basis,
                                              double* __restrict__ Qcur) {
  extern __shared__ double inv[];  // [nb]: 1 / b_j as b_j, 0 where inactive
  for (int bi = threadIdx.x >> 6; bi < nb; bi += RB / 64) {  // one wave per chain
    double s = 0;
    for (int i = threadIdx.x & 63; i < npart; i += 64) s += part[(long long)bi * npart + i];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
    if (threadIdx.x & 63) continue;
    const double bj = sqrt(fmax(s, 0.0));
    double sc = fmax(scale[(long long)(j - 1) * nb + bi], fabs(a[(long long)bi * m + j - 1]));
    if (j > 1) sc = fmax(sc, b[(long long)bi * (m + 1) + j - 1]);
    const int was = active[(long long)(j - 1) * nb + bi], is = was && bj > tol * sc ? 1 : 0;
    inv[bi] = is ? bj : 0.0;
    if (blockIdx.x == 0) {
      b[(long long)bi * (m + 1) + j] = bj;
      scale[(long long)j * nb + bi] = was ? sc : scale[(long long)(j - 1) * nb + bi];
      active[(long long)j * nb + bi] = is;
      if (was && !is) steps[bi] = j;
    }
  }
  __syncthreads();
  const long long t = (long long)blockIdx.x * RB + threadIdx.x;
  if (t >= N * nb) return;
  const long long I = t / nb;
  const int bi = (int)(t % nb);
  double vr = 0, vi = 0;
  if (inv[bi] != 0.0) {
    const double2 v = reinterpret_cast<const double2*>(w)[bi * N + I];
    vr = v.x / inv[bi];
    vi = v.y / inv[bi];
  }
  Qcur[2 * t] = vr;
  Qcur[2 * t + 1] = vi;
  if (j < m) reinterpret_cast<double2*>(basis)[(long long)bi * m * N + (long long)j * N + I] = double2{vr, vi};
}

// continued fraction, one thread per (chain, frequency)
__global__ void cont_frac(int nb, int m, int n_w, const double* __restrict__ a, const double* __restrict__ b,
                          const int* __restrict__ steps, const double* __restrict__ omega, double eta, double scale,
                          double* __restrict__ S) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nb * n_w) return;
  const int bi = t / n_w, iw = t % n_w;
  const int n = steps[bi];
  if (n <= 0) {
    S[t] = 0.0;
    return;
  }
  const double zr = omega[iw], zi = eta;
  const double* ab = a + (long long)bi * m;
  const double* bb = b + (long long)bi * (m + 1);
  double gr = zr - ab[n - 1], gi = zi;
  for (int j = n - 1; j >= 1; --j) {
    const double den = gr * gr + gi * gi;
    const double b2 = bb[j] * bb[j];
    // g = z - a_j - b_j^2 / g
    const double qr = b2 * gr / den, qi = -b2 * gi / den;
    gr = zr - ab[j - 1] - qr;
    gi = zi - qi;
  }
  const double den = gr * gr + gi * gi;
  const double fi = -bb[0] * bb[0] * gi / den;  // Im(b0^2 / g)
  S[t] = -fi * scale;
}

}  // namespace
}  // namespace bse

using namespace bse;

extern "C" bse_status bse_haydock_spectrum(bse_plan* plan, const void* P, int32_t nb, int32_t n_steps,
                                           const double* omega, int32_t n_w, double eta, double* S, double* a,
                                           double* b, int32_t* steps_done, void* basis_out, void* hip_stream) {
  set_error("");
  if (!plan || !P || !omega || !S || !a || !b || !steps_done) {
    set_error("bse_haydock_spectrum: NULL argument");
    return BSE_EINVAL;
  }
  Plan* p = &plan->impl;
  if (nb <= 0 || nb > p->max_nb || n_steps <= 0 || n_w <= 0 || !(eta > 0.0)) {
    set_error("bse_haydock_spectrum: need 1 <= nb <= max_nb, n_steps > 0, n_w > 0, eta > 0");
    return BSE_EINVAL;
  }
  if ((long long)n_steps > p->N) {
    set_error("bse_haydock_spectrum: n_steps exceeds the dimension");
    return BSE_ESHAPE;
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  const long long N = p->N;
  const int m = n_steps;
  const double tol = 1e-12;
  const int nblk = (int)std::min<long long>(1024, (N + RB - 1) / RB);

  struct Bufs {
    double *basis = nullptr, *Q = nullptr, *Wb = nullptr, *w = nullptr, *da = nullptr, *db = nullptr, *h = nullptr,
           *part = nullptr, *dom = nullptr, *dS = nullptr, *scl = nullptr;
    int *act = nullptr, *stp = nullptr;
    bool own_basis = false;
    ~Bufs() {
      if (own_basis) dfree(basis);
      dfree(Q);
      dfree(Wb);
      dfree(w);
      dfree(da);
      dfree(db);
      dfree(h);
      dfree(part);
      dfree(dom);
      dfree(dS);
      dfree(scl);
      dfree(act);
      dfree(stp);
    }
  } B;
  // the recurrence reads the basis 16 bytes at a time: a caller's buffer aligned to its doubles only is filled at the end
  const bool in_place = basis_out && (reinterpret_cast<uintptr_t>(basis_out) & 15) == 0;
  if (in_place) {
    B.basis = (double*)basis_out;
  } else {
    BSE_TRY(dmalloc((void**)&B.basis, 16 * (size_t)nb * m * N));
    B.own_basis = true;
  }
  BSE_TRY(dmalloc((void**)&B.Q, 16 * (size_t)N * nb));
  BSE_TRY(dmalloc((void**)&B.Wb, 16 * (size_t)N * nb));
  BSE_TRY(dmalloc((void**)&B.w, 16 * (size_t)N * nb));
  BSE_TRY(dmalloc((void**)&B.da, 8 * (size_t)nb * m));
  BSE_TRY(dmalloc((void**)&B.db, 8 * (size_t)nb * (m + 1)));
  BSE_TRY(dmalloc((void**)&B.h, 16 * (size_t)nb * m));
  BSE_TRY(dmalloc((void**)&B.part, std::max<size_t>(16 * (size_t)nb * nblk, 8 * (size_t)nb * ((N + 63) / 64 + 1))));
  BSE_TRY(dmalloc((void**)&B.dom, 8 * (size_t)n_w));
  BSE_TRY(dmalloc((void**)&B.dS, 8 * (size_t)nb * n_w));
  BSE_TRY(dmalloc((void**)&B.scl, 8 * (size_t)nb * (m + 1)));
  BSE_TRY(dmalloc((void**)&B.act, sizeof(int) * (size_t)nb * (m + 1)));
  BSE_TRY(dmalloc((void**)&B.stp, sizeof(int) * nb));
  BSE_TRY(zero_fill(B.da, 8 * (size_t)nb * m, st));
  BSE_TRY(zero_fill(B.db, 8 * (size_t)nb * (m + 1), st));
  BSE_TRY(zero_fill(B.scl, 8 * (size_t)nb, st));
  BSE_HIP(hipMemcpyAsync(B.dom, omega, 8 * (size_t)n_w, hipMemcpyHostToDevice, st));

  const unsigned gN = (unsigned)((N * nb + 255) / 256);
  const dim3 gV((unsigned)((N + RB - 1) / RB), nb);
  // b_0 = |p|   (P is [N][nb]: chain stride 1, element stride nb -> gather first)
  hipLaunchKernelGGL(lz_gather, dim3(gN), dim3(256), 0, st, N, nb, (const double*)P, B.w);
  hipLaunchKernelGGL(dotc_partial, dim3(nblk, nb), dim3(RB), 0, st, N, B.w, N, B.w, N, B.part);
  hipLaunchKernelGGL(dot_finalize, dim3(nb), dim3(RB), 0, st, nblk, B.part, B.db, (long long)(m + 1), 1);
  hipLaunchKernelGGL(lz_init, dim3(gN), dim3(256), 0, st, N, nb, m, (const double*)P, B.db, B.basis, B.Q, B.act,
                     B.stp);
  BSE_CHECK_LAUNCH();
  // One step: h = Q^H w (its last entry is a_j), w -= Q h, both once more (classical Gram-Schmidt twice; the first
  // pass takes the three-term part with it), then b_j, the breakdown test and q_{j+1}: five launches.  Small chains
  // read w from the apply block as it lies; larger ones gather it into rows first, or each of the j blocks of a
  // chain would read n_b times the lines it needs.  More than 128 partial norms are summed by a launch of their own.
  // At 4x4x4 (3 chains of 1024) the recurrence took 38 us per step in twelve launches, now 22.
  // Chains of up to 8192 transitions share the sum over the basis between four groups of threads (the blocks of 256
  // elements would be few).
  const bool direct = N * nb <= 16384, shared_sum = N <= 8192;
  const dim3 gS(shared_sum ? (unsigned)((N + RB / 4 - 1) / (RB / 4)) : gV.x, nb);
  const unsigned npart = gS.x;
  const bool norm = npart > 128;
  if (m > 3000) {  // h of a chain in LDS beyond the default limit
    BSE_HIP(hipFuncSetAttribute((const void*)lz_subtract<1>, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024));
    BSE_HIP(hipFuncSetAttribute((const void*)lz_subtract<4>, hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024));
  }
  auto subtract = [&](int j, const double* src, long long sb, long long si, double* part) {
    const size_t sh = 16 * (size_t)j;
    if (shared_sum)
      hipLaunchKernelGGL(lz_subtract<4>, gS, dim3(RB), sh, st, N, m, j, B.basis, B.h, src, sb, si, B.w, part);
    else
      hipLaunchKernelGGL(lz_subtract<1>, gS, dim3(RB), sh, st, N, m, j, B.basis, B.h, src, sb, si, B.w, part);
  };
  for (int j = 1; j <= m; ++j) {
    BSE_TRY(bse_apply(plan, B.Q, B.Wb, nb, hip_stream));
    StageMark sm_(p, BSE_STAGE_LANCZOS, st);
    if (!direct) hipLaunchKernelGGL(lz_gather, dim3(gN), dim3(256), 0, st, N, nb, B.Wb, B.w);
    const double* src = direct ? B.Wb : B.w;
    const long long sb = direct ? 1 : N, si = direct ? nb : 1;
    hipLaunchKernelGGL(lz_project, dim3(j, nb), dim3(RB), 0, st, N, m, j, B.basis, src, sb, si, B.h, B.da);
    subtract(j, src, sb, si, nullptr);
    hipLaunchKernelGGL(lz_project, dim3(j, nb), dim3(RB), 0, st, N, m, j, B.basis, B.w, N, 1LL, B.h, (double*)nullptr);
    subtract(j, B.w, N, 1, B.part);
    if (norm) hipLaunchKernelGGL(lz_norm, dim3(nb), dim3(RB), 0, st, (int)npart, B.part, B.part + (size_t)nb * npart);
    hipLaunchKernelGGL(lz_next, dim3(gN), dim3(RB), 8 * (size_t)nb, st, N, nb, m, j, tol, norm ? 1 : (int)npart,
                       norm ? B.part + (size_t)nb * npart : B.part, B.da, B.db, B.scl, B.act, B.stp, B.w, B.basis, B.Q);
    BSE_CHECK_LAUNCH();
  }
  {
    const int n = nb * n_w;
    hipLaunchKernelGGL(cont_frac, dim3((n + 255) / 256), dim3(256), 0, st, nb, m, n_w, B.da, B.db, B.stp, B.dom, eta,
                       1.0 / (M_PI * (double)p->Nk), B.dS);
    BSE_CHECK_LAUNCH();
  }
  if (basis_out && !in_place)
    BSE_HIP(hipMemcpyAsync(basis_out, B.basis, 16 * (size_t)nb * m * N, hipMemcpyDeviceToDevice, st));
  BSE_HIP(hipMemcpyAsync(S, B.dS, 8 * (size_t)nb * n_w, hipMemcpyDeviceToHost, st));
  BSE_HIP(hipMemcpyAsync(a, B.da, 8 * (size_t)nb * m, hipMemcpyDeviceToHost, st));
  BSE_HIP(hipMemcpyAsync(b, B.db, 8 * (size_t)nb * (m + 1), hipMemcpyDeviceToHost, st));
  BSE_HIP(hipMemcpyAsync(steps_done, B.stp, sizeof(int) * nb, hipMemcpyDeviceToHost, st));
  BSE_HIP(hipStreamSynchronize(st));
  for (int i = 0; i < nb; ++i)
    if (steps_done[i] < m) return BSE_INFO_BREAKDOWN;
  return BSE_OK;
}

// k-offset averaging (Sec. IV.A, k-point convergence): independent Haydock spectra on shifted dense meshes,
// S = sum_j w_j S_j.  Every plan must describe the same problem sizes (they differ in their bands).
extern "C" bse_status bse_offset_spectrum(bse_plan* const* plans, const void* const* P, const double* weights,
                                          int32_t n_off, int32_t nb, int32_t n_steps, const double* omega,
                                          int32_t n_w, double eta, double* S, int32_t* steps_done,
                                          void* hip_stream) {
  set_error("");
  if (!plans || !P || !weights || !omega || !S || n_off <= 0 || nb <= 0 || n_steps <= 0 || n_w <= 0) {
    set_error("bse_offset_spectrum: NULL argument or non-positive size");
    return BSE_EINVAL;
  }
  for (int j = 0; j < n_off; ++j) {
    if (!plans[j] || !P[j] || !std::isfinite(weights[j])) {
      set_error("bse_offset_spectrum: NULL plan / start block or non-finite weight at offset " + std::to_string(j));
      return BSE_EINVAL;
    }
    // the sizes as given: BF16x3 plans store n_ao and n_aux rounded up, and only where the copies fit
    const Plan &p = plans[0]->impl, &o = plans[j]->impl;
    const bse_dims &a = p.d, &b = o.d;
    if (a.nk[0] != b.nk[0] || a.nk[1] != b.nk[1] || a.nk[2] != b.nk[2] || a.nv != b.nv || a.nc != b.nc ||
        p.given_ao != o.given_ao || p.given_aux != o.given_aux) {
      set_error("bse_offset_spectrum: the plans describe different problem sizes");
      return BSE_ESHAPE;
    }
  }
  const size_t ns = (size_t)nb * n_w;
  std::vector<double> Sj(ns), a((size_t)nb * n_steps), b((size_t)nb * (n_steps + 1));
  std::vector<int32_t> steps(nb);
  for (size_t i = 0; i < ns; ++i) S[i] = 0.0;
  bool breakdown = false;
  for (int j = 0; j < n_off; ++j) {
    const bse_status s = bse_haydock_spectrum(plans[j], P[j], nb, n_steps, omega, n_w, eta, Sj.data(), a.data(),
                                              b.data(), steps.data(), nullptr, hip_stream);
    if (s != BSE_OK && s != BSE_INFO_BREAKDOWN) return s;
    breakdown = breakdown || s == BSE_INFO_BREAKDOWN;
    for (size_t i = 0; i < ns; ++i) S[i] += weights[j] * Sj[i];
    if (steps_done)
      for (int i = 0; i < nb; ++i) steps_done[(size_t)j * nb + i] = steps[i];
  }
  return breakdown ? BSE_INFO_BREAKDOWN : BSE_OK;
}

// the paper's offset set: the four classes of a 3x3x3 grid of offsets (units of the mesh spacing)
extern "C" bse_status bse_offset_set(int32_t* n, double* offsets, double* weights) {
  set_error("");
  if (!n) {
    set_error("bse_offset_set: NULL argument");
    return BSE_EINVAL;
  }
  static const double off[4][3] = {{0.0, 0.0, 0.0}, {1.0 / 3, 0.0, 0.0}, {1.0 / 3, 1.0 / 3, 0.0}, {2.0 / 3, 1.0 / 3, 0.0}};
  static const double wts[4] = {1.0 / 27, 8.0 / 27, 6.0 / 27, 12.0 / 27};
  *n = 4;
  for (int j = 0; j < 4; ++j) {
    if (offsets)
      for (int i = 0; i < 3; ++i) offsets[3 * j + i] = off[j][i];
    if (weights) weights[j] = wts[j];
  }
  return BSE_OK;
}
