// Separable Fourier sums between lattice vectors R and a product grid of q:
//   spread:  out[q][e] = sum_R w_R in[R][e] exp(+-2 pi i q.R)
//   gather:  out[R][e] = w_R sum_q in[q][e] exp(+-2 pi i q.R)
// for q = (q1[i], q2[j], q3[k]) listed with k fastest and R any set of distinct vectors in a box of at most
// 7 x 7 x 7.  One axis is summed after the other, so an 8x8x8 grid on a 5x5x5 box takes 10 complex products
// per output instead of 125 and the sums are bound by reading the input and writing the output once.
// At 8x8x8 on 5x5x5 with N_aux = 256 (668 MB in and out, 0.14 ms at the 4.4-5.1 TB/s of a large copy) the
// spread takes 0.145-0.175 ms and the gather 0.188 ms (0.233 with the loads of a step only); the phase table and FP64 GEMM took 0.86 and 0.88 ms.  Nothing
// is copied from the host or allocated: a 4x4x4 interpolation at N_aux = 64 takes 12 us against 43.
#include "bse_internal.h"
#include "fourier.h"

#include <algorithm>
#include <cmath>

namespace bse {

namespace {
// the box of the last two axes as the kernels are instantiated: 3, 5 or 7 on a side
int ft_square(const FtArgs& a) {
  const int m = std::max(a.r[1], a.r[2]);
  return m <= 3 ? 3 : (m <= 5 ? 5 : 7);
}
}  // namespace

bool ft_axes(FtArgs* a, int n_q, const double* q, int n_R, const int32_t* R, const double* w) {
  if (n_R > FT_MAXNR) return false;
  // q: the last axis runs while the first two coordinates stay, the middle one while the first stays
  int n3 = 1;
  while (n3 < n_q && q[3 * n3] == q[0] && q[3 * n3 + 1] == q[1]) ++n3;
  if (n3 > FT_MAXQ || n_q % n3) return false;
  int n2 = 1;
  while (n2 * n3 < n_q && q[3 * (size_t)n2 * n3] == q[0]) ++n2;
  if (n2 > FT_MAXQ || n_q % (n2 * n3)) return false;
  const int n1 = n_q / (n2 * n3);
  if (n1 > FT_MAXQ) return false;
  for (int i = 0; i < n1; ++i)
    for (int j = 0; j < n2; ++j)
      for (int k = 0; k < n3; ++k) {
        const double* p = q + 3 * ((size_t)(i * n2 + j) * n3 + k);
        if (p[0] != q[3 * (size_t)i * n2 * n3] || p[1] != q[3 * (size_t)j * n3 + 1] || p[2] != q[3 * (size_t)k + 2])
          return false;
      }
  a->n[0] = n1;
  a->n[1] = n2;
  a->n[2] = n3;
  for (int i = 0; i < n1; ++i) a->q[0][i] = q[3 * (size_t)i * n2 * n3];
  for (int j = 0; j < n2; ++j) a->q[1][j] = q[3 * (size_t)j * n3 + 1];
  for (int k = 0; k < n3; ++k) a->q[2][k] = q[3 * (size_t)k + 2];
  // R: the distinct values of each axis
  for (int x = 0; x < 3; ++x) {
    int v[FT_MAXR], m = 0;
    for (int r = 0; r < n_R; ++r) {
      const int t = R[3 * r + x];
      int s = 0;
      while (s < m && v[s] != t) ++s;
      if (s < m) continue;
      if (m == FT_MAXR || t > 30000 || t < -30000) return false;
      v[m++] = t;
    }
    std::sort(v, v + m);
    a->r[x] = m;
    for (int s = 0; s < m; ++s) a->Rv[x][s] = (short)v[s];
  }
  const int ns = ft_square(*a);
  for (int s = 0; s < FT_BOX; ++s) a->map[s] = -1;
  for (int r = 0; r < n_R; ++r) {
    int s[3];
    for (int x = 0; x < 3; ++x) {
      s[x] = 0;
      while (a->Rv[x][s[x]] != R[3 * r + x]) ++s[x];
    }
    short& slot = a->map[(s[0] * ns + s[1]) * ns + s[2]];
    if (slot >= 0) return false;  // a vector listed twice
    slot = (short)r;
    a->w[r] = w ? w[r] : 1.0;
  }
  a->nR = n_R;
  return true;
}

namespace {

struct Z {
  double x, y;
};
__device__ __forceinline__ void fma_z(Z& a, const double2 p, const Z b) {
  a.x = fma(p.x, b.x, fma(-p.y, b.y, a.x));
  a.y = fma(p.x, b.y, fma(p.y, b.x, a.y));
}

// outputs are not read again here: past the caches, which keep the input
typedef double dbl2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void store_nt(double2* p, const Z v) {
  __builtin_nontemporal_store(dbl2{v.x, v.y}, reinterpret_cast<dbl2*>(p));
}

// exp(sign 2 pi i q R) of each axis, [q][NS] per axis (columns beyond the axis' R are zero), the three axes after each
// other in LDS; from a table made once where the caller keeps one (the sines take 2 us of a small sum)
template <int NS>
__device__ __forceinline__ void ft_phases(const FtArgs& a, double sign, const double2* __restrict__ tab, double2* p1,
                                          double2* p2, double2* p3) {
  if (tab) {
    const int n = a.n[0] * FT_MAXR + (a.n[1] + a.n[2]) * NS;
    for (int t = threadIdx.x; t < n; t += blockDim.x) p1[t] = tab[t];
    __syncthreads();
    return;
  }
  for (int x = 0; x < 3; ++x) {
    double2* p = x == 0 ? p1 : (x == 1 ? p2 : p3);
    const int ns = x == 0 ? FT_MAXR : NS;
    for (int t = threadIdx.x; t < a.n[x] * ns; t += blockDim.x) {
      const int i = t / ns, r = t % ns;
      double2 v = {0.0, 0.0};
      if (r < a.r[x]) {
        double y = a.q[x][i] * (double)a.Rv[x][r];
        y -= rint(y);
        sincospi(2.0 * sign * y, &v.y, &v.x);
      }
      p[t] = v;
    }
  }
  __syncthreads();
}

// Spread.  A block stages in[R][te consecutive e] (weighted) in LDS, the whole tile's loads in flight together
// and each input read from memory once; a thread owns one e and every (256 / te)-th q1.  For its q1 it sums the
// R1 axis into A[R2][R3] in registers, then two q2 at a time into B[R3], so that each LDS read of a phase of the
// last axis serves two outputs.
// MODE 0: c128 out, 1: c64 out, 2: max |sum - ref| (component-wise) into out as a non-negative double's bits.
// Input: c128 rows of E (planar = 0), or re / im planes per group of `group` elements, [R][E / group][2][group],
// summed over nsplit partial arrays split_stride apart.
template <int NS, int MODE>
__global__ __launch_bounds__(256) void ft_spread(FtArgs a, double sign, int te, const double* __restrict__ in,
                                                 long long E, int planar, long long group, int nsplit,
                                                 long long split_stride, void* __restrict__ out,
                                                 const double* __restrict__ ref, const double2* tab) {
  extern __shared__ double2 ft_lds[];
  const int n1 = a.n[0], n2 = a.n[1], n3 = a.n[2];
  double2* const W = ft_lds;  // [nR + 1][te], the last row zero (the box slots without an R)
  double2* const p1 = W + (a.nR + 1) * te;
  double2* const p2 = p1 + n1 * FT_MAXR;
  double2* const p3 = p2 + n2 * NS;
  const long long e0 = (long long)blockIdx.x * te;
#pragma unroll 8
  for (int t = threadIdx.x; t < a.nR * te; t += blockDim.x) {
    const int r = t / te;
    const long long e = e0 + t % te;
    double2 v = {0.0, 0.0};
    if (e < E) {
      if (planar) {
        const double* s = in + 2 * (long long)r * E + (e / group) * 2 * group + e % group;
#pragma unroll 8
        for (int q = 0; q < nsplit; ++q) {
          v.x += s[q * split_stride];
          v.y += s[q * split_stride + group];
        }
      } else {
        v = reinterpret_cast<const double2*>(in)[(long long)r * E + e];
      }
    }
    W[t] = double2{a.w[r] * v.x, a.w[r] * v.y};
  }
  for (int t = threadIdx.x; t < te; t += blockDim.x) W[a.nR * te + t] = double2{0.0, 0.0};
  ft_phases<NS>(a, sign, tab, p1, p2, p3);
  const int el = threadIdx.x % te, qstep = blockDim.x / te;
  const long long e = e0 + el;
  double dmax = 0.0;
  for (int i1 = threadIdx.x / te; i1 < n1 && e < E; i1 += qstep) {
    Z A[NS][NS];
#pragma unroll
    for (int y = 0; y < NS; ++y)
#pragma unroll
      for (int z = 0; z < NS; ++z) A[y][z] = Z{0.0, 0.0};
    for (int x = 0; x < a.r[0]; ++x) {
      const double2 p = p1[i1 * FT_MAXR + x];
      const short* map = a.map + x * NS * NS;
#pragma unroll
      for (int y = 0; y < NS; ++y)
#pragma unroll
        for (int z = 0; z < NS; ++z) {
          const int r = map[y * NS + z];
          const double2 v = W[(r < 0 ? a.nR : r) * te + el];
          fma_z(A[y][z], p, Z{v.x, v.y});
        }
    }
    for (int j = 0; j < n2; j += 2) {
      const int j2 = j + 1 < n2 ? j + 1 : j;
      Z B0[NS], B1[NS];
#pragma unroll
      for (int z = 0; z < NS; ++z) B0[z] = B1[z] = Z{0.0, 0.0};
#pragma unroll
      for (int y = 0; y < NS; ++y) {
        const double2 pa = p2[j * NS + y], pb = p2[j2 * NS + y];
#pragma unroll
        for (int z = 0; z < NS; ++z) {
          fma_z(B0[z], pa, A[y][z]);
          fma_z(B1[z], pb, A[y][z]);
        }
      }
      for (int k = 0; k < n3; ++k) {
        Z s0{0.0, 0.0}, s1{0.0, 0.0};
#pragma unroll
        for (int z = 0; z < NS; ++z) {
          const double2 p = p3[k * NS + z];
          fma_z(s0, p, B0[z]);
          fma_z(s1, p, B1[z]);
        }
        const long long o0 = ((long long)(i1 * n2 + j) * n3 + k) * E + e;
        const long long o1 = ((long long)(i1 * n2 + j2) * n3 + k) * E + e;
        if constexpr (MODE == 0) {
          double2* c = reinterpret_cast<double2*>(out);
          store_nt(c + o0, s0);
          if (j2 != j) store_nt(c + o1, s1);
        } else if constexpr (MODE == 1) {
          float2* c = reinterpret_cast<float2*>(out);
          c[o0] = float2{(float)s0.x, (float)s0.y};
          if (j2 != j) c[o1] = float2{(float)s1.x, (float)s1.y};
        } else {
          const double2 r0 = reinterpret_cast<const double2*>(ref)[o0], r1 = reinterpret_cast<const double2*>(ref)[o1];
          dmax = max_or_nan(dmax, max_or_nan(fabs(s0.x - r0.x), fabs(s0.y - r0.y)));
          dmax = max_or_nan(dmax, max_or_nan(fabs(s1.x - r1.x), fabs(s1.y - r1.y)));
        }
      }
    }
  }
  if constexpr (MODE == 2) {
    for (int o = 32; o > 0; o >>= 1) dmax = max_or_nan(dmax, __shfl_down(dmax, o));
    if ((threadIdx.x & 63) == 0)
      atomicMax((unsigned long long*)out, (unsigned long long)__double_as_longlong(fabs(dmax)));
  }
}

// Gather.  A thread owns one e (te per block, rows of 16 te bytes) and one q1 of a round of 256 / te: it reads
// each input once and sums the last two axes into D[R2][R3] in registers, two q2 and four q3 at a time (each phase
// read serves two products, the next step's eight loads are in flight).  The R1 axis is then summed over the round's
// q1 through LDS, one R2 at a time, with the first loads of the block's next round or tile in flight; rounds after the
// first add to the outputs the same thread wrote before.
// Output: c128 rows of E, or re and im planes of E each ([R][2][E]) when planar.
template <int NS>
__global__ __launch_bounds__(256) void ft_gather(FtArgs a, double sign, int te, const double* __restrict__ in,
                                                 long long E, int planar, double* __restrict__ out,
                                                 const double2* tab) {
  extern __shared__ double2 ft_lds[];
  const int n1 = a.n[0], n2 = a.n[1], n3 = a.n[2];
  const int el = threadIdx.x % te, ql = threadIdx.x / te, nq = blockDim.x / te;
  double2* const X = ft_lds;  // [nq][NS][te], one R2 of D
  double2* const p1 = X + nq * NS * te;
  double2* const p2 = p1 + n1 * FT_MAXR;
  double2* const p3 = p2 + n2 * NS;
  long long e = (long long)blockIdx.x * te + el;  // of the tile in hand, which starts at e - el < E
  int i0 = 0;
  const int nk = (n3 + 3) / 4, steps = (n2 + 1) / 2 * nk;
  const double2* g;
  bool on;  // the thread has a column in this round
  auto place = [&](long long e, int i0) {
    on = i0 + ql < n1 && e < E;
    g = reinterpret_cast<const double2*>(in) + (long long)(on ? i0 + ql : 0) * n2 * n3 * E + (on ? e : 0);
  };
  double2 u[2][4], v[2][4];
  auto load = [&](int o, int s) {
    const int j = 2 * (s / nk), k0 = 4 * (s % nk);
    const double2* ga = g + (long long)j * n3 * E;
    const double2* gb = j + 1 < n2 ? ga + (long long)n3 * E : ga;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const long long at = (long long)min(k0 + k, n3 - 1) * E;
      u[o][k] = ga[at];
      v[o][k] = gb[at];
    }
  };
  place(e, i0);
  if (on) load(0, 0);
  ft_phases<NS>(a, sign, tab, p1, p2, p3);
  while (e - el < E) {
    Z D[NS][NS];
#pragma unroll
    for (int y = 0; y < NS; ++y)
#pragma unroll
      for (int z = 0; z < NS; ++z) D[y][z] = Z{0.0, 0.0};
    if (on) {
      Z C0[NS], C1[NS];
      auto step = [&](int o, int s) {
        const int j = 2 * (s / nk), k0 = 4 * (s % nk);
        if (k0 == 0) {
#pragma unroll
          for (int z = 0; z < NS; ++z) C0[z] = C1[z] = Z{0.0, 0.0};
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k0 + k >= n3) break;
#pragma unroll
          for (int z = 0; z < NS; ++z) {
            const double2 p = p3[(k0 + k) * NS + z];
            fma_z(C0[z], p, Z{u[o][k].x, u[o][k].y});
            fma_z(C1[z], p, Z{v[o][k].x, v[o][k].y});
          }
        }
        if (k0 + 4 < n3) return;
        const bool two = j + 1 < n2;
        if (!two) {
#pragma unroll
          for (int z = 0; z < NS; ++z) C1[z] = Z{0.0, 0.0};
        }
#pragma unroll
        for (int y = 0; y < NS; ++y) {
          const double2 pa = p2[j * NS + y], pb = p2[(two ? j + 1 : j) * NS + y];
#pragma unroll
          for (int z = 0; z < NS; ++z) {
            fma_z(D[y][z], pa, C0[z]);
            fma_z(D[y][z], pb, C1[z]);
          }
        }
      };
      for (int s = 0; s < steps; s += 2) {
        load(1, min(s + 1, steps - 1));
        step(0, s);
        if (s + 1 >= steps) break;
        if (s + 2 < steps) load(0, s + 2);
        step(1, s + 1);
      }
    }
    const bool same = i0 + nq < n1;
    const long long e2 = same ? e : e + (long long)gridDim.x * te;
    place(e2, same ? i0 + nq : 0);
    if (on) load(0, 0);
    const int live = min(nq, n1 - i0);
#pragma unroll
    for (int y = 0; y < NS; ++y) {
      if (y >= a.r[1]) break;
      __syncthreads();
#pragma unroll
      for (int z = 0; z < NS; ++z) X[(ql * NS + z) * te + el] = double2{D[y][z].x, D[y][z].y};
      __syncthreads();
      for (int it = ql; it < a.r[0] * a.r[2]; it += nq) {
        const int x = it / a.r[2], z = it % a.r[2];
        const int r = a.map[(x * NS + y) * NS + z];
        if (r < 0 || e >= E) continue;
        Z s{0.0, 0.0};
        for (int q = 0; q < live; ++q) {
          const double2 v = X[(q * NS + z) * te + el];
          fma_z(s, p1[(i0 + q) * FT_MAXR + x], Z{v.x, v.y});
        }
        const double w = a.w[r];
        double* o = out + 2 * (long long)r * E;
        double* const re = planar ? o + e : o + 2 * e;
        double* const im = planar ? o + E + e : o + 2 * e + 1;
        *re = i0 ? *re + w * s.x : w * s.x;
        *im = i0 ? *im + w * s.y : w * s.y;
      }
    }
    e = e2;
    i0 = same ? i0 + nq : 0;
  }
}

template <int NS>
__global__ __launch_bounds__(256) void ft_table(FtArgs a, double sign, double2* __restrict__ out) {
  extern __shared__ double2 ft_lds[];
  double2* const p2 = ft_lds + a.n[0] * FT_MAXR;
  ft_phases<NS>(a, sign, nullptr, ft_lds, p2, p2 + a.n[1] * NS);
  const int n = a.n[0] * FT_MAXR + (a.n[1] + a.n[2]) * NS;
  for (int t = threadIdx.x; t < n; t += blockDim.x) out[t] = ft_lds[t];
}

template <int NS, int MODE>
bse_status spread_go(const FtArgs& a, double sign, const double* in, long long E, int planar, long long group,
                     int nsplit, long long split_stride, void* out, const double* ref, const double2* tab, hipStream_t st) {
  // 32 e per block (512-byte rows) while the tile leaves room for two blocks on a CU, 16 for the larger R sets
  // and while 32 would leave CUs without a block
  const int te = (a.nR <= 128 && E >= 32 * 512) ? 32 : 16;
  const int bs = 256;
  const size_t lds = 16 * ((size_t)(a.nR + 1) * te + (size_t)a.n[0] * FT_MAXR + (size_t)(a.n[1] + a.n[2]) * NS);
  if (lds > 64 * 1024)
    BSE_HIP(hipFuncSetAttribute((const void*)ft_spread<NS, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                160 * 1024));
  hipLaunchKernelGGL((ft_spread<NS, MODE>), dim3((unsigned)((E + te - 1) / te)), dim3(bs), lds, st, a, sign, te, in, E,
                     planar, group, nsplit, split_stride, out, ref, tab);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

template <int NS>
bse_status spread_ns(const FtArgs& a, double sign, const double* in, long long E, int planar, long long group,
                     int nsplit, long long split_stride, int mode, void* out, const double* ref, const double2* tab,
                     hipStream_t st) {
  if (mode == 0) return spread_go<NS, 0>(a, sign, in, E, planar, group, nsplit, split_stride, out, ref, tab, st);
  if (mode == 1) return spread_go<NS, 1>(a, sign, in, E, planar, group, nsplit, split_stride, out, ref, tab, st);
  return spread_go<NS, 2>(a, sign, in, E, planar, group, nsplit, split_stride, out, ref, tab, st);
}

}  // namespace

bse_status ft_spread_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, long long group,
                            int nsplit, long long split_stride, int mode, void* out, const double* ref,
                            hipStream_t st, const double* table) {
  const int ns = ft_square(a);
  const double2* tab = reinterpret_cast<const double2*>(table);
  if (ns <= 3) return spread_ns<3>(a, sign, in, E, planar, group, nsplit, split_stride, mode, out, ref, tab, st);
  if (ns <= 5) return spread_ns<5>(a, sign, in, E, planar, group, nsplit, split_stride, mode, out, ref, tab, st);
  return spread_ns<7>(a, sign, in, E, planar, group, nsplit, split_stride, mode, out, ref, tab, st);
}

bse_status ft_gather_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, double* out,
                            hipStream_t st, const double* table) {
  const int ns = ft_square(a);
  const double2* tab = reinterpret_cast<const double2*>(table);
  // as the spread: 32 e per block while that leaves every CU two blocks
  const int te = E >= 32 * 512 ? 32 : 16;
  const int bs = 256;
  const size_t lds = 16 * ((size_t)(bs / te) * ns * te + (size_t)a.n[0] * FT_MAXR + (size_t)(a.n[1] + a.n[2]) * ns);
  // two blocks per CU (their registers allow no more), each over its share of the tiles
  const dim3 grid((unsigned)std::min<long long>(512, (E + te - 1) / te)), block(bs);
  if (ns <= 3)
    hipLaunchKernelGGL(ft_gather<3>, grid, block, lds, st, a, sign, te, in, E, planar, out, tab);
  else if (ns <= 5)
    hipLaunchKernelGGL(ft_gather<5>, grid, block, lds, st, a, sign, te, in, E, planar, out, tab);
  else
    hipLaunchKernelGGL(ft_gather<7>, grid, block, lds, st, a, sign, te, in, E, planar, out, tab);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

size_t ft_table_bytes(const FtArgs& a) {
  return 16 * ((size_t)a.n[0] * FT_MAXR + (size_t)(a.n[1] + a.n[2]) * ft_square(a));
}

bse_status ft_table_launch(const FtArgs& a, double sign, double* out, hipStream_t st) {
  const int ns = ft_square(a);
  const size_t lds = ft_table_bytes(a);
  if (ns <= 3)
    hipLaunchKernelGGL(ft_table<3>, dim3(1), dim3(256), lds, st, a, sign, (double2*)out);
  else if (ns <= 5)
    hipLaunchKernelGGL(ft_table<5>, dim3(1), dim3(256), lds, st, a, sign, (double2*)out);
  else
    hipLaunchKernelGGL(ft_table<7>, dim3(1), dim3(256), lds, st, a, sign, (double2*)out);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

}  // namespace bse
