// Separable Fourier sums between lattice vectors R and a product grid of q:
//   spread:  out[q][e] = sum_R w_R in[R][e] exp(+-2 pi i q.R)
//   gather:  out[R][e] = w_R sum_q in[q][e] exp(+-2 pi i q.R)
// for q = (q1[i], q2[j], q3[k]) listed with k fastest and R any set of distinct vectors in a box of at most
// 7 x 7 x 7.  One axis is summed after the other, so an 8x8x8 grid on a 5x5x5 box takes 10 complex products
// per output instead of 125 and the sums are bound by reading the input and writing the output once.
// At 8x8x8 on 5x5x5 with N_aux = 256 (668 MB in and out, 0.14 ms at the 4.4-5.1 TB/s of a large copy) the
// spread takes 0.145-0.175 ms and the gather 0.188 ms (0.233 with the loads of a step only); the phase table and FP64
// GEMM took 0.86 and 0.88 ms.  Nothing is copied from the host or allocated: a 4x4x4 interpolation at N_aux = 64 takes
// 12 us against 43.
#include "bse_internal.h"
#include "fourier.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace bse {

namespace {
// the box of the last two axes as the kernels are instantiated: each 1, 3, 5 or 7 (with one size for both a plane of R
// cost up to five times its sums: 12x12x1 q on 7x7x1 R, N_aux 300, spread 526 us with 7 x 7 and 60 with 7 x 1, gather 446
// and 95; the phase table and GEMM 239 and 202)
int ft_side(const FtArgs& a, int x) { return a.r[x] / 2 * 2 + 1; }
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
  const int ny = ft_side(*a, 1), nz = ft_side(*a, 2);
  for (int s = 0; s < FT_BOX; ++s) a->map[s] = -1;
  for (int r = 0; r < n_R; ++r) {
    int s[3];
    for (int x = 0; x < 3; ++x) {
      s[x] = 0;
      while (a->Rv[x][s[x]] != R[3 * r + x]) ++s[x];
    }
    short& slot = a->map[(s[0] * ny + s[1]) * nz + s[2]];
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

// exp(sign 2 pi i q R) of each axis, [q][7], [q][ny] and [q][nz] (columns beyond the axis' R are zero), the three axes
// after each other in LDS; from a table made once where the caller keeps one (the sines take 2 us of a small sum)
__device__ __forceinline__ void ft_phases(const FtArgs& a, double sign, const double2* __restrict__ tab, int ny, int nz,
                                          double2* p1) {
  if (tab) {
    const int n = a.n[0] * FT_MAXR + a.n[1] * ny + a.n[2] * nz;
    for (int t = threadIdx.x; t < n; t += blockDim.x) p1[t] = tab[t];
    __syncthreads();
    return;
  }
  for (int x = 0; x < 3; ++x) {
    const int ns = x == 0 ? FT_MAXR : (x == 1 ? ny : nz);
    for (int t = threadIdx.x; t < a.n[x] * ns; t += blockDim.x) {
      const int i = t / ns, r = t % ns;
      double2 v = {0.0, 0.0};
      if (r < a.r[x]) {
        double y = a.q[x][i] * (double)a.Rv[x][r];
        y -= rint(y);
        sincospi(2.0 * sign * y, &v.y, &v.x);
      }
      p1[t] = v;
    }
    p1 += a.n[x] * ns;
  }
  __syncthreads();
}

// Few q1 leave rows of threads without one: the pairs of q2 of each q1 are then shared between this many of them (by the
// spread where there are more than four rows per q1, by the gather for fewer than four q1: with more the sharing costs what
// it gives).
int ft_parts(int rows, int n1, int n2) { return std::min(std::max(1, rows / n1), (n2 + 1) / 2); }

// Spread.  A block stages in[R][te consecutive e] (weighted) in LDS, the whole tile's loads in flight together
// and each input read from memory once; a thread owns one e and every (256 / te)-th q1 (or part of its q2).  For its q1
// it sums the R1 axis into A[R2][R3] in registers, then two q2 at a time into B[R3], so that each LDS read of a phase of
// the last axis serves two outputs.
// MODE 0: c128 out, 1: c64 out, 2: max |sum - ref| (component-wise) into out as a non-negative double's bits.
// Input: c128 rows of E (planar = 0), or re / im planes per group of `group` elements, [R][E / group][2][group],
// summed over nsplit partial arrays split_stride apart.
template <int NY, int NZ, int MODE>
__global__ __launch_bounds__(256) void ft_spread(FtArgs a, double sign, int te, int parts, const double* __restrict__ in,
                                                 long long E, int planar, long long group, int nsplit,
                                                 long long split_stride, void* __restrict__ out,
                                                 const double* __restrict__ ref, const double2* tab) {
  extern __shared__ double2 ft_lds[];
  const int n1 = a.n[0], n2 = a.n[1], n3 = a.n[2];
  double2* const W = ft_lds;  // [nR + 1][te], the last row zero (the box slots without an R)
  double2* const p1 = W + (a.nR + 1) * te;
  double2* const p2 = p1 + n1 * FT_MAXR;
  double2* const p3 = p2 + n2 * NY;
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
  ft_phases(a, sign, tab, NY, NZ, p1);
  const int el = threadIdx.x % te, qstep = blockDim.x / te;
  const long long e = e0 + el;
  double dmax = 0.0;
  for (int it = threadIdx.x / te; it < n1 * parts && e < E; it += qstep) {
    const int i1 = parts == 1 ? it : it / parts, part = parts == 1 ? 0 : it % parts;
    Z A[NY][NZ];
#pragma unroll
    for (int y = 0; y < NY; ++y)
#pragma unroll
      for (int z = 0; z < NZ; ++z) A[y][z] = Z{0.0, 0.0};
    for (int x = 0; x < a.r[0]; ++x) {
      const double2 p = p1[i1 * FT_MAXR + x];
      const short* map = a.map + x * NY * NZ;
#pragma unroll
      for (int y = 0; y < NY; ++y)
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          const int r = map[y * NZ + z];
          const double2 v = W[(r < 0 ? a.nR : r) * te + el];
          fma_z(A[y][z], p, Z{v.x, v.y});
        }
    }
    for (int j = 2 * part; j < n2; j += 2 * parts) {
      const int j2 = j + 1 < n2 ? j + 1 : j;
      Z B0[NZ], B1[NZ];
#pragma unroll
      for (int z = 0; z < NZ; ++z) B0[z] = B1[z] = Z{0.0, 0.0};
#pragma unroll
      for (int y = 0; y < NY; ++y) {
        const double2 pa = p2[j * NY + y], pb = p2[j2 * NY + y];
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          fma_z(B0[z], pa, A[y][z]);
          fma_z(B1[z], pb, A[y][z]);
        }
      }
      for (int k = 0; k < n3; ++k) {
        Z s0{0.0, 0.0}, s1{0.0, 0.0};
#pragma unroll
        for (int z = 0; z < NZ; ++z) {
          const double2 p = p3[k * NZ + z];
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

// R2 of D that go through LDS at a time: all of a small box (fewer barriers: 12x12x1 on 7x7x1, N_aux 300, 118 -> 95 us),
// one of a larger
constexpr int ft_turn(int ny, int nz) { return ny * nz <= 9 ? ny : 1; }

// Gather.  A thread owns one e (te per block, rows of 16 te bytes) and one q1 (or part of its q2) of a round of 256 / te:
// it reads each input once and sums the last two axes into D[R2][R3] in registers, two q2 and four q3 at a time (each phase
// read serves two products, the next step's eight loads are in flight).  The R1 axis is then summed over the round's
// q1 through LDS, with the first loads of the block's next round or tile in flight; rounds after the
// first add to the outputs the same thread wrote before.
// Output: c128 rows of E, or re and im planes of E each ([R][2][E]) when planar.
// SPLIT: q2 shared between rows (without it what depends on the part is known, and stays in scalar registers).
template <int NY, int NZ, bool SPLIT>
__global__ __launch_bounds__(256, NY * NZ <= 25 ? 2 : 1) void ft_gather(FtArgs a, double sign, int te, int shared,
                                                                        const double* __restrict__ in, long long E,
                                                                        int planar, double* __restrict__ out,
                                                                        const double2* tab) {
  extern __shared__ double2 ft_lds[];
  const int n1 = a.n[0], n2 = a.n[1], n3 = a.n[2];
  const int el = threadIdx.x % te, ql = threadIdx.x / te, nq = blockDim.x / te;
  constexpr int YB = ft_turn(NY, NZ);
  double2* const X = ft_lds;  // [nq][YB][NZ][te], YB R2 of D
  double2* const p1 = X + nq * YB * NZ * te;
  double2* const p2 = p1 + n1 * FT_MAXR;
  double2* const p3 = p2 + n2 * NY;
  long long e = (long long)blockIdx.x * te + el;  // of the tile in hand, which starts at e - el < E
  // row i of a round: q1 i / parts, part i % parts of its q2
  const int parts = SPLIT ? shared : 1, rows = n1 * parts;
  int i0 = 0, part = 0, steps = 0;
  const int nk = (n3 + 3) / 4;
  const double2* g;
  bool on;  // the thread has a column in this round
  auto place = [&](long long e, int i0) {
    on = i0 + ql < rows && e < E;
    const int i = on ? i0 + ql : 0;
    part = SPLIT ? i % parts : 0;
    steps = ((n2 + 1) / 2 - part + parts - 1) / parts * nk;
    g = reinterpret_cast<const double2*>(in) + (long long)(i / parts) * n2 * n3 * E + (on ? e : 0);
  };
  double2 u[2][4], v[2][4];
  auto load = [&](int o, int s) {
    const int j = 2 * (part + s / nk * parts), k0 = 4 * (s % nk);
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
  ft_phases(a, sign, tab, NY, NZ, p1);
  while (e - el < E) {
    Z D[NY][NZ];
#pragma unroll
    for (int y = 0; y < NY; ++y)
#pragma unroll
      for (int z = 0; z < NZ; ++z) D[y][z] = Z{0.0, 0.0};
    if (on) {
      Z C0[NZ], C1[NZ];
      auto step = [&](int o, int s) {
        const int j = 2 * (part + s / nk * parts), k0 = 4 * (s % nk);
        if (k0 == 0) {
#pragma unroll
          for (int z = 0; z < NZ; ++z) C0[z] = C1[z] = Z{0.0, 0.0};
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (k0 + k >= n3) break;
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
            const double2 p = p3[(k0 + k) * NZ + z];
            fma_z(C0[z], p, Z{u[o][k].x, u[o][k].y});
            fma_z(C1[z], p, Z{v[o][k].x, v[o][k].y});
          }
        }
        if (k0 + 4 < n3) return;
        const bool two = j + 1 < n2;
        if (!two) {
#pragma unroll
          for (int z = 0; z < NZ; ++z) C1[z] = Z{0.0, 0.0};
        }
#pragma unroll
        for (int y = 0; y < NY; ++y) {
          const double2 pa = p2[j * NY + y], pb = p2[(two ? j + 1 : j) * NY + y];
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
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
    const bool same = i0 + nq < rows;
    const long long e2 = same ? e : e + (long long)gridDim.x * te;
    place(e2, same ? i0 + nq : 0);
    if (on) load(0, 0);
    const int live = min(nq, rows - i0);
#pragma unroll
    for (int y0 = 0; y0 < NY; y0 += YB) {
      if (y0 >= a.r[1]) break;
      __syncthreads();
#pragma unroll
      for (int y = 0; y < YB; ++y)
#pragma unroll
        for (int z = 0; z < NZ; ++z) X[((ql * YB + y) * NZ + z) * te + el] = double2{D[y0 + y][z].x, D[y0 + y][z].y};
      __syncthreads();
      const int ny = YB == 1 ? 1 : a.r[1];
      for (int it = ql; it < a.r[0] * ny * a.r[2]; it += nq) {
        const int z = it % a.r[2], xy = it / a.r[2], x = xy / ny, y = YB == 1 ? 0 : xy % ny;
        const int r = a.map[(x * NY + y0 + y) * NZ + z];
        if (r < 0 || e >= E) continue;
        Z s{0.0, 0.0};
        for (int q = 0; q < live; ++q) {
          const double2 v = X[((q * YB + y) * NZ + z) * te + el];
          fma_z(s, p1[(i0 + q) / parts * FT_MAXR + x], Z{v.x, v.y});
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

__global__ __launch_bounds__(256) void ft_table(FtArgs a, double sign, int ny, int nz, double2* __restrict__ out) {
  extern __shared__ double2 ft_lds[];
  ft_phases(a, sign, nullptr, ny, nz, ft_lds);
  const int n = a.n[0] * FT_MAXR + a.n[1] * ny + a.n[2] * nz;
  for (int t = threadIdx.x; t < n; t += blockDim.x) out[t] = ft_lds[t];
}

// go(NY, NZ) with the box of the last two axes as constants
template <typename F>
bse_status with_sides(const FtArgs& a, F go) {
  auto one = [&](auto ny) -> bse_status {
    switch (ft_side(a, 2)) {
      case 1: return go(ny, std::integral_constant<int, 1>());
      case 3: return go(ny, std::integral_constant<int, 3>());
      case 5: return go(ny, std::integral_constant<int, 5>());
      default: return go(ny, std::integral_constant<int, 7>());
    }
  };
  switch (ft_side(a, 1)) {
    case 1: return one(std::integral_constant<int, 1>());
    case 3: return one(std::integral_constant<int, 3>());
    case 5: return one(std::integral_constant<int, 5>());
    default: return one(std::integral_constant<int, 7>());
  }
}

}  // namespace

bse_status ft_spread_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, long long group,
                            int nsplit, long long split_stride, int mode, void* out, const double* ref,
                            hipStream_t st, const double* table) {
  const double2* tab = reinterpret_cast<const double2*>(table);
  // 32 e per block (512-byte rows) while the tile leaves room for two blocks on a CU, 16 for the larger R sets
  // and while 32 would leave CUs without a block; more where q1 and the pairs of q2 are fewer than the rows of threads
  int te = (a.nR <= 128 && E >= 32 * 512) ? 32 : 16;
  while (te >= 32 && te < 256 && 256 / te >= a.n[0] * (a.n[1] + 1) && E >= 2 * te * 448 && (a.nR + 1) * te <= 1536) te *= 2;
  const size_t lds = 16 * (size_t)(a.nR + 1) * te + ft_table_bytes(a);
  const dim3 grid((unsigned)((E + te - 1) / te));
  const int parts = 256 / te / a.n[0] > 4 ? ft_parts(256 / te, a.n[0], a.n[1]) : 1;
  return with_sides(a, [&](auto ny, auto nz) -> bse_status {
    auto go = [&](auto kern) -> bse_status {
      if (lds > 64 * 1024)
        BSE_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
      hipLaunchKernelGGL(kern, grid, dim3(256), lds, st, a, sign, te, parts, in, E, planar, group, nsplit, split_stride,
                         out, ref, tab);
      BSE_CHECK_LAUNCH();
      return BSE_OK;
    };
    constexpr int NY = decltype(ny)::value, NZ = decltype(nz)::value;
    return mode == 0 ? go(ft_spread<NY, NZ, 0>) : mode == 1 ? go(ft_spread<NY, NZ, 1>) : go(ft_spread<NY, NZ, 2>);
  });
}

bse_status ft_gather_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, double* out,
                            hipStream_t st, const double* table) {
  const double2* tab = reinterpret_cast<const double2*>(table);
  // as the spread: 32 e per block while that leaves every CU two blocks; 16 where all q1 are then in one round (12x12x12 on
  // 5x5x5, N_aux 200: 317 -> 262 us); more for fewer than five q1 while 448 blocks are left (1x10x2 on 1x5x3, N_aux 394: 70
  // us with 32, the GEMM 46, and below that with 256)
  int te = E >= 32 * 512 && !(a.n[0] > 8 && a.n[0] <= 16) ? 32 : 16;
  while (te >= 32 && te < 256 && 256 / te >= 2 * a.n[0] && E >= 2 * te * 448) te *= 2;
  const int ny = ft_side(a, 1), nz = ft_side(a, 2);
  const size_t lds = 16 * (size_t)256 * ft_turn(ny, nz) * nz + ft_table_bytes(a);
  return with_sides(a, [&](auto ny, auto nz) -> bse_status {
    constexpr int NY = decltype(ny)::value, NZ = decltype(nz)::value;
    // as many blocks as the registers allow on the CUs (two for the boxes of 5 x 5), each over its share of the tiles
    constexpr int PER_CU = NY * NZ <= 3 ? 4 : NY * NZ <= 9 && NZ < 7 ? 3 : 2;
    const dim3 grid((unsigned)std::min<long long>(256 * PER_CU, (E + te - 1) / te));
    const int parts = a.n[0] < 4 ? ft_parts(256 / te / 2, a.n[0], a.n[1]) : 1;
    if (parts > 1)
      hipLaunchKernelGGL((ft_gather<NY, NZ, true>), grid, dim3(256), lds, st, a, sign, te, parts, in, E, planar, out, tab);
    else
      hipLaunchKernelGGL((ft_gather<NY, NZ, false>), grid, dim3(256), lds, st, a, sign, te, 1, in, E, planar, out, tab);
    BSE_CHECK_LAUNCH();
    return BSE_OK;
  });
}

size_t ft_table_bytes(const FtArgs& a) {
  return 16 * ((size_t)a.n[0] * FT_MAXR + (size_t)a.n[1] * ft_side(a, 1) + (size_t)a.n[2] * ft_side(a, 2));
}

bse_status ft_table_launch(const FtArgs& a, double sign, double* out, hipStream_t st) {
  hipLaunchKernelGGL(ft_table, dim3(1), dim3(256), ft_table_bytes(a), st, a, sign, ft_side(a, 1), ft_side(a, 2),
                     (double2*)out);
  BSE_CHECK_LAUNCH();
  return BSE_OK;
}

}  // namespace bse
