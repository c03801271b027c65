// Separable Fourier sums between a set of lattice vectors and a product grid of q (fourier.hip).
#pragma once

#include "bse_internal.h"

namespace bse {

constexpr int FT_MAXQ = 24;   // grid points per axis
constexpr int FT_MAXR = 7;    // distinct R components per axis
constexpr int FT_BOX = FT_MAXR * FT_MAXR * FT_MAXR + 1;
constexpr int FT_MAXNR = 256;

// the larger of two non-negative numbers, a NaN above all: as bits it then passes an atomicMax too
__device__ __forceinline__ double max_or_nan(double a, double b) { return a > b || a != a ? a : b; }

// the axes of a sum, passed to the kernels by value (no table in device memory): under 4 KiB
struct FtArgs {
  int n[3], r[3], nR;
  double q[3][FT_MAXQ];       // fractional q of each axis
  short Rv[3][FT_MAXR + 1];   // R components of each axis, ascending
  double w[FT_MAXNR];         // weight of each listed R
  short map[FT_BOX];          // box slot (R1, R2, R3), the last two axes padded to odd sizes -> listed R or -1
};
static_assert(sizeof(FtArgs) <= 3600, "kernel argument");

// true when the q list is a product grid (last axis fastest) and the R are distinct vectors of a small box;
// w == nullptr: unit weights
bool ft_axes(FtArgs* a, int n_q, const double* q, int n_R, const int32_t* R, const double* w);

// out[q][e] = sum_R w_R in[R][e] exp(sign 2 pi i q.R).  mode 0: c128 out, 1: c64 out, 2: max |out - ref|.
// planar input: [R][E / group][2][group] doubles, summed over nsplit arrays split_stride doubles apart.
bse_status ft_spread_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, long long group,
                            int nsplit, long long split_stride, int mode, void* out, const double* ref, hipStream_t st,
                            const double* table = nullptr);
// out[R][e] = w_R sum_q in[q][e] exp(sign 2 pi i q.R); planar: out as [R][2][E]
bse_status ft_gather_launch(const FtArgs& a, double sign, const double* in, long long E, int planar, double* out,
                            hipStream_t st, const double* table = nullptr);
// the phases of the axes for one sign, as the kernels take them from `table`
size_t ft_table_bytes(const FtArgs& a);
bse_status ft_table_launch(const FtArgs& a, double sign, double* out, hipStream_t st);

}  // namespace bse
