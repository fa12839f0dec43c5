// The k x k float64 steps of the factor refresh (k_small.hip): CholeskyQR's
// Cholesky and R^-1, and the Rayleigh-Ritz eigensolver, up to k = 256.
#pragma once

#include "gift_internal.h"

namespace gift {

// One member's k x k step: partial products in, factor or eigenpairs out.
struct SmallJob {
  const float *part;     // [ks][k][k] split-K partials of the k x k product
  float *out;            // R^-1 (Cholesky) or V (eigensolver), [k][k] row-major
  float *theta;          // eigenvalues [k] (eigensolver)
  double *W;             // [k][k + 1] float64 scratch
  double *aux;           // [2k + 64] float64 scratch
  int ks, k;
  float *rout;           // optional R [k][k] (Cholesky, upper triangular)
  double *sum;           // [k][k] float64: the summed partials (k_sum), or null: part is the sum
  int *flags;            // [kJacobiSweeps] sweep flags of the eigensolver
};

constexpr int kSmallMax = 256;      // k of the register-tile kernels
constexpr int kJacobiSweeps = 10;   // block Jacobi sweeps launched before the finishing kernel

// Columns count as orthogonal once |<p,q>| <= 1e-10 |p| |q|: B comes from
// float32 products (relative noise ~1e-7), so rotating further changes nothing
// the codec can see.  Sweeps stop after the first one whose largest rotated
// |<p,q>| / (|p| |q|) is at most kJacobiLast: the next sweep would leave only
// about its square.
constexpr double kJacobiTol = 1e-10;
constexpr double kJacobiLast = 1e-6;

// sum[i][j] = the partials' sum in float64, z in order, averaged with its
// transpose, for the jobs jobs[0 .. count) of k <= kmax
gift_status launch_k_sum(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax, int kernel_family);
// Cholesky of the jobs' sums (k <= kmax <= kSmallMax): eig = false: R^-1 (and
// R) in float32; eig = true: W[j][i] = column j of the Cholesky factor L of
// sum + delta I (aux[k] = delta), sweep flags cleared
gift_status launch_chol_tiles(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax, bool eig);
// Eigenpairs of jobs of 64 < k <= kmax <= kSmallMax whose sums are ready
gift_status launch_eig_blocks(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax);

}  // namespace gift
