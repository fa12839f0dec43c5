// The k x k float64 steps of the factor refresh on matrix-core tiles: the
// Cholesky factorisation and inverse of CholeskyQR (k <= 256) and the
// Rayleigh-Ritz eigensolver (64 < k <= 256).
//
// Both are chains of dependent steps on a matrix that one workgroup can hold,
// so what bounds them is the latency of a step, not arithmetic (the 256 x 256
// Cholesky is 5.6 Mflop).  The design takes steps out of the chain: the
// factorisation advances 16 columns per step instead of one, and the
// eigensolver's rounds run in LDS on pairs of column blocks, several
// workgroups per matrix.
//
// v_mfma_f64_16x16x4_f64: lane (n, g) = (lane % 16, lane / 16) supplies
// A[n][4 s + g] and B[4 s + g][n] in step s and holds D[4 v + g][n] in result
// register v.  A result tile's registers are therefore the B operand of the
// next product as they stand, and the A operand of its transpose: tiles go
// from register to matrix core with no rearrangement.

#include <type_traits>

#include "k_small.h"

namespace gift {
namespace {

typedef double doublex4 __attribute__((ext_vector_type(4)));

// 1 / sqrt(x): the hardware estimate (relative error 3.3e-8 measured) and one
// third-order step, which leaves its cube
__device__ __forceinline__ double rsqrt64(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  return fma(y * e, fma(0.375, e, 0.5), y);
}

__device__ __forceinline__ double rcp64(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}

__device__ __forceinline__ double readlane64(double v, int lane) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// lane S of each 16-lane row to the whole row
template <int S>
__device__ __forceinline__ double row_bcast(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + S, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + S, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

// v + (v of the lane R places further down the 16-lane row)
template <int R>
__device__ __forceinline__ double row_ror_add(double v) {
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + R, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + R, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}

// Sum over the 16 lanes of a row; every lane ends with the same bits.
__device__ __forceinline__ double row_sum(double v) {
  v = row_ror_add<8>(v);
  v = row_ror_add<4>(v);
  v = row_ror_add<2>(v);
  return row_ror_add<1>(v);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// ---------------------------------------------------------------------------
// Sum of the split-K partials, averaged with its transpose: a workgroup takes
// the 32 x 32 tiles (a, b) and (b, a), a <= b.  The consumer reads the upper
// triangle and whole diagonal tiles, so the lower tiles are not written.
// (The reads that one workgroup made for a whole matrix, 4 MB at k = 256 and
// 16 partials, are spread over 36 of them.)
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sum_kernel(const SmallJob *jobs) {
  __shared__ double lower[32][33];
  const SmallJob J = jobs[blockIdx.y];
  const int k = J.k, nt = (k + 31) / 32;
  if (!J.sum || (int)blockIdx.x >= nt * (nt + 1) / 2) return;   // (no sum: one partial, read as it is)
  int b = 0, at = (int)blockIdx.x;   // column tile b holds tiles (0 .. b, b)
  while (at > b) at -= ++b;
  const int a = at;
  const int c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
  const int64_t kk = (int64_t)k * k;
  auto total = [&](int row, int col) {
    double s = 0.0;
    if (row < k && col < k)
      for (int z = 0; z < J.ks; ++z) s += (double)J.part[z * kk + (int64_t)row * k + col];
    return s;
  };
#pragma unroll
  for (int u = 0; u < 4; ++u) lower[r0 + 8 * u][c] = total(32 * b + r0 + 8 * u, 32 * a + c);
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = 32 * a + r0 + 8 * u, col = 32 * b + c;
    const double s = a == b ? lower[r0 + 8 * u][c] : total(row, col);
    if (row < k && col < k) J.sum[(int64_t)row * k + col] = 0.5 * (s + lower[c][r0 + 8 * u]);
  }
}

// ---------------------------------------------------------------------------
// Cholesky in 16 x 16 register tiles, upper form G = R^T R.  NT / 2 waves;
// wave w owns the tile columns w and NT - 1 - w (NT + 1 tiles of the upper
// triangle for every wave) in registers.  Panel step p:
//   the owner of column p factors the diagonal tile in its registers, 16
//   column steps with the inverse alongside (Gauss-Jordan on [L | I]), and
//   leaves L_pp^-1 in LDS;
//   every wave forms R_pi = L_pp^-1 A_pi of its columns i > p and shares it
//   through LDS;
//   every wave updates A_qi -= R_pq^T R_pi.
// A pivot is max(G_jj, 1e-12 tr/k); rows and columns past k are the identity.
// The inverse Z = L^-1 (R^-1 = Z^T) goes by block columns, again NT + 1 tiles
// per wave: Z_ij = -L_ii^-1 sum_l R_li^T Z_lj, the tiles R_li of a step read
// back from memory through LDS one step ahead.
// A wave's two tile columns share one array of NT + 1 register tiles (slots),
// whose coordinates are wave-uniform: as two arrays of fixed rows they would
// take 3 NT / 2.  (136 registers of tiles at NT = 16; with the prefetched tiles
// of the inverse 148 bytes per lane go to scratch all the same.)
//
// Twelve matrices of k = 256 took 3.9 ms as a column-at-a-time kernel on
// global memory, 24 of k = 128 0.20 ms one column at a time in registers; this
// kernel 0.16 and 0.057 ms.
// ---------------------------------------------------------------------------
template <int NT>
__global__ __launch_bounds__(32 * NT) __attribute__((amdgpu_waves_per_eu(1, 2))) void chol_tile_kernel(
    const SmallJob *jobs, int eig) {
  constexpr int H = NT / 2;
  __shared__ double li[NT][16][17];            // L_pp^-1
  __shared__ double panel[2][NT][4][64];       // a panel's tiles, registers as they are
  __shared__ double red[2][H];
  const SmallJob J = jobs[blockIdx.x];
  const int k = J.k, nt = (k + 15) / 16;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 15, g = lane >> 4;
  const int ca = wave, cb = NT - 1 - wave;
  double t[NT + 1][4];                         // slots 0 .. ca: tiles (s, ca), then (s - ca - 1, cb)
  auto slot_row = [&](int s) { return s <= ca ? s : s - ca - 1; };
  auto slot_col = [&](int s) { return s <= ca ? ca : cb; };
  double trace = 0.0, squares = 0.0;
#pragma unroll
  for (int s = 0; s <= NT; ++s) {
    const int p = slot_row(s), i = slot_col(s);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * p + 4 * v + g, c = 16 * i + n;
      const bool in = r < k && c < k;
      const int lo = r < c ? r : c, hi = r < c ? c : r;
      const int64_t at = in ? (int64_t)lo * k + hi : 0;
      const double x = J.sum ? J.sum[at] : (double)J.part[at];
      t[s][v] = in ? x : (r == c ? 1.0 : 0.0);
      if (in) {
        squares += (p == i ? 1.0 : 2.0) * x * x;
        if (r == c) trace += x;
      }
    }
  }
  trace = wave_sum(trace);
  squares = wave_sum(squares);
  if (lane == 0) {
    red[0][wave] = trace;
    red[1][wave] = squares;
  }
  __syncthreads();
  trace = squares = 0.0;
#pragma unroll
  for (int w = 0; w < H; ++w) {
    trace += red[0][w];
    squares += red[1][w];
  }
  if (eig) {
    // a shift of 1e-5 |B|_F makes the factor of a Rayleigh-Ritz matrix exist
    // (the split-bf16 products of Q A at k <= 128 take an eigenvalue of 0 to
    // -1.2e-6 |B|_F at most, over spectra of one, ten, equal and i^-1.2
    // eigenvalues at dimensions 256 to 2816, random and all-positive bases;
    // float32 ones to a tenth of that); eigenvectors do not move, and the
    // finishing kernel takes it off the eigenvalues
    const double delta = 1e-5 * sqrt(squares);
#pragma unroll
    for (int s = 0; s <= NT; ++s)
      if (slot_row(s) == slot_col(s))
#pragma unroll
        for (int v = 0; v < 4; ++v) t[s][v] += 4 * v + g == n && 16 * slot_col(s) + n < k ? delta : 0.0;
    if (tid == 0) J.aux[k] = delta;
    if (tid < kJacobiSweeps) J.flags[tid] = 0;
  }
  const double floor = 1e-12 * (trace > 0.0 ? trace : 0.0) / k + 1e-300;

  // R tile (p, i) to where the caller wants it
  auto emit_r = [&](int p, int i, const double (&x)[4]) {
    float *const rf = J.rout;
    if (!eig && !rf) return;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * p + 4 * v + g, c = 16 * i + n;
      if (r < k && c < k) {
        if (eig) J.W[(int64_t)r * k + c] = x[v];
        else rf[(int64_t)r * k + c] = (float)x[v];
      }
    }
  };
  // the tile's registers to memory, for the inverse
  auto keep = [&](int p, int i, const double (&x)[4]) {
    double2 *q = reinterpret_cast<double2 *>(J.W + ((int64_t)(i * (i - 1) / 2 + p) * 64 + lane) * 4);
    q[0] = make_double2(x[0], x[1]);
    q[1] = make_double2(x[2], x[3]);
  };
  auto factor = [&](int p, double (&y)[4]) {
    double x[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = 4 * v + g == n ? 1.0 : 0.0;
    auto step = [&](auto sc) {
      constexpr int s = decltype(sc)::value, v0 = s / 4, g0 = s % 4;
      // row s of the tile and of the inverse to every 16-lane row
      const double row = __shfl(y[v0], n + 16 * g0), xrow = __shfl(x[v0], n + 16 * g0);
      const double d0 = readlane64(y[v0], s + 16 * g0);
      const double rs = rsqrt64(d0 > floor ? d0 : floor);
      const double rr = row * rs, xr = xrow * rs;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        if (4 * v + 3 <= s) continue;          // rows at or above s are final
        const double l = row_bcast<s>(y[v]) * (4 * v + g > s ? rs : 0.0);
        y[v] = fma(-l, rr, y[v]);
        x[v] = fma(-l, xr, x[v]);
      }
      if (g == g0) {
        y[v0] = rr;
        x[v0] = xr;
      }
    };
#define GIFT_STEP(S) step(std::integral_constant<int, S>{})
    GIFT_STEP(0); GIFT_STEP(1); GIFT_STEP(2); GIFT_STEP(3); GIFT_STEP(4); GIFT_STEP(5); GIFT_STEP(6); GIFT_STEP(7);
    GIFT_STEP(8); GIFT_STEP(9); GIFT_STEP(10); GIFT_STEP(11); GIFT_STEP(12); GIFT_STEP(13); GIFT_STEP(14);
    GIFT_STEP(15);
#undef GIFT_STEP
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (n < 4 * v + g) y[v] = 0.0;
      if (n > 4 * v + g) x[v] = 0.0;
      li[p][4 * v + g][n] = x[v];
    }
    emit_r(p, p, y);
  };
  // L_pp^-1 y, the panel's R tile of column i, shared and kept
  auto solve = [&](int p, int i, double (&y)[4]) {
    doublex4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(li[p][n][4 * s + g], y[s], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      y[v] = acc[v];
      panel[0][i][v][lane] = acc[v];
    }
    emit_r(p, i, y);
    if (!eig) keep(p, i, y);
  };
  // y -= a^T r
  auto update = [&](const double (&a)[4], const double (&r)[4], double (&y)[4]) {
    doublex4 acc = {y[0], y[1], y[2], y[3]};
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], -r[s], acc, 0, 0, 0);
#pragma unroll
    for (int v = 0; v < 4; ++v) y[v] = acc[v];
  };

  // (the step is one piece of code: the tiles of row p come out of their
  // registers by a chain of scalar branches)
  for (int p = 0; p < nt; ++p) {
    double ra[4] = {0.0, 0.0, 0.0, 0.0}, rb[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s <= NT; ++s)
      if (slot_row(s) == p) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (s <= ca) ra[v] = t[s][v];
          else rb[v] = t[s][v];
        }
      }
    if (ca == p) factor(p, ra);
    if (cb == p) factor(p, rb);
    __syncthreads();
    if (ca > p && ca < nt) solve(p, ca, ra);
    if (cb > p && cb < nt) solve(p, cb, rb);
    __syncthreads();
#pragma unroll
    for (int s = 0; s <= NT; ++s) {
      const int q = slot_row(s);
      if (q > p && slot_col(s) < nt) {
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = panel[0][q][u][lane];
        if (s <= ca) update(a, ra, t[s]);
        else update(a, rb, t[s]);
      }
    }
  }

  // zeros below the diagonal tiles of R
  if (eig || J.rout) {
    const double zero[4] = {0.0, 0.0, 0.0, 0.0};
    for (int p = ca + 1; p < nt; ++p) emit_r(p, ca, zero);
    for (int p = cb + 1; p < nt; ++p) emit_r(p, cb, zero);
  }
  if (eig) return;

  // ------------------------------------------------------------------ inverse
  // slots 0 .. NT - 1 - ca: Z tiles (ca + s, ca), then (cb + s - (NT - ca), cb)
  auto inv_row = [&](int s) { return s < NT - ca ? ca + s : cb + s - (NT - ca); };
  auto inv_col = [&](int s) { return s < NT - ca ? ca : cb; };
#pragma unroll
  for (int s = 0; s <= NT; ++s)
#pragma unroll
    for (int v = 0; v < 4; ++v) t[s][v] = inv_row(s) == inv_col(s) && inv_row(s) < nt ? li[inv_row(s)][4 * v + g][n] : 0.0;
  // tiles (0 .. i - 1, i) of step i: one after another in memory
  constexpr int PER = (NT - 1 + H - 1) / H;    // tiles a wave fetches per step
  double2 pre[PER][2];
  auto fetch = [&](int i) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int l = wave + H * u;
      if (l < i) {
        const double2 *q = reinterpret_cast<const double2 *>(J.W + ((int64_t)(i * (i - 1) / 2 + l) * 64 + lane) * 4);
        pre[u][0] = q[0];
        pre[u][1] = q[1];
      }
    }
  };
  __syncthreads();   // the kept tiles of every wave
  fetch(1 < nt ? 1 : 0);
  for (int i = 1; i < nt; ++i) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int l = wave + H * u;
      if (l < i) {
        panel[i & 1][l][0][lane] = pre[u][0].x;
        panel[i & 1][l][1][lane] = pre[u][0].y;
        panel[i & 1][l][2][lane] = pre[u][1].x;
        panel[i & 1][l][3][lane] = pre[u][1].y;
      }
    }
    if (i + 1 < nt) fetch(i + 1);
    __syncthreads();
    doublex4 sa = {0.0, 0.0, 0.0, 0.0}, sb = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s <= NT; ++s) {
      const int l = inv_row(s);
      if (l < i) {
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = panel[i & 1][l][u][lane];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (s < NT - ca) sa = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], t[s][u], sa, 0, 0, 0);
          else sb = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], t[s][u], sb, 0, 0, 0);
        }
      }
    }
    doublex4 da = {0.0, 0.0, 0.0, 0.0}, db = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const double a = li[i][n][4 * u + g];
      da = __builtin_amdgcn_mfma_f64_16x16x4f64(a, sa[u], da, 0, 0, 0);
      db = __builtin_amdgcn_mfma_f64_16x16x4f64(a, sb[u], db, 0, 0, 0);
    }
#pragma unroll
    for (int s = 1; s <= NT; ++s)
      if (inv_row(s) == i && inv_col(s) < i) {
#pragma unroll
        for (int v = 0; v < 4; ++v) t[s][v] = s < NT - ca ? -da[v] : -db[v];
      }
  }
  // R^-1 = Z^T: tile (i, j) of Z transposed, zeros below the diagonal tiles
  auto emit_inv = [&](int i, int j, const double (&z)[4]) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = 16 * j + n, c = 16 * i + 4 * v + g;
      if (r < k && c < k) J.out[(int64_t)r * k + c] = (float)z[v];
    }
  };
  const double zero[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s <= NT; ++s) emit_inv(inv_row(s), inv_col(s), t[s]);
  for (int i = 0; i < ca; ++i) emit_inv(i, ca, zero);
  for (int i = 0; i < cb; ++i) emit_inv(i, cb, zero);
}

// ---------------------------------------------------------------------------
// One-sided Jacobi on the columns of the Cholesky factor L of B + delta I
// (Veselic and Hari): rotating the columns of L until they are mutually
// orthogonal gives L V = U diag(sigma) with U the eigenvectors of B and
// sigma^2 - delta its eigenvalues.  The cosines between columns of L are
// B_pq / sqrt(B_pp B_qq), small from the start when B is nearly diagonal (a
// warm refresh), where those between columns of B itself grow with
// sqrt(B_pp / B_qq): fewer sweeps.
//
// Round-robin over blocks of 32 columns: a launch is one round, a workgroup
// one block pair, its 64 columns in LDS.  16 lanes hold one column pair; the
// left column of a pair stays in their registers for the 32 rounds against
// the right block, so a round reads and writes one column per pair.  Round 0
// of a sweep also takes the pairs inside both blocks.  Every pair is met once
// per sweep, as in one workgroup walking the whole matrix, but the rounds of
// disjoint block pairs run side by side and none of them touches global
// memory.  A warm refresh of 12 factors at k = 256: 23.1 ms with one workgroup
// per matrix on global memory, 2.1 ms here (10 sweeps launched); 24 factors at
// k = 128: 1.6 ms (one workgroup, LDS) against 0.75 ms.
// Squared norms are carried through the rotations and formed anew by every
// launch.
// ---------------------------------------------------------------------------
constexpr int kJB = 32;                        // columns per block

// rotation for columns of squared norms alpha, beta and inner product gamma != 0
__device__ __forceinline__ void rotation(double alpha, double beta, double gamma, double &c, double &s, double &t) {
  const double d = beta - alpha, w = 2.0 * gamma;
  const double x = fma(d, d, w * w);
  const double h = x * rsqrt64(x);             // sqrt((beta - alpha)^2 + 4 gamma^2)
  t = w * rcp64((d >= 0.0 ? h : -h) + d);
  c = rsqrt64(fma(t, t, 1.0));
  s = c * t;
}

template <int EL>
__global__ __launch_bounds__(512) void jacobi_block_kernel(const SmallJob *jobs, int sweep, int round) {
  constexpr int S = 16 * EL + 16;              // column stride: neighbours 128 bytes apart in the banks
  __shared__ double col[2 * kJB][S];
  __shared__ double norm2[2 * kJB];
  __shared__ int big;
  const SmallJob J = jobs[blockIdx.y];
  const int k = J.k, nb = ((k + kJB - 1) / kJB + 1) & ~1;   // blocks, even (the last may be empty)
  if (round >= nb - 1 || (int)blockIdx.x >= nb / 2) return;
  if (sweep > 0 && J.flags[sweep - 1] == 0) return;         // orthogonal after the sweep before
  int bp, bq;
  if (blockIdx.x == 0) {
    bp = round;
    bq = nb - 1;
  } else {
    bp = (round + (int)blockIdx.x) % (nb - 1);
    bq = (round - (int)blockIdx.x + nb - 1) % (nb - 1);
  }
  const int tid = threadIdx.x, grp = tid >> 4, l16 = tid & 15;
  const int cp = bp * kJB + grp, cq = bq * kJB + grp;       // this group's columns in memory
  double a[EL], b[EL];
  const double delta = J.aux[k];
  if (tid == 0) big = 0;
  auto square = [&](const double (&x)[EL]) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int e = 0; e < EL; e += 2) {
      s0 = fma(x[e], x[e], s0);
      s1 = fma(x[e + 1], x[e + 1], s1);
    }
    return row_sum(s0 + s1);
  };
#pragma unroll
  for (int e = 0; e < EL; ++e) {
    const int r = l16 + 16 * e;
    a[e] = r < k && cp < k ? J.W[(int64_t)cp * k + r] : 0.0;
    b[e] = r < k && cq < k ? J.W[(int64_t)cq * k + r] : 0.0;
  }
  double alpha = square(a);
  {
    const double beta = square(b);
#pragma unroll
    for (int e = 0; e < EL; ++e) {
      col[grp][l16 + 16 * e] = a[e];
      col[kJB + grp][l16 + 16 * e] = b[e];
    }
    if (l16 == 0) {
      norm2[grp] = alpha;
      norm2[kJB + grp] = beta;
    }
  }
  __syncthreads();
  bool any_big = false;
  // orthogonality is judged against the eigenvalues themselves, without the
  // shift (down to 1e-3 delta, below the noise of B)
  const double low = 1e-3 * delta;
  auto scale = [&](double al, double be) {
    const double p = al - delta > low ? al - delta : low, q = be - delta > low ? be - delta : low;
    return p * q;
  };
  constexpr double tol2 = kJacobiTol * kJacobiTol, last2 = kJacobiLast * kJacobiLast;
  auto dot = [&](const double (&x)[EL], const double (&y)[EL]) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int e = 0; e < EL; e += 2) {
      s0 = fma(x[e], y[e], s0);
      s1 = fma(x[e + 1], y[e + 1], s1);
    }
    return row_sum(s0 + s1);
  };

  if (round == 0) {
    // pairs inside the blocks: groups 0-15 in block p, 16-31 in block q
    const int side = grp >> 4, pi = grp & 15;
    const int c0 = (side ? bq : bp) * kJB;
    for (int rd = 0; rd < kJB - 1; ++rd) {
      int p, q;
      if (pi == 0) {
        p = rd;
        q = kJB - 1;
      } else {
        p = (rd + pi) % (kJB - 1);
        q = (rd - pi + kJB - 1) % (kJB - 1);
      }
      if (p > q) {
        const int t = p;
        p = q;
        q = t;
      }
      if (c0 + q < k) {
        double *const x = col[side * kJB + p] + l16, *const y = col[side * kJB + q] + l16;
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          a[e] = x[16 * e];
          b[e] = y[16 * e];
        }
        const double al = norm2[side * kJB + p], be = norm2[side * kJB + q];
        const double gamma = dot(a, b), g2 = gamma * gamma, sc = scale(al, be);
        if (g2 > tol2 * sc && g2 > 0.0) {
          double c, s, t;
          rotation(al, be, gamma, c, s, t);
#pragma unroll
          for (int e = 0; e < EL; ++e) {
            x[16 * e] = c * a[e] - s * b[e];
            y[16 * e] = s * a[e] + c * b[e];
          }
          if (l16 == 0) {
            norm2[side * kJB + p] = al - t * gamma;
            norm2[side * kJB + q] = be + t * gamma;
          }
          any_big = any_big || g2 > last2 * sc;
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int e = 0; e < EL; ++e) a[e] = col[grp][l16 + 16 * e];
    alpha = norm2[grp];
  }

  for (int s0 = 0; s0 < kJB; ++s0) {
    const int q = (grp + s0) & (kJB - 1);
    if (cp < k && bq * kJB + q < k) {
      double *const y = col[kJB + q] + l16;
#pragma unroll
      for (int e = 0; e < EL; ++e) b[e] = y[16 * e];
      const double beta = norm2[kJB + q];
      const double gamma = dot(a, b), g2 = gamma * gamma, sc = scale(alpha, beta);
      if (g2 > tol2 * sc && g2 > 0.0) {
        double c, s, t;
        rotation(alpha, beta, gamma, c, s, t);
#pragma unroll
        for (int e = 0; e < EL; ++e) {
          y[16 * e] = s * a[e] + c * b[e];
          a[e] = c * a[e] - s * b[e];
        }
        alpha -= t * gamma;
        if (l16 == 0) norm2[kJB + q] = beta + t * gamma;
        any_big = any_big || g2 > last2 * sc;
      }
    }
    __syncthreads();
  }
  if (any_big && l16 == 0) big = 1;
#pragma unroll
  for (int e = 0; e < EL; ++e) {
    const int r = l16 + 16 * e;
    if (r < k && cp < k) J.W[(int64_t)cp * k + r] = a[e];
    if (r < k && cq < k) J.W[(int64_t)cq * k + r] = col[kJB + grp][r];
  }
  __syncthreads();
  if (tid == 0 && big) atomicOr(&J.flags[sweep], 1);
}

// Sorted eigenpairs from the orthogonal columns.  A matrix whose last
// launched sweep still rotated noticeably (none seen in practice) is finished
// here first, by the one workgroup.
__global__ __launch_bounds__(1024) void jacobi_finish_kernel(const SmallJob *jobs) {
  __shared__ int any_big;
  __shared__ double norms[kSmallMax];
  __shared__ int perm[kSmallMax];
  const SmallJob J = jobs[blockIdx.x];
  const int k = J.k, tid = threadIdx.x, l16 = tid & 15, grp = tid >> 4;
  const double delta = J.aux[k];
  if (J.flags[kJacobiSweeps - 1] != 0) {
    const int kp = (k + 1) & ~1;
    constexpr double tol2 = kJacobiTol * kJacobiTol, last2 = kJacobiLast * kJacobiLast;
    for (int sweep = 0; sweep < 30; ++sweep) {
      if (tid == 0) any_big = 0;
      __syncthreads();
      for (int rd = 0; rd < kp - 1; ++rd) {
        for (int pi = grp; pi < kp / 2; pi += 64) {
          int p = pi == 0 ? rd : (rd + pi) % (kp - 1);
          int q = pi == 0 ? kp - 1 : (rd - pi + kp - 1) % (kp - 1);
          if (p > q) {
            const int t = p;
            p = q;
            q = t;
          }
          if (q >= k) continue;
          double *const x = J.W + (int64_t)p * k, *const y = J.W + (int64_t)q * k;
          double al = 0.0, be = 0.0, ga = 0.0;
          for (int r = l16; r < k; r += 16) {
            al = fma(x[r], x[r], al);
            be = fma(y[r], y[r], be);
            ga = fma(x[r], y[r], ga);
          }
          al = row_sum(al);
          be = row_sum(be);
          ga = row_sum(ga);
          const double sc = al * be;
          if (ga * ga > tol2 * sc && ga * ga > 0.0) {
            double c, s, t;
            rotation(al, be, ga, c, s, t);
            for (int r = l16; r < k; r += 16) {
              const double u = x[r], w = y[r];
              x[r] = c * u - s * w;
              y[r] = s * u + c * w;
            }
            if (l16 == 0 && ga * ga > last2 * sc) any_big = 1;
          }
        }
        __syncthreads();
      }
      const int again = any_big;
      __syncthreads();
      if (!again) break;
    }
  }
  for (int c = grp; c < k; c += 64) {
    double s = 0.0;
    for (int r = l16; r < k; r += 16) s = fma(J.W[(int64_t)c * k + r], J.W[(int64_t)c * k + r], s);
    s = row_sum(s);
    if (l16 == 0) norms[c] = s;
  }
  __syncthreads();
  // (a NaN norm ranks last: the ranks are a permutation whatever the norms)
  for (int j = tid; j < k; j += 1024) {
    const double v = norms[j], kv = v == v ? v : -1.0;
    int rank = 0;
    for (int l = 0; l < k; ++l) {
      const double ku = norms[l] == norms[l] ? norms[l] : -1.0;
      rank += (ku > kv) || (ku == kv && l < j);
    }
    J.theta[rank] = (float)(v - delta);
    perm[rank] = j;
  }
  __syncthreads();
  for (int t = tid; t < k * k; t += 1024) {
    const int i = t / k, c = t - i * k;
    const double v = norms[perm[c]];
    J.out[t] = (float)(J.W[(int64_t)perm[c] * k + i] * (v > 0.0 ? rsqrt64(v) : 0.0));
  }
}

}  // namespace

gift_status launch_k_sum(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax, int kernel_family) {
  if (count <= 0) return GIFT_OK;
  const int nt = (kmax + 31) / 32;
  ProfileScope prof(ctx, kernel_family);
  hipLaunchKernelGGL(k_sum_kernel, dim3(nt * (nt + 1) / 2, count), dim3(256), 0, ctx->stream, jobs);
  return check_launch("k_sum_kernel");
}

gift_status launch_chol_tiles(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax, bool eig) {
  if (count <= 0) return GIFT_OK;
  ProfileScope prof(ctx, eig ? GIFT_KERNEL_EIG : GIFT_KERNEL_CHOL);
  if (kmax <= 128)
    hipLaunchKernelGGL(chol_tile_kernel<8>, dim3(count), dim3(256), 0, ctx->stream, jobs, eig ? 1 : 0);
  else
    hipLaunchKernelGGL(chol_tile_kernel<16>, dim3(count), dim3(512), 0, ctx->stream, jobs, eig ? 1 : 0);
  return check_launch("chol_tile_kernel");
}

gift_status launch_eig_blocks(gift_ctx *ctx, const SmallJob *jobs, int count, int kmax) {
  if (count <= 0) return GIFT_OK;
  gift_status st = launch_chol_tiles(ctx, jobs, count, kmax, true);
  if (st != GIFT_OK) return st;
  ProfileScope prof(ctx, GIFT_KERNEL_EIG);
  const int nb = ((kmax + kJB - 1) / kJB + 1) & ~1;
  for (int sweep = 0; sweep < kJacobiSweeps; ++sweep)
    for (int round = 0; round < nb - 1; ++round) {
      const dim3 grid(nb / 2, count);
      if (kmax <= 128)
        hipLaunchKernelGGL(jacobi_block_kernel<8>, grid, dim3(512), 0, ctx->stream, jobs, sweep, round);
      else
        hipLaunchKernelGGL(jacobi_block_kernel<16>, grid, dim3(512), 0, ctx->stream, jobs, sweep, round);
    }
  hipLaunchKernelGGL(jacobi_finish_kernel, dim3(count), dim3(1024), 0, ctx->stream, jobs);
  return check_launch("jacobi kernels");
}

}  // namespace gift
