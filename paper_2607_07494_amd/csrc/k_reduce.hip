// Dequantize-accumulate over the N data-parallel ranks held on this GPU
// (eq. dp_grad_avg; Algorithm 1's AllReduce_SUM followed by Dequantize / N,
// with each rank dequantized by its own block scale).
//
// mean[e] = fl32(acc / N), acc = fl32(acc + fl32(val(q_j[e]) * s_j[block(e)]))
// for j = 0..N-1 in order.  The translation unit is compiled without FMA
// contraction, so the result is bit-for-bit the sequence above.
//
// Layout: one workgroup (256 lanes) covers 16 rows x 64 V columns, lane t row
// t/16 and the four columns 4*(t%16).. of each 64.  The loads of U ranks are the
// only ones a lane has in flight, so narrow workgroups, many of them, where
// there are ranks to load together (V = 1, U = 4: 1001 x 2731, six ranks: 28 us
// with wide ones and one rank's load at a time, 17 here).  Up to three ranks
// are too few for that: the workgroup's start and end outweigh its loads, and
// wide ones with a rank at a time are faster (V = 4, U = 1: 3000 x 2001, one /
// two / three ranks 23.1 / 22.3 / 22.6 -> 15.6 / 16.9 / 18.1 us; 8191 x 4095
// 102 / 106 / 110 -> 56 / 63 / 72).  Block scales of the tile are staged in LDS.

#include "fp8_e4m3.h"
#include "gift_internal.h"

namespace gift {
namespace {

constexpr int kRows = 16, kThreads = 256;
constexpr int kMaxScales = 4096;

struct RArgs {
  const uint8_t *codes;
  const float *scales;
  float *mean;
  int64_t m, n;
  int64_t br, bc;
  int nbr, nbc;
  int N;
};

// accesses at any byte's / float's address: rows of an odd length start
// anywhere, and the memory path takes a wide access there as one
typedef uint32_t u32u __attribute__((aligned(1)));
typedef float float4u __attribute__((ext_vector_type(4), aligned(4)));

template <int V, int U>
__global__ __launch_bounds__(kThreads) void reduce_kernel(const RArgs p) {
  constexpr int kCols = 64 * V;
  __shared__ float lds_s[kMaxScales];
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.y * kRows, j0 = (int64_t)blockIdx.x * kCols;
  const int64_t i1 = i0 + kRows < p.m ? i0 + kRows : p.m;
  const int64_t j1 = j0 + kCols < p.n ? j0 + kCols : p.n;
  // (rows and columns fit 31 bits: 32-bit divisions)
  const uint32_t br = (uint32_t)p.br, bc = (uint32_t)p.bc;
  const int bi0 = (int)((uint32_t)i0 / br), bj0 = (int)((uint32_t)j0 / bc);
  const int nlbj = (int)((uint32_t)(j1 - 1) / bc) - bj0 + 1;
  const int64_t nlb = (int64_t)((int)((uint32_t)(i1 - 1) / br) - bi0 + 1) * nlbj;
  const int64_t nblk = (int64_t)p.nbr * p.nbc;
  const bool staged = nlb * p.N <= kMaxScales;
  if (staged) {
    for (int t = tid; t < (int)nlb * p.N; t += kThreads) {
      const int j = t / (int)nlb, l = t % (int)nlb;
      const int64_t bi = bi0 + l / nlbj, bj = bj0 + l % nlbj;
      lds_s[t] = p.scales[j * nblk + bi * p.nbc + bj];
    }
  }
  __syncthreads();

  const int64_t gi = i0 + tid / 16;
  if (gi >= p.m) return;
  const int q = tid % 16;
  const int lbi = (int)((uint32_t)gi / br) - bi0;
  const int64_t mn = p.m * p.n;
  const float fN = (float)p.N;
  if (V == 1 && j0 + 4 * q >= p.n) return;
  bool full[V];
  int lbl[V][4];   // local block of each column
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int64_t gj = j0 + 64 * v + 4 * q;
    full[v] = gj + 3 < p.n;
    int lbj = (int)((uint32_t)gj / bc);
    int64_t edge = (int64_t)(lbj + 1) * bc;
    lbj -= bj0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (gj + e == edge && gj + e < p.n) {
        ++lbj;
        edge += bc;
      }
      lbl[v][e] = lbi * nlbj + lbj;
    }
  }
  float acc[V][4];
#pragma unroll
  for (int v = 0; v < V; ++v)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[v][e] = 0.f;
  const int64_t off = gi * p.n + j0 + 4 * q;
  auto load = [&](int j, int v) {
    const uint8_t *c = p.codes + j * mn + off + 64 * v;
    if (full[v]) return (uint32_t)*reinterpret_cast<const u32u *>(c);
    uint32_t word = 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j0 + 64 * v + 4 * q + e < p.n) word |= (uint32_t)c[e] << (8 * e);
    return word;
  };
  // U ranks' codes in flight together (rank order kept in the sums)
  for (int j0r = 0; j0r < p.N; j0r += U) {
    uint32_t word[U][V];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) word[u][v] = load(j0r + u < p.N ? j0r + u : p.N - 1, v);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (j0r + u >= p.N) break;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        if (V > 1 && j0 + 64 * v + 4 * q >= p.n) continue;
        float d[4];
        e4m3_decode4(word[u][v], d);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int l = lbl[v][e];
          const float s = staged ? lds_s[(j0r + u) * (int)nlb + l]
                                 : p.scales[(j0r + u) * nblk + (int64_t)(bi0 + l / nlbj) * p.nbc + bj0 + l % nlbj];
          const float val = d[e] * s;
          acc[v][e] = acc[v][e] + val;
        }
      }
    }
  }
  float *out = p.mean + off;
#pragma unroll
  for (int v = 0; v < V; ++v) {
    if (full[v]) {
      const float4u o = {acc[v][0] / fN, acc[v][1] / fN, acc[v][2] / fN, acc[v][3] / fN};
      *reinterpret_cast<float4u *>(out + 64 * v) = o;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (j0 + 64 * v + 4 * q + e < p.n) out[64 * v + e] = acc[v][e] / fN;
    }
  }
}

}  // namespace

gift_status launch_reduce(gift_ctx *ctx, const uint8_t *codes, const float *scales, int32_t N,
                          int64_t m, int64_t n, BlockGeom g, float *mean) {
  if (m <= 0 || n <= 0) return GIFT_OK;
  if (stream_eligible(m, n, g, mean, codes, nullptr, nullptr))
    return launch_stream_reduce(ctx, codes, scales, N, m, n, g, mean);
  RArgs a{};
  a.codes = codes;
  a.scales = scales;
  a.mean = mean;
  a.m = m;
  a.n = n;
  a.br = g.br;
  a.bc = g.bc;
  a.nbr = g.nbr;
  a.nbc = g.nbc;
  a.N = N;
  ProfileScope prof(ctx, GIFT_KERNEL_REDUCE);
  // (three ranks one after the other only where there are workgroups enough to
  // cover the waits, two per CU: 1001 x 2731 13.4 -> 12.0 us, 700 x 515 6.0 -> 7.1)
  const int64_t wide = (m + kRows - 1) / kRows * ((n + 255) / 256);
  const bool four = N <= 2 || (N == 3 && wide >= 512);
  const int cols = four ? 256 : 64;
  const dim3 grid((unsigned)((n + cols - 1) / cols), (unsigned)((m + kRows - 1) / kRows));
  if (four)
    hipLaunchKernelGGL((reduce_kernel<4, 1>), grid, dim3(kThreads), 0, ctx->stream, a);
  else
    hipLaunchKernelGGL((reduce_kernel<1, 4>), grid, dim3(kThreads), 0, ctx->stream, a);
  return check_launch("reduce_kernel");
}

}  // namespace gift
