// Dequantize-accumulate over the N data-parallel ranks held on this GPU
// (eq. dp_grad_avg; Algorithm 1's AllReduce_SUM followed by Dequantize / N,
// with each rank dequantized by its own block scale).
//
// mean[e] = fl32(acc / N), acc = fl32(acc + fl32(val(q_j[e]) * s_j[block(e)]))
// for j = 0..N-1 in order.  The translation unit is compiled without FMA
// contraction, so the result is bit-for-bit the sequence above.
//
// Layout: one workgroup (256 lanes) covers 16 rows x 64 columns, lane t row
// t/16 and the four columns 4*(t%16)..: the ranks' loads of a lane are the only
// ones it has in flight, so narrow workgroups, many of them (1001 x 2731, six
// ranks: 28 us at 256 columns and one rank's load at a time).  Block scales of
// the tile are staged in LDS.

#include "fp8_e4m3.h"
#include "gift_internal.h"

namespace gift {
namespace {

constexpr int kRows = 16, kCols = 64, kThreads = 256;
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

__global__ __launch_bounds__(kThreads) void reduce_kernel(const RArgs p) {
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
  const int64_t gj = j0 + 4 * q;
  if (gj >= p.n) return;
  {
    const bool full = gj + 3 < p.n;
    int lbl[4];   // local block of each column
    {
      int lbj = (int)((uint32_t)gj / bc);
      int64_t edge = (int64_t)(lbj + 1) * bc;
      lbj -= bj0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (gj + e == edge && gj + e < p.n) {
          ++lbj;
          edge += bc;
        }
        lbl[e] = lbi * nlbj + lbj;
      }
    }
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    const int64_t off = gi * p.n + gj;
    auto load = [&](int j) {
      const uint8_t *c = p.codes + j * mn + off;
      if (full) return (uint32_t)*reinterpret_cast<const u32u *>(c);
      uint32_t word = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (gj + e < p.n) word |= (uint32_t)c[e] << (8 * e);
      return word;
    };
    // four ranks' codes in flight together (rank order kept in the sums)
    for (int j0r = 0; j0r < p.N; j0r += 4) {
      uint32_t word[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) word[u] = load(j0r + u < p.N ? j0r + u : p.N - 1);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (j0r + u >= p.N) break;
        float d[4];
        e4m3_decode4(word[u], d);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float s =
              staged ? lds_s[(j0r + u) * (int)nlb + lbl[e]]
                     : p.scales[(j0r + u) * nblk + (int64_t)(bi0 + lbl[e] / nlbj) * p.nbc + bj0 + lbl[e] % nlbj];
          const float val = d[e] * s;
          acc[e] = acc[e] + val;
        }
      }
    }
    float *out = p.mean + off;
    if (full) {
      const float4u o = {acc[0] / fN, acc[1] / fN, acc[2] / fN, acc[3] / fN};
      *reinterpret_cast<float4u *>(out) = o;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (gj + e < p.n) out[e] = acc[e] / fN;
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
  dim3 grid((unsigned)((n + kCols - 1) / kCols), (unsigned)((m + kRows - 1) / kRows));
  hipLaunchKernelGGL(reduce_kernel, grid, dim3(kThreads), 0, ctx->stream, a);
  return check_launch("reduce_kernel");
}

}  // namespace gift
