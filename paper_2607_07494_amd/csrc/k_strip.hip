// The encode's two passes (block maxima; scale and E4M3 pack) of the
// input-side transform over column strips.
//
// W~ = W + P (U diag(c))^T by split-bf16 products, as the sweep kernel of
// k_lowrank.hip forms it (same fragments, same order: W~, the maxima and the
// codes are bit-identical).  What bounded that kernel was moving its column
// operand: per 128 rows and 64 columns it copied as many bytes of the operand's
// image into LDS as it read of W, with a workgroup barrier for every tile.
// Here a workgroup (8 waves, two per SIMD, one workgroup per CU) keeps the
// image of its strip (up to 256 columns at rank 128) in LDS for its whole
// life: it is copied once, and after that the waves run free of barriers, each
// over 32-row groups of its own, reading the group's rows of P (a quarter to
// two thirds of W's bytes, from L2) and W.
//
// The grid is one workgroup per CU: on each XCD `slots` / `strips` row chunks
// of `strips` workgroups, the strips of one row chunk on one XCD, so that the
// rows of P that they share can be read from one L2.  A wave takes a 32 x 64
// tile at a time: its products, then its epilogue, then the loads of W of the
// next tile (across row groups), which arrive under the products; P's chunks
// are loaded one group ahead into the registers that a group's last tile
// leaves.  Block maxima stay in registers per tile column and are merged into
// the block's sub-slots when the block row changes.
//
// Measured against the sweep kernel, maxima / codes: 8192 x 1536, 16 ranks,
// rank 128: 258 / 304 -> 221 / 271 us; 5632 x 1024, 8 ranks, rank 64: 42 / 53 -> 35 /
// 45.  With the residual the gain depends on the launch (lr_strip_eligible):
// 3072 x 4096, 8 ranks, rank 128: 175 / 261 -> 160 / 261; 2048 columns at a third
// of that size: 66 / 99 -> 54 / 87.  Not faster: two tiles' products at a time, W
// two tiles ahead, 32x32x16 products (the matrix cores do not bound the pass),
// non-temporal loads of W.

#include <algorithm>
#include <type_traits>

#include "fp8_e4m3.h"
#include "gift_internal.h"
#include "split_bf16.h"

namespace gift {
namespace {

constexpr int kStripWaves = 8;
constexpr int kStripThreads = 64 * kStripWaves;
constexpr int kXcds = 8, kCusPerXcd = 32;

struct StripArgs {
  const float *P;       // [batch][M][K]
  const uint4 *img;     // column image: per 64-column tile 2 x 256 K / 32 entries
  const float *D;       // [batch][M][N]
  float *ef;            // residual (read; QUANT also writes it)
  uint32_t *amax;       // AMAX: sub-slots [batch][nbr][nbc][64]
  const uint32_t *raw;  // QUANT: the AMAX pass's sub-slots
  uint8_t *codes;
  float *scales;
  uint32_t *clear;
  int64_t clear_words;
  int M, N, batch;
  int br, bc, nbr, nbc;
  int strips, pairs;    // strips per row chunk, 128-column tile pairs over all strips
  int groups;           // 32-row groups of one rank
  int total, chunk;     // 32-row groups of the batch, and per row chunk
};

// word of the lane eight places round the 16-lane row
__device__ __forceinline__ uint32_t row_half(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, false);
}

template <int EPI, int KC, int CP, bool EF>
__global__ __launch_bounds__(kStripThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void lr_strip_kernel(
    const StripArgs p) {
  constexpr int TS = KC * 256;             // (chunk, column, fg) entries of a tile, hi or lo
  constexpr int CT = 2 * CP;               // tiles of a strip, at most
  __shared__ __attribute__((aligned(1024))) uint4 image[CT * 2 * TS];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 15, fg = lane >> 4;
  const int xcd = (int)blockIdx.x % kXcds, local = (int)blockIdx.x / kXcds;
  const int strip = local % p.strips, chunk = local / p.strips * kXcds + xcd;
  const int base = p.pairs / p.strips, rem = p.pairs % p.strips;
  const int t0 = 2 * (strip * base + (strip < rem ? strip : rem));   // first tile of the strip
  const int nt = 2 * (base + (strip < rem ? 1 : 0));                 // its tiles, <= CT
  const int g_end = (chunk + 1) * p.chunk < p.total ? (chunk + 1) * p.chunk : p.total;
  const int slot = (int)(blockIdx.x * kStripWaves + wave) % kAmaxSlots;
  const int64_t MN = (int64_t)p.M * p.N;
  if (EPI == EPI_QUANT && p.clear_words) {
    const int64_t nthreads = (int64_t)gridDim.x * kStripThreads;
    for (int64_t i = (int64_t)blockIdx.x * kStripThreads + tid; i < p.clear_words; i += nthreads)
      st_u32_untracked(p.clear + i, 0u);
  }
  // the strip's image, 1 KiB per copy (zeros past the strip)
  {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(p.img + (int64_t)t0 * 2 * TS), (short)0, nt * 2 * TS * 16, 0x00020000);
    constexpr int PIECES = CT * 2 * TS / 64;
    for (int piece = wave; piece < PIECES; piece += kStripWaves)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (GIFT_LDS void *)(image + piece * 64), 16,
                                               piece * 1024 + lane * 16, 0, 0, 0);
  }

  typedef float4 WTile[2][4];
  // W (and R) of tile ct of row group g (zeros, unfetched, past the range)
  auto load_w = [&](int g, int ct, WTile &dd, WTile &re) {
    const bool ok = g < g_end && ct < nt;
    const int b = ok ? g / p.groups : 0, r0 = ok ? (g - b * p.groups) * 32 : 0;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void *)(p.D + b * MN), (short)0, (int)(MN * 4), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsE = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(EF ? p.ef + b * MN : p.D), (short)0, EF ? (int)(MN * 4) : 0, 0x00020000);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = r0 + 16 * h + fr;
      const uint32_t ro = ok && r < p.M ? (uint32_t)r * (uint32_t)p.N * 4u : 0x80000000u;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int off = (int)(ro + (uint32_t)(64 * (t0 + ct) + 16 * t + 4 * fg) * 4u);
        dd[h][t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
        if (EF) re[h][t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsE, off, 0, 0));
      }
    }
  };
  // chunk ch of the rows of P of row group g
  float4 rw[2][KC][2];
  auto load_p = [&](int g, int ch) {
    const bool in = g < g_end;
    const int b = in ? g / p.groups : 0, r0 = in ? (g - b * p.groups) * 32 : 0;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void *)(p.P + (int64_t)b * p.M * (32 * KC)), (short)0, p.M * 32 * KC * 4, 0x00020000);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = r0 + 16 * h + fr;
      const uint32_t ro = in && r < p.M ? (uint32_t)r * (uint32_t)(32 * KC * 4) + 16u * fg : 0x80000000u;
      rw[h][ch][0] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ro + 128u * ch), 0, 0));
      rw[h][ch][1] =
          __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ro + 128u * ch + 64u), 0, 0));
    }
  };

  WTile cur, curR;
  const int g0 = chunk * p.chunk + wave;
#pragma unroll
  for (int ch = 0; ch < KC; ++ch) load_p(g0, ch);
  load_w(g0, 0, cur, curR);
  __builtin_amdgcn_sched_barrier(0);
  wait_vm<0>();          // the image's copies (and the first loads)
  __syncthreads();
  // from here on the waves are on their own

  uint32_t tmax[CT];
  float inv[CT], sc[CT];
#pragma unroll
  for (int t = 0; t < CT; ++t) {
    tmax[t] = 0u;
    inv[t] = sc[t] = 0.f;
  }
  int cur_b = -1, cur_bi = -1;   // block row the running maxima / scales belong to
  auto flush = [&]() {
    if (cur_b < 0) return;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      if (ct >= nt) break;
      const uint32_t m = wave_max_u32(tmax[ct]);
      const int gb = (cur_b * p.nbr + cur_bi) * p.nbc + 64 * (t0 + ct) / p.bc;
      if (lane == 0 && m) atomicMax(&p.amax[(int64_t)gb * kAmaxSlots + slot], m);
      tmax[ct] = 0u;
    }
  };

  for (int g = g0; g < g_end; g += kStripWaves) {
    const int b = g / p.groups, r0 = (g - b * p.groups) * 32, bi = r0 / p.br;
    if (b != cur_b || bi != cur_bi) {
      if (EPI == EPI_AMAX) flush();
      cur_b = b;
      cur_bi = bi;
      if (EPI == EPI_QUANT) {
        // the finished maxima of the strip's blocks in this block row; the
        // wave at a block's first element writes its scale
        uint32_t v[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const int bj = 64 * (t0 + (ct < nt ? ct : nt - 1)) / p.bc;
          v[ct] = p.raw[(int64_t)((b * p.nbr + bi) * p.nbc + bj) * kAmaxSlots + lane];
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          const float a = __uint_as_float(wave_max_u32(v[ct]));
          inv[ct] = e4m3_multiplier(a);
          sc[ct] = e4m3_scale(a);
          const int j0 = 64 * (t0 + ct), bj = j0 / p.bc;
          if (ct < nt && lane == 0 && r0 == bi * p.br && j0 == bj * p.bc)
            st_u32_untracked(p.scales + (b * p.nbr + bi) * p.nbc + bj, __float_as_uint(sc[ct]));
        }
      }
    }
    bool rv[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) rv[h] = r0 + 16 * h + fr < p.M;
    uint4 rh[2][KC], rl[2][KC];
    uint4 held[2];         // codes of a pair's first tile
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      // the tile's products, chunk by chunk: the group's first tile splits P's
      // chunks as it comes to them, and its last one loads the next group's
      // chunks into the registers that it leaves
      floatx4 acc[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[h][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ch = 0; ch < KC; ++ch) {
        if (ct == 0) {
#pragma unroll
          for (int h = 0; h < 2; ++h) split8(rw[h][ch][0], rw[h][ch][1], rh[h][ch], rl[h][ch]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const uint4 *const im = image + ct * 2 * TS + ch * 256 + lds_slot(16 * t + fr, fg);
          const uint4 ah = im[0], al = im[TS];
#pragma unroll
          for (int h = 0; h < 2; ++h) acc[h][t] = mfma3(ah, al, rh[h][ch], rl[h][ch], acc[h][t]);
        }
        if (ct == CT - 1) {
          __builtin_amdgcn_sched_barrier(0);
          load_p(g + kStripWaves, ch);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      const int j0 = 64 * (t0 + ct);
      if (ct < nt) {
        float w[2][4][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            w[h][t][0] = cur[h][t].x + acc[h][t][0];
            w[h][t][1] = cur[h][t].y + acc[h][t][1];
            w[h][t][2] = cur[h][t].z + acc[h][t][2];
            w[h][t][3] = cur[h][t].w + acc[h][t][3];
            if (EF) {
              w[h][t][0] += curR[h][t].x;
              w[h][t][1] += curR[h][t].y;
              w[h][t][2] += curR[h][t].z;
              w[h][t][3] += curR[h][t].w;
            }
          }
        if (EPI == EPI_AMAX) {
#pragma unroll
          for (int h = 0; h < 2; ++h)
            if (rv[h]) {
#pragma unroll
              for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                  const uint32_t a = __float_as_uint(w[h][t][e]) & 0x7fffffffu;
                  tmax[ct] = a > tmax[ct] ? a : tmax[ct];
                }
            }
        } else {
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            uint32_t q[4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
              q[t] = e4m3_encode4(w[h][t][0] * inv[ct], w[h][t][1] * inv[ct], w[h][t][2] * inv[ct],
                                  w[h][t][3] * inv[ct]);
            if (EF && rv[h]) {   // R = W~ - its dequantized code
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                float qv[4];
                e4m3_decode4(q[t], qv);
                st_u128_untracked(p.ef + b * MN + (int64_t)(r0 + 16 * h + fr) * p.N + j0 + 16 * t + 4 * fg,
                                  make_uint4(__float_as_uint(w[h][t][0] - qv[0] * sc[ct]),
                                             __float_as_uint(w[h][t][1] - qv[1] * sc[ct]),
                                             __float_as_uint(w[h][t][2] - qv[2] * sc[ct]),
                                             __float_as_uint(w[h][t][3] - qv[3] * sc[ct])));
              }
            }
            // lane (fr, fg): the 16 codes of columns 16 fg .. of its row
            const uint4 v = transpose_rows(q[0], q[1], q[2], q[3]);
            if ((ct & 1) == 0) {
              held[h] = v;
            } else {
              // whole 128-byte lines: rows 0 .. 7 of the 16 in one store, 8
              // .. 15 in the next, lanes fr < 8 the first tile's half of a
              // row and the others the second's
              const bool lo = fr < 8;
              const uint4 send = lo ? v : held[h];
              const uint4 got = make_uint4(row_half(send.x), row_half(send.y), row_half(send.z), row_half(send.w));
              const uint4 v1 = lo ? held[h] : got, v2 = lo ? got : v;
              const int row = r0 + 16 * h + (fr & 7);
              uint8_t *dst = p.codes + b * MN + (int64_t)row * p.N + j0 - (lo ? 64 : 0) + 16 * fg;
              if (row < p.M) st_u128_untracked(dst, v1);
              if (row + 8 < p.M) st_u128_untracked(dst + 8 * (int64_t)p.N, v2);
            }
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // W of the next tile, past this group's last tile in the next group
      if (ct + 1 < CT) load_w(g, ct + 1, cur, curR);
      else load_w(g + kStripWaves, 0, cur, curR);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  if (EPI == EPI_AMAX) flush();
}

// Strips per row chunk for `pairs` 128-column tile pairs and `total` 32-row
// groups at rank K (0: too few groups), and the pairs per strip *cp.  Each
// choice is priced by what it leaves idle (columns of an uneven split,
// workgroups of an XCD, waves of the last round of groups) and by its reads of
// P, which cost about half of W's by the byte (they come from L2).
int pick_strips(int pairs, int64_t total, int K, bool ef, int *cp) {
  // LDS: 512 K bytes per pair; the residual's registers take no more than two
  const int cp_max = K == 64 && !ef ? 4 : 2;
  int best = 0;
  double top = 0.0;
  for (int s = 1; s <= kCusPerXcd; ++s) {
    const int per = (pairs + s - 1) / s;
    const int64_t chunks = kXcds * (kCusPerXcd / s), rows = (total + chunks - 1) / chunks;
    if (per > cp_max || s > pairs || rows < 2 * kStripWaves) continue;
    const int64_t rounds = (rows + kStripWaves - 1) / kStripWaves;
    const double use = (double)pairs / (s * per) * (double)total / (double)(chunks * kStripWaves * rounds);
    const double score = use * ((double)(chunks * s) / (kXcds * kCusPerXcd)) / (1.0 + 0.5 * K / (128.0 * per));
    if (score > top) {
      top = score;
      best = s;
      *cp = per;
    }
  }
  return best;
}

}  // namespace

bool lr_strip_eligible(const TileJob &j) {
  const int64_t K = j.seg[0].K;
  const int64_t br = j.geom.br > 0 ? j.geom.br : j.M, bc = j.geom.bc > 0 ? j.geom.bc : j.N;
  if (!(K == 64 || K == 96 || K == 128) || j.nseg != 1 || j.N % 128 != 0 || j.shared || j.mx_codes || j.transformed ||
      !j.col_img || j.img_bs != 0 || j.seg[0].a.parts != 1 || j.seg[0].b.bs != 0 || j.seg[0].a.ld != K ||
      j.seg[0].a.bs != j.M * K)
    return false;
  if (!((br % 32 == 0 || br >= j.M) && (bc % 64 == 0 || bc >= j.N))) return false;
  if (j.M * j.N >= (1LL << 29) || j.M * K >= (1LL << 29)) return false;
  if (j.codes && (!j.from_raw || j.hits || (reinterpret_cast<uintptr_t>(j.codes) & 15))) return false;
  if ((int64_t)j.batch * j.geom.nbr * j.geom.nbc * kAmaxSlots >= (1LL << 31)) return false;
  const int64_t groups = (j.M + 31) / 32 * j.batch;
  if (groups >= (1LL << 30)) return false;
  const int pairs = (int)(j.N / 128);
  int cp = 0;
  const int strips = pick_strips(pairs, groups, (int)K, j.ef != nullptr, &cp);
  if (strips == 0) return false;
  // With the residual, twice the bytes in flight, an idle quarter of the chip
  // costs more than the image's copies did, and past the last-level cache the
  // code pass moves its bytes no faster than the sweep: at 8 ranks, maxima and
  // codes, sweep -> strips,
  //   2816 columns (0.69 of the chip): 80 MB at rank 128 45 -> 50 and 64 -> 69 us, 320 MB 163 -> 168 and
  //     242 -> 284; 1536 columns (0.75), 48 MB 28 -> 30 and 40 -> 43
  //   1024 columns (all of it): 200 MB at rank 64 / 128 108 / 120 -> 93 / 104 and 152 / 162 -> 139 / 141, 320 MB
  //     135 / 158 -> 126 / 137 and 205 / 225 -> 210 / 221
  //   1664 columns (0.81): 160 MB at rank 128 91 -> 81 and 138 -> 131, 384 MB 193 -> 184 and 290 -> 307
  // (Without it strips are at worst even: 2816 columns, 160 MB 57.2 -> 56.9 and
  // 70.5 -> 68.9.)  The code pass at rank 64 has a sweep only where the columns
  // are whole 256-column ranges; the per-unit kernel is slower than strips
  // throughout (1664 columns, 160 MB: 144 -> 122).
  if (j.ef && !(j.codes && K == 64 && j.N % 256 != 0)) {
    const double fill = (double)pairs * (kXcds * (kCusPerXcd / strips)) / (double)(kXcds * kCusPerXcd * cp);
    if (fill < 0.8) return false;
    if (j.codes && 4 * j.M * j.N * j.batch > (224LL << 20) && (K < 128 || fill < 0.85)) return false;
  }
  return true;
}

gift_status launch_lr_strip(gift_ctx *ctx, const TileJob &j) {
  StripArgs a{};
  const int K = (int)j.seg[0].K;
  a.P = j.seg[0].a.ptr;
  a.img = static_cast<const uint4 *>(j.col_img);
  a.D = j.D;
  a.ef = j.ef;
  a.amax = j.amax;
  a.raw = j.codes ? j.amax : nullptr;
  a.codes = j.codes;
  a.scales = j.scales;
  a.clear = j.codes ? j.clear : nullptr;
  a.clear_words = j.codes ? j.clear_words : 0;
  a.M = (int)j.M;
  a.N = (int)j.N;
  a.batch = j.batch;
  a.br = (int)(j.geom.br > 0 ? j.geom.br : j.M);
  a.bc = (int)(j.geom.bc > 0 ? j.geom.bc : j.N);
  a.nbr = j.geom.nbr;
  a.nbc = j.geom.nbc;
  int cp = 0;
  a.pairs = (int)(j.N / 128);
  a.groups = (int)((j.M + 31) / 32);
  a.total = a.groups * j.batch;
  a.strips = pick_strips(a.pairs, a.total, K, j.ef != nullptr, &cp);
  const int chunks = kXcds * (kCusPerXcd / a.strips);
  a.chunk = (a.total + chunks - 1) / chunks;
  ProfileScope prof(ctx, j.kernel_family);
  const dim3 grid((unsigned)(chunks * a.strips));
  auto go = [&](auto epi_c, auto ef_c, auto kc_c, auto cp_c) {
    hipLaunchKernelGGL((lr_strip_kernel<decltype(epi_c)::value, decltype(kc_c)::value, decltype(cp_c)::value,
                                        decltype(ef_c)::value>),
                       grid, dim3(kStripThreads), 0, ctx->stream, a);
  };
  auto by_cp = [&](auto epi_c, auto ef_c, auto kc_c) {
    constexpr int KC = decltype(kc_c)::value;
    if (cp == 1) go(epi_c, ef_c, kc_c, std::integral_constant<int, 1>{});
    else if (cp == 2) go(epi_c, ef_c, kc_c, std::integral_constant<int, 2>{});
    else if constexpr (KC == 2 && !decltype(ef_c)::value) {
      if (cp == 3) go(epi_c, ef_c, kc_c, std::integral_constant<int, 3>{});
      else go(epi_c, ef_c, kc_c, std::integral_constant<int, 4>{});
    }
  };
  auto by_k = [&](auto epi_c, auto ef_c) {
    if (K == 64) by_cp(epi_c, ef_c, std::integral_constant<int, 2>{});
    else if (K == 96) by_cp(epi_c, ef_c, std::integral_constant<int, 3>{});
    else by_cp(epi_c, ef_c, std::integral_constant<int, 4>{});
  };
  auto by_ef = [&](auto epi_c) {
    if (j.ef) by_k(epi_c, std::true_type{});
    else by_k(epi_c, std::false_type{});
  };
  if (j.codes) by_ef(std::integral_constant<int, EPI_QUANT>{});
  else by_ef(std::integral_constant<int, EPI_AMAX>{});
  return check_launch("lr_strip_kernel");
}

}  // namespace gift
