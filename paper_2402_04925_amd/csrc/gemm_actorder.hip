// Act-order product for more than 64 rows on gfx950 (and sorted rows whose
// groups are not whole 32-row steps): the weights are dequantized once, row by
// row through g_idx, into 16-bit values in MFMA operand order, and multiplied
// by a dense MFMA kernel.
//
// The per-row metadata costs eight (scale, zero) lookups per packed word. In
// launches of 64 rows (the decode kernels) every launch pays them again and
// streams all weights again: 6144 x 6144 at M = 512, 8 launches of 77 us. Here
// they are paid once, and the dense kernel has no VALU work per weight; the
// price is 2 K N bytes written and read, in chunks of columns that stay in the
// 256 MB last-level cache. Each weight is s (q - z) rounded once to the
// element type, as the decode kernels do.
#include "kernels_common.h"

#include <algorithm>
#include <type_traits>

namespace tpdq {
namespace {

constexpr int kDqCols = 64;      // columns per workgroup: one wave's lanes
constexpr int kDqWaves = 16;
constexpr size_t kDqLdsMax = 80 * 1024;  // two workgroups per CU

// W16: 16-byte records [16-column tile][32-row step][lane l] of the columns
// from col0: column 16 t + l % 16, rows 32 s + 8 (l / 16) .. +7 in order, zero
// past K. A wave takes one word row at 64 columns, so the row's group is
// wave-uniform (scalar g_idx loads) and its metadata are 64 neighbouring
// entries: of LDS, staged per workgroup (META_LDS), or of global memory.
// Bound by the 2 K N bytes it writes.
template <int DT, int LAYOUT, bool META_LDS>
__global__ __launch_bounds__(kDqWaves * 64) void k_dequant16(GemmArgs a, int col0, int ncols,
                                                             uint16_t* __restrict__ W) {
  extern __shared__ __align__(16) uint32_t meta[];  // [num_groups][64]: scale bits | z << 16
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int cl = (int)blockIdx.x * kDqCols + lane;  // column of the chunk
  const int c = min(col0 + cl, a.N - 1);
  const int ng = a.num_groups;
  auto entry = [&](int g) {
    const uint32_t sv = a.sc[(int64_t)g * a.lds + c];
    const uint32_t zw = a.qz[(int64_t)g * a.ldz + (c >> 3)];
    return sv | ((((zw >> (4 * (c & 7))) & 0xFu) + (uint32_t)a.zoff) << 16);
  };
  if constexpr (META_LDS) {
    for (int g = wave; g < ng; g += kDqWaves) meta[g * 64 + lane] = entry(g);
    __syncthreads();
  }
  const int kw = a.K >> 3;
  const int nquads = 4 * ((a.K + 127) >> 7);
  const UnpackConsts<DT> kc;
  const int64_t nsteps = nquads;
  u4_t* out = (u4_t*)W + (int64_t)(cl >> 4) * nsteps * 64 + (lane & 15);
  const uint32_t gmax = (uint32_t)(ng - 1);
  // quad q = 4 b + kq: word rows 4 (4 b + u) + kq, u = 0 .. 3 (the four words
  // of one 16-byte piece of the tiled order)
  for (int q = (int)blockIdx.y * kDqWaves + wave; q < nquads; q += kDqWaves * (int)gridDim.y) {
    const int b = q >> 2, kq = q & 3;
    uint32_t w[4];
    if constexpr (LAYOUT == TPDQ_LAYOUT_TILED) {
      const u4_t v = *(const u4_t*)(a.qw + (int64_t)(c >> 4) * a.ldq + 256 * b + 4 * (16 * kq + (c & 15)));
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = v[u];
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int r = 4 * (4 * b + u) + kq;
        w[u] = r < kw ? a.qw[(int64_t)r * a.ldq + c] : 0u;
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = 4 * (4 * b + u) + kq;
      u4_t v = {0u, 0u, 0u, 0u};
      if (r < kw) {
        uint32_t g[8];
        if (a.g_idx) {
#pragma unroll
          for (int t = 0; t < 8; ++t) g[t] = (uint32_t)a.g_idx[8 * r + t];
        } else {
#pragma unroll
          for (int t = 0; t < 8; ++t) g[t] = (uint32_t)(8 * r + t) / (uint32_t)a.G;
        }
        uint32_t z[8], s[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int gt = (int)min(g[t], gmax);
          const uint32_t e = META_LDS ? meta[gt * 64 + lane] : entry(gt);
          z[t] = e >> 16;
          s[t] = e & 0xFFFFu;
        }
        constexpr bool NAT = LAYOUT == TPDQ_LAYOUT_TILED;
        v = dequant_rows<NAT, DT>(kc, w[u], z, s);
        if constexpr (!NAT) {  // x0 x4, x1 x5, x2 x6, x3 x7 -> x0 .. x7
          v = u4_t{__builtin_amdgcn_perm(v.y, v.x, 0x05040100u), __builtin_amdgcn_perm(v.w, v.z, 0x05040100u),
                   __builtin_amdgcn_perm(v.y, v.x, 0x07060302u), __builtin_amdgcn_perm(v.w, v.z, 0x07060302u)};
        }
      }
      if (cl < ncols) out[(int64_t)(4 * b + u) * 64 + 16 * kq] = v;
    }
  }
}

struct DenseArgs {
  const uint16_t* X;   // [M][ldx]
  int64_t ldx;
  int M, K, N;         // N: the chunk's columns
  const uint16_t* W;   // W16 of the chunk (GATED: gate)
  const uint16_t* Wu;  // GATED: up
  uint16_t* Y;         // [M][ldy], the chunk's first column
  int64_t ldy;
  float* part;         // ks > 1: [ks][(gate, up)][M][N]
  int ks;
};

// Dense MFMA GEMM on W16: 8 waves (two per SIMD), a workgroup computes 16 RT
// rows x 512 columns (GATED: 256 of gate and of up). As in k_prefill the
// activations go to LDS in operand order, one 128-row block ahead (two
// stages, one barrier per block). The weights are not shared between waves,
// so they go straight to registers, each 16-byte record reloaded with the
// record R steps on as soon as its MFMAs are issued: no waits but each
// record's own. R = 4 steps in flight per wave with 64-row tiles, 2 with
// 128-row ones (whose steps take twice as long; 4 would spill).
template <int RT, int DT, bool GATED>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void k_dense16(DenseArgs a) {
  constexpr int NW = 8, NT = 4, R = RT == 8 ? 2 : 4;
  constexpr int AREC = RT * 4 / NW;           // activation records per wave and block
  constexpr int STAGE = RT * 4 * 64 * 16;
  constexpr int CWAVE = GATED ? 32 : 64;
  extern __shared__ __align__(16) unsigned char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j = lane & 15;
  const int kq = lane >> 4;
  const int nbm = (a.M + 16 * RT - 1) / (16 * RT);
  const int ks = a.ks > 1 ? a.ks : 1;
  const int ntl = (int)(gridDim.x / ks);
  const int lt = xcd_tile(blockIdx.x, gridDim.x);
  const int kidx = lt / ntl;
  const int tl = lt - kidx * ntl;
  const int bn = tl / nbm;
  const int row0 = (tl - bn * nbm) * 16 * RT;
  const int cw = (bn * NW + wave) * CWAVE;  // the wave's first column
  const int nblk = (a.K + 127) >> 7;
  const int kb0 = (int)((int64_t)nblk * kidx / ks);
  const int kb1 = (int)((int64_t)nblk * (kidx + 1) / ks);
  const int bl = nblk - 1;
  const uint32_t tile_bytes = (uint32_t)nblk * 4096u;
  const uint32_t wbytes = (uint32_t)((a.N + 15) / 16) * tile_bytes;

  uint32_t offA[AREC], offAt[AREC], offW[NT];
#pragma unroll
  for (int k = 0; k < AREC; ++k) {
    const int rec = AREC * wave + k, rt = rec >> 2, u = rec & 3;
    offA[k] = ((uint32_t)(16 * rt + j) * (uint32_t)a.ldx + (uint32_t)(32 * u + 8 * kq)) * 2u;
    offAt[k] = 128 * bl + 32 * u + 8 * kq < a.K ? offA[k] : kOutOfRange;  // octets past K: zeros
  }
#pragma unroll
  for (int i = 0; i < NT; ++i)
    offW[i] = (uint32_t)((cw >> 4) + (GATED ? i & 1 : i)) * tile_bytes + (uint32_t)lane * 16u;
  const uint32_t xbytes = (uint32_t)(a.M - row0) * (uint32_t)a.ldx * 2u;

  auto dma_a = [&](int b, int st, int k) {
    const __amdgpu_buffer_rsrc_t r = buffer_rsrc(a.X + (int64_t)row0 * a.ldx + 128 * b,
                                                 b < kb1 ? xbytes - 256u * (uint32_t)b : 0u);
    dma_to_lds<16>(r, smem + st * STAGE + (AREC * wave + k) * 1024, b == bl ? offAt[k] : offA[k]);
  };
  auto load_w = [&](int b, int u, int i) {
    const uint16_t* w = GATED && i >= 2 ? a.Wu : a.W;
    const __amdgpu_buffer_rsrc_t r =
        buffer_rsrc(w + (int64_t)2048 * b, b < kb1 ? wbytes - 4096u * (uint32_t)b : 0u);
    return buffer_load16(r, offW[i] + 1024u * (uint32_t)u);
  };

  f4_t acc[RT][NT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < NT; ++i) acc[r][i] = f4_t{0.f, 0.f, 0.f, 0.f};

  u4_t w[R][NT];
#pragma unroll
  for (int k = 0; k < AREC; ++k) dma_a(kb0, 0, k);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < R; ++u)
#pragma unroll
    for (int i = 0; i < NT; ++i) {
      w[u][i] = load_w(kb0, u, i);  // in the loop's order, or its first wait is for all
      __builtin_amdgcn_sched_barrier(0);
    }
  int st = 0;
#pragma unroll 1
  for (int b = kb0; b < kb1; ++b) {
    // this wave's activation records of block b have landed: the weight loads
    // issued after the last of them (R NT before the first block, then one per
    // slot from the last record's) may be in flight
    constexpr int LATER = R * NT < 17 - AREC ? R * NT : 17 - AREC;
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::"n"(LATER) : "memory");
    const u4_t* ab = (const u4_t*)(smem + st * STAGE);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      u4_t av[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) av[r] = ab[(r * 4 + u) * 64 + lane];
#pragma unroll
      for (int i = 0; i < NT; ++i) {
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r][i] = mfma_k32<DT>(av[r], w[u % R][i], acc[r][i]);
        // the wait above counts these: one weight load per slot, behind the
        // slot's activation record; the scheduling barriers keep them there
        // (left to the scheduler the loads sink to the end of the block and
        // are waited for at once), LDS reads and scalar work may cross
        if (4 * u + i < AREC) dma_a(b + 1, st ^ 1, 4 * u + i);
        if (4 * u + i < AREC) __builtin_amdgcn_sched_barrier(0);
        w[u % R][i] = load_w(b + (u + R) / 4, (u + R) % 4, i);
        __builtin_amdgcn_sched_barrier(0x106);
      }
    }
    st ^= 1;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the last block: let them land

  const size_t plane = (size_t)a.M * a.N;
  float* part = a.part + (size_t)kidx * (GATED ? 2 : 1) * plane;
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < (GATED ? 2 : NT); ++i) {
      const int c = cw + 16 * i + j;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = row0 + 16 * r + 4 * kq + e;
        if (row < a.M && c < a.N) {
          if (ks > 1) {
            part[(int64_t)row * a.N + c] = acc[r][i][e];
            if constexpr (GATED) part[plane + (int64_t)row * a.N + c] = acc[r][i + 2][e];
          } else if constexpr (GATED) {
            a.Y[(int64_t)row * a.ldy + c] = float_to_bits<DT>(silu_mul(acc[r][i][e], acc[r][i + 2][e]));
          } else {
            a.Y[(int64_t)row * a.ldy + c] = float_to_bits<DT>(acc[r][i][e]);
          }
        }
      }
    }
}

template <int DT, int LAYOUT>
hipError_t launch_dequant_t(const GemmArgs& a, int col0, int ncols, uint16_t* W, hipStream_t s) {
  const size_t lds = (size_t)a.num_groups * kDqCols * 4;
  const int gx = (ncols + kDqCols - 1) / kDqCols;
  const int nquads = 4 * ((a.K + 127) / 128);
  // about two workgroups per CU; every one stages its columns' metadata
  const int gy = std::max(1, std::min(512 / gx, nquads / kDqWaves));
  if (lds <= kDqLdsMax) {
    auto k = k_dequant16<DT, LAYOUT, true>;
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kDqLdsMax);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(gx, gy), dim3(kDqWaves * 64), lds, s, a, col0, ncols, W);
  } else {
    auto k = k_dequant16<DT, LAYOUT, false>;
    hipLaunchKernelGGL(k, dim3(gx, gy), dim3(kDqWaves * 64), 0, s, a, col0, ncols, W);
  }
  return hipGetLastError();
}

hipError_t launch_dequant(const GemmArgs& a, int layout, int col0, int ncols, uint16_t* W, hipStream_t s) {
  const bool tiled = layout == TPDQ_LAYOUT_TILED;
  if (a.dt == kBF16)
    return tiled ? launch_dequant_t<kBF16, TPDQ_LAYOUT_TILED>(a, col0, ncols, W, s)
                 : launch_dequant_t<kBF16, TPDQ_LAYOUT_GPTQ>(a, col0, ncols, W, s);
  return tiled ? launch_dequant_t<kF16, TPDQ_LAYOUT_TILED>(a, col0, ncols, W, s)
               : launch_dequant_t<kF16, TPDQ_LAYOUT_GPTQ>(a, col0, ncols, W, s);
}

template <int RT, int DT, bool GATED>
hipError_t launch_dense_t(const DenseArgs& a, hipStream_t s) {
  constexpr int lds = 2 * RT * 4096;
  auto k = k_dense16<RT, DT, GATED>;
  const int bn = GATED ? 256 : 512;
  const int grid = ((a.M + 16 * RT - 1) / (16 * RT)) * ((a.N + bn - 1) / bn) * a.ks;
  hipLaunchKernelGGL(k, dim3(grid), dim3(512), lds, s, a);
  return hipGetLastError();
}

hipError_t launch_dense(const DenseArgs& a, int rt, int dt, bool gated, hipStream_t s) {
  auto go = [&](auto d) {
    constexpr int DT = decltype(d)::value;
    if (rt == 8) return gated ? launch_dense_t<8, DT, true>(a, s) : launch_dense_t<8, DT, false>(a, s);
    return gated ? launch_dense_t<4, DT, true>(a, s) : launch_dense_t<4, DT, false>(a, s);
  };
  const hipError_t e = dt == kBF16 ? go(std::integral_constant<int, kBF16>()) : go(std::integral_constant<int, kF16>());
  if (e != hipSuccess || a.ks == 1) return e;
  return launch_splitk_reduce(a.part, a.ks, a.M, a.N, a.Y, a.ldy, dt, gated, s);
}

// Bytes of 16-bit weights per column (of one projection).
int64_t col_bytes(int K) { return (int64_t)((K + 127) / 128) * 256; }

}  // namespace

// Microseconds of the dense kernel over one chunk, as mtile_cost counts its own
// (per block and round 2.45 us with 128-row tiles, where MFMA bounds it, 2.0 with
// 64-row ones, where the weight records through L1 do: 128 KiB per block and CU).
static double dense_cost(int M, int N, int nblk, int rt, int ks, bool gated) {
  return tiles_us(M, N, nblk, rt, ks, gated, 4.0, rt == 8 ? 2.45 : 2.0, 4.0, 4.5e6);
}

// Microseconds of the act-order call in launches of 64 rows (k_rowmeta), fitted
// within 10% to 1,700 GEMMs of 256 to 16384 rows and columns: per launch and round
// of one workgroup per CU, its blocks' dequantization and its row tiles.
static double decode_cost(int M, int N, int nblk, bool gated) {
  const int rounds = ((N + kTileN - 1) / kTileN + 255) / 256;
  double us = 0.0;
  for (int m = M; m > 0; m -= kDecodeMaxM) {
    const int tiles = m <= kTileM ? 1 : m <= 2 * kTileM ? 2 : 4;
    us += 5.6 + rounds * (0.1 + nblk * (0.04 + 0.08 * tiles) * (gated ? 2 : 1));
  }
  return us;
}

bool plan_dense16(int M, int64_t ldx, const tpdq_w4* w, bool gated, size_t budget, DensePlan* p) {
  const int K = w->K, N = w->N;
  const int64_t lim = (int64_t)1 << 31;
  if (M <= kDecodeMaxM || K % 8 != 0 || ldx % 8 != 0 || (int64_t)M * ldx * 2 >= lim) return false;
  const int64_t cb = col_bytes(K) * (gated ? 2 : 1);
  const int step = 512;
  DensePlan q{};
  // columns per chunk: whole 512-column tiles, the chunks of equal size
  int64_t fit = (int64_t)(std::min(budget, kDenseChunkBytes) / (size_t)cb);
  const int npad = (N + 15) / 16 * 16;
  if (fit < npad) {
    fit = fit / step * step;
    if (fit < step) return false;
    const int chunks = (int)((npad + fit - 1) / fit);
    q.ncols = std::min<int64_t>(fit, ((npad + chunks - 1) / chunks + step - 1) / step * step);
  } else {
    q.ncols = N;
  }
  q.w_bytes = align_up((size_t)((q.ncols + 15) / 16 * 16) * (size_t)cb);
  const int nblk = (K + 127) / 128;
  // as in plan_mtile: the choice without a limit, where the workspace holds it
  double us = 0.0;
  for (size_t limit : {SIZE_MAX, budget}) {
    double best = 1e30;
    for (int rt : {8, 4})
      for (int ks = 1; ks <= std::max(1, nblk / 4); ++ks) {
        const size_t part = ks > 1 ? align_up((size_t)ks * M * q.ncols * (gated ? 8 : 4)) : 0;
        if (part && (q.w_bytes + part > limit || part > kDenseChunkBytes / 2)) break;
        const double cost = dense_cost(M, q.ncols, nblk, rt, ks, gated);
        if (cost < 0.98 * best) {
          best = cost;
          q.rt = rt;
          q.ks = ks;
          q.part_bytes = part;
        }
      }
    us = 8.3 + ((N + q.ncols - 1) / q.ncols) * 0.76 * best + 0.92e-6 * K * N * (gated ? 2 : 1);
    if (q.w_bytes + q.part_bytes <= budget) break;
  }
  if (q.w_bytes > budget) return false;
  // two to four launches on a small layer may cost less than dequantizing it:
  // 1512 x 3208 at M = 65 24.7 us dense, 17.4 in two launches (of 1,700 sizes the
  // choice is 0.7% from the better one on average, dense alone 8%; 15% for what
  // decode_cost does not know, the metadata of a row shard's many groups)
  if (M <= kRowsMaxM && us > 1.15 * decode_cost(M, N, nblk, gated)) return false;
  *p = q;
  return true;
}

hipError_t launch_dense16(const GemmArgs& a, const DensePlan& p, int layout, char* ws, hipStream_t s) {
  const bool gated = a.qw_up != nullptr;
  uint16_t* W = (uint16_t*)ws;
  uint16_t* Wu = (uint16_t*)(ws + p.w_bytes / 2);
  for (int c0 = 0; c0 < a.N; c0 += p.ncols) {
    const int nc = std::min(p.ncols, a.N - c0);
    hipError_t e = launch_dequant(a, layout, c0, nc, W, s);
    if (e != hipSuccess) return e;
    if (gated) {
      GemmArgs u = a;
      u.qw = a.qw_up;
      u.sc = a.sc_up;
      u.qz = a.qz_up;
      e = launch_dequant(u, layout, c0, nc, Wu, s);
      if (e != hipSuccess) return e;
    }
    DenseArgs d{};
    d.X = a.X;
    d.ldx = a.ldx;
    d.M = a.M;
    d.K = a.K;
    d.N = nc;
    d.W = W;
    d.Wu = Wu;
    d.Y = a.Y + c0;
    d.ldy = a.ldy;
    d.part = (float*)(ws + p.w_bytes);
    d.ks = p.ks;
    e = launch_dense(d, p.rt, a.dt, gated, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tpdq
