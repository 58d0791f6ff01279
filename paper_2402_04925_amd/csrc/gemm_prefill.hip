// W4A16 dequantize-and-multiply for prefill-sized batches on gfx950: sorted
// rows (the ordered path of Alg. 3, group of row k = k / G), tiled weights.
//
// At M in the thousands the product is a dense contraction and the MFMA pipe
// bounds it (2 M K N flops against K N / 2 bytes of weights), so the kernel
// is a register-blocked MFMA GEMM:
//   * a workgroup of 8 waves (two per SIMD, so that one wave's waits are
//     covered by the other's MFMAs) computes a 128 x 512 tile of Y; each wave
//     owns 64 columns over all 128 rows (8 row tiles x 4 column tiles of
//     v_mfma_f32_16x16x32_f16), so that each dequantized weight fragment
//     feeds 8 MFMAs and the unpack and scaling cost about 2 VALU per MFMA;
//   * K advances one 128-row block at a time (4 MFMA steps of 32 rows);
//   * every operand goes from global memory straight to LDS (buffer loads
//     with the LDS bit, one record of 64 lanes per instruction): activations
//     laid out as the A operand, the wave's weights as they are tiled (one
//     16-byte record per lane and 16-column tile: the B operand), the scales
//     and zeros of the wave's columns; nothing is staged through registers,
//     so the loop keeps one copy of the accumulators;
//   * two stages: block b + 1 is loaded while block b is multiplied, its
//     loads issued one after each column tile's MFMAs (a burst of them at
//     the start of a block stalls the issuing waves); one barrier per block
//     hands a stage from its loads to its readers and back.
// The waits are explicit: before block b each wave waits for its own loads
// of block b (the most recent ones), and the barrier then makes every wave's
// LDS writes visible.
// Dequantizing to fp16 before the MFMA rounds each weight once (relative
// error 2^-12). With bf16 activations the weight is formed in fp32 and rounded
// once to bf16 (relative error 2^-9), about four times the VALU work of fp16.
// Most 64-row tiles (EXACT, see k_prefill) keep q - z in the MFMAs and scale in
// fp32 as the decode kernels do, for 6% more time than rounded weights in fp16 (6144
// x 6144, G = 128, M = 512, no K split: 94.5 us against 88.7; bf16 is faster than
// rounded; groups of 64 and 32 cost 25 and 55% more per block than G = 128): they
// also serve what would otherwise run in decode launches of 64 rows. Gated
// Llama-70B TP=8 MLP at M = 1000, bf16: 514 -> 220 us (gate and up in one launch
// at 0.9 PFLOP/s).
#include "kernels_common.h"

#include <algorithm>

namespace tpdq {
namespace {

constexpr int kPWT = 4;    // column tiles per wave
constexpr int kPWwave = kPWT * 64 * 16;
// metadata records of 256 bytes per wave and block: two of scales and one of
// zeros (64 columns), or gated one of each for 32 columns of gate and of up
__host__ __device__ constexpr int pf_meta(bool gated) { return (gated ? 4 : 3) * 256; }
// LDS per stage with RT row tiles and NW waves: activations
// [RT row tiles][4 steps][64 lanes] x 16 B, then per wave its weights
// [4 tiles][64 lanes] x 16 B and its metadata
__host__ __device__ constexpr int pf_stage(int rt, int nw, bool gated) {
  return rt * 4 * 64 * 16 + nw * (kPWwave + pf_meta(gated));
}

__device__ __forceinline__ u4_t dequant_scaled(const UnpackConsts<kF16>& kc, uint32_t w, uint32_t z1024,
                                               uint32_t z64, uint32_t s2) {
  const h8_t d = unpack_sub(kc, w, z1024, z64);
  const h2_t s = as_h2(s2);
  const h8_t sv = {s.x, s.y, s.x, s.y, s.x, s.y, s.x, s.y};
  return __builtin_bit_cast(u4_t, d * sv);
}

// bf16: s (q - z) = (128 + q) s - (128 + z) s with zs = (128 + z) s; both
// products are exact in fp32 (8 significant bits each), so one FMA gives
// s (q - z) exactly and the conversion rounds it once.
__device__ __forceinline__ u4_t dequant_scaled_bf16(const UnpackConsts<kBF16>& kc, uint32_t w,
                                                    float s, float zs) {
  const u4_t b = unpack_bias_bf16(kc, w);
  u4_t r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = pack2<kBF16>(__builtin_fmaf(as_f32(b[i] << 16), s, -zs),
                        __builtin_fmaf(as_f32(b[i] & 0xFFFF0000u), s, -zs));
  return r;
}

// bf16, EXACT: an infinite x, or a finite one past about 2e36, makes both of a
// group's sums infinite and their difference NaN. The elements that came out
// not finite (bits of `again`, see k_prefill) are summed again here with every
// weight s (q - z) rounded to bf16, as the 128-row tiles take them, so that each
// product has its own sign and size; what is finite keeps its bits. One wave for
// itself, straight from global memory, a tile at a time: for rare inputs only,
// so nothing of it may cost the kernel registers.
template <int SPG, int RT, bool GATED>
__device__ __forceinline__ void round_not_finite(const GemmArgs& a, uint64_t again, int row0, int cw, int kb0,
                                                 int kb1, float* part) {
  constexpr int COLT = GATED ? 2 : kPWT;
  // counted anew: threadIdx held through the kernel's loop is a register it has not
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const int j = lane & 15, kq = lane >> 4;
  const size_t plane = (size_t)a.M * a.N;
  const UnpackConsts<kBF16> kc;
#pragma unroll 1
  for (int t = 0; t < RT * COLT; ++t) {
    const int r = t / COLT, i = t % COLT;
    uint32_t bits = (uint32_t)(again >> ((r * kPWT + i) * 4)) & 15u;
    if (GATED) bits |= (uint32_t)(again >> ((r * kPWT + i + 2) * 4)) & 15u;
    if (!__any(bits != 0)) continue;
    const int c = cw + 16 * i + j;
    const bool cok = c < a.N;
    f4_t v[2] = {f4_t{0.f, 0.f, 0.f, 0.f}, f4_t{0.f, 0.f, 0.f, 0.f}};
    const int m = row0 + 16 * r + j;  // the lane's row of the A operand
#pragma unroll 1
    for (int s = 4 * kb0; s < 4 * kb1; ++s) {
      const int k0 = 32 * s + 8 * kq;
      u4_t x = {0u, 0u, 0u, 0u};
      if (m < a.M && k0 < a.K) x = *(const u4_t*)(a.X + (int64_t)m * a.ldx + k0);
      const int64_t g = s / SPG;
#pragma unroll
      for (int p = 0; p < (GATED ? 2 : 1); ++p) {
        uint32_t w = 0u, zc = 0u;
        float sf = 0.f;
        if (cok && 32 * s < a.K) {
          w = (p ? a.qw_up : a.qw)[(int64_t)(c >> 4) * a.ldq + 256 * (s >> 2) + 4 * lane + (s & 3)];
          sf = bits_to_float<kBF16>((p ? a.sc_up : a.sc)[g * a.lds + c]);
          zc = (((p ? a.qz_up : a.qz)[g * a.ldz + (c >> 3)] >> (4 * (c & 7))) & 0xFu) + (uint32_t)a.zoff;
        }
        v[p] = mfma_k32<kBF16>(x, dequant_scaled_bf16(kc, w, sf, (128.f + (float)zc) * sf), v[p]);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int row = row0 + 16 * r + 4 * kq + e;
      if (!((bits >> e) & 1u) || row >= a.M || !cok) continue;
      if (a.ks > 1) {
        part[(int64_t)row * a.N + c] = v[0][e];
        if constexpr (GATED) part[plane + (int64_t)row * a.N + c] = v[1][e];
      } else {
        a.Y[(int64_t)row * a.ldy + c] = float_to_bits<kBF16>(GATED ? silu_mul(v[0][e], v[1][e]) : v[0][e]);
      }
    }
  }
}

// RT row tiles (16 RT rows of Y per workgroup), NW waves (64 columns each). With a.ks > 1 the workgroup covers one of ks
// contiguous ranges of 128-row blocks of K and writes its fp32 partial tile
// to a.part[split][M][N] (k_splitk_reduce sums the splits); else it writes
// fp16 Y.
// Two waves per SIMD (the 8-wave workgroup):
// 256 registers per lane, with the accumulators in the architectural VGPRs
// (no accumulator copies between loop iterations).
//
// EXACT (64-row tiles; the 128-row ones round, and 64-row ones of groups of 32
// and 64 on large weights): the MFMAs take q - z (bf16: 128 + q), exact in the element type, into
// a second set of accumulators, and every group closes with its scale in fp32
// (bf16: and its zero, against the group's sum of X from one more MFMA per row
// tile), as the decode kernels do: no weight is rounded. Twice the
// accumulators, so RT = 4; per MFMA 9 / 4 VALU of unpacking and, at G = 128,
// one of scaling (bf16 two).
// GATED (EXACT): Y = silu(X W) * (X W_up). A wave's four column tiles are 32
// columns of gate (tiles 0, 1) and the same 32 of up (tiles 2, 3), so that the
// epilogue has both products of an element in one lane; split partials are
// [split][gate, up][M][N].
template <int SPG, int NW, int RT, int DT, bool EXACT = false, bool GATED = false>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void k_prefill(GemmArgs a) {
  static_assert(!EXACT || RT <= 4, "two accumulators per output");
  static_assert(!GATED || EXACT, "the gated product keeps its weights exact");
  // groups per 128-row block: G = 32, 64, 128 -> 4, 2, 1; G = 256 -> one
  // group spans two blocks (each block loads it)
  constexpr int GPK = SPG >= 4 ? 1 : 4 / SPG;
  // scale records per wave and block (two groups of 64 columns in each;
  // gated: four groups of 32 columns, one record for gate, one for up)
  constexpr int NSD = GATED ? 2 : (GPK + 1) / 2;
  constexpr int NZ = GATED ? 2 : 1;
  constexpr int CWAVE = GATED ? 32 : 64;  // output columns per wave
  static_assert((RT * 4) % NW == 0, "activation records split evenly over the waves");
  constexpr int AREC = RT * 4 / NW;   // activation records per wave and block
  // loads per wave and block: activations, scales, zeros, weights
  constexpr int LPB = AREC + NSD + NZ + kPWT;
  constexpr int STAGE = pf_stage(RT, NW, GATED);
  constexpr int MWAVE = pf_meta(GATED);
  constexpr int ZOFF = 512;  // the zeros behind the scales in a wave's metadata
  constexpr int ABYTES = RT * 4 * 64 * 16;
  constexpr int BM = 16 * RT;
  constexpr int BN = CWAVE * NW;
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = lane & 15;
  const int kq = lane >> 4;
  const int nbm = (a.M + BM - 1) / BM;
  const int ks = a.ks > 1 ? a.ks : 1;
  const int ntl = (int)(gridDim.x / ks);  // output tiles
  // consecutive workgroups (one XCD) take neighbouring tiles of one split:
  // they share its activations in L2
  const int lt = xcd_tile(blockIdx.x, gridDim.x);
  const int kidx = lt / ntl;
  const int tl = lt - kidx * ntl;
  const int bn = tl / nbm;
  const int bm = tl - bn * nbm;
  const int row0 = bm * BM;
  const int col0 = bn * BN;
  const int cw = col0 + CWAVE * wave;
  const int nblk_all = (a.K + 127) >> 7;
  // this workgroup's blocks [kb0, kb1)
  const int kb0 = (int)((int64_t)nblk_all * kidx / ks);
  const int kb1 = (int)((int64_t)nblk_all * (kidx + 1) / ks);
  const int ng = a.num_groups;
  const int ntiles = (a.N + kTileN - 1) / kTileN;
  const UnpackConsts<DT> kc;

  // sources: rows past M, groups past the last one and tiles past N load
  // zeros from the resource bounds
  // per-lane parts of the offsets
  // activations: record (rt, u) of block b, lane l = row 16 rt + l % 16,
  // columns 128 b + 32 u + 8 (l / 16) .. +7
  const uint32_t x_lane = ((uint32_t)j * (uint32_t)a.ldx + 8u * (uint32_t)kq) * 2u;
  const uint32_t x_rt = 16u * (uint32_t)a.ldx * 2u;
  // scales: record d, lane l = group 2 d + l / 32, columns 2 (l % 32), +1;
  // gated: record of gate or up, lane l = group l / 16, columns 2 (l % 16), +1
  const int sg = GATED ? lane >> 4 : lane >> 5, scol = 2 * (GATED ? lane & 15 : lane & 31);
  const uint32_t s_lane = (uint32_t)sg * (uint32_t)a.lds * 2u + (uint32_t)(cw + scol) * 2u;
  // zeros: lane l = group l / 8, word l % 8 of the wave's 8 (gated l / 4, l % 4)
  const int zg = GATED ? lane >> 2 : lane >> 3, zw0 = GATED ? lane & 3 : lane & 7;
  const uint32_t z_lane = ((uint32_t)zg * (uint32_t)a.ldz + (uint32_t)((cw >> 3) + zw0)) * 4u;
  const bool z_used = zg < GPK;
  // weights: tile (cw / 16 + i), block b: lane l's 16 bytes
  const uint32_t w_lane = ((uint32_t)(cw >> 4) * (uint32_t)a.ldq + 4u * (uint32_t)lane) * 4u;
  const uint32_t w_tile = (uint32_t)a.ldq * 4u;

  // per-lane offsets inside one block's window of each source, the same for
  // every block; the window (a buffer resource: base and size in scalar
  // registers) moves with the block, so a load needs no per-block vector
  // arithmetic. Blocks past the workgroup's range get an empty window: their
  // loads return zeros and cost no traffic.
  const int bl = nblk_all - 1;
  uint32_t offA[AREC], offAt[AREC], offS[NSD], offW[kPWT];
#pragma unroll
  for (int k = 0; k < AREC; ++k) {
    const int rec = AREC * wave + k, rt = rec >> 2, u = rec & 3;
    offA[k] = x_lane + (uint32_t)rt * x_rt + (uint32_t)(32 * u) * 2u;
    // the last block: the lane's octet loads zeros past K (the padding of X
    // past K is never read)
    offAt[k] = 128 * bl + 32 * u + 8 * kq < a.K ? offA[k] : kOutOfRange;
  }
#pragma unroll
  for (int d = 0; d < NSD; ++d)
    offS[d] = GATED ? (sg < GPK ? s_lane : kOutOfRange)
                    : (2 * d + sg < GPK ? s_lane + (uint32_t)(2 * d) * (uint32_t)a.lds * 2u : kOutOfRange);
  const uint32_t offZ = z_used ? z_lane : kOutOfRange;
#pragma unroll
  for (int i = 0; i < kPWT; ++i) offW[i] = w_lane + (uint32_t)(GATED ? i & 1 : i) * w_tile;
  const uint32_t xbytes = (uint32_t)(a.M - row0) * (uint32_t)a.ldx * 2u;
  const uint32_t wbytes = (uint32_t)ntiles * (uint32_t)a.ldq * 4u;

  // load k (0 <= k < LPB) of block b into LDS stage st; each item is exactly
  // one load (the wait counts rely on it)
  auto dma_item = [&](int b, int st, int k) {
    unsigned char* sb = smem + st * STAGE;
    unsigned char* wb = sb + ABYTES + wave * (kPWwave + MWAVE);
    unsigned char* mb = wb + kPWwave;
    const int g0 = (128 * b) / (32 * SPG);
    const bool bok = b < kb1;
    if (k < AREC) {
      const int rec = AREC * wave + k;
      const __amdgpu_buffer_rsrc_t r = buffer_rsrc(a.X + (int64_t)row0 * a.ldx + 128 * b,
                                                   bok ? xbytes - 256u * (uint32_t)b : 0u);
      dma_to_lds<16>(r, sb + rec * 1024, b == bl ? offAt[k] : offA[k]);
    } else if (k < AREC + NSD) {
      const int d = k - AREC;
      const uint16_t* sc = GATED && d == 1 ? a.sc_up : a.sc;
      const __amdgpu_buffer_rsrc_t r = buffer_rsrc(sc + (int64_t)g0 * a.lds,
                                                   bok ? (uint32_t)(ng - g0) * (uint32_t)a.lds * 2u : 0u);
      dma_to_lds<4>(r, mb + d * 256, offS[d]);
    } else if (k < AREC + NSD + NZ) {
      const int d = k - AREC - NSD;
      const uint32_t* qz = GATED && d == 1 ? a.qz_up : a.qz;
      const __amdgpu_buffer_rsrc_t r = buffer_rsrc(qz + (int64_t)g0 * a.ldz,
                                                   bok ? (uint32_t)(ng - g0) * (uint32_t)a.ldz * 4u : 0u);
      dma_to_lds<4>(r, mb + ZOFF + d * 256, offZ);
    } else {
      const int i = k - AREC - NSD - NZ;
      const uint32_t* qw = GATED && i >= 2 ? a.qw_up : a.qw;
      const __amdgpu_buffer_rsrc_t r = buffer_rsrc(qw + (int64_t)256 * b,
                                                   bok ? wbytes - 1024u * (uint32_t)b : 0u);
      dma_to_lds<16>(r, wb + i * 1024, offW[i]);
    }
  };
  auto issue = [&](int b, int st) {
#pragma unroll
    for (int k = 0; k < LPB; ++k) dma_item(b, st, k);
  };

  f4_t acc[RT][kPWT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < kPWT; ++i) acc[r][i] = f4_t{0.f, 0.f, 0.f, 0.f};
  f4_t gacc[EXACT ? RT : 1][EXACT ? kPWT : 1];   // EXACT: the open group
  f4_t xsum[EXACT && DT == kBF16 ? RT : 1];
  const f4_t fz = {0.f, 0.f, 0.f, 0.f};
  const u4_t ones = {kBf16OnePair, kBf16OnePair, kBf16OnePair, kBf16OnePair};
  // block in stage st; the loads of block bn go out one after each column
  // tile's MFMAs, into stage sn
  auto compute = [&](int b, int st, int bnext, int sn) {
    const u4_t* ab = (const u4_t*)(smem + st * STAGE);
    const u4_t* wb = (const u4_t*)(smem + st * STAGE + ABYTES + wave * (kPWwave + MWAVE));
    const unsigned char* mb = (const unsigned char*)wb + kPWwave;
    u4_t w[kPWT];
#pragma unroll
    for (int i = 0; i < kPWT; ++i) w[i] = wb[i * 64 + lane];
    uint32_t z1024[kPWT], z64[kPWT], s2[kPWT];
    float sf[kPWT], zs[kPWT];  // bf16, rounded weights
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool open = SPG >= 4 ? u == 0 : (u % SPG) == 0;
      // the MFMAs' first step of a group, and its last (G = 256: a group is
      // blocks 2g and 2g + 1, cut where the workgroup's range is)
      const bool first = SPG <= 4 ? open : u == 0 && ((b & 1) == 0 || b == kb0);
      const bool last = SPG <= 4 ? (u % (SPG <= 4 ? SPG : 4)) == (SPG <= 4 ? SPG : 4) - 1
                                 : u == 3 && ((b & 1) == 1 || b == kb1 - 1);
      const int gi = SPG >= 4 ? 0 : u / SPG;
      // scale bits and zero code of column j of tile i in this block's group
      auto meta_of = [&](int i, uint32_t& sv, uint32_t& zc) {
        const int c = 16 * (GATED ? i & 1 : i) + j;
        const int ms = GATED ? (i >> 1) * 256 + gi * 64 : gi * 128;  // record and group
        const int mz = ZOFF + (GATED ? (i >> 1) * 256 + gi * 16 : gi * 32);
        sv = *(const uint16_t*)(mb + ms + 2 * c);
        const uint32_t zw = *(const uint32_t*)(mb + mz + 4 * (c >> 3));
        zc = ((zw >> (4 * (c & 7))) & 0xFu) + (uint32_t)a.zoff;  // up to 16
      };
      if (open) {
#pragma unroll
        for (int i = 0; i < kPWT; ++i) {
          uint32_t sv, zc;
          meta_of(i, sv, zc);
          if constexpr (DT == kBF16) {
            if constexpr (!EXACT) {
              sf[i] = bits_to_float<kBF16>(sv);
              zs[i] = (128.f + (float)zc) * sf[i];
            }
          } else {
            z1024[i] = (0x6400u | zc) * 0x10001u;
            z64[i] = (0x5400u | (zc << 4)) * 0x10001u;
            s2[i] = sv * 0x10001u;
          }
        }
      }
      u4_t av[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) av[r] = ab[(r * 4 + u) * 64 + lane];
#pragma unroll
      for (int i = 0; i < kPWT; ++i) {
        u4_t bv;
        if constexpr (EXACT)
          bv = unpack_step<DT>(kc, w[i][u], z1024[i], z64[i]);
        else if constexpr (DT == kBF16)
          bv = dequant_scaled_bf16(kc, w[i][u], sf[i], zs[i]);
        else
          bv = dequant_scaled(kc, w[i][u], z1024[i], z64[i], s2[i]);
#pragma unroll
        for (int r = 0; r < RT; ++r) {
          if constexpr (EXACT)
            gacc[r][i] = mfma_k32<DT>(av[r], bv, first ? fz : gacc[r][i]);
          else
            acc[r][i] = mfma_k32<DT>(av[r], bv, acc[r][i]);
        }
        if (4 * u + i < LPB) dma_item(bnext, sn, 4 * u + i);
      }
      if constexpr (EXACT) {
        if constexpr (DT == kBF16) {
#pragma unroll
          for (int r = 0; r < RT; ++r) xsum[r] = mfma_k32<DT>(av[r], ones, first ? fz : xsum[r]);
        }
        if (last) {
          // the group's scale (and zero) are read again here: held since the
          // group's first step they would cost registers the kernel has not
#pragma unroll
          for (int i = 0; i < kPWT; ++i) {
            uint32_t sv, zc;
            meta_of(i, sv, zc);
            const float sc = bits_to_float<DT>(sv);
            const float zt = 128.f + (float)zc;
#pragma unroll
            for (int r = 0; r < RT; ++r) {
              if constexpr (DT == kBF16)
                acc[r][i] += sc * (gacc[r][i] - zt * xsum[r]);
              else
                acc[r][i] += sc * gacc[r][i];
            }
          }
        }
      }
    }
  };

  issue(kb0, 0);
  int st = 0;
#pragma unroll 1
  for (int b = kb0; b < kb1; ++b) {
    // this wave's loads of block b have landed and its LDS reads of block b - 1
    // are done; the barrier then publishes every wave's block b and frees the
    // stage that receives the next block
    asm volatile("s_waitcnt vmcnt(0)\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    compute(b, st, b + 1, st == 0 ? 1 : st - 1);
    st = st == 1 ? 0 : st + 1;
  }
  // the loads past the last block (zeros) still write LDS: let them land
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

  // epilogue: acc[r][i] of lane (j, kq) holds rows 4 kq .. +3 of row tile r,
  // column j of the wave's tile i
  const size_t plane = (size_t)a.M * a.N;
  float* part = a.part + (size_t)kidx * (GATED ? 2 : 1) * plane;
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int i = 0; i < (GATED ? 2 : kPWT); ++i) {
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
  if constexpr (EXACT && DT == kBF16) {
    uint64_t again = 0;  // element e of tile i, row tile r: bit (r kPWT + i) 4 + e
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
      for (int i = 0; i < kPWT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (!__builtin_isfinite(acc[r][i][e])) again |= 1ull << ((r * kPWT + i) * 4 + e);
    if (__any(again != 0)) round_not_finite<SPG, RT, GATED>(a, again, row0, cw, kb0, kb1, part);
  }
}

// Y[m][n] = round(sum over s of part[s][m][n]) to the element type, the splits added in order s =
// 0, 1, ... (the result does not depend on which split finished first). Four
// columns per thread: one 16-byte load per split, one 8-byte store (N % 4 ==
// 0 and 16-byte aligned rows; otherwise one column per thread).
// GATED: the partials are [s][gate, up][M][N] and Y = silu(gate) * up.
template <int DT, bool GATED>
__global__ __launch_bounds__(256) void k_splitk_reduce(const float* __restrict__ part, int ks, int M,
                                                       int N, uint16_t* __restrict__ Y, int64_t ldy) {
  const int64_t plane = (int64_t)M * N;
  const int64_t step = GATED ? 2 * plane : plane;
  if ((N & 3) == 0 && (ldy & 3) == 0) {
    const int n4 = N >> 2;
    const int64_t total = (int64_t)M * n4;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
      const int m = (int)(i / n4);
      const int c0 = (int)(i - (int64_t)m * n4) * 4;
      const float* src = part + (int64_t)m * N + c0;
      f4_t v = *(const f4_t*)src;
      for (int s = 1; s < ks; ++s) v += *(const f4_t*)(src + s * step);
      if constexpr (GATED) {
        src += plane;
        f4_t u = *(const f4_t*)src;
        for (int s = 1; s < ks; ++s) u += *(const f4_t*)(src + s * step);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = silu_mul(v[e], u[e]);
      }
      const uint32_t lo = pack2<DT>(v[0], v[1]);
      const uint32_t hi = pack2<DT>(v[2], v[3]);
      *(uint2*)(Y + (int64_t)m * ldy + c0) = make_uint2(lo, hi);
    }
    return;
  }
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < plane;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int m = (int)(i / N);
    const int c = (int)(i - (int64_t)m * N);
    float v = part[i];
    for (int s = 1; s < ks; ++s) v += part[s * step + i];
    if constexpr (GATED) {
      float u = part[plane + i];
      for (int s = 1; s < ks; ++s) u += part[s * step + plane + i];
      v = silu_mul(v, u);
    }
    Y[(int64_t)m * ldy + c] = float_to_bits<DT>(v);
  }
}

__global__ __launch_bounds__(256) void k_gather_rows(const uint16_t* __restrict__ X, int64_t ldx,
                                                     int K, const int32_t* __restrict__ perm,
                                                     uint16_t* __restrict__ Xp) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint16_t* xl = (uint16_t*)smem;
  const int m = blockIdx.x;
  const uint16_t* xr = X + (int64_t)m * ldx;
  const int kw = K >> 3;
  for (int o = threadIdx.x; o < kw; o += blockDim.x) *(u4_t*)(xl + 8 * o) = *(const u4_t*)(xr + 8 * o);
  __syncthreads();
  const uint32_t kmax = (uint32_t)(K - 1);
  for (int o = threadIdx.x; o < kw; o += blockDim.x) {
    const u4_t p0 = *(const u4_t*)(perm + 8 * o);
    const u4_t p1 = *(const u4_t*)(perm + 8 * o + 4);
    uint32_t x[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      x[e] = xl[min(p0[e], kmax)];
      x[e + 4] = xl[min(p1[e], kmax)];
    }
    *(u4_t*)(Xp + (int64_t)m * K + 8 * o) =
        u4_t{x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16)};
  }
}

}  // namespace

// The tile and split at prefill sizes. Measured on 6144 x 6144, 8192 x 3584 and
// 3584 x 8192 at M = 300 to 1500 with G = 128, per block 128 x 512 tiles 2.8 us
// (bf16 3.2), 64 x 512 ones 1.9 (2.5). Groups of 32 and 64 make the 64-row tiles
// dearer (prefill_us has the figures) and are not counted here: by time alone
// some of their sizes would take 128-row tiles, whose weights are rounded, where
// they have exact ones now (3584 x 8192, bf16, G = 32, M = 1000: 106 us exact, 78
// rounded).
static double mtile_cost(int M, int N, int nblk, int rt, int ks, bool gated, int dt) {
  const double tb = dt == kBF16 ? (rt == 8 ? 3.2 : 2.5) : (rt == 8 ? 2.8 : 1.9);
  return tiles_us(M, N, nblk, rt, ks, gated, 4.0, tb, 4.0, 4.5e6);
}

// With the group size, where the choice is between kernels of one precision:
// fitted within 3.3% to 530 GEMMs of those sizes and 4096 x 11008 at M = 100 to
// 1500. Exact 64-row tiles close every group; rounded 128-row ones load its
// metadata and spill.
static double prefill_us(int M, int N, int nblk, int rt, int ks, bool gated, int dt, int spg) {
  // G = 32, 64, 128, 256
  static constexpr double block[2][2][4] = {{{2.6, 2.1, 1.7, 1.75}, {3.95, 3.75, 2.7, 2.7}},
                                            {{3.2, 2.4, 2.0, 1.95}, {3.5, 3.65, 3.1, 3.1}}};
  const double tb = block[dt == kBF16][rt == 8][spg == 1 ? 0 : spg == 2 ? 1 : spg == 4 ? 2 : 3];
  return tiles_us(M, N, nblk, rt, ks, gated, 7.7, tb, 2.8, 8.8e6);
}

bool plan_mtile(int M, int64_t ldx, const tpdq_w4* w, int meta, int dt, bool gated, bool optional,
                size_t part_budget, MtilePlan* p) {
  if (meta != kMetaGroup || w->layout != TPDQ_LAYOUT_TILED) return false;
  const int K = w->K, N = w->N, G = w->group_size;
  if (M < kMtileMinM || K % 8 != 0 || G <= 0 || G % 32 != 0) return false;
  const int spg = G / 32;
  if (!(spg == 1 || spg == 2 || spg == 4 || spg == 8)) return false;
  // activation rows on 16 bytes, scale rows on 4 (the LDS loads move 16 and
  // 4 bytes per lane)
  if (ldx % 8 != 0 || w->ld_s % 2 != 0 || ((uintptr_t)w->scales & 3) != 0) return false;
  // byte offsets of the buffer loads are 32-bit
  const int64_t lim = (int64_t)1 << 31;
  const int64_t ntiles = (N + kTileN - 1) / kTileN;
  if (!(ntiles * w->ld_q * 4 < lim && (int64_t)M * ldx * 2 < lim &&
        (int64_t)w->num_groups * w->ld_s * 2 < lim && (int64_t)w->num_groups * w->ld_z * 4 < lim))
    return false;
  MtilePlan q{};
  q.ks = 1;
  q.gated = gated;
  const int nblk = (K + 127) / 128;
  const bool big = !gated && (int64_t)K * N >= kMtileMinWeights;
  if (big && M < kPrefillMinM) {
    // 64 x 512 tiles, 8 waves (two per SIMD, one workgroup per CU), K split as
    // far as the workgroups still fit the kMtileSlots CUs in one round.
    // Llama-70B TP=1 at M = 64 (MLP): 109.5 us with 64 x 256 tiles of 4 waves
    // in 512 slots (two per CU), 106.3 us here (GEMM2 52.4 -> 48.9 us: 8 waves
    // share one copy of the activations); more splits than fit one round are
    // slower (8 waves in 320 slots: GEMM1 280 workgroups, 144 us), and so is
    // one wave per SIMD. Groups of 32 and 64 close four times and twice a block
    // and keep rounded weights here (8192 x 28672 at M = 64, exact / rounded:
    // G = 32 63.1 / 60.3 us, G = 64 55.4 / 54.3, G = 128 49.3 / 51.7)
    auto cut = [&](int rt) {
      MtilePlan c = q;
      const int tiles = ((M + 16 * rt - 1) / (16 * rt)) * ((N + 511) / 512);
      c.rt = rt;
      c.exact = rt == 4 && spg > 2;
      c.ks = std::max(1, std::min(kMtileSlots / tiles, nblk / 4));
      if ((int64_t)c.ks * M * N * 4 >= lim) c.ks = 1;
      return c;
    };
    *p = cut(4);
    // more than one 64-row tile: 128-row tiles halve the activations' share of
    // a CU's bytes, for twice the partials (8192 x 28672 and 28672 x 8192 at M
    // = 128: 84.8 and 81.9 us -> 77.1 and 76.7), not over few columns, where the
    // splits are many (53248 x 2048, G = 64, at M = 160 68 -> 80)
    if (M > 64 && optional) {
      const MtilePlan c = cut(8);
      if (mtile_part_bytes(c, M, N) <= part_budget &&
          prefill_us(M, N, nblk, 8, c.ks, false, dt, spg) < prefill_us(M, N, nblk, 4, p->ks, false, dt, spg))
        *p = c;
    }
    return true;
  }
  // the gated product and smaller weights below prefill sizes keep their
  // weights exact (64-row tiles), as the decode kernels that otherwise run
  // them do
  const bool exact = gated || M < kPrefillMinM;
  if (exact && (!optional || M <= kDecodeMaxM)) return false;
  // 128 x 512 tiles over the whole K, or 64 x 512 ones, or either with K
  // split, whichever fills the CUs better (mtile_cost); Llama-70B TP=8 GEMM2
  // at M = 1000: 128 tiles of 128 x 512 on 256 CUs 84.7 us, 256 of 64 x 512
  // 67.8 us; 6144 x 6144 at M = 512: 133.6 us, 57.5 us with 64-row tiles and
  // K split 2
  // Chosen without a limit on the workspace first, so that every workspace that
  // holds the choice gives the same one (a workspace that other calls have made
  // larger must not change the order of a call's sums).
  for (size_t budget : {SIZE_MAX, part_budget}) {
    double best = 1e30;
    for (int rt : {8, 4}) {
      if (exact && rt == 8) continue;
      for (int ks = 1; ks <= std::max(1, nblk / 4); ++ks) {
        MtilePlan c = q;
        c.rt = rt;
        c.ks = ks;
        c.exact = rt == 4;
        if (ks > 1 && (!optional || mtile_part_bytes(c, M, N) > budget ||
                       (int64_t)ks * M * N * (gated ? 8 : 4) >= lim))
          break;
        const double cost = M < kPrefillMinM ? prefill_us(M, N, nblk, rt, ks, gated, dt, spg)
                                             : mtile_cost(M, N, nblk, rt, ks, gated, dt);
        if (cost < 0.98 * best) {
          best = cost;
          c.cost = cost;
          *p = c;
        }
      }
    }
    if (mtile_part_bytes(*p, M, N) <= part_budget) break;
  }
  return true;
}

size_t mtile_part_bytes(const MtilePlan& p, int M, int N) {
  return p.ks > 1 ? align_up((size_t)p.ks * M * N * (p.gated ? 8 : 4)) : 0;
}

hipError_t launch_mtile_k(void (*k)(GemmArgs), int rt, bool gated, const GemmArgs& a, int ks, hipStream_t s) {
  const int lds = 2 * pf_stage(rt, 8, gated);
  hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  const int bn = gated ? 256 : 512;
  const int grid = ((a.M + 16 * rt - 1) / (16 * rt)) * ((a.N + bn - 1) / bn) * ks;
  hipLaunchKernelGGL(k, dim3(grid), dim3(512), lds, s, a);
  return hipGetLastError();
}

template <int RT, int DT, bool EXACT, bool GATED>
hipError_t launch_mtile_t(const GemmArgs& a, int ks, hipStream_t s) {
  typedef void (*Kern)(GemmArgs);
  Kern k = nullptr;
  switch (a.G / 32) {
    case 1: k = k_prefill<1, 8, RT, DT, EXACT, GATED>; break;
    case 2: k = k_prefill<2, 8, RT, DT, EXACT, GATED>; break;
    case 4: k = k_prefill<4, 8, RT, DT, EXACT, GATED>; break;
    case 8: k = k_prefill<8, 8, RT, DT, EXACT, GATED>; break;
  }
  return k ? launch_mtile_k(k, RT, GATED, a, ks, s) : hipErrorInvalidValue;
}

template <int DT>
hipError_t launch_mtile_dt(const GemmArgs& a, const MtilePlan& p, hipStream_t s) {
  if (p.rt == 4 && !p.exact) {  // groups of 32 and 64 only (plan_mtile)
    if (p.gated) return hipErrorInvalidValue;
    if (a.G == 32) return launch_mtile_k(k_prefill<1, 8, 4, DT, false, false>, 4, false, a, p.ks, s);
    return a.G == 64 ? launch_mtile_k(k_prefill<2, 8, 4, DT, false, false>, 4, false, a, p.ks, s)
                     : hipErrorInvalidValue;
  }
  if (p.rt == 4)
    return p.gated ? launch_mtile_t<4, DT, true, true>(a, p.ks, s) : launch_mtile_t<4, DT, true, false>(a, p.ks, s);
  return p.rt == 8 && !p.exact && !p.gated ? launch_mtile_t<8, DT, false, false>(a, p.ks, s)
                                           : hipErrorInvalidValue;
}

hipError_t launch_mtile(const GemmArgs& a0, const MtilePlan& p, float* part, hipStream_t s) {
  GemmArgs a = a0;
  a.ks = p.ks;
  a.part = part;
  if (p.ks > 1 && !part) return hipErrorInvalidValue;
  const hipError_t e = a.dt == kBF16 ? launch_mtile_dt<kBF16>(a, p, s) : launch_mtile_dt<kF16>(a, p, s);
  if (e != hipSuccess || p.ks == 1) return e;
  return launch_splitk_reduce(part, p.ks, a.M, a.N, a.Y, a.ldy, a.dt, p.gated, s);
}

hipError_t launch_splitk_reduce(const float* part, int ks, int M, int N, uint16_t* Y, int64_t ldy,
                                int dt, bool gated, hipStream_t s) {
  const int64_t total = (int64_t)M * N / 4 + 1;
  const int blocks = (int)std::min<int64_t>((total + 255) / 256, 16384);
  auto go = [&](auto k) {
    hipLaunchKernelGGL(k, dim3(blocks), dim3(256), 0, s, part, ks, M, N, Y, ldy);
    return hipGetLastError();
  };
  if (dt == kBF16) return gated ? go(k_splitk_reduce<kBF16, true>) : go(k_splitk_reduce<kBF16, false>);
  return gated ? go(k_splitk_reduce<kF16, true>) : go(k_splitk_reduce<kF16, false>);
}

hipError_t launch_gather_rows(const uint16_t* X, int64_t ldx, int M, int K, const int32_t* perm,
                              uint16_t* Xp, hipStream_t s) {
  const size_t lds = (size_t)K * 2;
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k_gather_rows,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_gather_rows, dim3(M), dim3(256), lds, s, X, ldx, K, perm, Xp);
  return hipGetLastError();
}

}  // namespace tpdq
