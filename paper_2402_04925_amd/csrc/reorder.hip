// Offline reorder on gfx950: Alg. 1 (P = argsort(g_idx), g_opt = g_idx[P])
// and the permutations of the packed weights and their metadata (section 2.2:
// W1[P1, P2], W2[P2]).
//
// The sort is a counting sort: with off[g] the number of rows in groups
// before g (an exclusive scan of the group counts, which the validation pass
// computes anyway), the sorted position of row i is
//   off[g_idx[i]] + #{ j < i : g_idx[j] == g_idx[i] }
// (ascending groups, ties by ascending row: the stable order). For Eq. 3's
// groups off[g] = g G. One workgroup per group sweeps g_idx in row order and
// ranks the group's members with wave ballots, so the result does not depend
// on scheduling.
#include "tpdq_internal.h"

namespace tpdq {
namespace {

__global__ void k_fill_u32(uint32_t* p, size_t n, uint32_t v) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// flag bit 0: a g_idx value out of [0, num_groups); bit 1: a group whose
// count differs from what Eq. 3 gives (set by k_check_counts). LDS: a
// workgroup counts its rows there first, since under act-order the rows of a
// group lie in every workgroup and their global atomics on one counter
// serialise (K = 28672, 224 groups: 14.2 us, all rows on global counters).
template <bool LDS>
__global__ void k_count_groups(const int32_t* __restrict__ g_idx, int K, int num_groups,
                               uint32_t* __restrict__ counts, uint32_t* __restrict__ flag) {
  extern __shared__ uint32_t local[];
  if (LDS) {
    for (int g = threadIdx.x; g < num_groups; g += blockDim.x) local[g] = 0u;
    __syncthreads();
  }
  uint32_t* c = LDS ? local : counts;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < K; i += gridDim.x * blockDim.x) {
    const uint32_t g = (uint32_t)g_idx[i];
    if (g >= (uint32_t)num_groups)
      atomicOr(flag, 1u);
    else
      atomicAdd(c + g, 1u);
  }
  if (LDS) {
    __syncthreads();
    for (int g = threadIdx.x; g < num_groups; g += blockDim.x)
      if (local[g]) atomicAdd(counts + g, local[g]);
  }
}

// Eq. 3 with a permutation phi of 0..K-1: G rows in every group but the last,
// which holds K - (num_groups - 1) G (a partial group when G does not divide K)
__global__ void k_check_counts(const uint32_t* __restrict__ counts, int num_groups, int G, int K,
                               uint32_t* __restrict__ flag) {
  for (int g = blockIdx.x * blockDim.x + threadIdx.x; g < num_groups; g += gridDim.x * blockDim.x) {
    const uint32_t want = g == num_groups - 1 ? (uint32_t)(K - (num_groups - 1) * G) : (uint32_t)G;
    if (counts[g] != want) atomicOr(flag, 2u);
  }
}

// counts -> exclusive prefix sums, in place (one workgroup: 256 counts per
// pass into LDS, scanned serially there by thread 0, which carries the
// running total from pass to pass)
__global__ __launch_bounds__(256) void k_scan_counts(uint32_t* __restrict__ counts, int num_groups) {
  __shared__ uint32_t buf[256];
  uint32_t carry = 0;
  for (int c0 = 0; c0 < num_groups; c0 += 256) {
    const int g = c0 + (int)threadIdx.x;
    buf[threadIdx.x] = g < num_groups ? counts[g] : 0u;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int i = 0; i < 256; ++i) {
        const uint32_t v = buf[i];
        buf[i] = carry;
        carry += v;
      }
    }
    __syncthreads();
    if (g < num_groups) counts[g] = buf[threadIdx.x];
    __syncthreads();
  }
}

// One workgroup (16 waves) per group g; offs from k_scan_counts. Each pass of
// the workgroup covers 4096 rows, four neighbouring ones per thread: the
// sweep is a serial chain of passes (two barriers and an L2 round trip each),
// so few long passes beat many short ones (K = 28672, 224 groups: 112 passes
// of 256 rows 57 us).
__global__ __launch_bounds__(1024) void k_rank_group(const int32_t* __restrict__ g_idx, int K,
                                                     const uint32_t* __restrict__ offs, int num_groups,
                                                     int32_t* __restrict__ P,
                                                     int32_t* __restrict__ g_sorted) {
  __shared__ int wave_count[2][16];
  const int g = blockIdx.x;
  const int first = (int)offs[g];
  const int end = g + 1 < num_groups ? (int)offs[g + 1] : K;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int base = 0;  // members of group g already placed (rows before this chunk)
  int buf = 0;
  for (int c0 = 0; c0 < K; c0 += 4096) {
    const int i = c0 + 4 * threadIdx.x;  // K % 8 == 0, g_idx 16-byte aligned
    int4 v = make_int4(-1, -1, -1, -1);
    if (i < K) v = *(const int4*)(g_idx + i);
    const bool hit[4] = {v.x == g, v.y == g, v.z == g, v.w == g};
    // hits of the lower lanes (all four rows), and of the whole wave
    int below = 0, mine = 0;
    const unsigned long long lower = (1ull << lane) - 1ull;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned long long m = __ballot(hit[e]);
      below += __popcll(m & lower);
      mine += __popcll(m);
    }
    if (lane == 0) wave_count[buf][wave] = mine;
    __syncthreads();  // the other buffer is free again one barrier later
    int before = base, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      const int n = wave_count[buf][w];
      if (w < wave) before += n;
      total += n;
    }
    int r = first + before + below;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (hit[e]) {
        if (r < end) {
          P[r] = i + e;
          g_sorted[r] = g;
        }
        ++r;
      }
    }
    base += total;
    buf ^= 1;
  }
}

// One output word: rows P_row[8r .. 8r+7] of source column cs; nibble t of
// the result = nibble (i & 7) of src word [i >> 3][cs], i = P_row[8r + t].
__device__ __forceinline__ uint32_t gather_word(const uint32_t* __restrict__ src, int64_t ld_src,
                                                int K, const int32_t* __restrict__ Prow, int r,
                                                uint32_t cs) {
  if (!Prow) return src[(int64_t)r * ld_src + cs];
  const uint32_t kmax = (uint32_t)(K - 1);
  uint32_t out = 0;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const uint32_t i = min((uint32_t)Prow[8 * r + t], kmax);
    const uint32_t w = src[(int64_t)(i >> 3) * ld_src + cs];
    out |= ((w >> (4 * (i & 7))) & 0xFu) << (4 * t);
  }
  return out;
}

// GPTQ-layout output: dst[r][c] = W[P_row, P_col] word.
__global__ void k_permute_qweight(const uint32_t* __restrict__ src, int64_t ld_src, int K, int N,
                                  const int32_t* __restrict__ Prow, const int32_t* __restrict__ Pcol,
                                  uint32_t* __restrict__ dst) {
  const int64_t words = (int64_t)(K / 8) * N;
  const uint32_t nmax = (uint32_t)(N - 1);
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < words;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int r = (int)(idx / N);
    const int c = (int)(idx - (int64_t)r * N);
    const uint32_t cs = Pcol ? min((uint32_t)Pcol[c], nmax) : (uint32_t)c;
    dst[idx] = gather_word(src, ld_src, K, Prow, r, cs);
  }
}

// A GPTQ word (row 8r + i at bits 4i) in the tiled nibble order: row 8r + i
// at bits 4 (i >> 1) + 16 (i & 1), the even rows in the low half-word and the
// odd rows in the high one.
__device__ __forceinline__ uint32_t interleave_nibbles(uint32_t w) {
  uint32_t out = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) out |= ((w >> (4 * i)) & 0xFu) << (4 * (i >> 1) + 16 * (i & 1));
  return out;
}

// Tiled output: dst[t][256 b + 4 l + u] = word [4 (4 b + u) + kq][16 t + j]
// with its nibbles interleaved, l = 16 kq + j; words past K or N are zero.
__global__ void k_permute_qweight_tiled(const uint32_t* __restrict__ src, int64_t ld_src, int K,
                                        int N, const int32_t* __restrict__ Prow,
                                        const int32_t* __restrict__ Pcol,
                                        uint32_t* __restrict__ dst) {
  const int64_t ld = tiled_ld(K);
  const int ntiles = (N + 15) / 16;
  const int64_t words = (int64_t)ntiles * ld;
  const uint32_t nmax = (uint32_t)(N - 1);
  const int kw = K / 8;
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < words;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int t = (int)(idx / ld);
    const int o = (int)(idx - (int64_t)t * ld);
    const int b = o >> 8;
    const int l = (o >> 2) & 63;
    const int u = o & 3;
    const int r = 4 * (4 * b + u) + (l >> 4);
    const int c = 16 * t + (l & 15);
    uint32_t v = 0u;
    if (r < kw && c < N) {
      const uint32_t cs = Pcol ? min((uint32_t)Pcol[c], nmax) : (uint32_t)c;
      v = interleave_nibbles(gather_word(src, ld_src, K, Prow, r, cs));
    }
    dst[idx] = v;
  }
}

// ---------------------------------------------------------------------------
// Row and column gather of a whole layer through LDS.
//
// Both permutations are random, so a word-at-a-time gather from global memory
// touches a 128-byte line for every 4-byte word, eight times per output word
// (the kernels above on the Llama-70B W1, 8192 x 28672: 3.4 ms). The gather is
// HBM work (read and write K N / 2 bytes) once the random accesses happen in
// LDS instead, in two passes:
//   1. k_permute_cols: a workgroup holds one source word row (N words) in LDS
//      and writes it with its columns in the new order;
//   2. k_permute_rows: a workgroup holds CW columns of every word row in LDS
//      and writes their words with the rows in the new order.
// Measured on that W1: 66 + 55 us (3.6 and 4.3 TB/s read + write), where the
// word-by-word kernel took 3.4 ms; the whole reorder of the layer pair
// 3791 -> 295 us.
// Pass 1 writes into the destination, each 16-column tile's words inside the
// memory of that same tile, and pass 2 reads all of them before it writes its
// tile, so no scratch is needed. Without a column permutation pass 2 reads the
// source directly.
// ---------------------------------------------------------------------------
constexpr int kPermThreads = 1024;

// TILED: word row r of columns 16 t .. 16 t + 15 goes to words 16 r .. 16 r + 15
// of destination tile t (pass 2 puts them in the tiled order); else dst[r][c].
// Neighbouring word rows run on one XCD, whose L2 merges their 64-byte pieces.
template <bool TILED>
__global__ __launch_bounds__(kPermThreads) void k_permute_cols(
    const uint32_t* __restrict__ src, int64_t ld_src, int K, int N, const int32_t* __restrict__ Pcol,
    uint32_t* __restrict__ dst) {
  extern __shared__ __align__(16) uint32_t row[];
  const int nb = (int)gridDim.x;
  const int r = nb % 8 ? (int)blockIdx.x : (int)(blockIdx.x % 8) * (nb / 8) + (int)(blockIdx.x / 8);
  const uint32_t* sr = src + (int64_t)r * ld_src;
  for (int c = 4 * threadIdx.x; c < N; c += 4 * kPermThreads)  // N % 8 == 0, 16-byte aligned rows
    *(uint4*)(row + c) = *(const uint4*)(sr + c);
  __syncthreads();
  const uint32_t nmax = (uint32_t)(N - 1);
  const int64_t ld = tiled_ld(K);
  for (int c = threadIdx.x; c < N; c += kPermThreads) {
    const uint32_t v = row[min((uint32_t)Pcol[c], nmax)];
    if (TILED)
      dst[(int64_t)(c >> 4) * ld + 16 * r + (c & 15)] = v;
    else
      dst[(int64_t)r * N + c] = v;
  }
}

// quad_perm lane exchanges (lane ^ 1, lane ^ 2)
__device__ __forceinline__ uint32_t quad_xor1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t quad_xor2(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);
}

// 4 x 4 transpose over the four lanes of a quad: lane u holds a[0..3] of row u
// and ends with column u.
__device__ __forceinline__ void quad_transpose(uint32_t (&a)[4], int u) {
#pragma unroll
  for (int h = 0; h < 4; h += 2) {
    const uint32_t r = quad_xor1((u & 1) ? a[h] : a[h + 1]);
    if (u & 1) a[h] = r; else a[h + 1] = r;
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const uint32_t r = quad_xor2((u & 2) ? a[h] : a[h + 2]);
    if (u & 2) a[h] = r; else a[h + 2] = r;
  }
}

// CW columns (16, or 8 when 16 columns of all rows don't fit in LDS) of every
// word row. IN_PLACE: they are pass 1's output in dst, else src's. A thread
// builds four neighbouring columns of one word row (one 16-byte LDS read per
// source row and one set of row addresses for the four); in the tiled order
// the four lanes of a quad hold steps u = 0 .. 3 and transpose, so that every
// lane stores 16 bytes.
template <int CW, bool TILED, bool IN_PLACE>
__global__ __launch_bounds__(kPermThreads) void k_permute_rows(
    const uint32_t* __restrict__ src, int64_t ld_src, int K, int N, const int32_t* __restrict__ Prow,
    uint32_t* dst) {
  static_assert(CW == 16 || (CW == 8 && !(TILED && IN_PLACE)),
                "a tile is one workgroup's where its words are overwritten");
  constexpr int Q = CW / 4;
  extern __shared__ __align__(16) uint4 words[];  // [K / 8][Q]
  const int nb = (int)gridDim.x;
  const int cg = nb % 8 ? (int)blockIdx.x : (int)(blockIdx.x % 8) * (nb / 8) + (int)(blockIdx.x / 8);
  const int c0 = cg * CW;
  const int kw = K >> 3;
  const int64_t ld = tiled_ld(K);
  uint32_t* tile = dst + (int64_t)(c0 >> 4) * ld;
  for (int i = threadIdx.x; i < kw * Q; i += kPermThreads) {
    const int r = i / Q, q = i % Q;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (c0 + 4 * q < N) {
      if (IN_PLACE && TILED)
        v = *(const uint4*)(tile + 16 * r + 4 * q);
      else if (IN_PLACE)
        v = *(const uint4*)(dst + (int64_t)r * N + c0 + 4 * q);
      else
        v = *(const uint4*)(src + (int64_t)r * ld_src + c0 + 4 * q);
    }
    words[i] = v;
  }
  __syncthreads();
  const uint32_t kmax = (uint32_t)(K - 1);
  const int rows = TILED ? 16 * ((K + 127) >> 7) : kw;  // the tiled order pads the last block
  for (int i = threadIdx.x; i < rows * Q; i += kPermThreads) {
    // TILED: i = ((4 b + kq) Q + q) 4 + u, word row 4 (4 b + u) + kq; a quad
    // of lanes covers u = 0 .. 3 (rows * Q is a multiple of 4)
    const int u = i & 3;
    const int q = TILED ? (i >> 2) % Q : i % Q;
    const int bk = TILED ? (i >> 2) / Q : 0;
    const int b = bk >> 2, kq = bk & 3;
    const int r = TILED ? 4 * (4 * b + u) + kq : i / Q;
    uint32_t o[4] = {0u, 0u, 0u, 0u};
    if (r < kw) {
      const uint4 p0 = *(const uint4*)(Prow + 8 * r);
      const uint4 p1 = *(const uint4*)(Prow + 8 * r + 4);
      const uint32_t p[8] = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const uint32_t k = min(p[t], kmax);
        const uint4 w = words[(k >> 3) * Q + q];
        const uint32_t sh = 4u * (k & 7u);
        // row 8r + t: bits 4t, or 4 (t / 2) + 16 (t % 2) in a tiled word
        const int to = TILED ? 4 * (t >> 1) + 16 * (t & 1) : 4 * t;
        o[0] |= ((w.x >> sh) & 0xFu) << to;
        o[1] |= ((w.y >> sh) & 0xFu) << to;
        o[2] |= ((w.z >> sh) & 0xFu) << to;
        o[3] |= ((w.w >> sh) & 0xFu) << to;
      }
    }
    if (TILED) {
      quad_transpose(o, u);  // lane u: column 4 q + u, steps 0 .. 3
      const int l = 16 * kq + (c0 & 15) + 4 * q + u;
      *(uint4*)(tile + 256 * b + 4 * l) = make_uint4(o[0], o[1], o[2], o[3]);
    } else if (c0 + 4 * q < N) {
      *(uint4*)(dst + (int64_t)r * N + c0 + 4 * q) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}

// dst[g][c] = src[g][P_col[c]] (2-byte elements; fp16 or bf16 bits).
__global__ void k_permute_scales(const uint16_t* __restrict__ src, int64_t ld_src, int ng, int N,
                                 const int32_t* __restrict__ Pcol, uint16_t* __restrict__ dst) {
  const int64_t total = (int64_t)ng * N;
  const uint32_t nmax = (uint32_t)(N - 1);
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int g = (int)(idx / N);
    const int c = (int)(idx - (int64_t)g * N);
    const uint32_t cs = Pcol ? min((uint32_t)Pcol[c], nmax) : (uint32_t)c;
    dst[idx] = src[(int64_t)g * ld_src + cs];
  }
}

// Zero codes packed along N: nibble t of dst word [g][cw] = zero of column
// P_col[8 cw + t] of group g.
__global__ void k_permute_qzeros(const uint32_t* __restrict__ src, int64_t ld_src, int ng, int N,
                                 const int32_t* __restrict__ Pcol, uint32_t* __restrict__ dst) {
  const int nw = N / 8;
  const int64_t total = (int64_t)ng * nw;
  const uint32_t nmax = (uint32_t)(N - 1);
  for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
       idx += (int64_t)gridDim.x * blockDim.x) {
    const int g = (int)(idx / nw);
    const int cw = (int)(idx - (int64_t)g * nw);
    uint32_t out = 0;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t c = Pcol ? min((uint32_t)Pcol[8 * cw + t], nmax) : (uint32_t)(8 * cw + t);
      const uint32_t w = src[(int64_t)g * ld_src + (c >> 3)];
      out |= ((w >> (4 * (c & 7))) & 0xFu) << (4 * t);
    }
    dst[idx] = out;
  }
}

int grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 8192) b = 8192;
  if (b < 1) b = 1;
  return (int)b;
}

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_u32, dim3(grid_for((int64_t)n)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_gidx_validate(const ReorderLayer& L, uint32_t* counts, uint32_t* flag,
                                hipStream_t s) {
  // counters in LDS where they fit 16 KiB: 4096 rows per workgroup
  if (L.num_groups <= 4096)
    hipLaunchKernelGGL(k_count_groups<true>, dim3((L.K + 4095) / 4096), dim3(1024),
                       (size_t)L.num_groups * 4, s, L.g_idx, L.K, L.num_groups, counts, flag);
  else
    hipLaunchKernelGGL(k_count_groups<false>, dim3(grid_for(L.K)), dim3(256), 0, s, L.g_idx, L.K,
                       L.num_groups, counts, flag);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || L.G == 0) return e;  // G == 0: groups of any size
  hipLaunchKernelGGL(k_check_counts, dim3(grid_for(L.num_groups)), dim3(256), 0, s, counts,
                     L.num_groups, L.G, L.K, flag);
  return hipGetLastError();
}

hipError_t launch_gidx_rank(const ReorderLayer& L, uint32_t* offs, hipStream_t s) {
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(256), 0, s, offs, L.num_groups);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_rank_group, dim3(L.num_groups), dim3(1024), 0, s, L.g_idx, L.K, offs,
                     L.num_groups, L.P, L.g_sorted);
  return hipGetLastError();
}

namespace {
template <typename Kern, typename... Args>
hipError_t launch_lds(Kern k, int grid, size_t lds, hipStream_t s, Args... args) {
  if (lds > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kLdsMax);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3(grid), dim3(kPermThreads), lds, s, args...);
  return hipGetLastError();
}

template <bool TILED>
hipError_t permute_through_lds(const uint32_t* src, int64_t ld_src, int K, int N, const int32_t* Prow,
                               const int32_t* Pcol, uint32_t* dst, bool* done, hipStream_t s) {
  const size_t rows16 = (size_t)(K / 8) * 64, rows8 = (size_t)(K / 8) * 32;
  *done = true;
  if (Pcol && (size_t)N * 4 <= kLdsMax && rows16 <= kLdsMax) {
    hipError_t e = launch_lds(k_permute_cols<TILED>, K / 8, (size_t)N * 4, s, src, ld_src, K, N, Pcol, dst);
    if (e != hipSuccess) return e;
    return launch_lds(k_permute_rows<16, TILED, true>, (N + 15) / 16, rows16, s, src, ld_src, K, N, Prow,
                      dst);
  }
  // 16 columns where two workgroups then share a CU, else 8 (a tiled tile is
  // then two workgroups', its last half zeros where N ends inside it)
  if (!Pcol && rows16 <= kLdsMax / 2)
    return launch_lds(k_permute_rows<16, TILED, false>, (N + 15) / 16, rows16, s, src, ld_src, K, N, Prow,
                      dst);
  if (!Pcol && rows8 <= kLdsMax)
    return launch_lds(k_permute_rows<8, TILED, false>, TILED ? 2 * ((N + 15) / 16) : N / 8, rows8, s, src,
                      ld_src, K, N, Prow, dst);
  *done = false;
  return hipSuccess;
}
}  // namespace

hipError_t launch_permute_qweight(const uint32_t* src, int64_t ld_src, int K, int N,
                                  const int32_t* Prow, const int32_t* Pcol, uint32_t* dst,
                                  int dst_layout, hipStream_t s) {
  // gathers whose rows and columns fit in LDS; what is larger (with a column
  // permutation K > 20480 or N > 40960, else K > 40960) and the plain
  // repacking (no row permutation: already coalesced) word by word, as what
  // is not on 16 bytes (the caller's P and outputs may be on any word)
  const uintptr_t at = (uintptr_t)src | (uintptr_t)Prow | (uintptr_t)dst;
  // ... and as small layers, whose gathers hit the caches and whose reorder the
  // host's launches bound (pairs of K x N and N x K, word by word / through
  // LDS: 1024 x 1024 93 / 119 us, 4096 x 2048 114-120 / 123, 4096 x 4096 171 / 117)
  const bool large = (int64_t)K * N >= (int64_t)12 << 20;
  if (Prow && large && at % 16 == 0 && ld_src % 4 == 0 && K % 8 == 0 && N % 8 == 0) {
    bool done = false;
    const hipError_t e =
        dst_layout == TPDQ_LAYOUT_TILED
            ? permute_through_lds<true>(src, ld_src, K, N, Prow, Pcol, dst, &done, s)
            : permute_through_lds<false>(src, ld_src, K, N, Prow, Pcol, dst, &done, s);
    if (done || e != hipSuccess) return e;
  }
  if (dst_layout == TPDQ_LAYOUT_TILED) {
    const int64_t words = (int64_t)((N + 15) / 16) * tiled_ld(K);
    hipLaunchKernelGGL(k_permute_qweight_tiled, dim3(grid_for(words)), dim3(256), 0, s, src, ld_src,
                       K, N, Prow, Pcol, dst);
  } else {
    hipLaunchKernelGGL(k_permute_qweight, dim3(grid_for((int64_t)(K / 8) * N)), dim3(256), 0, s,
                       src, ld_src, K, N, Prow, Pcol, dst);
  }
  return hipGetLastError();
}

hipError_t launch_permute_scales(const uint16_t* src, int64_t ld_src, int ng, int N,
                                 const int32_t* Pcol, uint16_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_permute_scales, dim3(grid_for((int64_t)ng * N)), dim3(256), 0, s, src,
                     ld_src, ng, N, Pcol, dst);
  return hipGetLastError();
}

hipError_t launch_permute_qzeros(const uint32_t* src, int64_t ld_src, int ng, int N,
                                 const int32_t* Pcol, uint32_t* dst, hipStream_t s) {
  hipLaunchKernelGGL(k_permute_qzeros, dim3(grid_for((int64_t)ng * (N / 8))), dim3(256), 0, s, src,
                     ld_src, ng, N, Pcol, dst);
  return hipGetLastError();
}

}  // namespace tpdq
