// Grouped mixed-bit expert GEMM (Sec. 3.3.2: dequantization fused with the
// expert matrix products) for any number of tokens per expert, and the
// weighted combine (Fig. 1: outputs of the activated experts weighted by the
// gate).
//
// Positions are the (token, slot) pairs sorted by (expert, bit-width).  An
// expert's positions are cut, bit-width by bit-width, into blocks of at most
// 16 positions, and its blocks, in ascending bit-width, into chunks of at most
// kBlocks = 8.  One 4-wave workgroup computes one chunk against 128 weight
// rows; each wave owns 32 of the rows (W1/W3: 16 rows of W1 and the same 16 of
// W3; W2: 32 rows) and all of the chunk's positions.
//
// The weights never pass through LDS: a lane dequantizes the 32 columns of
// one plane word per row tile straight into the operands of four
// v_mfma_f32_16x16x32_bf16 (lane 16 q + i holds row i, columns 8 s .. 8 s + 7
// of run q of the step's 128 columns in product s).  Chunks mix bit-widths:
// planes are added lowest first, and the blocks of width b run their products
// right after plane b - 1, so the nest is dequantized once for every width of
// the chunk.  The activations of a step (128 columns of every position) are
// brought into LDS by the DMA engine one step ahead and shared by the waves;
// one barrier per step orders them.
//
// What bounds it: the vector ALU, issuing 63 to 78 % of the cycles at 301 to 512
// tokens (matrix pipe 11 to 14 %), then the waits of two waves per SIMD for one
// step's loads.  Dequantizing a pair of weights costs 3 packed operations for a
// plane by its sign, about half of that for the two or three planes that come by
// lookup, and 3 conversions per width, against one 16-cycle product per 16
// positions and 32 columns of 16 rows.
#include <type_traits>

#include "lookup.h"

namespace d2moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
using lookup::as_h2;
using lookup::as_u;
using lookup::h2;
using lookup::rotr;
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));

constexpr int kBlockPos = 16;                    // positions per block (MFMA columns)
constexpr int kBlocks = 8;                       // blocks per chunk
constexpr int kGemmWaves = 4;                    // waves per workgroup, one per SIMD
constexpr int kGemmThreads = 64 * kGemmWaves;
constexpr int kTileRows = 128;                   // weight rows per workgroup
constexpr int kStepK = 128;                      // reduction columns per step
constexpr int kBlockBytes = kBlockPos * kStepK * 2;  // one block's activations of a step
constexpr int kStageBytes = kBlocks * kBlockBytes;

#define D2MOE_GPTR(p) ((__attribute__((address_space(1))) void*)(p))
#define D2MOE_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// The work of a GEMM launch: chunk c of the routed experts is entry c of the
// table that chunk_kernel writes, or, with `table` NULL, chunk c of one bucket
// of `one_cnt` positions from `one_first` at `one_bits` bits of expert
// `one_expert`, one_blocks blocks per chunk.
struct GemmWork {
  const int32_t* table;    // chunk_kernel's; entry c in words 4 (c + 1) ..
  const int32_t* hist;     // [E][L]
  const int32_t* offsets;  // [E L + 1]
  int L;
  int one_first, one_cnt, one_bits, one_expert, one_blocks;
};

// Chunks of one expert with n[l] positions at the l-th bit-width.
// Register chunks: the expert's blocks, all bit-widths together, in as few
// chunks of at most kBlocks as hold them.  Tile chunks: the positions of each
// bucket in chunks of kTileChunk.
struct ChunkCount {
  int reg, cost, tiles;  // cost: of the register chunks (use_tiles)
};
__host__ __device__ inline int expert_blocks(const int32_t* n, int L, int b_min, ChunkCount* c) {
  int blocks = 0, widths = 0, top = 0;
  for (int l = 0; l < L; ++l) {
    blocks += (n[l] + kBlockPos - 1) / kBlockPos;
    c->tiles += (n[l] + kTileChunk - 1) / kTileChunk;
    widths += n[l] > 0;
    if (n[l] > 0) top = b_min + l;
  }
  const int reg = (blocks + kBlocks - 1) / kBlocks;
  c->reg += reg;
  c->cost += reg * (24 + 3 * top + 4 * widths);
  return blocks;
}

// Whether the layer's routed experts take the tile GEMM (all of them: with some
// on each, the two launches follow one another, each with its own tail, and at
// 8 experts of d 4096, d_ff 4096, one width of 4 bits, 130 positions per expert
// a step took 392 us with half of them on tiles, 280 on registers, 283 on tiles).
// A chunk dequantizes 128 rows, once for up to 256 positions of one width (tile)
// or 128 of any (register).  A register chunk of w widths up to b bits takes
// about (24 + 3 b + 4 w) / 48 of a tile chunk's time in W1/W3, and 0.4 of that in
// W2, whose reduction it takes in two groups where workgroups are few; about 256
// workgroups of W1/W3 and 384 of W2 run at once, so fewer take the time of that
// many.  Fitted to 1828 layers (E 1 to 64, d 512 to 5120, up to 384 positions per
// expert, one to seven widths, even and Zipf load): 0.2 % above the faster GEMM on
// average.  Tile / register, us per step: 8 experts of d 4096, d_ff 14336, 260 per
// expert, 8 bits 1651 / 2145 (tile), 4 bits 1368 / 1358 and widths 2, 4, 8 2207 /
// 2121 (register); 4 experts of d 1024, d_ff 2048, 260 per expert, 4 bits 115 / 86
// (register: 224 workgroups); 16 of d 2048, d_ff 1408, Zipf load, 180 per expert,
// each of one width, 176 / 208 (tile).
// From kTileAverage positions per expert on it is tiles whatever the counts, so
// that the register launch is left out.
constexpr int kTileAverage = 384;
// Bound on the tile chunks of a layer of T tokens, top-k, that would make at most
// `reg` register chunks; at 0 the tile launch is left out.  use_tiles keeps to it:
// as many tile chunks as register chunks are slower (with at most 128 tokens, and
// so positions per expert, there are no fewer), and so are tile chunks of few
// positions (64 experts, Zipf load, 45 per tile chunk 343 / 247).
__host__ __device__ inline int tile_bound(int T, int k, int reg) {
  if (T <= kBlocks * kBlockPos) return 0;
  return T * k / 48 < reg ? T * k / 48 : reg - 1;
}
__host__ __device__ inline bool use_tiles(const ChunkCount& c, int T, int k, int d, int d_ff) {
  if (c.tiles > tile_bound(T, k, c.reg)) return false;
  const long rows13 = (d_ff + kTileRows / 2 - 1) / (kTileRows / 2);
  const long rows2 = (d + kTileRows - 1) / kTileRows;
  auto at_least = [](long n, long least) { return n > least ? n : least; };
  const long reg = 5 * at_least(c.reg * rows13, 256) * d + 2 * at_least(c.reg * rows2, 384) * d_ff;
  const long tiles = 5 * (at_least(c.tiles * rows13, 256) * d + at_least(c.tiles * rows2, 384) * d_ff);
  return c.cost * reg > 48 * c.reg * tiles;
}

// Sum over the 64 lanes of a wave, in every lane (DPP row shifts, then the rows).
__device__ inline int wave_total(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
  return __builtin_amdgcn_readlane(v, 15) + __builtin_amdgcn_readlane(v, 31) +
         __builtin_amdgcn_readlane(v, 47) + __builtin_amdgcn_readlane(v, 63);
}

// Chunk table of the layer's GEMM from the routing histogram, in slots of four
// words: slot 0 = {register chunks, tile chunks}, one of them 0; then the chunks,
// a register chunk as {expert | blocks << 8, first block of the expert} (an
// expert's chunks are of even size), a tile chunk as {first position, positions,
// bit-width, expert}.
//
// Longest workgroups first: experts (buckets) of the largest bit-width, then of
// the most positions.  One workgroup of kChunkThreads threads, one per expert
// (E <= 64) and one per bucket (E L <= 512).  Workgroups past the first round n
// values of x to bf16 in xb instead: neither needs the other, and a launch of
// its own takes 2 us of a small fp32 layer's 45 (64 tokens of 256, d_ff 512).
constexpr int kChunkThreads = 512;
constexpr int kConvert = 4;  // values per thread
__global__ __launch_bounds__(kChunkThreads) void chunk_kernel(
    const int32_t* __restrict__ hist, const int32_t* __restrict__ offsets, int E, int L, int b_min,
    int T, int k, int d, int d_ff, bool all_tile, int32_t* __restrict__ table,
    const float* __restrict__ x, size_t n, uint16_t* __restrict__ xb) {
  if (blockIdx.x > 0) {  // workgroup-uniform
    const size_t i0 = (size_t)(blockIdx.x - 1) * (kChunkThreads * kConvert) + threadIdx.x;
#pragma unroll
    for (int i = 0; i < kConvert; ++i) {
      const size_t at = i0 + i * kChunkThreads;
      if (at < n) xb[at] = f2bf(x[at]);
    }
    return;
  }
  __shared__ int rkey[64], nreg[64];
  __shared__ ChunkCount total;
  __shared__ int tkey[kChunkThreads], ntile[kChunkThreads];
  const int j = threadIdx.x;
  int tot = 0;
  if (j < 64) {  // the first wave
    int n[8], mb = 0;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
      n[l] = j < E && l < L ? hist[j * L + l] : 0;
      if (n[l] > 0) mb = l + 1;
    }
    ChunkCount c{};
    tot = expert_blocks(n, 8, b_min, &c);
    rkey[j] = (mb << 24) + min(tot, (1 << 24) - 1);
    nreg[j] = c.reg;
    c = {wave_total(c.reg), wave_total(c.cost), wave_total(c.tiles)};
    if (j == 0) total = c;
  }
  __syncthreads();
  const ChunkCount sum = total;
  int first = 0;
  if (!all_tile && !use_tiles(sum, T, k, d, d_ff)) {  // workgroup-uniform
    if (j == 0) {
      table[0] = sum.reg;
      table[1] = 0;
    }
    if (j < E) {
      for (int o = 0; o < E; ++o)
        if (rkey[o] > rkey[j] || (rkey[o] == rkey[j] && o < j)) first += nreg[o];
      const int nc = nreg[j];
      for (int c = 0; c < nc; ++c) {
        const int b0 = (int)((long)c * tot / nc), b1 = (int)((long)(c + 1) * tot / nc);
        table[4 * (1 + first + c)] = j | (b1 - b0) << 8;
        table[4 * (1 + first + c) + 1] = b0;
      }
    }
    return;
  }
  const int nb = E * L;
  const int cnt = j < nb ? hist[j] : 0;
  ntile[j] = (cnt + kTileChunk - 1) / kTileChunk;
  tkey[j] = cnt > 0 ? ((j % L + 1) << 24) + min(cnt, (1 << 24) - 1) : 0;
  __syncthreads();
  for (int o = 0; o < nb; ++o)
    if (tkey[o] > tkey[j] || (tkey[o] == tkey[j] && o < j)) first += ntile[o];
  if (j == 0) {
    table[0] = 0;
    table[1] = sum.tiles;
  }
  for (int c = 0; c < ntile[j]; ++c) {
    int32_t* t = table + 4 * (1 + first + c);
    t[0] = offsets[j] + c * kTileChunk;
    t[1] = min(kTileChunk, cnt - c * kTileChunk);
    t[2] = b_min + j % L;
    t[3] = j / L;
  }
}

__device__ inline float silu(float a) { return a / (1.0f + __expf(-a)); }

__device__ inline uint32_t h2_splat(float v) {
  const _Float16 h = (_Float16)v;
  return as_u(h2{h, h});
}

// Reads of the DMA-filled LDS stages are inline assembly: with LDS DMA in
// flight the compiler would otherwise wait for every outstanding
// vector-memory instruction (draining the prefetch) before each of them.
// They are ordered by an explicit lgkmcnt wait in the same basic block, and
// re-bound after it.
__device__ inline uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// OFF is the instruction's unsigned 16-bit byte offset added to the address.
template <int OFF = 0>
__device__ inline void ld128(u32x4& v, uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
}
__device__ inline void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// f(integral_constant<int, i>) for i = 0 .. N-1, so that the index can be a
// template argument (an instruction offset) inside f.
template <int N, int I = 0, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Slot of 16-byte chunk 4 q + s (of 16) in the 256-byte LDS row of position r
// (of 16).  A 16-byte LDS read serves 16 lanes at a time: positions 0-3 and
// 12-15 of an even q with 4-11 of the odd one beside it, and the other half of
// each.  With q's two bits recoded to 0, 3, 1, 2 before the exclusive or, those
// 16 lanes fall in distinct banks; with q itself every read was a two-way
// conflict.
__device__ inline int slot_of_chunk(int q, int s, int r) {
  return (4 * (((q & 1) << 1) | ((q ^ (q >> 1)) & 1)) + s) ^ r;
}
// The chunk that slot `slot` of position r's row holds.
__device__ inline int chunk_at(int slot, int r) {
  const int v = slot ^ r, k = v >> 2;
  return 4 * ((k >> 1) | (((k ^ (k >> 1)) & 1) << 1)) + (v & 3);
}

// Source of the activation columns past the end of the reduction dimension.
__device__ __align__(16) const uint8_t zero_chunk[16] = {};

// Plane words, scales and zero point of one row tile that a lane dequantizes
// in one step: the word of plane p, the binary16 scale of plane p >= b_min,
// the base scale and the zero point.
struct RawTile {
  uint32_t w[8], sp[8], s1, z;
};

// One workgroup: chunk blockIdx.x / tiles against weight-row tile
// blockIdx.x % tiles (tiles fastest: consecutive workgroups, which the
// dispatcher deals round-robin to the 8 XCDs, share one chunk's activations).
//   in:  bf16 activations; position p reads row (perm ? perm[p] / kdiv : p)
//   SWIGLU: W is [2f][K] (w13); wave v holds W1 rows n0 + 16 v .. + 15 and the
//           same rows of W3 (f + ..), n0 = 64 tile; out = h [pos][f] bf16
//   else:   W is [N][K]; wave v holds rows n0 + 32 v .. + 31, n0 = 128 tile;
//           out = y [pos][N] fp32, the part blockIdx.y of gridDim.y of the
//           reduction in plane blockIdx.y (out_split values apart)
// BMIN > 0 fixes b_min at compile time (the common ladder starts at 2 bits);
// BMIN == 0 takes it from W.
// KS = 2 (the plain variant only): two such groups of four waves per workgroup,
// each with its own stages, take the first and the second half of the
// reduction, and the first adds the second's sums at the end.
template <int G, bool SWIGLU, int BMIN, int KS>
__global__ __launch_bounds__(KS * kGemmThreads) __attribute__((amdgpu_waves_per_eu(2)))
void bgemm_kernel(const uint16_t* __restrict__ in, int in_ld, const int32_t* __restrict__ perm,
                  int kdiv, MwqView W, GemmWork wk, int tiles, int f, int N,
                  void* __restrict__ out, int out_ld, size_t out_split) {
  __shared__ __attribute__((aligned(1024))) uint8_t xs_all[KS][2][kStageBytes];
  // first 16-byte unit of each position's activation row (kept in LDS rather
  // than in registers, and read before a step's DMA)
  __shared__ __attribute__((aligned(16))) uint32_t xrow_at[kBlockPos][kBlocks];
  __shared__ int blk_pos[kBlocks], blk_cnt[kBlocks], blk_bits[kBlocks];
  constexpr int BR = 2048 / G;   // rows per packed block
  constexpr int KPS = kStepK / G;  // packed blocks per step (1 or 2)

  const int chunk = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = wave_all & (kGemmWaves - 1), kg = KS > 1 ? wave_all / kGemmWaves : 0;
  uint8_t (&xs)[2][kStageBytes] = xs_all[kg];
  const int r = lane & 15, q = lane >> 4;
  const int b_min = BMIN > 0 ? BMIN : W.b_min;

  // ---- the chunk's blocks ----
  int expert, nblk;
  if (wk.table) {
    if (chunk >= wk.table[0]) return;
    const int e0 = wk.table[4 * (chunk + 1)];
    expert = e0 & 0xff;
    nblk = e0 >> 8;
    if (tid < kBlocks) {
      int b = wk.table[4 * (chunk + 1) + 1] + tid, pos = 0, cnt = 0, bits = 0;
      if (tid < nblk) {
        for (int l = 0; l < wk.L; ++l) {
          const int n = wk.hist[expert * wk.L + l], nb = (n + kBlockPos - 1) / kBlockPos;
          if (b < nb) {
            pos = wk.offsets[expert * wk.L + l] + kBlockPos * b;
            cnt = min(kBlockPos, n - kBlockPos * b);
            bits = b_min + l;
            break;
          }
          b -= nb;
        }
      }
      blk_pos[tid] = pos;
      blk_cnt[tid] = cnt;
      blk_bits[tid] = bits;
    }
  } else {
    expert = wk.one_expert;
    const int b0 = chunk * wk.one_blocks, all = (wk.one_cnt + kBlockPos - 1) / kBlockPos;
    nblk = min(wk.one_blocks, all - b0);
    if (nblk <= 0) return;
    if (tid < kBlocks) {
      const int at = kBlockPos * (b0 + tid);
      blk_pos[tid] = wk.one_first + at;
      blk_cnt[tid] = tid < nblk ? min(kBlockPos, wk.one_cnt - at) : 0;
      blk_bits[tid] = tid < nblk ? wk.one_bits : 0;
    }
  }
  __syncthreads();
  // widths in scalar registers: block i's in nibble i of `wid`, and the set
  uint32_t wid = 0, wset = 0;
  int bits = 0;
#pragma unroll
  for (int i = 0; i < kBlocks; ++i) {
    const int b = __builtin_amdgcn_readfirstlane(blk_bits[i]);
    wid |= (uint32_t)b << (4 * i);
    wset |= 1u << b;
    bits = b > bits ? b : bits;
  }

  // ---- activations: DMA instruction i moves this wave's four positions
  // 4 wave .. 4 wave + 3 of block i, 256 bytes of each, chunk c of a row at the
  // slot that slot_of_chunk gives it.  Positions past a block's end repeat its
  // last one (their results are not stored). ----
  const int K = W.cols;
  const int xrow = 4 * wave + q;            // row within the block
  const int xchunk = chunk_at(lane & 15, xrow);  // 16-byte chunk of the step this lane fetches
  if (tid < kBlockPos * kBlocks) {
    const int i = tid & (kBlocks - 1), row = tid / kBlocks, cnt = blk_cnt[i];
    const int pos = blk_pos[i] + min(row, max(cnt, 1) - 1);
    const int src = cnt > 0 ? (perm ? perm[pos] / kdiv : pos) : 0;
    xrow_at[row][i] = (uint32_t)((size_t)src * in_ld / 8);
  }
  __syncthreads();
  const int nall = (K + kStepK - 1) / kStepK;
  // this group's steps; both groups run `steps` of them (the second one's last
  // may be past its end: it only keeps the barriers in step)
  const int part = blockIdx.y * KS + kg, parts = gridDim.y * KS;
  const int it0 = SWIGLU ? 0 : (int)((long)part * nall / parts);
  const int it1 = SWIGLU ? nall : (int)((long)(part + 1) * nall / parts);
  int steps = it1 - it0;
  if (KS > 1) {
    const int o = blockIdx.y * KS + (kg ^ 1);
    steps = max(steps, (int)((long)(o + 1) * nall / parts) - (int)((long)o * nall / parts));
  }
  auto x_dma = [&](int it) {
    uint8_t* dst = xs[it & 1] + 1024 * wave;
    uint32_t xoff[kBlocks];
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) xoff[i] = xrow_at[xrow][i];
    const bool past = G < kStepK && kStepK * it + 8 * xchunk >= K;
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) {
      if (i < nblk) {
        const uint8_t* src = (const uint8_t*)in + (size_t)it * (2 * kStepK) +
                             ((size_t)xoff[i] + xchunk) * 16;
        if (G < kStepK) src = past ? zero_chunk : src;
        __builtin_amdgcn_global_load_lds(D2MOE_GPTR(src), D2MOE_LPTR(dst + kBlockBytes * i), 16, 0, 0);
      }
    }
  };

  // ---- weights: row tiles 0 and 1 of this wave, lane (r, q) row r of each,
  // columns 32 q .. 32 q + 31 of a step ----
  const int wn0 = tile * (SWIGLU ? 64 : kTileRows) + wave * (SWIGLU ? 16 : 32);
  const bool active = wn0 < (SWIGLU ? f : N);  // wave-uniform (f % 32 == 0, N % 64 == 0)
  const uint8_t *pbase[2], *sbase[2], *zbase[2];
  uint32_t poff[2], soff[2], zoff[2];
  const uint32_t pstep = (uint32_t)W.b_max * 256u * KPS, sstep = (uint32_t)W.levels() * BR * 2 * KPS,
                 zstep = BR * KPS;
  const uint32_t qblk = G < kStepK ? (uint32_t)(q >> 1) : 0u;  // packed block within the step
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int row0 = active ? (SWIGLU ? t * f + wn0 : wn0 + 16 * t) : 0;
    const size_t blk = W.block(expert, row0 / BR, 0);
    const int rr = row0 % BR + r;
    pbase[t] = (const uint8_t*)(W.planes + W.plane_word(blk, 0, 0));
    sbase[t] = (const uint8_t*)(W.scales + W.scale_idx(blk, 0, 0));
    zbase[t] = W.zeros + W.zero_idx(blk, 0);
    poff[t] = qblk * (W.b_max * 256u) + 4u * ((G < kStepK ? (q & 1) : q) * BR + rr);
    soff[t] = qblk * ((uint32_t)W.levels() * BR * 2) + 2u * rr;
    zoff[t] = qblk * BR + rr;
  }
  // A register of `raw` is loaded again for the next step as soon as this
  // step has used it.
  RawTile raw[2];
  const uint8_t *pb[2], *sb[2], *zb[2];  // of the step that is loaded
  uint32_t po[2], so[2], zo[2];
  auto at_step = [&](int it) {
    // the last step of a reduction dimension that ends in half a step: lanes
    // past the end read the first half again (and use scale 0)
    const bool past = G < kStepK && kStepK * it + 32 * q >= K;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      pb[t] = pbase[t] + (size_t)it * pstep;
      sb[t] = sbase[t] + (size_t)it * sstep;
      zb[t] = zbase[t] + (size_t)it * zstep;
      po[t] = past ? poff[t] - W.b_max * 256u : poff[t];
      so[t] = past ? soff[t] - (uint32_t)W.levels() * BR * 2 : soff[t];
      zo[t] = past ? zoff[t] - BR : zoff[t];
    }
  };
  auto load_base = [&](int t) {
    raw[t].s1 = *(const uint16_t*)(sb[t] + so[t]);
    raw[t].z = *(zb[t] + zo[t]);
  };
  auto load_plane = [&](int t, int p) {
    raw[t].w[p] = *(const uint32_t*)(pb[t] + po[t] + 256 * p);
    if (BMIN > 0) {
      if (p >= BMIN) raw[t].sp[p] = *(const uint16_t*)(sb[t] + so[t] + (p - BMIN + 1) * BR * 2);
    } else if (p >= 1) {  // below b_min the base scale is read and not used
      const int lev = p >= b_min ? p - b_min + 1 : 0;
      raw[t].sp[p] = *(const uint16_t*)(sb[t] + lev * (BR * 2) + so[t]);
    }
  };

  f32x4 acc[2][kBlocks];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int i = 0; i < kBlocks; ++i) acc[t][i] = f32x4{0.f, 0.f, 0.f, 0.f};

  uint32_t sh_m;  // opaque copy of the sign mask: keeps the and-or on registers
  asm volatile("" : "=v"(sh_m) : "0"(0x80008000u));
  uint32_t xaddr[4];  // LDS address of operand s of block 0, stage 0
#pragma unroll
  for (int s = 0; s < 4; ++s)
    xaddr[s] = lds_addr(xs[0]) + 256 * r + 16 * slot_of_chunk(q, s, r);

  // a group without steps still loads one (unused, within the matrix)
  x_dma(min(it0, nall - 1));
  at_step(min(it0, nall - 1));
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    raw[t] = RawTile{};
    if (active) {
      load_base(t);
#pragma unroll
      for (int p = 0; p < 8; ++p)
        if (p < bits) load_plane(t, p);
    }
  }
  for (int it = it0; it < it0 + steps; ++it) {
    // everything issued in the previous step has landed: this step's
    // activations (every wave's, after the barrier) and raw words.  The
    // barrier also ends every read of the stage that is filled next.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (KS > 1 && it >= it1) continue;
    if (!active) {
      if (it + 1 < it1) x_dma(it + 1);
      continue;
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#pragma unroll
      for (int p = 0; p < 8; ++p) asm volatile("" : "+v"(raw[t].w[p]), "+v"(raw[t].sp[p]));
      asm volatile("" : "+v"(raw[t].s1), "+v"(raw[t].z));
      if (G < kStepK && kStepK * it + 32 * q >= K) {
        raw[t].s1 = 0;
#pragma unroll
        for (int p = 0; p < 8; ++p) raw[t].sp[p] = 0;
      }
    }
    // the step that is loaded during this one (in the last step: this one
    // again, not used)
    const int nx = it + 1 < it1 ? it + 1 : it;
    if (nx != it) x_dma(nx);
    at_step(nx);
    // opaque in every step: the tests below stay scalar compares instead of
    // masks that are computed once and spilled
    asm volatile("" : "+s"(wid), "+s"(wset), "+s"(bits));
    const uint32_t xst = (it & 1) ? (uint32_t)kStageBytes : 0u;
    // With every plane read as a sign,
    //   W^_b = s1 (Q - z) + sum_{p>=b_min} s_p sigma_p
    //        = C + sum_{p<b} c_p (2 bit_p - 1),  c_p = s1 2^(p-1) for p < b_min,
    //          c_p = s_p for p >= b_min,  C = s1 ((2^b_min - 1) / 2 - z),
    // accumulated in binary16 from C (pairs of columns j, j + 16), then
    // rounded to bf16 for the products.  A shift puts bits j and j + 16 of a
    // plane word at the two sign positions and one and-or makes (+-c_p, +-c_p).
    // Planes 0 .. first - 1 come by lookup, with the same roundings, so that a
    // weight's value does not depend on the widths that share its chunk: no
    // width of the chunk ends before plane `first`.  The vector ALU bounds this
    // kernel; with it, ms per step: 64 experts top-6, 512 tokens at 2 to 8 bits
    // 0.392 -> 0.367, Mixtral shape 512 tokens at 5 to 8 bits 1.70 -> 1.57, 301
    // tokens 1.06 -> 1.00.
    h2 a[2][16], s1p[2], base_c[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const float s1 = h2f((uint16_t)raw[t].s1);
      const h2 C = as_h2(h2_splat(s1 * ((float)((1 << b_min) - 1) * 0.5f - (float)raw[t].z)));
      s1p[t] = as_h2(raw[t].s1 | (raw[t].s1 << 16));
      base_c[t] = C;
      load_base(t);
    }
    u32x4 X[4];  // operands of the block whose products are next
    static_for<4>([&](auto sc) {
      constexpr int S = decltype(sc)::value;
      ld128<0>(X[S], xaddr[S] + xst);
    });
    wait_lgkm();
#pragma unroll
    for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(X[s]));
    auto scale_pair = [&](int t, int p) {  // (c_p, c_p) of plane p
      const _Float16 k = (_Float16)((float)(1 << p) * 0.5f);
      const uint32_t base = as_u(s1p[t] * h2{k, k}), res = raw[t].sp[p] | (raw[t].sp[p] << 16);
      return p < b_min ? base : res;
    };
    const int run = __builtin_ctz(wset >> 1) + 1, first = run < 2 ? 0 : run < 3 ? 2 : 3;
    if (first == 3) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        lookup::planes3<true, 8>(a[t], raw[t].w[0], rotr(raw[t].w[1], 31), rotr(raw[t].w[2], 30),
                                 scale_pair(t, 0), scale_pair(t, 1), scale_pair(t, 2), base_c[t]);
        __builtin_amdgcn_sched_barrier(0);
        load_plane(t, 0);
        load_plane(t, 1);
        load_plane(t, 2);
      }
    } else if (first == 2) {
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        lookup::planes2<true, 8>(a[t], raw[t].w[0], rotr(raw[t].w[1], 31), scale_pair(t, 0),
                                 scale_pair(t, 1), base_c[t]);
        __builtin_amdgcn_sched_barrier(0);
        load_plane(t, 0);
        load_plane(t, 1);
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < 16; ++j) a[t][j] = base_c[t];
    }
    static_for<8>([&](auto pc) {
      constexpr int P = decltype(pc)::value;
      if (P < bits) {
        if (P > 2 || P >= first) {
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const uint32_t cp = scale_pair(t, P);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
              const uint32_t v = (sh_m & (raw[t].w[P] << (15 - j))) | cp;  // bit set -> -c_p
              a[t][j] = a[t][j] - as_h2(v);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_plane(t, P);
          }
        }
        if ((wset >> (P + 1)) & 1u) {
          // products of the blocks of width P + 1: operand s is columns
          // 8 s .. 8 s + 7 of the lane's run
          u32x4 wv[2][4];
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int s = 0; s < 2; ++s) {
              f2 fv[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) fv[j] = __builtin_convertvector(a[t][8 * s + j], f2);
#pragma unroll
              for (int d = 0; d < 4; ++d) {
                wv[t][s][d] = __builtin_bit_cast(
                    uint32_t, __builtin_convertvector(f2{fv[2 * d].x, fv[2 * d + 1].x}, b2));
                wv[t][2 + s][d] = __builtin_bit_cast(
                    uint32_t, __builtin_convertvector(f2{fv[2 * d].y, fv[2 * d + 1].y}, b2));
              }
              __builtin_amdgcn_sched_barrier(0);  // bounds the live conversions
            }
          }
          static_for<kBlocks>([&](auto bc) {
            constexpr int B = decltype(bc)::value;
            if (((wid >> (4 * B)) & 15u) == P + 1) {
              // the next block's operands are read during this block's
              // products (blocks run in order, whatever their widths)
              constexpr int NB = (B + 1) % kBlocks;
              static_for<4>([&](auto sc) {
                constexpr int S = decltype(sc)::value;
#pragma unroll
                for (int t = 0; t < 2; ++t)
                  acc[t][B] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                      __builtin_bit_cast(bf16x8, wv[t][S]), __builtin_bit_cast(bf16x8, X[S]),
                      acc[t][B], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                ld128<kBlockBytes * NB>(X[S], xaddr[S] + xst);
              });
              wait_lgkm();
#pragma unroll
              for (int s = 0; s < 4; ++s) asm volatile("" : "+v"(X[s]));
              // keeps each sum in its own registers: without it a chain of
              // products may start in registers that overlap its own sum's
              asm volatile("" : "+v"(acc[0][B]), "+v"(acc[1][B]));
            }
          });
        }
      }
    });
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (KS > 1) {
    // the second group's sums through its own stages, which no one reads now
    __syncthreads();
    f32x4* sums = (f32x4*)xs_all[KS - 1] + (size_t)wave * (2 * kBlocks * 64) + lane;
    static_assert(kGemmWaves * 2 * kBlocks * 64 * 16 <= 2 * kStageBytes, "the sums fit");
    if (kg != 0)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < kBlocks; ++i) sums[64 * (kBlocks * t + i)] = acc[t][i];
    __syncthreads();
    if (kg != 0) return;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int i = 0; i < kBlocks; ++i) acc[t][i] += sums[64 * (kBlocks * t + i)];
  }
  if (!active) return;

  // ---- epilogue: lane (r, q) holds position r of every block, rows 4 q ..
  // 4 q + 3 of both row tiles ----
  if constexpr (!SWIGLU) out = (float*)out + (size_t)blockIdx.y * out_split;
#pragma unroll
  for (int i = 0; i < kBlocks; ++i) {
    if (r < blk_cnt[i]) {
      const size_t pos = (size_t)(blk_pos[i] + r);
      if constexpr (SWIGLU) {
        uint32_t h[2];
#pragma unroll
        for (int d = 0; d < 2; ++d)
          h[d] = (uint32_t)f2bf(silu(acc[0][i][2 * d]) * acc[1][i][2 * d]) |
                 (uint32_t)f2bf(silu(acc[0][i][2 * d + 1]) * acc[1][i][2 * d + 1]) << 16;
        *(u32x2*)((uint16_t*)out + pos * out_ld + wn0 + 4 * q) = u32x2{h[0], h[1]};
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          *(f32x4*)((float*)out + pos * out_ld + wn0 + 16 * t + 4 * q) = acc[t][i];
      }
    }
  }
}

// fp32 activations are rounded to bf16 once for the GEMM's operand tiles.
__global__ void to_bf16_kernel(const float* __restrict__ in, size_t n, uint16_t* __restrict__ out) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = f2bf(in[i]);
}

// out[t][c] = sum_i w[t][i] * y[slot_of[t*k+i]][c] (+ the shared expert's
// output, the sum of its ys_parts partial planes), i ascending.  Four columns
// per thread, and the rows' loads are issued AHEAD (the power of two that holds
// k, at most 8) at a time before their sums: memory latency bounds it at one column and one load in flight.
// 2048 tokens of 4096, top-2: 31 -> 14.5 us; 512 tokens of 2048, top-6 with a
// shared expert: 15.5 -> 12.2; one token of 4096: 4.7 -> 4.4.
constexpr int kCombineThreads = 128;
template <typename TOUT, int AHEAD>
__global__ __launch_bounds__(kCombineThreads) void combine_kernel(
    const float* __restrict__ y, const float* __restrict__ ys, int ys_parts, size_t ys_split,
    const float* __restrict__ topk_w, const int32_t* __restrict__ slot_of, int k, int d,
    TOUT* __restrict__ out) {
  const int t = blockIdx.y;
  const int c = 4 * (blockIdx.x * blockDim.x + threadIdx.x);
  if (c >= d) return;  // d % 64 == 0
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  for (int i0 = 0; i0 < k; i0 += AHEAD) {
    f32x4 v[AHEAD];
    float w[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {  // past the last row: it again, not summed
      const int at = t * k + min(i0 + i, k - 1);
      v[i] = *(const f32x4*)(y + (size_t)slot_of[at] * d + c);
      w[i] = topk_w[at];
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
      if (i0 + i < k)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += w[i] * v[i][e];
  }
  if (ys) {
    // the shared expert's reduction parts, summed in order
    f32x4 sh = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int z = 0; z < ys_parts; ++z) sh += *(const f32x4*)(ys + z * ys_split + (size_t)t * d + c);
    acc += sh;
  }
  // the caller's buffer: aligned to its elements only
  typedef TOUT out4 __attribute__((ext_vector_type(4), aligned(sizeof(TOUT))));
  out4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if constexpr (sizeof(TOUT) == 2)
      o[e] = f2bf(acc[e]);
    else
      o[e] = acc[e];
  }
  *(out4*)(out + (size_t)t * d + c) = o;
}
hipError_t launch_combine(const float* y, const float* ys, int ys_parts, size_t ys_split,
                          const d2moe_routing* r, int T, int k, int d, d2moe_dtype xd, void* out,
                          hipStream_t s) {
  const int quads = d / 4, threads = quads < kCombineThreads ? (quads + 63) / 64 * 64 : kCombineThreads;
  const dim3 grid((quads + threads - 1) / threads, T);
  auto launch = [&](auto ahead) {
    constexpr int A = decltype(ahead)::value;
    if (xd == D2MOE_BF16)
      combine_kernel<uint16_t, A><<<grid, threads, 0, s>>>(y, ys, ys_parts, ys_split, r->topk_w,
                                                           r->slot_of, k, d, (uint16_t*)out);
    else
      combine_kernel<float, A><<<grid, threads, 0, s>>>(y, ys, ys_parts, ys_split, r->topk_w,
                                                        r->slot_of, k, d, (float*)out);
  };
  using std::integral_constant;
  k <= 1   ? launch(integral_constant<int, 1>{})
  : k <= 2 ? launch(integral_constant<int, 2>{})
  : k <= 4 ? launch(integral_constant<int, 4>{})
           : launch(integral_constant<int, 8>{});
  return hipGetLastError();
}

// One matrix's share of a nested delta: per packed block, planes [p0, p1) and
// scale levels [l0, l1), and the zero points with the first load, as 16-byte
// words at fixed strides (the canonical layout on both sides).
struct DeltaPart {
  const uint8_t *hp, *hs, *hz;  // host planes, scales, zeros of the expert (device addresses)
  uint8_t *dp, *ds, *dz;
  long nblk;
  int ppitch, spitch, zpitch;   // bytes per block
  int poff, soff;               // of the delta in a block
  int np, ns, nz;               // 16-byte words per block
};

// Copies the deltas of both matrices of an expert (blockIdx.y) by reading the
// pinned host memory from the device: the runs of a block are 256 bytes per
// plane and 32 to 224 bytes of scales, which the runtime's strided copies move
// at about two thirds of the link's rate.  Bound by the host link (57 GB/s).  A
// few workgroups with many consecutive words in flight each do best: 8 experts
// of d 2048, d_ff 5632, 18 units, whole step 5.2 ms with 32 x 8 words, 5.8 with
// 64 x 8, 7.8 with 8 x 16, 6.3 with 128 x 4 strided over the grid, and 6.1 with
// the strided copies.
constexpr int kDeltaThreads = 256, kDeltaWords = 8, kDeltaGroups = 32;
__global__ __launch_bounds__(kDeltaThreads) void copy_delta_kernel(DeltaPart a, DeltaPart b) {
  const DeltaPart& d = blockIdx.y ? b : a;
  const int per = d.np + d.ns + d.nz;
  constexpr int kRun = kDeltaThreads * kDeltaWords;  // consecutive words of a workgroup
  const long total = d.nblk * per;
  for (long i0 = (long)blockIdx.x * kRun + threadIdx.x; i0 < total; i0 += (long)gridDim.x * kRun) {
    u32x4 v[kDeltaWords];
    uint8_t* to[kDeltaWords];
#pragma unroll
    for (int q = 0; q < kDeltaWords; ++q) {
      const long i = i0 + q * kDeltaThreads;
      to[q] = nullptr;
      if (i < total) {
        const long blk = i / per;
        int w = (int)(i - blk * per);
        const uint8_t* from;
        size_t off;
        if (w < d.np) {
          off = (size_t)blk * d.ppitch + d.poff + 16 * w;
          from = d.hp, to[q] = d.dp;
        } else if ((w -= d.np) < d.ns) {
          off = (size_t)blk * d.spitch + d.soff + 16 * w;
          from = d.hs, to[q] = d.ds;
        } else {
          off = (size_t)blk * d.zpitch + 16 * (w - d.ns);
          from = d.hz, to[q] = d.dz;
        }
        to[q] += off;
        v[q] = *(const u32x4*)(from + off);
      }
    }
#pragma unroll
    for (int q = 0; q < kDeltaWords; ++q)
      if (to[q]) *(u32x4*)to[q] = v[q];
  }
}

// The part of (hm -> dm) for expert e, widths from .. to, at the device
// addresses `host` of hm's planes, scales and zeros.
DeltaPart delta_part(const uint8_t* const host[3], const d2moe_mwq* dm, int e, int from, int to) {
  const int BR = 2048 / dm->group, levels = dm->b_max - dm->b_min + 1;
  DeltaPart d;
  d.nblk = (long)(dm->rows / BR) * (dm->cols / dm->group);
  d.ppitch = dm->b_max * 256;
  d.spitch = levels * BR * 2;
  d.zpitch = BR;
  const int l0 = from == 0 ? 0 : from - dm->b_min + 1, l1 = to - dm->b_min + 1;
  d.poff = from * 256;
  d.soff = l0 * BR * 2;
  d.np = (to - from) * 16;
  d.ns = (l1 - l0) * BR / 8;
  d.nz = from == 0 ? BR / 16 : 0;
  const size_t eb = (size_t)e * d.nblk;
  d.hp = host[0] + eb * d.ppitch;
  d.hs = host[1] + eb * d.spitch;
  d.hz = host[2] + eb * d.zpitch;
  d.dp = (uint8_t*)dm->planes + eb * d.ppitch;
  d.ds = (uint8_t*)dm->scales + eb * d.spitch;
  d.dz = dm->zeros + eb * d.zpitch;
  return d;
}

// Device addresses of the host copy's three arrays, if the device can read all
// of each (within one pinned allocation: an array may go on past the end of the
// one that its first byte lies in) and both copies allow 16-byte words.
bool delta_addresses(const d2moe_mwq* hm, const d2moe_mwq* dm, const uint8_t* host[3]) {
  const void* const h[3] = {hm->planes, hm->scales, hm->zeros};
  const void* const d[3] = {dm->planes, dm->scales, dm->zeros};
  const size_t values = (size_t)hm->n_experts * hm->rows * hm->cols, groups = values / hm->group;
  const size_t bytes[3] = {values / 8 * hm->b_max, groups * (hm->b_max - hm->b_min + 1) * 2, groups};
  for (int i = 0; i < 3; ++i) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, h[i]) != hipSuccess) {
      (void)hipGetLastError();  // an address the runtime does not know: ordinary memory
      return false;
    }
    if (at.type != hipMemoryTypeHost || !at.devicePointer) return false;
    const uint8_t* dev =
        (const uint8_t*)at.devicePointer + ((const uint8_t*)h[i] - (const uint8_t*)at.hostPointer);
    if ((((uintptr_t)dev | (uintptr_t)d[i]) & 15u) != 0) return false;
    hipDeviceptr_t base = nullptr;
    size_t size = 0;
    if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)dev) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    const uintptr_t at_byte = (uintptr_t)dev - (uintptr_t)base;
    if ((uintptr_t)dev < (uintptr_t)base || at_byte > size || bytes[i] > size - at_byte) return false;
    host[i] = dev;
  }
  return true;
}

// The same copy for host memory that the device cannot read: planes
// [from, to) (the bit-widths' planes; from = 0: nothing present), the scale
// levels they add, and the zero points with the first load.  Both buffers are
// in the canonical tiled layout, so every copy is one strided rectangle (one
// row per (row block, group) block).
hipError_t copy_delta(const d2moe_mwq* hm, const d2moe_mwq* dm, int e, int from, int to,
                      hipStream_t io) {
  if (to <= from) return hipSuccess;
  const int BR = 2048 / dm->group, KB = dm->cols / dm->group;
  const size_t nblk = (size_t)(dm->rows / BR) * KB;
  const int levels = dm->b_max - dm->b_min + 1;
  const int p0 = from, p1 = to;
  const size_t ppitch = (size_t)dm->b_max * 256;
  const size_t poff = (size_t)e * nblk * ppitch + (size_t)p0 * 256;
  hipError_t err = hipMemcpy2DAsync((char*)dm->planes + poff, ppitch, (const char*)hm->planes + poff,
                                    ppitch, (size_t)(p1 - p0) * 256, nblk,
                                    hipMemcpyHostToDevice, io);
  if (err != hipSuccess) return err;
  const int l0 = from == 0 ? 0 : from - dm->b_min + 1, l1 = to - dm->b_min + 1;
  const size_t spitch = (size_t)levels * BR * 2;
  const size_t soff = (size_t)e * nblk * spitch + (size_t)l0 * BR * 2;
  err = hipMemcpy2DAsync((char*)dm->scales + soff, spitch, (const char*)hm->scales + soff, spitch,
                         (size_t)(l1 - l0) * BR * 2, nblk, hipMemcpyHostToDevice, io);
  if (err != hipSuccess) return err;
  if (from == 0) {
    const size_t zoff = (size_t)e * nblk * BR;
    err = hipMemcpyAsync(dm->zeros + zoff, hm->zeros + zoff, nblk * BR, hipMemcpyHostToDevice, io);
  }
  return err;
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

// Bound on the register chunks that n positions in at most L buckets of each of
// E experts can make.  A bucket of m positions has at most (m + 15) / 16 blocks,
// an expert of t blocks at most (t + 7) / 8 register chunks.
int chunk_bound(int n, int L, int E) {
  const long experts = E < n ? E : n, buckets = (long)E * L < n ? (long)E * L : n;
  const long blocks = (n + (kBlockPos - 1) * buckets) / kBlockPos;
  return (int)((blocks + (kBlocks - 1) * experts) / kBlocks);
}

// About how many register chunks there will be: one per active expert and one
// more per 256 positions.
int chunk_estimate(int T, int k, int E) {
  return (E < T * k ? E : T * k) + T * k / (2 * kBlocks * kBlockPos);
}

// Slots of four words of the chunk table: one per bucket (nb = 8 E, or n if
// fewer) and one per 256 positions.  Where every expert takes the tile GEMM by
// the average, a bucket of m positions has (m + 255) / 256 chunks, and one slot
// is left for the counts.  Otherwise n < kTileAverage E; m positions of an expert
// in l buckets make at most (m + 15 l) / 128 + 7 / 8 register chunks, n / 128 +
// 1.9 E + 1 slots in all, below 8 E, and tile chunks are used only if they are
// fewer.  With n < 8 E, an expert has at most a chunk per position.
int chunk_room(int n, int nb) { return (nb < n ? nb : n) + (n + 255) / 256; }

// The shared expert is one bucket of T positions, on the tile GEMM from here
// on (64 experts top-6, shared d_ff 5632 at 8 bits, ms per step register /
// tile: 0.39 / 0.42 at 512 tokens, 0.53 / 0.47 at 1024).
constexpr int kTileShared = 768;

// The shared expert is one bucket of T positions, so its launches are small.
// In the tile GEMM its positions are cut into as many equal chunks (multiples
// of 64, at most 256) as keep W1/W3 within one round of kFillWgs workgroups.
// In both GEMMs its W2 reduction is split into parts until W2 has about as many
// (each part at least 512 columns); the parts' partial sums are added by the
// combine.  A function of the sizes only, so the workspace layout and the
// launches agree.
constexpr int kFillWgs = 256;
void shared_plan(int T, int d, int shared_d_ff, int* cs, int* ksplit) {
  const long tiles13 = (shared_d_ff + kTileRows / 2 - 1) / (kTileRows / 2);
  long nch = kFillWgs / tiles13;
  const long most_ch = (T + 63) / 64;
  nch = nch < 1 ? 1 : (nch > most_ch ? most_ch : nch);
  int c = (int)(((T + nch - 1) / nch + 63) / 64 * 64);
  c = c > 256 ? 256 : (c < 64 ? 64 : c);
  *cs = c;
  const long wg2 = (long)((d + kTileRows - 1) / kTileRows) * ((T + c - 1) / c);
  const int steps2 = shared_d_ff / 32;
  int sp = (int)((kFillWgs + wg2 - 1) / wg2);
  const int most = steps2 / 16 > 1 ? steps2 / 16 : 1;
  *ksplit = sp < 1 ? 1 : (sp > most ? most : sp);
}

// n_ub: chunks of `wk` (a bound when it is the device's table).
template <int G, bool SWIGLU>
hipError_t run_gemm_g(const uint16_t* in, int in_ld, const int32_t* perm, int kdiv,
                      const MwqView& W, const GemmWork& wk, int n_ub, void* out, int out_ld,
                      hipStream_t s, int ksplit, size_t out_split, int n_chunks) {
  const int N = SWIGLU ? W.rows / 2 : W.rows;
  const int per = SWIGLU ? kTileRows / 2 : kTileRows;
  const int tiles = (N + per - 1) / per;
  const dim3 grid((unsigned)((long)n_ub * tiles), ksplit);
  const long n_wg = (long)n_chunks * tiles * ksplit;
  // W2 in two groups where its workgroups would fill less than about two thirds
  // of the GPU's 512 places for them (n_wg: about as many as there will be) and
  // each group still has a few steps.  Mixtral shape, ms per step in one group /
  // two: 70 tokens (256 workgroups of 112 steps) 0.99 / 0.93, 301 (320) 1.14 /
  // 1.06, 512 (384) 1.31 / 1.35.  At four steps (d_ff 512, 64 tokens of 256) the
  // launch takes 16.5 / 14.5 us.
  const bool two = !SWIGLU && n_wg <= 352 && W.cols / kStepK / ksplit >= 4;
  auto launch = [&](auto kernel, int threads) {
    kernel<<<grid, threads, 0, s>>>(in, in_ld, perm, kdiv, W, wk, tiles, N, N, out, out_ld,
                                    out_split);
  };
  constexpr int KS2 = SWIGLU ? 1 : 2;
  if (W.b_min == 2)
    two ? launch(bgemm_kernel<G, SWIGLU, 2, KS2>, KS2 * kGemmThreads)
        : launch(bgemm_kernel<G, SWIGLU, 2, 1>, kGemmThreads);
  else
    two ? launch(bgemm_kernel<G, SWIGLU, 0, KS2>, KS2 * kGemmThreads)
        : launch(bgemm_kernel<G, SWIGLU, 0, 1>, kGemmThreads);
  return hipGetLastError();
}
// n_ub bounds the chunks of `wk`, n_chunks is about how many there will be.
template <bool SWIGLU>
hipError_t run_gemm(const uint16_t* in, int in_ld, const int32_t* perm, int kdiv, const MwqView& W,
                    const GemmWork& wk, int n_ub, int n_chunks, void* out, int out_ld,
                    hipStream_t s, int ksplit = 1, size_t out_split = 0) {
  if (n_ub <= 0) return hipSuccess;
  return W.group == 128 ? run_gemm_g<128, SWIGLU>(in, in_ld, perm, kdiv, W, wk, n_ub, out, out_ld,
                                                  s, ksplit, out_split, n_chunks)
                        : run_gemm_g<64, SWIGLU>(in, in_ld, perm, kdiv, W, wk, n_ub, out, out_ld,
                                                 s, ksplit, out_split, n_chunks);
}

// The work of one bucket: `cnt` positions from `first` at `bits` bits of
// `expert`, in as few chunks as hold them, of even size.
GemmWork one_bucket(int first, int cnt, int bits, int expert, int* n_ub) {
  const int blocks = (cnt + kBlockPos - 1) / kBlockPos;
  const int nch = (blocks + kBlocks - 1) / kBlocks;
  const int per = nch > 0 ? (blocks + nch - 1) / nch : 1;
  *n_ub = (blocks + per - 1) / per;
  return GemmWork{nullptr, nullptr, nullptr, 0, first, cnt, bits, expert, per};
}

}  // namespace

FwdWorkspace fwd_workspace_layout(int T, int d, int d_ff, int E, int k, int shared_d_ff) {
  FwdWorkspace L;
  size_t off = 0;
  // chunk tables of the routed experts (at most 8 bit-widths per expert) and
  // of the shared expert
  L.chunk_n = chunk_room(T * k, E * 8);
  L.shared_chunk = 1;
  L.shared_ksplit = 1;
  if (shared_d_ff > 0) shared_plan(T, d, shared_d_ff, &L.shared_chunk, &L.shared_ksplit);
  const size_t room =
      (size_t)L.chunk_n + (shared_d_ff > 0 ? (T + L.shared_chunk - 1) / L.shared_chunk : 0);
  L.sched_off = off;  off += align256(16 * room);
  L.h_off = off;      off += align256(sizeof(uint16_t) * (size_t)T * k * d_ff);
  L.hs_off = off;     off += align256(sizeof(uint16_t) * (size_t)T * shared_d_ff);
  L.y_off = off;      off += align256(sizeof(float) * (size_t)T * k * d);
  L.ys_off = off;
  off += align256(sizeof(float) * (size_t)L.shared_ksplit * T * (shared_d_ff > 0 ? d : 0));
  L.xb_off = off;     off += align256(sizeof(uint16_t) * (size_t)T * d);
  const size_t nd = T <= kDecodeMaxTokens ? (size_t)T * k : 0;  // decode positions
  // decode work list: at most one run per active expert plus one per 8 positions
  // (runs of up to 16 positions need fewer)
  L.elist_off = off;  off += align256(sizeof(int32_t) * (4 * ((size_t)E + (nd + 7) / 8) + 4));
  const size_t nz = nd ? nd + 1 : 0;  // plus one all-zero activation slot
  L.xq13_off = off;   off += align256(nz * d * 2);
  const size_t nxs = nz ? nz + 24 : 0;  // info words, padded for 24-position reads
  L.xs13_off = off;   off += align256(nxs * sizeof(uint32_t));
  L.h32_off = off;    off += align256(nd * d_ff * sizeof(float));
  L.xq2_off = off;    off += align256(nz * d_ff * 2);
  L.xs2_off = off;    off += align256(nxs * sizeof(uint32_t));
  // partial maxima of |h|: one word per (position, 16-row block of d_ff)
  L.hmax_off = off;   off += align256(nd * ((size_t)(d_ff + 15) / 16) * sizeof(uint32_t));
  L.total = off;
  return L;
}

// Side stream of the calling host thread on the current device (created at
// its first concurrent forward there, default priority, kept until the
// process ends), and the events that fork work onto it from the caller's
// stream and join it back.  Per thread, so that calls from different host
// threads never wait on each other's events.
struct SideStream {
  hipStream_t s = nullptr;
  hipEvent_t fork = nullptr, join = nullptr;
};
constexpr int kMaxSideDevices = 64;
hipError_t side_stream(SideStream** out) {
  thread_local SideStream cache[kMaxSideDevices];
  int dev = 0;
  hipError_t err = hipGetDevice(&dev);
  if (err != hipSuccess) return err;
  if (dev < 0 || dev >= kMaxSideDevices) return hipErrorInvalidDevice;
  SideStream& ss = cache[dev];
  if (ss.fork == nullptr) {
    SideStream n;
    if ((err = hipStreamCreateWithFlags(&n.s, hipStreamNonBlocking)) != hipSuccess) return err;
    if ((err = hipEventCreateWithFlags(&n.join, hipEventDisableTiming)) != hipSuccess) return err;
    if ((err = hipEventCreateWithFlags(&n.fork, hipEventDisableTiming)) != hipSuccess) return err;
    ss = n;
  }
  *out = &ss;
  return hipSuccess;
}

// The layer with its expert weights streamed in (Sec. 3.4): units in the
// given order; each unit's nested delta is copied on `io`, and the unit's
// bucket is computed on `s` once that copy has landed (an event per unit), so
// the copy of the next unit overlaps the computation of this one.  The
// per-position arithmetic is that of the grouped GEMM path of
// launch_forward (how positions are grouped into blocks and chunks does not
// change a position's sums; which GEMM the layer takes does).
hipError_t launch_forward_streamed(const void* x, d2moe_dtype xd, int T, int d, int d_ff, int E,
                                   int k, const d2moe_mwq* hw13, const d2moe_mwq* hw2,
                                   const d2moe_mwq* w13, const d2moe_mwq* w2, uint8_t* resident,
                                   const d2moe_routing* r, const int32_t* hist_host,
                                   const d2moe_unit* units, int n_units, void* out, void* ws,
                                   hipStream_t s, hipStream_t io, const hipEvent_t* events) {
  const FwdWorkspace L = fwd_workspace_layout(T, d, d_ff, E, k, 0);
  char* base = (char*)ws;
  const int Lv = w13->b_max - w13->b_min + 1, b_min = w13->b_min;
  uint16_t* h = (uint16_t*)(base + L.h_off);
  float* y = (float*)(base + L.y_off);
  hipError_t err;
  // The copies follow what `s` holds already: work that reads the device copy
  // or still uses its memory (a fill, or a temporary that was there before).
  // events[0] carries that order and is recorded again for its unit below; a
  // wait keeps the record that it was enqueued after.
  bool loads = false;
  for (int i = 0; i < n_units; ++i) loads |= units[i].load_to > units[i].load_from;
  if (loads) {
    if ((err = hipEventRecord(events[0], s)) != hipSuccess) return err;
    if ((err = hipStreamWaitEvent(io, events[0], 0)) != hipSuccess) return err;
  }
  const uint16_t* xb = (const uint16_t*)x;
  if (T > 0 && xd == D2MOE_F32) {
    uint16_t* xw = (uint16_t*)(base + L.xb_off);
    const size_t n = (size_t)T * d;
    to_bf16_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const float*)x, n, xw);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    xb = xw;
  }
  // bucket offsets from the host counts (exclusive scan, expert major)
  int off[64 * 8 + 1];
  off[0] = 0;
  for (int i = 0; i < E * Lv; ++i) off[i + 1] = off[i] + hist_host[i];
  const MwqView W13 = view_of(w13), W2 = view_of(w2);
  // the same GEMM, and the same split of W2, as in launch_forward, so that a
  // position's sums are the same bit for bit
  int32_t* table = (int32_t*)(base + L.sched_off);
  const int n_chunks = chunk_estimate(T, k, E);
  ChunkCount sum{};
  for (int e = 0; e < E; ++e) expert_blocks(hist_host + e * Lv, Lv, b_min, &sum);
  const bool tile = (long)T * k >= (long)kTileAverage * E || use_tiles(sum, T, k, d, d_ff);
  const uint8_t *host13[3], *host2[3];
  const bool by_kernel = delta_addresses(hw13, w13, host13) && delta_addresses(hw2, w2, host2);
  for (int i = 0; i < n_units; ++i) {
    const d2moe_unit& u = units[i];
    if (by_kernel && u.load_to > u.load_from) {
      copy_delta_kernel<<<dim3(kDeltaGroups, 2), kDeltaThreads, 0, io>>>(
          delta_part(host13, w13, u.expert, u.load_from, u.load_to),
          delta_part(host2, w2, u.expert, u.load_from, u.load_to));
      if ((err = hipGetLastError()) != hipSuccess) return err;
    } else {
      if ((err = copy_delta(hw13, w13, u.expert, u.load_from, u.load_to, io)) != hipSuccess)
        return err;
      if ((err = copy_delta(hw2, w2, u.expert, u.load_from, u.load_to, io)) != hipSuccess)
        return err;
    }
    if ((err = hipEventRecord(events[i], io)) != hipSuccess) return err;
    if ((err = hipStreamWaitEvent(s, events[i], 0)) != hipSuccess) return err;
    if (resident[u.expert] < u.load_to) resident[u.expert] = (uint8_t)u.load_to;
    if (u.count <= 0) continue;
    const int first = off[u.expert * Lv + (u.bits - b_min)];
    if (tile) {
      err = launch_tile_bucket(xb, r->perm, k, w13, w2, first, u.count, u.bits, u.expert, table, h,
                               y, s);
      if (err != hipSuccess) return err;
      continue;
    }
    int n_ub;
    const GemmWork wk = one_bucket(first, u.count, u.bits, u.expert, &n_ub);
    err = run_gemm<true>(xb, d, r->perm, k, W13, wk, n_ub, n_chunks, h, d_ff, s);
    if (err != hipSuccess) return err;
    err = run_gemm<false>(h, d_ff, nullptr, 1, W2, wk, n_ub, n_chunks, y, d, s);
    if (err != hipSuccess) return err;
  }
  if (T == 0) return hipSuccess;
  return launch_combine(y, nullptr, 1, 0, r, T, k, d, xd, out, s);
}

hipError_t launch_forward(const void* x, d2moe_dtype xd, int T, int d, int d_ff, int E, int k,
                          const d2moe_mwq* w13, const d2moe_mwq* w2, const d2moe_routing* r,
                          const d2moe_mwq* sw13, const d2moe_mwq* sw2, int shared_bits,
                          int shared_d_ff, void* out, void* ws, hipStream_t s,
                          const hipEvent_t* events, bool concurrent) {
  if (T == 0) return hipSuccess;
  const bool has_shared = sw13 != nullptr;
  const FwdWorkspace L = fwd_workspace_layout(T, d, d_ff, E, k, has_shared ? shared_d_ff : 0);
  char* base = (char*)ws;
  const int Lv = w13->b_max - w13->b_min + 1;
  int32_t* table = (int32_t*)(base + L.sched_off);
  uint16_t* h = (uint16_t*)(base + L.h_off);
  uint16_t* hs = (uint16_t*)(base + L.hs_off);
  float* y = (float*)(base + L.y_off);
  float* ys = (float*)(base + L.ys_off);
  // bf16 activations for the grouped GEMM (fp32 inputs are rounded once)
  const uint16_t* xb = (const uint16_t*)x;
  const bool decode = decode_path_ok(w13, w2, T);
  const bool convert = xd == D2MOE_F32 && (has_shared || !decode);
  const size_t n = (size_t)T * d;
  uint16_t* xw = (uint16_t*)(base + L.xb_off);
  if (convert) {
    if (has_shared) {  // both chains read it; otherwise the chunk tables' launch writes it
      to_bf16_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((const float*)x, n, xw);
      hipError_t e0 = hipGetLastError();
      if (e0 != hipSuccess) return e0;
    }
    xb = xw;
  }

  hipError_t err;
  // Concurrency: the shared expert's chain runs on a side stream forked from
  // `s` (it writes its own workspace, hs / ys); the combine waits for it.  Not
  // with events: those time the kernels on `s`.
  const bool fork_shared = concurrent && !events && has_shared;
  SideStream* side = nullptr;
  if (fork_shared && (err = side_stream(&side)) != hipSuccess) return err;

  if (has_shared) {
    hipStream_t ss = s;
    if (fork_shared) {
      ss = side->s;
      if ((err = hipEventRecord(side->fork, s)) != hipSuccess) return err;
      if ((err = hipStreamWaitEvent(ss, side->fork, 0)) != hipSuccess) return err;
    }
    if (T >= kTileShared) {
      err = launch_tile_shared(xb, T, sw13, sw2, shared_bits, L.shared_chunk, L.shared_ksplit,
                               table + 4 * (size_t)L.chunk_n, hs, ys, ss);
      if (err != hipSuccess) return err;
    } else {
      int ns_ub;
      const GemmWork wk = one_bucket(0, T, shared_bits, 0, &ns_ub);
      err = run_gemm<true>(xb, d, nullptr, 1, view_of(sw13), wk, ns_ub, ns_ub, hs, shared_d_ff, ss);
      if (err != hipSuccess) return err;
      err = run_gemm<false>(hs, shared_d_ff, nullptr, 1, view_of(sw2), wk, ns_ub, ns_ub, ys, d, ss,
                            L.shared_ksplit, (size_t)T * d);
      if (err != hipSuccess) return err;
    }
    if (fork_shared && (err = hipEventRecord(side->join, ss)) != hipSuccess) return err;
  }

  if (decode) {
    DecodeBuffers db;
    db.elist = (int32_t*)(base + L.elist_off);
    db.xq13 = (uint8_t*)(base + L.xq13_off);
    db.xs13 = (uint32_t*)(base + L.xs13_off);
    db.h32 = (float*)(base + L.h32_off);
    db.xq2 = (uint8_t*)(base + L.xq2_off);
    db.xs2 = (uint32_t*)(base + L.xs2_off);
    db.hmax = (uint32_t*)(base + L.hmax_off);
    db.y = y;
    err = launch_decode_ffn(x, xd, T, d, d_ff, E, k, w13, w2, r, db, s, events);
    if (err != hipSuccess) return err;
  } else {
    const bool all_tile = (long)T * k >= (long)kTileAverage * E;
    constexpr int kPer = kChunkThreads * kConvert;
    const unsigned conv = convert && !has_shared ? (unsigned)((n + kPer - 1) / kPer) : 0;
    chunk_kernel<<<1 + conv, kChunkThreads, 0, s>>>(r->hist, r->offsets, E, Lv, w13->b_min,
                                                    T, k, d, d_ff, all_tile, table,
                                                    (const float*)x, n, xw);
    if ((err = hipGetLastError()) != hipSuccess) return err;
    const int n_ub = all_tile ? 0 : chunk_bound(T * k, Lv, E);
    const int nt_ub = all_tile ? L.chunk_n - 1 : tile_bound(T, k, n_ub);
    const int n_chunks = chunk_estimate(T, k, E);
    const GemmWork wk{table, r->hist, r->offsets, Lv, 0, 0, 0, 0, 0};
    if (events && (err = hipEventRecord(events[0], s)) != hipSuccess) return err;
    err = launch_tile_gemm13(xb, r->perm, k, w13, table + 1, table + 4, nt_ub, h, s);
    if (err != hipSuccess) return err;
    err = run_gemm<true>(xb, d, r->perm, k, view_of(w13), wk, n_ub, n_chunks, h, d_ff, s);
    if (err != hipSuccess) return err;
    if (events && (err = hipEventRecord(events[1], s)) != hipSuccess) return err;
    if (events && (err = hipEventRecord(events[2], s)) != hipSuccess) return err;
    err = launch_tile_gemm2(h, w2, table + 1, table + 4, nt_ub, y, s);
    if (err != hipSuccess) return err;
    err = run_gemm<false>(h, d_ff, nullptr, 1, view_of(w2), wk, n_ub, n_chunks, y, d, s);
    if (err != hipSuccess) return err;
    if (events && (err = hipEventRecord(events[3], s)) != hipSuccess) return err;
  }
  if (fork_shared && (err = hipStreamWaitEvent(s, side->join, 0)) != hipSuccess) return err;

  return launch_combine(y, has_shared ? ys : nullptr, L.shared_ksplit, (size_t)T * d, r, T, k, d, xd,
                        out, s);
}

}  // namespace d2moe
