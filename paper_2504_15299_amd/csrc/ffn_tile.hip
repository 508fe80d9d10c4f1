// Grouped mixed-bit expert GEMM for many positions per expert: chunks of up to
// 256 positions of one (expert, bit-width) bucket, one 4-wave workgroup per
// (chunk, 128 weight rows), two of them on a compute unit.  Each wave owns 64
// positions and all four share one dequantized weight tile in LDS, so a weight
// is dequantized once per 256 positions; the register kernel of ffn_gemm.hip
// dequantizes once per 128.  (An 8-wave variant of that kernel for 240
// positions, its waves exchanging operands through LDS, was no faster than this
// one: at one workgroup per compute unit its phases do not overlap.)
//
// Per reduction step of 32 columns (one plane word per row):
//   * the LDS DMA engine brings the raw planes, scales and zero points of a
//     later step into a ring shared by the workgroup, and each wave's
//     gathered activation rows of a later step into its own ring;
//   * the workgroup dequantizes the next step's 128 x 32 tile into bf16 while
//     each wave runs the current step's v_mfma_f32_16x16x32_bf16 products
//     (its positions x 128 rows, fp32 accumulation) from the other tile
//     buffer, the products interleaved with the dequantization's vector
//     instructions;
//   * one barrier per step orders the shared buffers.
// The W1/W3 variant puts 64 rows of W1 and the same 64 rows of W3 in one tile,
// so a lane holds a and c of the same output and applies SwiGLU in registers.
#include <type_traits>

#include "lookup.h"

namespace d2moe {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kWaveM = 64;                  // positions per wave
constexpr int kTileWaves = 4;               // waves per workgroup, one per SIMD
static_assert(kTileChunk == kTileWaves * kWaveM, "positions per chunk");
constexpr int kTileRows = 128;              // weight rows per workgroup
constexpr int kStepK = 32;                  // reduction columns per step
// The activation ring is two stages, one step of lookahead: it leaves LDS for
// the tiles, and the activations mostly come from L2.
constexpr int kXRing = 2;
constexpr int kXStage = kWaveM * kStepK * 2;  // bytes per wave and stage
// Raw stage layout at MB planes and LS scale levels (bytes): plane p at
// 512 p (one word per tile row), the scales of level l at 512 MB + 256 l (one
// binary16 per tile row), then the zero points (one byte per tile row).
// 16-byte DMA slots 0 .. raw_slots - 1 carry them; DMA instruction i of wave
// w moves slots 256 i + 64 w .. + 63.  The ring holds as many stages as fit
// kRawBytes, at most 8 (4 at 7 and 8 bits, 8 at 2 to 4), so the DMA runs
// further ahead of the dequantization when a step has less to read.
constexpr int kRawBytes = 25088;
constexpr int raw_zero_off(int MB, int LS) { return 512 * MB + 256 * LS; }
constexpr int raw_stage_bytes(int MB, int LS) { return raw_zero_off(MB, LS) + 128; }
constexpr int raw_slots(int MB, int LS) { return raw_stage_bytes(MB, LS) / 16; }
constexpr int raw_ring(int MB, int LS) {
  return kRawBytes / raw_stage_bytes(MB, LS) < 8 ? kRawBytes / raw_stage_bytes(MB, LS) : 8;
}
static_assert(raw_ring(8, 8) >= 4, "at least 4 raw stages");
constexpr int kRawDmas = 2;  // per wave and step
constexpr int kWTile = kTileRows * kStepK * 2;  // dequantized bf16 tile bytes

#define D2MOE_GPTR(p) ((__attribute__((address_space(1))) void*)(p))
#define D2MOE_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

__device__ inline float silu(float a) { return a / (1.0f + __expf(-a)); }

using lookup::as_h2;
using lookup::as_u;
using lookup::h2;
using lookup::rotr;
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t h2_splat(float v) {
  const _Float16 h = (_Float16)v;
  return as_u(h2{h, h});
}

// LDS accesses to the DMA-filled rings and to the shared tile are inline
// assembly: with LDS DMA in flight the compiler would otherwise wait for every
// outstanding vector-memory instruction (draining the prefetch) before each
// LDS access it cannot prove independent.  Reads are ordered by an explicit
// lgkmcnt wait and re-bound after it.
__device__ inline uint32_t lds_addr(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
// OFF is the instruction's unsigned 16-bit byte offset added to the address.
template <int OFF = 0>
__device__ inline void ld128(u32x4& v, uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
}
template <int OFF = 0>
__device__ inline void ld32(uint32_t& v, uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
}
template <int OFF = 0>
__device__ inline void ldu16(uint32_t& v, uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  asm volatile("ds_read_u16 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
}
template <int OFF = 0>
__device__ inline void ldu8(uint32_t& v, uint32_t a) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset");
  asm volatile("ds_read_u8 %0, %1 offset:%2" : "=v"(v) : "v"(a), "n"(OFF) : "memory");
}
__device__ inline void st64(uint32_t a, uint32_t x, uint32_t y) {
  asm volatile("ds_write_b64 %0, %1" ::"v"(a), "v"(u32x2{x, y}) : "memory");
}
__device__ inline void wait_lgkm() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
template <int N>
__device__ inline void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ inline void bar() { __builtin_amdgcn_s_barrier(); }

// 16-byte chunk q of tile row r sits at chunk q ^ ((r >> 2) & 3), so that the
// 16 rows one MFMA operand read touches fall in distinct banks.
__device__ inline uint32_t swz(int r, int q) { return (uint32_t)(r * 64 + ((q ^ ((r >> 2) & 3)) << 4)); }

// f(integral_constant<int, i>) for i = 0 .. N-1, so that the index can be a
// template argument (an instruction offset) inside f.
template <int N, int I = 0, typename F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// Registers of one step: raw words, scales and zero point of the tile row a
// thread dequantizes, and the MFMA operands of its wave.
struct StepRegs {
  uint32_t w[8];   // plane words
  uint32_t sp[8];  // binary16 scale of plane p (p >= b_min); register index = plane
  uint32_t s1, z;  // base scale and zero point
  u32x4 A[4], B[4], B2[4];  // B, B2: weight operands of tile rows 0..63, 64..127
  // Re-binds, after the covering wait, the registers the inline-asm LDS reads
  // of a step wrote: MB plane words, the scales of planes SPLO..MB-1, and
  // the operands of NA A, NB B and NB2 B2 reads.
  template <int MB, int SPLO, int NA, int NB, int NB2>
  __device__ __attribute__((always_inline)) inline void rebind() {
#pragma unroll
    for (int p = 0; p < MB; ++p) asm volatile("" : "+v"(w[p]));
#pragma unroll
    for (int p = SPLO; p < MB; ++p) asm volatile("" : "+v"(sp[p]));
    asm volatile("" : "+v"(s1));
    asm volatile("" : "+v"(z));
#pragma unroll
    for (int i = 0; i < NA; ++i) asm volatile("" : "+v"(A[i]));
#pragma unroll
    for (int i = 0; i < NB; ++i) asm volatile("" : "+v"(B[i]));
#pragma unroll
    for (int i = 0; i < NB2; ++i) asm volatile("" : "+v"(B2[i]));
  }
};

// Dequantization of 16 weights (columns j0 + j, j0 + 8 + j, j0 + 16 + j and
// j0 + 24 + j for j < 4) of a tile row at MB planes into bf16 pairs: o[2 c],
// o[2 c + 1] columns 8 c + j0 .. + 3.
// With every plane read as a sign,
//   W^_b = s1 (Q - z) + sum_{p>=b_min} s_p sigma_p
//        = C + sum_{p<b} c_p (2 bit_p - 1),  c_p = s1 2^(p-1) for p < b_min,
//          c_p = s_p for p >= b_min,  C = s1 ((2^b_min - 1) / 2 - z),
// accumulated in fp16 from C, then rounded to bf16 for the MFMA.  Planes come
// by threes and twos by lookup, a plane left over by its sign: shifting its
// word left by 15 - j puts bit j at bit 15 and bit j + 16 at bit 31, the sign
// positions of the two halves, and one and-or turns the pair into (+-c_p, +-c_p)
// (every scale is >= 0, so the sign bits of c_p are clear).
// Rows past the matrix edge are dequantized from whatever their stage holds:
// they only reach output columns that are not stored.
// At 8 bits the vector ALU, not the matrix pipe, bounds a step: 32 products are
// 512 cycles and the sign form of every plane was about 240 instructions of 4.
// With lookups about 185; ms per step, Mixtral shape, 2048 tokens: {2,4,8} bits
// 2.85 -> 2.67, {5,6,7,8} 3.88 -> 3.44; 64 experts top-6, 4096 tokens 1.36 -> 1.28.
// BMIN > 0 fixes b_min at compile time (the common ladder starts at 2 bits);
// BMIN == 0 takes it from `b_min_rt`.
template <int MB, int BMIN>
__device__ __attribute__((always_inline)) inline void dequant16(const StepRegs& R, int b_min_rt,
                                                                uint32_t sh_m, int j0,
                                                                uint32_t (&o)[8]) {
  const int b_min = BMIN > 0 ? BMIN : b_min_rt;
  const float s1 = h2f((uint16_t)R.s1);
  const h2 C = as_h2(h2_splat(s1 * ((float)((1 << b_min) - 1) * 0.5f - (float)R.z)));
  // base scale as a binary16 pair; the pair of a residual plane is its scale
  // bits duplicated, and that of a base plane p < b_min is s1 2^(p-1), a
  // power-of-two multiple in binary16
  const h2 s1p = as_h2(R.s1 | (R.s1 << 16));
  auto cp = [&](int p) {
    const _Float16 k = (_Float16)((float)(1 << p) * 0.5f);
    return p < b_min ? as_u(s1p * h2{k, k}) : (R.sp[p] | (R.sp[p] << 16));
  };
  auto w = [&](int p, int n) { return rotr(R.w[p], j0 + 32 - n); };
  h2 a[8];
  auto sign = [&](int p) {
    const uint32_t c = cp(p), wp = rotr(R.w[p], j0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[j] = a[j] - as_h2((sh_m & (wp << (15 - j))) | c);  // bit set -> -c_p
      a[4 + j] = a[4 + j] - as_h2((sh_m & (wp << (7 - j))) | c);
    }
  };
  if constexpr (MB == 1) {
#pragma unroll
    for (int j = 0; j < 8; ++j) a[j] = C;
    sign(0);
  } else if constexpr (MB == 2) {
    lookup::planes2<true, 4>(a, w(0, 0), w(1, 1), cp(0), cp(1), C);
  } else {
    lookup::planes3<true, 4>(a, w(0, 0), w(1, 1), w(2, 2), cp(0), cp(1), cp(2), C);
    if constexpr (MB >= 6)
      lookup::planes3<false, 4>(a, w(3, 0), w(4, 1), w(5, 2), cp(3), cp(4), cp(5), C);
    constexpr int P = MB >= 6 ? 6 : 3;
    if constexpr (MB == P + 2) lookup::planes2<false, 4>(a, w(P, 0), w(P + 1, 1), cp(P), cp(P + 1), C);
    if constexpr (MB == P + 1) sign(P);
  }
  // pairs of columns 16 apart to bf16 pairs of adjacent columns
  f2 f[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = __builtin_convertvector(a[j], f2);
  auto pk = [](float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{lo, hi}, b2));
  };
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    o[2 * c] = pk(f[4 * c].x, f[4 * c + 1].x);
    o[2 * c + 1] = pk(f[4 * c + 2].x, f[4 * c + 3].x);
    o[4 + 2 * c] = pk(f[4 * c].y, f[4 * c + 1].y);
    o[4 + 2 * c + 1] = pk(f[4 * c + 2].y, f[4 * c + 3].y);
  }
}
// Vector instructions of dequant16, about.
constexpr int dequant_ops(int mb) {
  constexpr int planes[9] = {0, 32, 34, 43, 68, 85, 93, 118, 135};
  return planes[mb] + mb + 45;
}

// One workgroup: chunk blockIdx.y (of *count) against weight-row tile
// blockIdx.x; chunk c is the four words at chunks + step c: first position,
// positions, bit-width, expert.  (step is 4 in every launch; as a constant it
// leaves the compiler another register allocation, 0.4 % slower at 2048 tokens of
// the Mixtral shape.)
//   in:  bf16 activations; position p reads row (perm ? perm[p] / kdiv : p)
//   SWIGLU: W is [2f][K] (w13); the tile holds W1 rows n0..n0+63 (tile rows
//           0..63) and W3 rows f+n0.. (tile rows 64..127); out = h [pos][f] bf16
//   else:   W is [N][K], out = y [pos][N] fp32
template <int G, bool SWIGLU>
__global__ __launch_bounds__(64 * kTileWaves)
__attribute__((amdgpu_waves_per_eu(2))) void tile_gemm_kernel(
    const uint16_t* __restrict__ in, int in_ld, const int32_t* __restrict__ perm, int kdiv,
    MwqView W, const int32_t* __restrict__ count, const int32_t* __restrict__ chunks, int step, int f, int N, void* __restrict__ out,
    int out_ld, size_t out_split) {
  constexpr int RD = kRawDmas;
  __shared__ __attribute__((aligned(16))) uint8_t xring[kXRing][kTileWaves][kXStage];
  __shared__ __attribute__((aligned(16))) uint8_t rraw[kRawBytes];  // ring of raw stages
  __shared__ __attribute__((aligned(16))) uint8_t wtile[2][kWTile];
  __shared__ __attribute__((aligned(16))) uint8_t dummy[1][16];
  constexpr int BR = 2048 / G, SPG = G / kStepK;  // rows per block, steps per group

  const int ci = blockIdx.y;
  if (count && ci >= *count) return;
  chunks += (long)step * ci;
  const int m_first = chunks[0], m_cnt = chunks[1], bits = chunks[2], expert = chunks[3];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * (SWIGLU ? kTileRows / 2 : kTileRows);
  // reduction part blockIdx.z of gridDim.z (the plain variant only): steps
  // [s_lo, s_lo + nsteps), partial sums to plane blockIdx.z of `out`
  const int K = W.cols, b_min = W.b_min;
  const int s_all = K / kStepK;
  const int s_lo = SWIGLU ? 0 : (int)((long)blockIdx.z * s_all / gridDim.z);
  const int nsteps = SWIGLU ? s_all : (int)((long)(blockIdx.z + 1) * s_all / gridDim.z) - s_lo;
  if (!SWIGLU) out = (float*)out + (size_t)blockIdx.z * out_split;
  const int nlev = bits - b_min + 1;
  const bool active = kWaveM * wave < m_cnt;  // wave-uniform
  // ---- raw weight DMA: 16-byte slot u of a stage laid out for MB planes
  // and LS scale levels ----
  // global row of tile row r
  auto grow = [&](int r) { return SWIGLU ? (r < 64 ? n0 + r : f + n0 + r - 64) : n0 + r; };
  auto row_ok = [&](int r) { return SWIGLU ? n0 + (r & 63) < f : n0 + r < N; };
  struct RawSlot {
    const uint8_t* src;  // address at step 0
    int sb, sc;          // bytes per group, per 32-column step
    bool real;
  };
  auto raw_slot = [&](int u, int MB, int LS) {
    RawSlot q{(const uint8_t*)W.planes, 0, 0, false};
    const int u1 = 32 * MB, u2 = u1 + 16 * LS;
    if (u < u1) {  // plane p = u / 32, tile rows 4 v .. 4 v + 3 of it
      const int p = u >> 5, v = u & 31;
      const int r = 4 * v;  // first tile row of the slot
      if (p < bits && row_ok(r)) {
        const int gr = grow(r);
        const size_t blk = W.block(expert, gr / BR, 0);
        q = {(const uint8_t*)(W.planes + W.plane_word(blk, p, gr % BR)), W.b_max * 64 * 4, BR * 4,
             true};
      }
    } else if (u < u2) {  // level l, tile rows 8 v .. 8 v + 7
      const int l = (u - u1) >> 4, v = (u - u1) & 15;
      const int r = 8 * v;
      if (l < nlev && row_ok(r)) {
        const int gr = grow(r);
        const size_t blk = W.block(expert, gr / BR, 0);
        q = {(const uint8_t*)(W.scales + W.scale_idx(blk, l, gr % BR)), W.levels() * BR * 2, 0,
             true};
      }
    } else if (u < u2 + 8) {  // zero points, tile rows 16 z .. 16 z + 15
      const int z = u - u2;
      const int r = 16 * z;
      if (row_ok(r)) {
        const int gr = grow(r);
        const size_t blk = W.block(expert, gr / BR, 0);
        q = {W.zeros + W.zero_idx(blk, gr % BR), BR, 0, true};
      }
    }
    return q;
  };

  // ---- activation DMA: an instruction moves 16 positions' 64-byte rows;
  // wave w stages its own 64 positions, instruction i the rows 16 i ..
  // 16 i + 15 (XD = 4 per step).
  constexpr int XD = 4;
  const uint16_t* xsrc[XD];
#pragma unroll
  for (int i = 0; i < XD; ++i) {
    const int rl = 16 * i + (lane >> 2);
    int pos = m_first + kWaveM * wave + rl;
    pos = pos < m_first + m_cnt ? pos : m_first + m_cnt - 1;
    const int src = perm ? perm[pos] / kdiv : pos;
    const int q = (lane & 3) ^ ((rl >> 2) & 3);
    xsrc[i] = in + (size_t)src * in_ld + 8 * q;
  }
  const bool xissue = active || lane == 0;
  auto x_dma = [&](int step) {
    const int st = s_lo + (step < nsteps ? step : nsteps - 1);
#pragma unroll
    for (int i = 0; i < XD; ++i) {
      uint8_t* dst = xring[step % kXRing][wave] + 1024 * i;
      if (xissue)
        __builtin_amdgcn_global_load_lds(D2MOE_GPTR(xsrc[i] + kStepK * st), D2MOE_LPTR(dst), 16,
                                         0, 0);
    }
  };

  // ---- dequantization: tile row dr, columns j0 .. j0 + 3 of every 8 ----
  const int dr = tid / 2, j0 = 4 * (tid % 2);
  uint32_t sh_m;  // opaque copy of the sign mask: keeps v_bfi on registers
  asm volatile("" : "=v"(sh_m) : "0"(0x80008000u));
  const int fr = lane & 15, fq = lane >> 4;

  f32x4 acc[4][8];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 8; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  // The step loop is compiled for the chunk's bit-width MB (and for b_min 2,
  // the common nest start, or any b_min) and separately for waves that
  // multiply and waves that only dequantize: every LDS read of a step, its
  // products and its dequantization then form one branch-free block, in which
  // the products are interleaved with the dequantization's vector
  // instructions so that the matrix pipe and the vector ALU overlap.
  auto run = [&](auto mb_c, auto bmin_c) {
    constexpr int MB = decltype(mb_c)::value, BMIN = decltype(bmin_c)::value;
    // scale levels reserved per stage: exact when b_min is fixed, else MB
    constexpr int LS = BMIN > 0 ? MB - BMIN + 1 : MB;
    constexpr int SB = raw_stage_bytes(MB, LS), NS = raw_slots(MB, LS);
    constexpr int kRawRing = raw_ring(MB, LS);
    constexpr int SOFF = 512 * MB, ZOFF = raw_zero_off(MB, LS);

    // instruction i of this wave: slots ubase + lane, ubase = 256 i + 64 wave.
    // Every wave issues RD raw DMAs per step (lane 0 at least), so that all
    // waves count the same memory instructions: lanes whose slot is past the
    // stage issue nothing, and an instruction with no slot of its own writes
    // the dummy area from lane 0.
    RawSlot rs[RD];
    bool rissue[RD];
#pragma unroll
    for (int i = 0; i < RD; ++i) {
      rs[i] = raw_slot(256 * i + 64 * wave + lane, MB, LS);
      rissue[i] = rs[i].real || lane == 0;
    }
    auto raw_dma = [&](int step) {
      const int st = s_lo + (step < nsteps ? step : nsteps - 1);  // past the end: reload, unused
#pragma unroll
      for (int i = 0; i < RD; ++i) {
        const int ubase = 256 * i + 64 * wave;  // wave-uniform
        const uint8_t* src = rs[i].src + (size_t)(st / SPG) * rs[i].sb + (st % SPG) * rs[i].sc;
        uint8_t* dst = ubase < NS ? &rraw[(step % kRawRing) * SB + 16 * ubase] : dummy[0];
        if (rissue[i])
          __builtin_amdgcn_global_load_lds(D2MOE_GPTR(src), D2MOE_LPTR(dst), 16, 0, 0);
      }
    };

    // ---- prologue: raw 0..kRawRing-1 and activations 0 in flight.
    // Issue order: raw 0 .. raw kRawRing-2, x 0, raw kRawRing-1; the wait leaves
    // the instructions after raw 0 outstanding (RD per raw stage, XD per
    // activation stage), i.e. raw 0 has landed.
#pragma unroll
    for (int i = 0; i + 1 < kRawRing; ++i) raw_dma(i);
    x_dma(0);
    raw_dma(kRawRing - 1);
    wait_vm<(kRawRing - 1) * RD + XD>();
    bar();

    StepRegs R;
    // One step: the products of `mstep` (if MMA) from the tile buffer and
    // activation stage written in earlier steps, and the dequantization of
    // tile `dstep` from its raw stage into the other tile buffer.  `dma`
    // issues the DMA of later steps once this step's LDS reads are issued, so
    // that its issue overlaps their latency (it writes only stages that this
    // step does not read).
    auto step = [&](int dstep, int mstep, auto mma_c, auto&& dma) {
      constexpr bool MMA = decltype(mma_c)::value;
      // one address register per access width: the stage base plus this
      // thread's row, with the plane, level and operand block as offsets
      const uint32_t rb = lds_addr(rraw + (dstep % kRawRing) * SB);
      const uint32_t rb4 = rb + 4 * dr, rb2 = rb + 2 * dr, rb1 = rb + dr;
      static_for<MB>([&](auto pc) {
        constexpr int P = decltype(pc)::value;
        ld32<512 * P>(R.w[P], rb4);
      });
      ldu16<SOFF>(R.s1, rb2);
      static_for<MB>([&](auto pc) {  // level p - b_min + 1 holds the scale of plane p
        constexpr int P = decltype(pc)::value;
        if constexpr (BMIN > 0) {
          if constexpr (P >= BMIN) ldu16<SOFF + 256 * (P - BMIN + 1)>(R.sp[P], rb2);
        } else if constexpr (P >= 1) {  // below b_min the base scale is read and not used
          const int lvl = P >= b_min ? P - b_min + 1 : 0;
          ldu16(R.sp[P], rb2 + SOFF + 256 * lvl);
        }
      });
      ldu8<ZOFF>(R.z, rb1);
      // a 16-row operand block m starts 1024 m bytes after block 0 (the
      // swizzle depends on the row within the block only)
      const uint32_t wb = lds_addr(wtile[mstep & 1]) + swz(fr, fq);
      if constexpr (MMA) {
        {
          const uint32_t xb = lds_addr(xring[mstep % kXRing][wave]) + swz(fr, fq);
          static_for<4>([&](auto mc) {
            constexpr int M = decltype(mc)::value;
            ld128<1024 * M>(R.A[M], xb);
            ld128<1024 * M>(R.B[M], wb);
            ld128<1024 * (4 + M)>(R.B2[M], wb);
          });
        }
      }
      dma();
      wait_lgkm();
      constexpr int NA = MMA ? 4 : 0;
      R.template rebind<MB, (BMIN > 0 ? BMIN : 1), NA, NA, NA>();
      constexpr int n_mfma = MMA ? 32 : 0;
      if constexpr (MMA) {
        {
#pragma unroll
          for (int mt = 0; mt < 4; ++mt)
#pragma unroll
            for (int nt = 0; nt < 8; ++nt)
              acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, R.A[mt]),
                  __builtin_bit_cast(bf16x8, nt < 4 ? R.B[nt] : R.B2[nt - 4]), acc[mt][nt], 0, 0, 0);
        }
      }
      const uint32_t wd = lds_addr(wtile[dstep & 1]);
      {
        uint32_t o[8];
        dequant16<MB, BMIN>(R, b_min, sh_m, j0, o);
#pragma unroll
        for (int c = 0; c < 4; ++c) st64(wd + swz(dr, c) + 2 * j0, o[2 * c], o[2 * c + 1]);
      }
      if constexpr (n_mfma > 0) {
        // one product, then its share of the dequantization's vector instructions
        constexpr int nv = (dequant_ops(MB) + n_mfma - 1) / n_mfma;
#pragma unroll
        for (int i = 0; i < n_mfma; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, nv, 0);
        }
      }
      wait_lgkm();
    };

    // Tile 0 first; then step s issues activations s+1 and raw s+kRawRing (XD
    // and RD instructions), dequantizes s+1 and multiplies s.  The
    // instructions issued after the activations of s, at the top of step s, are
    // the RD of raw s+kRawRing-1.  Raw s+1 was issued before the activations
    // of s (kRawRing > 3), so that wait makes both this wave's raw s+1 and its
    // activations of s ready; the barrier then makes every
    // wave's raw s+1 and tile s visible, and retires all reads of the stages
    // and the tile buffer that this step overwrites.  In the last step the
    // dequantization works on a reloaded stage and its tile is never read.
    step(0, 0, std::false_type{}, [] {});
    auto loop = [&](auto mma_c) {
      for (int s = 0; s < nsteps; ++s) {
        wait_vm<RD>();
        bar();
        step(s + 1, s, mma_c, [&] {
          x_dma(s + 1);
          raw_dma(s + kRawRing);
        });
      }
    };
    if (active)
      loop(std::true_type{});
    else
      loop(std::false_type{});
  };
  using std::integral_constant;
  if (b_min == 2) {
    switch (bits) {
#define D2MOE_CASE(MB) \
  case MB: run(integral_constant<int, MB>{}, integral_constant<int, 2>{}); break;
      D2MOE_CASE(2) D2MOE_CASE(3) D2MOE_CASE(4) D2MOE_CASE(5) D2MOE_CASE(6) D2MOE_CASE(7) D2MOE_CASE(8)
#undef D2MOE_CASE
      default: break;
    }
  } else {
    switch (bits) {
#define D2MOE_CASE(MB) \
  case MB: run(integral_constant<int, MB>{}, integral_constant<int, 0>{}); break;
      D2MOE_CASE(1) D2MOE_CASE(2) D2MOE_CASE(3) D2MOE_CASE(4) D2MOE_CASE(5) D2MOE_CASE(6)
      D2MOE_CASE(7) D2MOE_CASE(8)
#undef D2MOE_CASE
      default: break;
    }
  }
  wait_vm<0>();  // no DMA may still be writing this workgroup's LDS at exit

  // ---- epilogue ----
  if (!active) return;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = kWaveM * wave + 16 * mt + 4 * (lane >> 4) + r;
      if (m >= m_cnt) continue;
      const size_t pos = (size_t)(m_first + m);
      if (SWIGLU) {
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) {
          const int n = n0 + 16 * nt + (lane & 15);
          if (n >= f) continue;
          const float a = acc[mt][nt][r], c = acc[mt][nt + 4][r];
          ((uint16_t*)out)[pos * out_ld + n] = f2bf(silu(a) * c);
        }
      } else {
#pragma unroll
        for (int nt = 0; nt < 8; ++nt) {
          const int n = n0 + 16 * nt + (lane & 15);
          if (n >= N) continue;
          ((float*)out)[pos * out_ld + n] = acc[mt][nt][r];
        }
      }
    }
  }
}

// Chunk table of one bucket: cnt positions from `first` at `bits` bits of
// `expert`, in chunks of cs.
__global__ void tile_bucket_kernel(int first, int cnt, int bits, int expert, int cs, int n,
                                   int32_t* __restrict__ chunks) {
  for (int c = threadIdx.x; c < n; c += blockDim.x) {
    chunks[4 * c] = first + c * cs;
    chunks[4 * c + 1] = min(cs, cnt - c * cs);
    chunks[4 * c + 2] = bits;
    chunks[4 * c + 3] = expert;
  }
}

template <bool SWIGLU>
hipError_t run_tile_gemm(const uint16_t* in, int in_ld, const int32_t* perm, int kdiv,
                         const MwqView& W, const int32_t* count, const int32_t* chunks, int step,
                         int n_ub, int f, void* out,
                         int out_ld, hipStream_t s, int ksplit = 1, size_t out_split = 0) {
  if (n_ub <= 0) return hipSuccess;
  const int N = SWIGLU ? W.rows / 2 : W.rows;
  const int per = SWIGLU ? kTileRows / 2 : kTileRows;
  // weight-row tiles vary fastest: consecutive workgroups, which the
  // dispatcher deals round-robin to the 8 XCDs, share one chunk, so every
  // XCD's L2 holds the activations of the one or two chunks in flight
  // rather than of all of them
  const dim3 grid((N + per - 1) / per, n_ub, ksplit);
  auto kernel = W.group == 128 ? tile_gemm_kernel<128, SWIGLU> : tile_gemm_kernel<64, SWIGLU>;
  kernel<<<grid, 64 * kTileWaves, 0, s>>>(in, in_ld, perm, kdiv, W, count, chunks, step, f, N, out, out_ld,
                                         out_split);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_tile_shared(const uint16_t* x, int T, const d2moe_mwq* w13, const d2moe_mwq* w2,
                              int bits, int cs, int ksplit, int32_t* chunks, uint16_t* h, float* y,
                              hipStream_t s) {
  const int n = (T + cs - 1) / cs, f = w13->rows / 2, d = w2->rows;
  tile_bucket_kernel<<<1, 256, 0, s>>>(0, T, bits, 0, cs, n, chunks);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  err = run_tile_gemm<true>(x, w13->cols, nullptr, 1, view_of(w13), nullptr, chunks, 4, n, f, h, f, s);
  if (err != hipSuccess) return err;
  return run_tile_gemm<false>(h, f, nullptr, 1, view_of(w2), nullptr, chunks, 4, n, f, y, d, s,
                              ksplit, (size_t)T * d);
}

hipError_t launch_tile_bucket(const uint16_t* x, const int32_t* perm, int k, const d2moe_mwq* w13,
                              const d2moe_mwq* w2, int first, int cnt, int bits, int expert,
                              int32_t* chunks, uint16_t* h, float* y, hipStream_t s) {
  const int n = (cnt + kTileChunk - 1) / kTileChunk, f = w13->rows / 2, d = w2->rows;
  tile_bucket_kernel<<<1, 256, 0, s>>>(first, cnt, bits, expert, kTileChunk, n, chunks);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  err = run_tile_gemm<true>(x, w13->cols, perm, k, view_of(w13), nullptr, chunks, 4, n, f, h, f, s);
  if (err != hipSuccess) return err;
  return run_tile_gemm<false>(h, f, nullptr, 1, view_of(w2), nullptr, chunks, 4, n, f, y, d, s);
}

hipError_t launch_tile_gemm13(const uint16_t* x, const int32_t* perm, int k, const d2moe_mwq* w13,
                              const int32_t* count, const int32_t* chunks, int n_ub, uint16_t* h,
                              hipStream_t s) {
  const int f = w13->rows / 2;
  return run_tile_gemm<true>(x, w13->cols, perm, k, view_of(w13), count, chunks, 4, n_ub, f, h, f, s);
}

hipError_t launch_tile_gemm2(const uint16_t* h, const d2moe_mwq* w2, const int32_t* count,
                             const int32_t* chunks, int n_ub, float* y, hipStream_t s) {
  return run_tile_gemm<false>(h, w2->cols, nullptr, 1, view_of(w2), count, chunks, 4, n_ub, w2->cols,
                              y, w2->rows, s);
}

}  // namespace d2moe
