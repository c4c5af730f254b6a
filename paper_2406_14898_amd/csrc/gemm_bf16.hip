// bf16 GEMM for gfx950: C[m, n] (op)= sum_k A(m, k) B(n, k), fp32 accumulate.
//
// Same contract and epilogues as gemm.hip, specialised for the throughput
// path:
//   * large products: 256 x 256 output tile per workgroup, 8 waves (two per
//     SIMD, so one wave's LDS waits are covered by the other's matrix-core
//     work) of 128 x 64, reduction stages of 64 double-buffered in LDS
//     (132 KB): a DMA row segment is one full 128-byte line;
//   * products whose 256 x 256 tiles would leave most of the 256 CUs idle (a
//     few hundred tokens, narrow models), or whose last tile row would be
//     mostly empty, run on 192 x 256 tiles, or on 128 x 256 or 64 x 128 ones
//     with three stages in LDS, and cut the reduction into slices where the
//     tiles are still too few; row counts past whole rounds of large tiles put
//     the remaining rows on their own tile shape (plan_rows).  Hidden 4096,
//     FFN 16384, against 256 x 256 tiles for everything: 37 tokens QKV 83 ->
//     28 us, output projection 80 -> 14 us; 509 tokens 87 -> 59 and 87 -> 33
//     us; 2048 tokens FFN-down 319 -> 236 us; hidden 1280, 1458 tokens output
//     projection 34 -> 12 us;
//   * operands go from HBM/L2 straight into LDS with buffer loads in LDS-DMA
//     mode (no VGPR staging).  Buffer resources bound each operand, so rows
//     or reduction indices past the end read as zero (ragged token tails);
//   * each operand tile is a set of 1 KB DMA blocks of 8 rows (K-contiguous:
//     rows of 64 reduction indices, read by 16-byte fragment reads;
//     MN-contiguous: k-rows of 64 columns, read by transpose reads
//     (ds_read_b64_tr_b16: lane j of a 16-lane group receives four
//     consecutive-k values of column j when lane s points at
//     (k0 + s/4, c0 + 4 (s % 4)))).  Rows keep their global order inside;
//     which rows share a block, and the blocks' 16- or 32-byte offsets in
//     the bank map, keep the fragment reads free of bank conflicts;
//   * every fragment address is one per-lane base plus a compile-time
//     offset, which keeps the address arithmetic out of the VGPR budget;
//   * an LDS-DMA lane always writes to base + 16 * lane, so the placement is
//     chosen through the source addresses;
//   * one barrier per stage, placed between the two 32-wide halves: the
//     second half's fragments are already in registers when the barrier
//     releases the slot, so the next stage's loads and fragment reads overlap
//     matrix-core work.
#include <algorithm>
#include <cmath>

#include "common.h"
#include "kernels.h"

namespace flglm {
namespace {

constexpr int kBK = 64;
// LDS strides of the operand tiles' 1 KB DMA blocks (1056 bytes for the
// MN-contiguous layout, 1040 for the K-contiguous one)
constexpr int kMBlock = 528, kMCol = 8 * kMBlock, kKBlock = 520;

// Output tile of one workgroup: BM x BN by WM x WN waves of (16 kWTM) x
// (16 kWTN), a ring of S operand slots of a 64-wide reduction stage in LDS.
// ACC: row steps of the fp32 accumulator that the epilogue reads together.
template <int BM, int BN, int WM, int WN, int S, int OCC, int ACC = 8>
struct Tile {
  static constexpr int kAccSteps = ACC;
  static constexpr int kBM = BM, kBN = BN, kWM = WM, kWN = WN, kWaves = WM * WN, kThr = 64 * kWaves;
  static constexpr int kStages = S;
  static constexpr int kOcc = OCC;  // workgroups per CU the LDS holds
  static constexpr int kWTM = BM / (16 * WM), kWTN = BN / (16 * WN);
  static constexpr int kRegA = BM * 66, kRegB = BN * 66;  // elements, room for either layout's padding
  static constexpr int kSlot = kRegA + kRegB;
  static constexpr bool kBig = BM >= 192;  // one workgroup per CU, persistent
  // epilogue staging: the whole tile as fp32 where it fits, else one wave row at a time
  static constexpr int kPasses = BM * BN * 4 <= S * kSlot * 2 ? 1 : WM;
  static_assert(BM / kPasses * BN * 4 <= S * kSlot * 2, "staging");
};
using Tile256 = Tile<256, 256, 2, 4, 2, 1>;   // 132 KB
using Tile256w = Tile<256, 256, 2, 4, 2, 1, 4>;
using Tile192 = Tile<192, 256, 2, 4, 2, 1>;   // 116 KB
using Tile128 = Tile<128, 256, 2, 4, 3, 1>;   // 149 KB
// (six stages for reductions of 48 or more with one workgroup on a CU measured
// 0.93 to 1.08 of the time, 1.00 in the mean at 64 stages, operands from memory)
using Tile64 = Tile<64, 128, 1, 4, 3, 2>;     // 74 KB
// weight gradients: more workgroups per CU, so that one's fp32 read-modify-
// write epilogue runs beside the others' reductions
using Tile128w = Tile<128, 128, 2, 2, 2, 2>;  // 66 KB
using Tile64w = Tile<64, 128, 1, 4, 2, 3>;    // 50 KB
constexpr int EPI_PART = 7;  // fp32 partial sums of one reduction slice
typedef short i16x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))

struct G2Args {
  const bf16* A;
  const bf16* B;
  void* C;
  int M, N, K;
  long lda, ldb, ldc;
  const bf16* bias;
  const bf16* R;
  long ldr;
  bf16* C2;
  long ldc2;
  const bf16* Z;
  long ldz;
  // Split reduction: every tile's reduction is cut into `slices` slices whose
  // fp32 sums go to `part` (EPI_PART; token-major products [slices][M][N],
  // weight gradients [slices][tiles][BM][BN]); gemm_slices_kernel or
  // gemm_tile_slices_kernel adds them in slice order and runs the epilogue.
  float* part;
  int slices;
  int nb;  // rows of B that exist (see GemmDesc::b_rows)
  float res_scale;
  // EPI_GELU_BWD: per 256-row tile, the column sums of the stored C (fp32
  // [tiles_m][N]), or null
  float* colsum;
  // Weight gradients: the tiles [tile0, tile0 + tiles) of the work order are
  // this launch's (the others': all).
  int tile0, tiles;
};


__device__ __forceinline__ void dma16(i32x4 rs, uint32_t lds_inst_base, uint32_t voff) {
  dma_lds<16>(rs, lds_inst_base, voff);
}

// Per-lane source byte offsets (reduction index 0) of DMA instruction inst
// (0..31) of an operand tile.
// K-contiguous tile [256 rows][64]: 32 DMA blocks of 8 rows of 128 bytes at a
// stride of 1040 bytes, every row read in address order (as below).  Row
// r = 16 q + t sits in block b = (t & 7) + 8 (q >> 2), row 2 (q & 3) + (t >> 3):
// the 16 rows that one 16-lane fragment read touches (one 16-row group q)
// sit in 8 blocks (16-byte shifts 16 b) at two row parities, i.e. on 16
// distinct bank groups for 16 consecutive lanes.  The LDS serves a 16-byte
// read per cycle to the 16 lanes sharing lane bit 5 and the parity of bits
// 2-4, for which these reads are 2-way conflicted; a placement free of that
// (1056-byte blocks, row parities 512 bytes apart) measured no faster.
// Instruction inst fills block inst.
// ROWS = 192: a wave's six 16-row groups would straddle the 64-row sets, so
// the two wave rows' groups alternate instead (group place 2 j + w holds group
// 6 w + j): every fragment is again a wave base plus a constant.
template <int ROWS>
__device__ __forceinline__ uint32_t k_src(long ld, int inst, int lane) {
  const int slot = lane >> 3;
  int q = 4 * (inst >> 3) + (slot >> 1);
  if constexpr (ROWS == 192) q = 6 * (q & 1) + (q >> 1);
  const int row = 16 * q + (inst & 7) + 8 * (slot & 1);
  return (uint32_t)(row * ld + (lane & 7) * 8) * 2u;
}
// MN-contiguous tile: 4 column blocks of 64 columns (kMCol elements each),
// each 8 DMA blocks b of 8 k-rows of 128 bytes, at a stride of 1056 bytes.
// Every k-row is one DMA row segment read in address order: the texture
// addresser handles a permuted segment several times slower (counted as
// SQ_VMEM_TA_ADDR_FIFO_FULL), so bank spreading comes from where whole rows
// go instead of a swizzle inside them.  k-row k (k = c + 4 s0 + 8 p + 16 s1 +
// 32 h, each digit a bit) sits in block b = c + 4 h, row r = p + 2 s0 + 4 s1.
// A transpose read serves 32 lanes per cycle: k-rows kb .. kb+3 and
// kb+8 .. kb+11 (kb = 0, 4, 16, 20, + 32), 32 bytes each; these sit in four
// blocks (32-byte shifts 32 b) at two row parities: eight distinct bank
// groups.  Instruction inst fills block inst % 8 of column block inst / 8.
__device__ __forceinline__ uint32_t m_src(long ld, int inst, int lane) {
  const int blk = inst >> 3, b = inst & 7;
  const int krow = (b & 3) + 4 * ((lane >> 4) & 1) + 8 * ((lane >> 3) & 1) + 16 * (lane >> 5) + 32 * (b >> 2);
  return (uint32_t)((long)krow * ld + blk * 64 + (lane & 7) * 8) * 2u;
}
// LDS byte offset, inside an operand region, of DMA instruction inst
__device__ __forceinline__ uint32_t k_dst(int inst) { return (uint32_t)inst * (2u * kKBlock); }
__device__ __forceinline__ uint32_t m_dst(int inst) { return (uint32_t)((inst >> 3) * kMCol + (inst & 7) * kMBlock) * 2u; }

// Per-lane fragment bases (element offsets inside one operand tile).
// K-contiguous: fragment j of a wave (rows row0 + 16 j; a wave's fragments
// stay inside a 64-row group or start at one), reduction half c: lane (fr, fg) reads chunk fg + 4 c of row
// row0 + 16 j + fr.
__device__ __forceinline__ int frag_k_base(int row0, int fr, int fg) {
  return (fr & 7) * kKBlock + 64 * (fr >> 3) + 8 * fg + 8 * kKBlock * (row0 >> 6) + 128 * ((row0 >> 4) & 3);
}
// MN-contiguous: fragment j (columns col0 + 16 j), reduction half c: lane s
// of a 16-lane group points at k-row 8 g + s / 4 (block s / 4, row
// (g & 1) + 4 (g >> 1)), columns 4 (s % 4) of group j % 4 of column block
// col0 / 64 + j / 4; the second read is k + 4 (row + 2), half c = k + 32
// (block + 4).
__device__ __forceinline__ int frag_m_base(int col0, int fr, int fg) {
  return (col0 >> 6) * kMCol + 16 * ((col0 >> 4) & 3) + (fr >> 2) * kMBlock + ((fg & 1) + 4 * (fg >> 1)) * 64 +
         4 * (fr & 3);
}
template <int ROWS>
__device__ __forceinline__ int frag_k_base(int w, int rows, int fr, int fg) {
  return ROWS == 192 ? frag_k_base(16 * w, fr, fg) : frag_k_base(w * rows, fr, fg);
}
template <int ROWS>
__device__ __forceinline__ bf16x8 frag_k(const bf16* tile, int base, int c, int j) {
  const int off = ROWS == 192 ? 8 * kKBlock * (j >> 1) + 256 * (j & 1) : 8 * kKBlock * (j >> 2) + 128 * (j & 3);
  return __builtin_bit_cast(bf16x8, ld16(tile + base + off + 32 * c));
}
__device__ __forceinline__ bf16x8 frag_m(const bf16* tile, int base, int c, int j) {
  const bf16* p = tile + base + 16 * (j & 3) + kMCol * (j >> 2) + 4 * kMBlock * c;
  i16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS i16x4*)(p));
  i16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS i16x4*)(p + 128));
  return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// tanh-form GeLU via the logistic function: 0.5 (1 + tanh u) = sigma(2u), so
//   gelu(z)  = z sigma(2u),  u = sqrt(2/pi) (z + 0.044715 z^3)
//   gelu'(z) = sigma(2u) + 2 z sigma(2u) (1 - sigma(2u)) sqrt(2/pi) (1 + 3 * 0.044715 z^2)
// with sigma(v) = 1 / (1 + 2^(-v log2 e)) from the hardware exp2 and reciprocal
// (about 1 ulp each; exp2 saturates to 0 / inf, which gives sigma = 1 / 0).
__device__ __forceinline__ float sigmoid2u(float z) {
  const float c2 = 2.0f * 0.7978845608028654f * kLog2e, a = 0.044715f;
  const float e = __builtin_amdgcn_exp2f(-c2 * (z + a * z * z * z));
  return __builtin_amdgcn_rcpf(1.0f + e);
}
__device__ __forceinline__ float gelu2(float z) { return z * sigmoid2u(z); }
__device__ __forceinline__ float gelu2_grad(float z) {
  const float c = 0.7978845608028654f, a = 0.044715f;
  const float s = sigmoid2u(z);
  return s + 2.0f * c * z * s * (1.0f - s) * (1.0f + 3.0f * a * z * z);
}

// Work order: workgroup wg runs on XCD wg % 8, and each XCD takes a contiguous
// range of work items, one reduction slice of the launch's tiles after
// another, so that an XCD reads few slices of A (K = 16384 in four to eight
// slices: 1-3 % faster than a tile's slices side by side).
__device__ __forceinline__ int work_id(int wg, int nwg) {
  constexpr int kXcd = 8;
  const int q = nwg / kXcd, r = nwg % kXcd;
  const int x = wg % kXcd, j = wg / kXcd;
  return (x < r) ? x * (q + 1) + j : r * (q + 1) + (x - r) * q + j;
}
// Tiles walk bands of kBand tile rows column by column (kAlongN: bands of tile
// columns row by row).
template <int kBand, bool kAlongN>
__device__ __forceinline__ void tile_coords(int tile, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int ta = kAlongN ? tiles_n : tiles_m, tb = kAlongN ? tiles_m : tiles_n;
  const int per_band = kBand * tb;
  const int band = tile / per_band;
  const int first = band * kBand;
  const int size = min(ta - first, kBand);
  const int in_band = tile - band * per_band;
  const int a = first + in_band % size, b = in_band / size;
  tm = kAlongN ? b : a;
  tn = kAlongN ? a : b;
}

// Output tiles of a product.
template <class TL>
__host__ __device__ __forceinline__ int tile_count(const G2Args& a) {
  return ((a.M + TL::kBM - 1) / TL::kBM) * (a.N / TL::kBN);
}

// Bare workgroup barrier: a fence would also wait for DMA stages in flight.
__device__ __forceinline__ void wg_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Epilogue of one BM x BN tile from the wave accumulators acc[i][j] (wave tile
// rows 16 kWTM (wave % WM) + 16 j, columns 16 kWTN (wave / WM) + 16 i), with
// the LDS at stg (the S operand slots, free: every wave is past its operand
// reads) as staging.  The accumulators go to LDS as fp32, [BM / NP][BN] in each
// of NP passes: the whole tile where it fits, else one wave row at a time (a
// 256 x 256 tile: two halves of 128 KB).  Then a lane owns eight consecutive
// columns (group cg = lane % (BN / 8)) and the 512 / BN row groups of a wave
// take successive rows, so bias, residual, GeLU-input and output rows are read
// and written contiguously, 16 bytes per lane, two or four rows per wave
// instruction (a lane of the matrix core holds 4 columns of 16 different rows,
// which as direct stores cost more than the reduction for K = 4096; a CU's
// store instructions cost about the same at 8 and at 16 bytes per lane, so the
// wide form halves the row loop's memory instructions).  Staging puts
// 16-byte chunk c of row r at c ^ (r & 15) ^ ((c >> 4) & 1): the row writes
// of the matrix-core lanes and the 16-lane reads of even (or odd) chunks
// both hit 16 distinct bank groups.
__device__ __forceinline__ int stg_swz(int r, int c) { return c ^ (r & 15) ^ ((c >> 4) & 1); }

template <class TL, int EPI, int STEPS>
__device__ __forceinline__ void tile_epilogue(const G2Args& p, const f32x4 (&acc)[TL::kWTN][TL::kWTM], float* stg,
                                              int tm, int m0, int n0, int tid) {
  constexpr int kWaves = TL::kWaves, kWTM = TL::kWTM, kWTN = TL::kWTN, kBN = TL::kBN, NP = TL::kPasses;
  constexpr int kLpr = kBN / 8, kRpi = 64 / kLpr;  // lanes per row, rows per wave instruction
  constexpr int kRows = TL::kBM / NP, kSteps = kRows / (kWaves * kRpi);
  asm volatile("" : "+v"(tid));  // keeps the epilogue's per-lane values out of the main loop's live range
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave % TL::kWM, wn = wave / TL::kWM;
  const int fr = lane & 15, fg = lane >> 4;
  const int sh = lane / kLpr, cg = lane % kLpr;
  const int n = n0 + 8 * cg;
  float bias[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  // EPI_GELU_BWD with colsum: this lane's eight columns over its rows (the
  // stored, rounded values), in row order
  float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU) {
    Vec8<bf16> b;
    b.load(p.bias + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) bias[e] = b.get(e);
  }
#pragma unroll
  for (int half = 0; half < NP; ++half) {
    const int mbase = m0 + half * kRows + wave;
    if (NP == 1 || wm == half) {
#pragma unroll
      for (int j = 0; j < kWTM; ++j) {
        const int r = (NP == 1 ? wm * 16 * kWTM : 0) + 16 * j + fr;
#pragma unroll
        for (int i = 0; i < kWTN; ++i) {
          const int c = (wn * 16 * kWTN + 16 * i + 4 * fg) >> 2;
          st16(stg + r * kBN + (stg_swz(r, c) << 2), __builtin_bit_cast(u32x4, acc[i][j]));
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();
    // Rows wave + kWaves q, q = kRpi t + sh (t = 0 .. kSteps - 1), in batches
    // of steps whose global loads are issued together before their first use.
    constexpr int kB = kSteps % STEPS == 0 ? STEPS : kSteps < STEPS ? kSteps : kSteps / 2;
    static_assert(kSteps % kB == 0, "whole batches");
#pragma unroll
    for (int t0 = 0; t0 < kSteps; t0 += kB) {
      Vec8<bf16> ext[kB];
      Vec8<float> cacc[kB];
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const long m = mbase + (kRpi * (t0 + u) + sh) * kWaves;
        if (m < p.M) {
          if constexpr (EPI == EPI_BIAS_RES || EPI == EPI_RES) ext[u].load(p.R + m * p.ldr + n);
          if constexpr (EPI == EPI_GELU_BWD) ext[u].load(p.Z + m * p.ldz + n);
          if constexpr (EPI == EPI_ACC_F32) cacc[u].load(static_cast<float*>(p.C) + m * p.ldc + n);
        }
      }
#pragma unroll
      for (int u = 0; u < kB; ++u) {
        const int q = kRpi * (t0 + u) + sh;
        const int r = wave + q * kWaves;
        const long m = mbase + q * kWaves;
        if (m >= p.M) break;
        const u32x4 raw0 = ld16(stg + r * kBN + (stg_swz(r, 2 * cg) << 2));
        const u32x4 raw1 = ld16(stg + r * kBN + (stg_swz(r, 2 * cg + 1) << 2));
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = __uint_as_float(raw0[e]) + bias[e];
          v[4 + e] = __uint_as_float(raw1[e]) + bias[4 + e];
        }
        if constexpr (EPI == EPI_PART) {
          Vec8<float> o;
          o.set(v);
          o.store(static_cast<float*>(p.C) + m * p.ldc + n);
        } else if constexpr (EPI == EPI_ACC_F32) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = cacc[u].get(e) + v[e];
          cacc[u].set(o);
          cacc[u].store(static_cast<float*>(p.C) + m * p.ldc + n);
        } else {
          if constexpr (EPI == EPI_BIAS_RES || EPI == EPI_RES) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += p.res_scale * ext[u].get(e);
          }
          if constexpr (EPI == EPI_GELU_BWD) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= gelu2_grad(ext[u].get(e));
          }
          Vec8<bf16> o;
          o.set(v);
          if (EPI != EPI_BIAS_GELU || p.C) o.store(static_cast<bf16*>(p.C) + m * p.ldc + n);
          if constexpr (EPI == EPI_GELU_BWD) {
#pragma unroll
            for (int e = 0; e < 8; ++e) csum[e] += o.get(e);
          }
          if constexpr (EPI == EPI_BIAS_GELU) {
            float g[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) g[e] = gelu2(v[e]);
            Vec8<bf16> og;
            og.set(g);
            og.store(p.C2 + m * p.ldc2 + n);
          }
        }
      }
    }
    // the second half, or the next tile's loads, overwrite the staging area
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    wg_barrier();
  }
  if constexpr (EPI == EPI_GELU_BWD && TL::kBM == kColsumRows) {
    if (p.colsum) {
      // the sixteen half-waves' partial column sums, added in (wave, half)
      // order (the operand tiles are free: every wave passed the barrier)
      float* cs = stg;
      float* mine = cs + (wave * kRpi + sh) * kBN + 8 * cg;
      st16(mine, __builtin_bit_cast(u32x4, f32x4{csum[0], csum[1], csum[2], csum[3]}));
      st16(mine + 4, __builtin_bit_cast(u32x4, f32x4{csum[4], csum[5], csum[6], csum[7]}));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wg_barrier();
      if (tid < kBN) {
        float t = 0.f;
#pragma unroll
        for (int w2 = 0; w2 < kRpi * kWaves; ++w2) t += cs[w2 * kBN + tid];
        p.colsum[(long)tm * p.N + n0 + tid] = t;
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      wg_barrier();  // the next tile's loads overwrite cs
    }
  }
}

// Row steps of the epilogue whose global reads are issued together: 8 for the
// residual epilogues (a 128-row half's whole share: 6 % faster on the 41447 x
// 4096 x 4096 output projection than 4), 4 elsewhere (8 measured no faster).
// The fp32 accumulator: 8 on small tiles, whose short weight gradients wait for
// these reads (4096 x 16384 over 509 tokens on 128 x 128 tiles: 154 us with 2,
// 148 with 4, 136 with 8); on 256-row tiles 4, and 8 from eight rounds of tiles
// on (with 2, 4 and 8: 130528 x 4096 over 733 tokens 1354, 1334, 1323 us; 4096 x
// 4096 over 900 57.0, 56.8, 59.4; 16384 x 4096 over 1295 259, 265, 278).
// Reading it before the reduction instead was slower (88 -> 103 us, 12288 x
// 4096 over 509 tokens): the first operand stages then queue behind it.
template <int EPI, class TL>
constexpr int epi_steps() {
  if (EPI == EPI_ACC_F32) return TL::kAccSteps;
  return EPI == EPI_BIAS_RES || EPI == EPI_RES ? 8 : 4;
}

// One work item (output tile, reduction slice) of a product; smem holds at
// least TL's operand slots and every thread of the workgroup takes part.
template <bool AK, bool BKc, int EPI, class TL>
__device__ __forceinline__ void gemm_item(const G2Args& p, bf16* smem, int wi, int nwork) {
  constexpr int kBM = TL::kBM, kBN = TL::kBN, kThr = TL::kThr, kWaves = TL::kWaves;
  constexpr int kWTM = TL::kWTM, kWTN = TL::kWTN, kSlot = TL::kSlot, kStages = TL::kStages;
  const int tiles_m = (p.M + kBM - 1) / kBM, tiles_n = p.N / kBN;
  const int nk = (p.K + kBK - 1) / kBK;
  int tm, tn;
  // Bands of 4 tile rows for the forward and dgrad products on 256 x 256
  // tiles (the 32 tiles one XCD holds span 4 row panels of A and 8 column
  // panels of B): 1.5-3 % faster than 8 (16: 5-18 % slower than 8).  Their
  // weight gradients are 0.6 % faster with 8.  Weight gradients on smaller
  // tiles walk bands of tile columns: the C rows that run together are then
  // read and written as 4 KB runs (4096 x 16384 x 256 tokens: 116 us against
  // 159 in bands of tile rows).
  constexpr bool kWgrad = !AK && !BKc;
  const int tiles = kWgrad ? p.tiles : tiles_m * tiles_n;
  const int id = work_id(wi, nwork), slice = id / tiles, tile = id - slice * tiles;
  tile_coords<TL::kBig && !kWgrad ? 4 : 8, kWgrad && !TL::kBig>((kWgrad ? p.tile0 : 0) + tile, tiles_m, tiles_n, tm,
                                                                tn);
  const int kt0 = p.slices == 1 ? 0 : (int)((long)nk * slice / p.slices);
  const int kt1 = p.slices == 1 ? nk : (int)((long)nk * (slice + 1) / p.slices);
  // Per-lane values are rederived in every tile (the opaque copy keeps the
  // compiler from hoisting them out of the tile loop, where they would stay
  // live across the whole body and spill).
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int lane = tid & 63, wave = tid >> 6;
  // wave tile: rows wm * 16 kWTM .., columns wn * 16 kWTN ..
  const int wm = wave % TL::kWM, wn = wave / TL::kWM;
  const int fr = lane & 15, fg = lane >> 4;
  const int m0 = tm * kBM, n0 = tn * kBN;

  // Resources: K-contiguous -> base at the tile's first row, bound = its
  // valid rows; MN-contiguous -> base at the tile's first column, bound = the
  // rest of the buffer (reduction indices >= K read as zero).
  i32x4 ra, rb;
  if constexpr (AK) {
    const int rows = min(kBM, p.M - m0);
    ra = buf_rsrc(p.A + (long)m0 * p.lda, (uint32_t)((long)rows * p.lda * 2));
  } else {
    ra = buf_rsrc(p.A + m0, (uint32_t)(((long)p.K * p.lda - m0) * 2));
  }
  if constexpr (BKc) {
    // rows of B past p.nb (a padded N) do not exist: num_records 0 for a
    // tile wholly past them, so nothing is read there
    const int rows = p.nb > n0 ? min(kBN, p.nb - n0) : 0;
    rb = buf_rsrc(p.B + (long)n0 * p.ldb, (uint32_t)((long)rows * p.ldb * 2));
  } else {
    rb = buf_rsrc(p.B + n0, (uint32_t)(((long)p.nb * p.ldb - n0) * 2));
  }
  // DMA bookkeeping.  Each stage takes one DMA instruction per 8 rows of an
  // operand (32 for a 256-row tile).  Forward and dgrad: every wave issues an
  // equal share, instruction i of wave w being instruction kWaves i + w of
  // the tile.  Weight gradient on 256 x 256 tiles: waves 0-3
  // issue 8 per operand (instruction 4 i + w) and waves 4-7 none.  Waves w
  // and w + 4 share a SIMD, so each SIMD then pairs a loading wave with one
  // that only computes: a load stalled on the texture unit's address queue
  // holds up only the loading wave's matrix instructions while the other
  // wave's instructions keep the matrix core busy (3 % faster on the wgrad; the forward
  // and dgrad products measured within +-1 %).  k_dst / m_dst are linear in
  // the instruction index for these wave numbers, so a wave adds its own
  // offset once.  The per-lane source offsets are fixed up to the stage's
  // reduction offset, added per stage.
  constexpr bool kLoaders = TL::kBig && kWgrad;
  constexpr int kDmaStride = kLoaders ? 4 : kWaves;  // tile instruction stride between a wave's DMAs
  constexpr int kDmaA = kBM / 8 / kDmaStride, kDmaB = kBN / 8 / kDmaStride;  // per stage per loading wave
  constexpr int kDma = kDmaA + kDmaB;
  const bool loader = !kLoaders || wave < 4;
  const int wq = kLoaders ? (wave & 3) : wave;
  const uint32_t lds0 = FL_LDS_ADDR(&smem[0]);
  const uint32_t lds_a = __builtin_amdgcn_readfirstlane(lds0 + (AK ? k_dst(wq) : m_dst(wq)));
  const uint32_t lds_b =
      __builtin_amdgcn_readfirstlane(lds0 + TL::kRegA * 2 + (BKc ? k_dst(wq) : m_dst(wq)));
  uint32_t voa[kDmaA], vob[kDmaB];
#pragma unroll
  for (int i = 0; i < kDmaA; ++i)
    voa[i] = AK ? k_src<kBM>(p.lda, i * kDmaStride + wq, lane) : m_src(p.lda, i * kDmaStride + wq, lane);
#pragma unroll
  for (int i = 0; i < kDmaB; ++i)
    vob[i] = BKc ? k_src<kBN>(p.ldb, i * kDmaStride + wq, lane) : m_src(p.ldb, i * kDmaStride + wq, lane);
  // byte offset of reduction index k0 along each operand
  auto kstep_a = [&](int k0) { return AK ? (uint32_t)k0 * 2u : (uint32_t)((long)k0 * p.lda * 2); };
  auto kstep_b = [&](int k0) { return BKc ? (uint32_t)k0 * 2u : (uint32_t)((long)k0 * p.ldb * 2); };
  // DMA instruction g (A 0 .. kDmaA-1, then B) of this wave for stage kt, into slot
  auto dma_one = [&](int kt, int slot, int g) {
    const uint32_t slot_off = (uint32_t)slot * (kSlot * 2);
    if (g < kDmaA) {
      const int o = kDmaStride * g;
      dma16(ra, lds_a + slot_off + (AK ? k_dst(o) : m_dst(o)), voa[g] + kstep_a(kt * kBK));
    } else {
      const int o = kDmaStride * (g - kDmaA);
      dma16(rb, lds_b + slot_off + (BKc ? k_dst(o) : m_dst(o)), vob[g - kDmaA] + kstep_b(kt * kBK));
    }
  };
  auto issue = [&](int kt, int slot) {
    if (loader) {
#pragma unroll
      for (int g = 0; g < kDma; ++g) dma_one(kt, slot, g);
    }
  };
  const int abase = AK ? frag_k_base<kBM>(wm, 16 * kWTM, fr, fg) : frag_m_base(wm * 16 * kWTM, fr, fg);
  const int bbase = BKc ? frag_k_base<kBN>(wn, 16 * kWTN, fr, fg) : frag_m_base(wn * 16 * kWTN, fr, fg);

  f32x4 acc[kWTN][kWTM];
#pragma unroll
  for (int i = 0; i < kWTN; ++i)
#pragma unroll
    for (int j = 0; j < kWTM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto rd_a = [&](int slot, int c, int j) {
    const bf16* as = smem + slot * kSlot;
    return AK ? frag_k<kBM>(as, abase, c, j) : frag_m(as, abase, c, j);
  };
  auto rd_b = [&](int slot, int c, int i) {
    const bf16* bs = smem + slot * kSlot + TL::kRegA;
    return BKc ? frag_k<kBN>(bs, bbase, c, i) : frag_m(bs, bbase, c, i);
  };
  // fragments of reduction half c of the stage in slot `slot`
  auto load_frags = [&](int slot, int c, bf16x8 (&af)[kWTM], bf16x8 (&bf)[kWTN]) {
#pragma unroll
    for (int i = 0; i < kWTN; ++i) bf[i] = rd_b(slot, c, i);
#pragma unroll
    for (int j = 0; j < kWTM; ++j) af[j] = rd_a(slot, c, j);
  };
  auto mma_all = [&](const bf16x8 (&af)[kWTM], const bf16x8 (&bf)[kWTN]) {
#pragma unroll
    for (int j = 0; j < kWTM; ++j)
#pragma unroll
      for (int i = 0; i < kWTN; ++i) acc[i][j] = mma16(bf[i], af[j], acc[i][j]);
  };
  // bare barrier: a fence would also wait for the younger stage in flight
  auto barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  if (kt1 > kt0) {
  // Stage kt lives in slot (kt - kt0) % kStages.  Prologue: kStages stages in
  // flight; once the first is visible, read its first half.
#pragma unroll
  for (int u = 0; u < kStages; ++u)
    if (u == 0 || kt0 + u < kt1) issue(kt0 + u, u);
  // the first stage's loads done: the younger ones may stay in flight
  if (kt1 - kt0 >= kStages)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 1) * kDma) : "memory");
  else
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  barrier();
  bf16x8 fa0[kWTM], fb0[kWTN], fa1[kWTM], fb1[kWTN];
  load_frags(0, 0, fa0, fb0);
  int slot = 0;
  // Main loop, one stage per iteration, in two halves of 32 reductions.  The
  // issue order is fixed by scheduling barriers: each group of four matrix
  // instructions (one A fragment against the four B fragments) is preceded
  // by one or two fragment reads for the next half and, in the second half,
  // by one (each wave) or two (loading waves of the wgrad) of the DMA
  // instructions for stage kt + kStages, so the memory pipes are fed steadily
  // instead of in bursts that stall issue.
  // The last stage is peeled so that every path through the body passes the
  // barrier (the compiler then never waits for next-half reads early).
  for (int kt = kt0; kt < kt1 - 1; ++kt) {
    const int next = kStages == 2 ? slot ^ 1 : slot + 1 == kStages ? 0 : slot + 1;
#pragma unroll
    for (int j = 0; j < kWTM; ++j) {
      fa1[j] = rd_a(slot, 1, j);
      if (j < kWTN) fb1[j] = rd_b(slot, 1, j);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);  // the matrix group wins issue over the other wave's memory ops
#pragma unroll
      for (int i = 0; i < kWTN; ++i) acc[i][j] = mma16(fb0[i], fa0[j], acc[i][j]);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    // stage kt+1 landed (own loads; the stages behind it may stay in flight)
    // and every wave has finished reading slot kt: refill it with stage kt +
    // kStages, read stage kt+1's first half
    if (kStages > 2 && kt + kStages <= kt1)
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStages - 2) * kDma) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    barrier();
    const bool more = kt + kStages < kt1;
#pragma unroll
    for (int j = 0; j < kWTM; ++j) {
      if (more && loader) {
#pragma unroll
        for (int g = j * kDma / kWTM; g < (j + 1) * kDma / kWTM; ++g) dma_one(kt + kStages, slot, g);
      }
      fa0[j] = rd_a(next, 0, j);
      if (j < kWTN) fb0[j] = rd_b(next, 0, j);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < kWTN; ++i) acc[i][j] = mma16(fb1[i], fa1[j], acc[i][j]);
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
    }
    slot = next;
  }
  load_frags(slot, 1, fa1, fb1);
  mma_all(fa0, fb0);
  mma_all(fa1, fb1);
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  barrier();  // every wave is done with the operand tiles
  if constexpr (EPI == EPI_PART) {
    G2Args q = p;
    if constexpr (kWgrad) {  // the slice's own dense tile, addressed from the product's first element
      q.C = p.part + ((long)slice * p.tiles + tile) * (kBM * kBN) - ((long)m0 * kBN + n0);
      q.ldc = kBN;
    } else {
      q.C = p.part + (long)slice * p.M * p.N;
      q.ldc = p.N;
    }
    tile_epilogue<TL, EPI, epi_steps<EPI, TL>()>(q, acc, reinterpret_cast<float*>(&smem[0]), tm, m0, n0, tid);
  } else {
    tile_epilogue<TL, EPI, epi_steps<EPI, TL>()>(p, acc, reinterpret_cast<float*>(&smem[0]), tm, m0, n0, tid);
  }
}

template <bool AK, bool BKc, int EPI, class TL>
__global__ void __launch_bounds__(TL::kThr, TL::kOcc * TL::kWaves / 4) gemm_bf16_kernel(G2Args p) {
  __shared__ __attribute__((aligned(1024))) bf16 smem[TL::kStages * TL::kSlot];  // [slot][A | B]
  const int nwork = (!AK && !BKc ? p.tiles : tile_count<TL>(p)) * p.slices;
  // Persistent where the grid is smaller than the work (256 x 256 tiles: one
  // workgroup per CU); a tile's epilogue stores drain while the next item's
  // first stages load.
  for (int wi = blockIdx.x; wi < nwork; wi += gridDim.x) gemm_item<AK, BKc, EPI, TL>(p, smem, wi, nwork);
}

// The input gradient d (NN) and the weight gradient w (TN) of one linear layer
// and, with `bias`, its bias gradient (+= the column sums of the layer's output
// gradient) in one launch.  All three only read that gradient.
struct PairArgs {
  G2Args d, w;
  int nd, nw;        // their work items
  int chunk, share;  // of each segment of workgroups: items of d, then of w
  float* bias;       // [w.M], or null
};
template <int EPI, class TD, class TW>
__global__ void __launch_bounds__(256, TD::kOcc < TW::kOcc ? TD::kOcc : TW::kOcc) gemm_pair_kernel(PairArgs p) {
  static_assert(TD::kThr == 256 && TW::kThr == 256, "workgroup");
  constexpr int kD = TD::kStages * TD::kSlot, kW = TW::kStages * TW::kSlot;
  __shared__ __attribute__((aligned(1024))) bf16 smem[kD > kW ? kD : kW];
  const int seg = p.chunk + p.share, nseg = (p.nd + p.chunk - 1) / p.chunk;
  const int b = blockIdx.x;
  if (b < nseg * seg) {
    const int s = b / seg, r = b - s * seg;
    if (r < p.chunk) {
      const int wi = s * p.chunk + r;
      if (wi < p.nd) gemm_item<true, false, EPI, TD>(p.d, smem, wi, p.nd);
    } else {
      const int wi = s * p.share + r - p.chunk;
      if (wi < p.nw) gemm_item<false, false, EPI_ACC_F32, TW>(p.w, smem, wi, p.nw);
    }
  } else {
    colsum_cols<bf16, 4>(p.w.A, p.w.lda, p.w.K, (b - nseg * seg) * 64, p.bias, reinterpret_cast<float*>(smem));
  }
}

// v = the sum over `slices` slices, `stride` floats apart, of eight values, in
// slice order.
__device__ __forceinline__ void sum_slices(const float* src, long stride, int slices, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = 0.f;
  for (int s0 = 0; s0 < slices; s0 += 4) {
    Vec8<float> x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < slices) x[u].load(src + (s0 + u) * stride);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (s0 + u < slices) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] += x[u].get(e);
      }
  }
}

// C += the reduction slices of a weight gradient's tiles (fp32
// [slices][tiles][256][256], in slice order); eight columns per lane, 32
// workgroups per tile.
__global__ void __launch_bounds__(256) gemm_tile_slices_kernel(G2Args p) {
  constexpr int kBM = Tile256::kBM, kBN = Tile256::kBN, kPer = kBM * kBN / (8 * 256);
  const int tile = blockIdx.x / kPer;
  const int at = ((blockIdx.x % kPer) * 256 + threadIdx.x) * 8, r = at / kBN, c = at % kBN;
  int tm, tn;
  tile_coords<8, false>(p.tile0 + tile, (p.M + kBM - 1) / kBM, p.N / kBN, tm, tn);
  const long m = (long)tm * kBM + r;
  if (m >= p.M) return;
  float* out = static_cast<float*>(p.C) + m * p.ldc + tn * kBN + c;
  Vec8<float> o;
  o.load(out);
  float v[8];
  sum_slices(p.part + (long)tile * (kBM * kBN) + at, (long)p.tiles * (kBM * kBN), p.slices, v);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] += o.get(e);
  o.set(v);
  o.store(out);
}

// Sums the reduction slices of a whole product (fp32 [slices][M][N], in slice
// order) and applies the epilogue; eight columns per lane.
template <int EPI>
__global__ void __launch_bounds__(256) gemm_slices_kernel(G2Args p) {
  const long idx = (long)blockIdx.x * 256 + threadIdx.x;
  const int ng = p.N / 8;
  const long m = idx / ng;
  if (m >= p.M) return;
  const int n = (int)(idx % ng) * 8;
  float v[8];
  sum_slices(p.part + m * p.N + n, (long)p.M * p.N, p.slices, v);
  if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_RES || EPI == EPI_BIAS_GELU) {
    Vec8<bf16> b;
    b.load(p.bias + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += b.get(e);
  }
  if constexpr (EPI == EPI_BIAS_RES || EPI == EPI_RES) {
    Vec8<bf16> r;
    r.load(p.R + m * p.ldr + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += p.res_scale * r.get(e);
  }
  if constexpr (EPI == EPI_GELU_BWD) {
    Vec8<bf16> z;
    z.load(p.Z + m * p.ldz + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= gelu2_grad(z.get(e));
  }
  Vec8<bf16> o;
  o.set(v);
  if (EPI != EPI_BIAS_GELU || p.C) o.store(static_cast<bf16*>(p.C) + m * p.ldc + n);
  if constexpr (EPI == EPI_BIAS_GELU) {
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) g[e] = gelu2(v[e]);
    Vec8<bf16> og;
    og.set(g);
    og.store(p.C2 + m * p.ldc2 + n);
  }
}

// Compute units of the current device (one persistent workgroup each; a
// multiple of the 8 XCDs on MI355X, which the tile order relies on).
int num_cus() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
  if (cached[dev] == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cached[dev] = n - n % 8 > 0 ? n - n % 8 : n;
  }
  return cached[dev];
}

// Estimated time (us) of an NT or NN product of M rows on 64-, 128-, 192- or
// 256-row tiles with its reduction in s slices, fitted to a sweep on MI355X (M
// 16 .. 6000, N and K of hidden 1280 and 4096, every tile and slice count): a
// 64-wide stage takes 0.45 us with one 64-row workgroup on a CU and 0.64 with
// two, 0.79 for a 128-row one and 1.31 for a 256-row one; slices cost the
// round trip of their fp32 sums and a launch.  192-row tiles are taken as 0.79
// of a 256-row one, as measured on long products, where the clock falls as more
// CUs are busy (1295 x 130560 x 4096: 1244 us against 1375); short ones reach
// 0.77.  The sweep's operands were in cache and its epilogue a plain store: the
// estimate sees neither the operands' way from memory, which the smaller tiles
// read more often, nor the epilogues' further reads and writes, nor the clock.
// plan_rows allows for that where it matters.
double part_us(int M, int N, int K, int tile, int s) {
  const double n = (double)(K / kBK) / s;
  const long items = (long)((M + tile - 1) / tile) * (N / (tile == 64 ? 128 : 256)) * s;
  const double rounds = (double)((items + 255) / 256);
  double t;
  if (tile == 64) {
    const long full = items / 512, rem = items % 512;
    // (full rounds stay behind each other's stores)
    t = 2.0 + 1.5 * full + 0.97 * (rem > 0) + n * (0.64 * full + (rem > 256 ? 0.64 : rem > 0 ? 0.449 : 0.0));
  } else if (tile == 128) {
    t = 2.4 + rounds * (4.5 + 0.791 * n);
  } else {
    t = 3.7 + rounds * (tile == 192 ? 9.4 + 1.035 * n : 11.9 + 1.31 * n);
  }
  t = std::max(t, 4.5 + 2.0 * N * (double)K / 7.03e6);
  if (s > 1) {
    const double bytes = 8.0 * s * M * (double)N;
    t += 4.3 + std::min(bytes, 21e6) / 4.37e6 + std::max(bytes - 21e6, 0.0) / 6.39e6;
  }
  return t;
}

// The same with the column sums of C where they are asked for: whole 256-row
// tiles form them in their epilogue, the others in another pass over C.
double part_us(const GemmDesc& d, int M, int tile, int s) {
  const bool pass = d.colsum && (tile != kColsumRows || s > 1);
  return part_us(M, d.N, d.K, tile, s) + (pass ? 4.0 + 2.0 * M * (double)d.N / 4.5e6 : 0.0);
}

// fp32 sums of one slice of a 256 x 256 tile
constexpr size_t kTileBytes = (size_t)Tile256::kBM * Tile256::kBN * 4;
constexpr int kTiles[] = {64, 128, 192, 256};
constexpr int kSlices[] = {1, 2, 3, 4, 5, 6, 8, 12, 16};

// Whether M rows may run in s slices: as far as the scratch allows, of at
// least two stages each.  192-row tiles are not sliced (1295 x 4096 x 130560 in
// two slices 1346 us, on 256- and 128-row tiles in four and five 1208).
bool slices_fit(const GemmDesc& d, int M, int tile, int s) {
  const size_t bytes = d.part ? d.part_bytes : 0;
  return s == 1 || (tile != 192 && (size_t)s * M * d.N * 4 <= bytes && 2 * s <= d.K / kBK);
}

// Best single launch for M rows on tiles of at most `most` rows by the estimate.
double best_part(const GemmDesc& d, int M, int most, GemmPart* out) {
  double best = 1e30;
  for (int tile : kTiles)
    for (int s : kSlices) {
      if (tile > most || !slices_fit(d, M, tile, s)) break;
      const double t = part_us(d, M, tile, s);
      if (t < best) {
        best = t;
        *out = GemmPart{M, tile, s};
      }
    }
  return best;
}

// NT / NN: one launch over all rows, or two: as many whole rounds of large
// tiles as fill every CU, and the remaining rows on the shape that suits them.
// Other tiles than 256-row ones read the operands more often, which the
// estimate does not see: where 256-row tiles fill most of the chip, their
// estimate has to be a tenth lower, in forward products of up to eight stages,
// which are bound by their stores, a quarter (us, the smaller tiles that the
// plain estimate takes against 256-row ones, operands from memory: 6000 x 11520
// x 3840 485 / 444, 12000 x 10240 x 3840 847 / 790, 41447 x 768 x 256 41.7 /
// 35.4, 8192 x 2048 x 512 36.4 / 31.0; whole rounds of 256-row tiles and the
// rest apart against one launch of 192-row tiles: 18000 x 4096 x 16384 1846 /
// 2103, 4409 x 16384 x 4096 509 / 549).  Not for few rows against the columns,
// where A, the operand read again, stays in cache (600 x 130560 x 4096: 128-row
// tiles 629, 256 and 344 rows apart 667).
int plan_rows(const GemmDesc& d, bool forward, GemmPart (&parts)[2]) {
  const int nt = d.N / 256;
  const bool large = (long)((d.M + 255) / 256) * nt >= 160 && 32L * d.M >= d.N;
  const double small = !large ? 1.0 : forward && d.K <= 8 * kBK ? 1.0 / 0.75 : 1.0 / 0.9;
  double best = 1e30;
  int n = 1;
  for (int tile : kTiles)
    for (int s : kSlices) {
      if (!slices_fit(d, d.M, tile, s)) break;
      const double t = part_us(d, d.M, tile, s) * (tile == 256 && s == 1 ? 1.0 : small);
      if (t < best) {
        best = t;
        parts[0] = GemmPart{d.M, tile, s};
      }
    }
  if (d.M <= 256) return n;
  for (int tile : kTiles)
    for (int s = 1; tile > 64 && s <= 4; ++s) {
      const long rows_t = d.M / tile;  // whole tile rows
      const long k = rows_t * nt * s / 256 * 256 / ((long)nt * s);
      int m1 = (int)(k * tile);
      if (d.colsum) m1 = m1 / kColsumRows * kColsumRows;  // the second launch starts a block of column sums
      if (m1 <= 0 || m1 >= d.M || !slices_fit(d, m1, tile, s)) continue;
      GemmPart rest;
      // (5 % for what the estimate does not see; also keeps the choice of rows
      // that are close to whole rounds anyway)
      const double t = (part_us(d, m1, tile, s) + best_part(d, d.M - m1, 128, &rest)) / 0.95 *
                       (tile == 256 && s == 1 ? 1.0 : small);
      if (t < best) {
        best = t;
        parts[0] = GemmPart{m1, tile, s};
        parts[1] = rest;
        n = 2;
      }
    }
  return n;
}

// All tiles of the product, or those that the arguments name.
template <bool AK, bool BKc, int EPI, class TL>
hipError_t launch_tile(G2Args a, hipStream_t st) {
  if (a.tiles == 0) a.tiles = tile_count<TL>(a);
  const int items = a.tiles * a.slices;
  const int cus = num_cus();
  const int grid = TL::kBig && items > cus ? cus : items;
  hipLaunchKernelGGL((gemm_bf16_kernel<AK, BKc, EPI, TL>), dim3(grid), dim3(TL::kThr), 0, st, a);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_slices(const G2Args& a, hipStream_t st) {
  const long groups = (long)a.M * (a.N / 8);
  hipLaunchKernelGGL((gemm_slices_kernel<EPI>), dim3((unsigned)((groups + 255) / 256)), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <bool AK, bool BKc, int EPI, class TL>
hipError_t launch_rows(const G2Args& a, hipStream_t st) {
  if (a.slices == 1) return launch_tile<AK, BKc, EPI, TL>(a, st);
  hipError_t e = launch_tile<AK, BKc, EPI_PART, TL>(a, st);
  return e != hipSuccess ? e : launch_slices<EPI>(a, st);
}

G2Args make_args(const GemmDesc& d, bool bk) {
  G2Args a;
  a.A = (const bf16*)d.A; a.B = (const bf16*)d.B; a.C = d.C;
  a.M = d.M; a.N = d.N; a.K = d.K; a.lda = d.lda; a.ldb = d.ldb; a.ldc = d.ldc;
  a.bias = (const bf16*)d.bias; a.R = (const bf16*)d.R; a.ldr = d.ldr;
  a.C2 = (bf16*)d.C2; a.ldc2 = d.ldc2; a.Z = (const bf16*)d.Z; a.ldz = d.ldz;
  a.part = d.part; a.slices = 1; a.tile0 = 0; a.tiles = 0;
  a.nb = gemm_b_rows(bk, d);
  a.res_scale = d.res_scale;
  a.colsum = nullptr;
  return a;
}

// Forward and input-gradient products (rows = tokens).
template <bool BKc, int EPI>
hipError_t launch_tokens(const GemmDesc& d, hipStream_t st) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  GemmPart parts[2];
  int n = 1;
  if (d.tile) parts[0] = GemmPart{d.M, d.tile, d.slices};
  else n = plan_rows(d, BKc, parts);
  long m0 = 0;
  for (int i = 0; i < n; ++i) {
    G2Args a = make_args(d, BKc);
    a.M = parts[i].rows;
    a.slices = parts[i].slices;
    a.A += m0 * d.lda;
    const long cb = sizeof(bf16) * m0 * d.ldc;
    if (a.C) a.C = static_cast<char*>(a.C) + cb;
    if (a.R) a.R += m0 * d.ldr;
    if (a.C2) a.C2 += m0 * d.ldc2;
    if (a.Z) a.Z += m0 * d.ldz;
    float* colsum = EPI == EPI_GELU_BWD && d.colsum ? d.colsum + m0 / kColsumRows * d.N : nullptr;
    // only whole 256-row tiles form the column sums in their epilogue
    const bool fused = parts[i].tile == 256 && parts[i].slices == 1;
    if (fused) a.colsum = colsum;
    hipError_t e = parts[i].tile == 256   ? launch_rows<true, BKc, EPI, Tile256>(a, st)
                   : parts[i].tile == 192 ? launch_rows<true, BKc, EPI, Tile192>(a, st)
                   : parts[i].tile == 128 ? launch_rows<true, BKc, EPI, Tile128>(a, st)
                                          : launch_rows<true, BKc, EPI, Tile64>(a, st);
    if (e == hipSuccess && colsum && !fused)
      e = colsum_partial(DT_BF16, 0, a.C, d.ldc, nullptr, nullptr, nullptr, a.M, d.N, colsum, nullptr, st);
    if (e != hipSuccess) return e;
    m0 += parts[i].rows;
  }
  return hipSuccess;
}

// Estimated time (us) of a weight gradient on 64-, 128- or 256-row tiles, the
// 256-row tiles past whole rounds of 256 in s reduction slices: fitted to a
// sweep on MI355X with operands from memory (hidden 256 to 4096, FFN up to 16384
// wide, vocabularies of 32000 to 130528, 37 to 41447 tokens, every tile and
// slice count).  Choosing by it comes within 0.3 % (geometric mean; 10 % at
// worst) of the fastest choice.  Short reductions are bound by the fp32
// read-modify-write of C, which the small tiles' two or three workgroups per CU
// overlap with reductions (16384 x 4096 over 509 tokens: 64-row tiles 154 us, 128
// 155, 256 194; over 1295 277, 250, 257); long ones by the matrix cores, best fed
// by 256-row tiles (over 8192: 1964, 1069, 880), where few tiles are cut into
// slices instead of leaving CUs idle (1024 x 1024 over 41447 tokens: 64-row tiles
// 301, 256-row ones in 16 slices 94; 3072 x 12288, 64 tiles past two rounds,
// whole 2838, in 4 slices 2280).
double wgrad_us(int M, int N, int K, int tile, int s) {
  const double n = (K + kBK - 1) / kBK;
  const long items = (long)((M + tile - 1) / tile) * (N / (tile == 256 ? 256 : 128));
  if (tile == 64) {
    if (items <= 256) return 7.5 + 0.41 * n;  // one workgroup on a CU
    if (items <= 512) return 8.1 + 0.73 * n;  // two
    return 6.9 + std::max(1.0, items / 768.0) * (7.0 + 0.95 * n * (1.0 + 0.002 * n));
  }
  if (tile == 128) {
    const long full = items / 512, rem = items % 512;
    const double two = 12.5 + 0.87 * n, one = 6.2 + 0.8 * n;  // workgroups on a CU
    const double tail = rem == 0 ? 0.0 : rem <= 256 ? one : two;
    return 5.5 + std::max(items > 256 ? two : tail, full * two + 0.9 * tail + 0.1 * rem / 512.0 * two);
  }
  const long full = items / 256, rem = items % 256;
  const double t = 4.1 + 6.0 * std::min(full, 4L) + full * (26.0 + 1.38 * n);
  if (rem == 0) return t;
  if (s == 1) return t + 10.6 + 20.0 * rem / 256.0 + 1.38 * n;
  return t + 14.6 + 12.0 * rem * s / 256.0 + 1.38 * std::ceil(n / s) + rem * (0.022 * s + 0.1);
}

struct WgradPlan {
  int tile, slices;
};
WgradPlan plan_wgrad(const GemmDesc& d) {
  if (d.tile) return WgradPlan{d.tile, d.slices};
  WgradPlan best{256, 1};
  double t = wgrad_us(d.M, d.N, d.K, 256, 1);
  const int rem = (int)((long)((d.M + 255) / 256) * (d.N / 256) % 256), nk = (d.K + kBK - 1) / kBK;
  const size_t bytes = d.part ? d.part_bytes : 0;
  for (int s : kSlices) {
    // one round of slices of at least two stages each, as far as the scratch allows
    if (s == 1 || rem == 0) continue;
    if (rem * s > 256 || 2 * s > nk || (size_t)rem * s * kTileBytes > bytes) break;
    const double u = wgrad_us(d.M, d.N, d.K, 256, s);
    if (u < t) {
      t = u;
      best = WgradPlan{256, s};
    }
  }
  for (int tile : {64, 128}) {
    // (2 % for what the estimate does not see)
    const double u = 1.02 * wgrad_us(d.M, d.N, d.K, tile, 1);
    if (u < t) {
      t = u;
      best = WgradPlan{tile, 1};
    }
  }
  return best;
}

// Weight gradients (reduction over the tokens).
hipError_t launch_wgrad(const GemmDesc& d, hipStream_t st) {
  if (d.M <= 0 || d.N <= 0) return hipSuccess;
  const G2Args a = make_args(d, false);
  const WgradPlan pl = plan_wgrad(d);
  if (pl.tile == 256) {
    const int tiles = tile_count<Tile256>(a), rem = tiles % 256;
    auto whole = [&](const G2Args& x) {
      return tiles >= 8 * 256 ? launch_tile<false, false, EPI_ACC_F32, Tile256>(x, st)
                              : launch_tile<false, false, EPI_ACC_F32, Tile256w>(x, st);
    };
    if (pl.slices == 1 || rem == 0) return whole(a);
    G2Args b = a;
    b.tiles = tiles - rem;
    hipError_t e = b.tiles ? whole(b) : hipSuccess;
    if (e != hipSuccess) return e;
    b.tile0 = b.tiles; b.tiles = rem; b.slices = pl.slices;
    if ((e = launch_tile<false, false, EPI_PART, Tile256>(b, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(gemm_tile_slices_kernel, dim3(32 * rem), dim3(256), 0, st, b);
    return hipGetLastError();
  }
  if (pl.tile == 128) return launch_tile<false, false, EPI_ACC_F32, Tile128w>(a, st);
  if (tile_count<Tile64>(a) <= 512) return launch_tile<false, false, EPI_ACC_F32, Tile64>(a, st);
  return launch_tile<false, false, EPI_ACC_F32, Tile64w>(a, st);
}

// The pair kernel's tile heights for both products and slices for d.
struct PairPlan {
  int tile_d, slices, tile_w;
};

template <int EPI, class TD, class TW>
hipError_t launch_pair_tiles(const G2Args& d, const G2Args& w, float* bias, hipStream_t st) {
  PairArgs a;
  a.d = d; a.w = w; a.bias = bias;
  a.d.tiles = tile_count<TD>(d);
  a.w.tiles = tile_count<TW>(w);
  a.nd = a.d.tiles * d.slices;
  a.nw = a.w.tiles;
  a.chunk = std::min(num_cus(), (a.nd + 7) / 8 * 8);
  const int nseg = (a.nd + a.chunk - 1) / a.chunk;
  a.share = ((a.nw + nseg - 1) / nseg + 7) / 8 * 8;
  const int grid = nseg * (a.chunk + a.share) + (bias ? w.M / 64 : 0);
  hipLaunchKernelGGL((gemm_pair_kernel<EPI, TD, TW>), dim3(grid), dim3(256), 0, st, a);
  return hipGetLastError();
}

template <int EPI>
hipError_t launch_pair(const PairPlan& pl, const G2Args& d, const G2Args& w, float* bias, hipStream_t st) {
  if (pl.tile_d == 64)
    return pl.tile_w == 64 ? launch_pair_tiles<EPI, Tile64w, Tile64w>(d, w, bias, st)
                           : launch_pair_tiles<EPI, Tile64w, Tile128w>(d, w, bias, st);
  return pl.tile_w == 64 ? launch_pair_tiles<EPI, Tile128w, Tile64w>(d, w, bias, st)
                         : launch_pair_tiles<EPI, Tile128w, Tile128w>(d, w, bias, st);
}

// Tile heights, slices and whether one launch is the faster form, from a sweep
// of every choice on MI355X (rows 9 .. 2048; hidden 256 to 4096, FFN 2.6 to 4
// times as wide).  The input gradient wants about as many items as there are
// CUs, each of six stages or more; the weight gradient's items fill in behind.
// One launch against the products apart (us): hidden 1280, FFN 3328, 1458 rows
// FFN-down 51 / 61, FFN-up 51 / 67, 1024 rows QKV 50 / 56; hidden 4096 output
// projection 512 rows 72 / 81, 1024 rows 96 / 109; 64 rows FFN-down 135 / 145.
// Wide layers of more rows are bound by the matrix cores and by the weight
// gradient's traffic, where the larger tiles of the separate launches win
// (hidden 4096 FFN-up: 340 rows 182 / 194, 384 rows 187 / 200, 448 rows 263 /
// 215, 640 rows 284 / 260; output projection: 1024 rows 96 / 109, 1200 rows 125 /
// 114; hidden 3072 output projection: 2048 rows 95 / 107).
bool plan_pair(const GemmDesc& d, const GemmDesc& w, PairPlan* pl) {
  if (d.tile) {
    *pl = PairPlan{d.tile, d.slices, w.tile};
    return true;
  }
  const long n64 = (long)((d.M + 63) / 64) * (d.N / 128), n128 = (long)((d.M + 127) / 128) * (d.N / 128);
  const long w128 = (long)((w.M + 127) / 128) * (w.N / 128);
  const int stages = d.K / kBK;
  // (820 x 2048 x 8192, 128 stages: 208 unsliced 64-row items 122 us, 112 of 128
  // rows in two slices 95)
  pl->tile_d = d.M < 200 || (n64 < 256 && (stages < 32 || (n64 >= 200 && stages <= 64))) ? 64 : 128;
  const long n = pl->tile_d == 64 ? n64 : n128;
  pl->slices = (int)std::max(1L, std::min({8L, (long)stages / 6, 256 / n}));
  while (pl->slices > 1 && (!d.part || (size_t)pl->slices * d.M * d.N * 4 > d.part_bytes)) --pl->slices;
  pl->tile_w = (w128 > 512 && d.M < 200) || (w128 < 200 && d.M > 900) ? 64 : 128;
  return d.M <= (w128 <= 768 ? kColsumDirectRows : w128 <= 1024 ? 1024 : 384);
}

}  // namespace

bool gemm_bf16_pair_ok(int epi, const GemmDesc& d, const GemmDesc& w) {
  PairPlan pl;
  return (epi == EPI_STORE || epi == EPI_GELU_BWD) && d.M > 0 && w.M > 0 && gemm_bf16_dma_ok(GEMM_NN, d) &&
         gemm_bf16_dma_ok(GEMM_TN, w) && plan_pair(d, w, &pl);
}

hipError_t gemm_bf16_pair(int epi, const GemmDesc& d, const GemmDesc& w, float* bias, hipStream_t st) {
  PairPlan pl;
  if (!gemm_bf16_pair_ok(epi, d, w) || !plan_pair(d, w, &pl) || (bias && w.M % 64 != 0)) return hipErrorInvalidValue;
  G2Args a = make_args(d, false);
  a.slices = pl.slices;
  const G2Args b = make_args(w, false);
  if (pl.slices > 1) {
    hipError_t e = launch_pair<EPI_PART>(pl, a, b, bias, st);
    if (e != hipSuccess) return e;
    return epi == EPI_STORE ? launch_slices<EPI_STORE>(a, st) : launch_slices<EPI_GELU_BWD>(a, st);
  }
  return epi == EPI_STORE ? launch_pair<EPI_STORE>(pl, a, b, bias, st) : launch_pair<EPI_GELU_BWD>(pl, a, b, bias, st);
}

size_t gemm_part_bytes() { return (size_t)64 << 20; }

// Shapes the DMA kernel takes: N a multiple of 256, K-contiguous operands
// with K a multiple of 64, and every buffer offset below 2^31 bytes.
bool gemm_bf16_dma_ok(GemmLayout layout, const GemmDesc& d) {
  constexpr int kBM = 256, kBN = 256;
  if (d.N % kBN != 0 || d.M <= 0) return false;
  const bool ak = layout != GEMM_TN, bk = layout == GEMM_NT;
  if ((ak || bk) && d.K % kBK != 0) return false;
  const long lim = 1L << 31;
  if (!ak && (long)d.K * d.lda * 2 >= lim) return false;
  if (!bk && (long)d.K * d.ldb * 2 >= lim) return false;
  if (ak && (long)kBM * d.lda * 2 >= lim) return false;
  if (bk && (long)kBN * d.ldb * 2 >= lim) return false;
  return true;
}

bool gemm_fuses_colsum(DType dt, GemmLayout layout, int epi, const GemmDesc& d) {
  return dt == DT_BF16 && layout == GEMM_NN && epi == EPI_GELU_BWD && Tile256::kBM == kColsumRows &&
         gemm_bf16_dma_ok(layout, d);
}

int gemm_bf16_plan(GemmLayout layout, const GemmDesc& d, GemmPart (&parts)[2]) {
  if (layout != GEMM_TN) return plan_rows(d, layout == GEMM_NT, parts);
  const WgradPlan pl = plan_wgrad(d);
  parts[0] = GemmPart{d.M, pl.tile, pl.slices};
  return 1;
}

bool gemm_epilogue_colsum(const GemmDesc& d) {
  GemmPart parts[2];
  return plan_rows(d, false, parts) == 1 && parts[0].tile == 256 && parts[0].slices == 1;
}

hipError_t gemm_bf16_dma(GemmLayout layout, int epi, const GemmDesc& d, hipStream_t st) {
  switch (layout) {
    case GEMM_NT:
      switch (epi) {
        case EPI_STORE: return launch_tokens<true, EPI_STORE>(d, st);
        case EPI_BIAS: return launch_tokens<true, EPI_BIAS>(d, st);
        case EPI_BIAS_RES: return launch_tokens<true, EPI_BIAS_RES>(d, st);
        case EPI_BIAS_GELU: return launch_tokens<true, EPI_BIAS_GELU>(d, st);
      }
      break;
    case GEMM_NN:
      switch (epi) {
        case EPI_STORE: return launch_tokens<false, EPI_STORE>(d, st);
        case EPI_GELU_BWD: return launch_tokens<false, EPI_GELU_BWD>(d, st);
        case EPI_RES: return launch_tokens<false, EPI_RES>(d, st);
      }
      break;
    case GEMM_TN:
      if (epi == EPI_ACC_F32) return launch_wgrad(d, st);
      break;
  }
  return hipErrorInvalidValue;
}

}  // namespace flglm
