// Expert FFN of one ESP shard, forward and backward (Section II-A "Experts": weights (M,H) and
// (H,M) around an activation; hidden dimension sharded as Y = sum_p W2^(p) f(W1^(p) X),
// Section II-B, which ESP applies to experts).
//
// Six grouped GEMMs (one group per local expert g, all experts in one launch):
//   forward   Z  = X  * W1[:, h0:h0+H_l]        kind NN   epilogue: store Z and Act = GeLU(Z)
//             Y  = Act * W2[h0:h0+H_l, :]       kind NN
//   backward  dA = dY * W2[h0:h0+H_l, :]^T      kind NT   epilogue: dZ = dA * GeLU'(Z), Act = GeLU(Z)
//             dW2[h0:h0+H_l, :] = Act^T * dY    kind TN   (reduction over the expert's n_src*C rows)
//             dW1[:, h0:h0+H_l] = X^T * dZ      kind TN
//             dX = dZ * W1[:, h0:h0+H_l]^T      kind NT
//
// Activation-type operands live in the AlltoAll receive layout [n_src, G, C, ld]: the rows of
// expert g are n_src separate chunks of C rows.  The kernels address "virtual row" r of expert
// g at physical row ((r / C) * G + g) * C + r % C, so no permutation pass is needed and only
// the last row tile of an expert is ragged.
//
// bf16 path: one kernel, MFMA (v_mfma_f32_16x16x32_bf16 in the two largest tiles but for weight gradients of few k tiles,
// v_mfma_f32_32x32x16_bf16 in the others) with fp32 accumulation, over a family of tiles from 256 x 256 down to 32 x 64
// (described in front of gemm_dma_tile; plan_tiles chooses).  Global memory goes straight to LDS (buffer_load ... lds) in
// k tiles of 64; operands whose memory layout has k as the slow index stay in that layout in LDS and are read with the
// transposing LDS load, so no transpose pass exists.  The MFMA is issued with the operands swapped (D^T = B^T A^T) so that a
// lane ends up with 4 consecutive output columns.
//
// Row counts (capacity padding): the row-tiled GEMMs take an expert's rows in compacted order, the occupied rows of
// all its chunks first, so that only ceil(occupied / tile) row tiles are multiplied however the occupancy is spread
// over the chunks; the weight gradients skip the k tiles of a chunk that lie behind its count, and from four chunks on pack the
// occupied rows.
//
// fp32 path: a kernel on the fp64 matrix cores (fp64 accumulation), row counts used the same way.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace {

using namespace moe;

enum { KIND_NN = 1, KIND_NT = 2, KIND_TN = 3 };
enum { EPI_STORE = 0, EPI_GELU = 1, EPI_DGELU = 2, EPI_PART = 3 };   // EPI_PART: fp32 partial sums of a split reduction

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  void* C2;         // second output (the activation GeLU(Z)) for EPI_GELU
  const void* Zin;  // saved pre-activation for EPI_DGELU
  const int32_t* cnt;  // optional [n_src, G]: rows of chunk (s, g) at or beyond min(cnt, Cc) are zero padding
  // fused dispatch (NN GEMMs, n_src = 1): A is the token matrix and row r of expert g is the token
  // gather[g * Cc + r] / gather_k (the gate's inverse slot map; negative = empty slot, a zero row)
  const int32_t* gather;
  int gather_k;
  uint32_t gather_magic;  // ceil(2^32 / gather_k): v / gather_k = umulhi(v, magic) for v < 2^29 (gather_k <= 8)
  int64_t gather_rows;    // rows of the token matrix
  int G, n_src;
  int Cc;           // rows per chunk (capacity C)
  int R;            // n_src * Cc: virtual rows per expert
  int Mdim, Ndim, Kdim;
  int64_t lda, ldb, ldc;             // leading dimensions, elements
  int64_t b_goff, c_goff;            // per-expert stride of weight-type operands, elements
  int64_t b_off, c_off;              // constant offset of the ESP slice, elements
  int tiles_m, tiles_n, total_tiles;
  int run_mask;                      // tile order (xcd_tile): ~31: the XCDs take runs of 32 tiles in turn; 0: a range each
  uint64_t a_bytes, b_bytes;         // bf16 path: byte sizes of the A and B tensors (buffer descriptors)
  int splits;                        // EPI_PART: parts of the reduction; part q of every expert's matrix in
  float* part;                       // [splits, G, Mdim, Ndim]
};

__device__ __forceinline__ int64_t phys_row(int r, int g, int G, int Cc) {
  const int s = r / Cc;
  return ((int64_t)s * G + g) * Cc + (r - s * Cc);
}

// Row of the A operand that virtual row r of expert g is read from: its place in the received layout,
// or, with a gather map, the token that the slot holds (-1: an empty slot, read as zeros).
__device__ __forceinline__ int64_t a_src_row(const GemmArgs& p, int r, int g) {
  if (p.gather == nullptr) return phys_row(r, g, p.G, p.Cc);
  const int iv = p.gather[(int64_t)g * p.Cc + r];
  if (iv < 0) return -1;
  const int64_t tok = iv / p.gather_k;
  return tok < p.gather_rows ? tok : -1;   // an index past the token matrix is treated as an empty slot
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA kernel
// ------------------------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// The epilogue's 16-byte accesses go through buffer descriptors: a lane that must not load or store passes an offset
// beyond num_records, which reads as zeros and stores nothing, without a branch.  (The requests of the k loop go through
// descriptors too, but always lie inside their tensor: see gemm_dma_tile.)
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t OOB = 0xFFFFFFF0u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
template <bool STREAM = false>   // STREAM: non-temporal hint, for data read here for the last time
__device__ __forceinline__ uint4 ldb16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, STREAM ? 2 : 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// coefficients written by fit_gelu_poly.py (this directory)
__device__ constexpr float GELU_PHI[9] = {3.989023268e-01f, -6.634449214e-02f, 9.815968573e-03f, -1.108560129e-03f,
                                          9.341852274e-05f, -5.626405255e-06f, 2.255412426e-07f, -5.327701835e-09f,
                                          5.564777111e-11f};
__device__ constexpr float GELU_DG[10] = {7.977564335e-01f, -2.653926015e-01f, 5.909253657e-02f, -9.040454403e-03f,
                                          9.965471691e-04f, -7.936266047e-05f, 4.432653895e-06f, -1.634905260e-07f,
                                          3.552443228e-09f, -3.426744305e-11f};
// GeLU pieces for the bf16 epilogues, transcendental-free: on |z| <= 4.25 the odd parts of
//   Phi(z) - 1/2            (Phi = standard normal CDF, GeLU(z) = z Phi(z))   and
//   GeLU'(z) - 1/2 = Phi(z) + z phi(z) - 1/2
// are odd minimax polynomials in z (9 and 10 coefficients, fitted in fp64 and evaluated by Horner in
// fp32); outside that range z is clamped, where both functions are within 2e-4 of their limits.
// Evaluated in fp32: |GeLU error| < 5e-5 (relative 1e-5 for large z), |GeLU' error| < 1.7e-4, both far
// below the bf16 rounding of the stored result (2^-9 relative).
__device__ __forceinline__ float gelu_poly(float z) {
  const float zc = __builtin_amdgcn_fmed3f(z, -4.25f, 4.25f);
  const float u = zc * zc;
  float q = fmaf(GELU_PHI[8], u, GELU_PHI[7]);
#pragma unroll
  for (int i = 6; i >= 0; --i) q = fmaf(q, u, GELU_PHI[i]);
  const float cdf = __builtin_amdgcn_fmed3f(fmaf(zc, q, 0.5f), 0.0f, 1.0f);
  return z * cdf;
}
__device__ __forceinline__ float gelu_grad_poly(float z) {
  const float zc = __builtin_amdgcn_fmed3f(z, -4.25f, 4.25f);
  const float u = zc * zc;
  float q = fmaf(GELU_DG[9], u, GELU_DG[8]);
#pragma unroll
  for (int i = 7; i >= 0; --i) q = fmaf(q, u, GELU_DG[i]);
  return fmaf(zc, q, 0.5f);
}

// Epilogue, staged through LDS so that global memory sees 16-byte accesses in
// which consecutive lanes cover a contiguous run of a row (the MFMA result layout alone gives
// 8-byte pieces strided across 32 rows).  Each wave owns a private slice of the (now idle) stage
// memory: per 32-row block it writes bf16 results in [32][CW] row-major form (CW = columns of the
// wave tile, row pitch 2 CW + 16 bytes), reads them back row-wise and stores them; the GeLU
// epilogue stages its second output, and the GeLU' epilogue the saved pre-activation it reads, the
// same way.  Global memory is addressed through buffer descriptors with 32-bit byte offsets, so
// the code is branch-free: a row or column outside the problem gets an out-of-range offset, which
// the hardware drops (stores) or answers with zeros (loads).
// STREAM = the non-temporal hint, for tensors that are not read again soon (the saved pre-activation,
// the weight gradients): they then do not push the weights and the live activations out of the
// last-level cache, which the next GEMMs read their operands from.
template <bool STREAM = false>
__device__ __forceinline__ void stb16(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, const uint4& v) {
  const u32x4_t q = {v.x, v.y, v.z, v.w};
  __builtin_amdgcn_raw_buffer_store_b128(q, r, (int)byte_off, 0, STREAM ? 2 : 0);
}
// The accumulators come in MFMA blocks of MR x MR; a 32 x 32 piece of the wave tile is four groups of 4 consecutive
// columns per lane either way (quad()).
template <int MR> struct AccBlock;
template <> struct AccBlock<32> { typedef f32x16_t type; };
template <> struct AccBlock<16> { typedef f32x4_t type; };
template <int KIND, int EPI, int MR, int MB, int NBK, int AM, int AN>
__device__ __forceinline__ void store_tile_lds(const GemmArgs& p, typename AccBlock<MR>::type (&acc)[AM][AN],
                                               char* wave_lds, int g, int mwave, int mshift, int nbase,
                                               const uint32_t (&out_off)[2], int lane) {
  constexpr int CW = 32 * NBK;            // columns of the wave tile
  constexpr int PITCH_B = 2 * CW + 16;    // staged row pitch, bytes
  constexpr int BUF = 32 * PITCH_B;
  constexpr int LPR = CW / 8;             // lanes per row in the row-wise phase (16 bytes each)
  constexpr int RPI = 64 / LPR;           // rows per instruction
  constexpr int NT_ = 32 / RPI;           // instructions per 32-row block
  char* buf0 = wave_lds;          // first output (or staged Z on the way in)
  char* buf1 = wave_lds + BUF;    // second output
  const int rl = lane / LPR;      // row-wise phase: row RPI t + rl, 16-byte chunk lane % LPR
  const int cc = lane % LPR;
  const int ncol = nbase + cc * 8;
  const bool col_ok = ncol < p.Ndim;

  // descriptors: the activation tensors as a whole, or (weight gradients) this expert's matrix from
  // the first element of the shard on
  __amdgpu_buffer_rsrc_t rC, rC2, rZ;
  if (KIND == KIND_TN) {
    const uint32_t bytes = (uint32_t)(((int64_t)(p.Mdim - 1) * p.ldc + p.Ndim) * 2);
    rC = make_rsrc(reinterpret_cast<bf16_t*>(p.C) + ((int64_t)g * p.c_goff + p.c_off), bytes);
    rC2 = rC; rZ = rC;
  } else {
    const uint32_t bytes = (uint32_t)((uint64_t)p.n_src * p.G * p.Cc * (uint64_t)p.ldc * 2);
    rC = make_rsrc(p.C, bytes);
    rC2 = make_rsrc(EPI == EPI_GELU ? p.C2 : p.C, bytes);
    rZ = make_rsrc(EPI == EPI_DGELU ? p.Zin : p.C, bytes);
  }
  // byte offset of (row, ncol) for the rows this lane touches in the row-wise phase, or OOB: rows of a weight
  // gradient are a constant number of leading dimensions apart; for activations the lanes hold the offsets of the
  // wave tile's rows (lane, lane + 64), which are handed round
  uint32_t off[MB][NT_];
  if (KIND == KIND_TN) {
    const uint32_t ldc2 = (uint32_t)p.ldc * 2u;
    const uint32_t base = ((uint32_t)(mwave + mshift + rl) * (uint32_t)p.ldc + (uint32_t)ncol) * 2u;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int t = 0; t < NT_; ++t) {
        const int d = i * 32 + RPI * t;
        off[i][t] = (mwave + mshift + d + rl < p.Mdim && col_ok) ? base + (uint32_t)d * ldc2 : OOB;
      }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int t = 0; t < NT_; ++t) {
        const int d = mshift + i * 32 + RPI * t;   // multiple of RPI: d + rl stays within one half of the wave tile
        const uint32_t o = (uint32_t)__shfl((int)(d < 64 ? out_off[0] : out_off[1]), (d & 63) + rl, 64);
        off[i][t] = (o != OOB && col_ok) ? o + (uint32_t)ncol * 2u : OOB;   // even: bit 0 marks a row of zeros
      }
  }
  uint4 zq_next[EPI == EPI_DGELU ? NT_ : 1];
  if (EPI == EPI_DGELU) {
#pragma unroll
    for (int t = 0; t < NT_; ++t) zq_next[t] = ldb16<true>(rZ, off[0][t] & ~1u);
  }
  // accumulator phase, group q4 of block j: MR = 32: row lane % 32, 4 columns at 32 j + 8 q4 + 4 (lane / 32);
  // MR = 16: row 16 (q4 / 2) + lane % 16, 4 columns at 32 j + 16 (q4 % 2) + 4 (lane / 16)
  static_assert(AM == MB * 32 / MR && AN == NBK * 32 / MR, "accumulator blocks of the wave tile");
  const int acc_off = (lane & (MR - 1)) * PITCH_B + (lane / MR) * 8;
  auto quad = [&](int i, int j, int q4, int e) -> float {
    if constexpr (MR == 32) return acc[i][j][q4 * 4 + e];
    else return acc[2 * i + (q4 >> 1)][2 * j + (q4 & 1)][e];
  };
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    if (EPI == EPI_DGELU) {  // bring in the saved pre-activation, row-wise; the next block's is requested first
#pragma unroll
      for (int t = 0; t < NT_; ++t) *reinterpret_cast<uint4*>(buf0 + (RPI * t + rl) * PITCH_B + cc * 16) = zq_next[t];
      if (i + 1 < MB) {
#pragma unroll
        for (int t = 0; t < NT_; ++t) zq_next[t] = ldb16<true>(rZ, off[i + 1][t] & ~1u);
      }
    }
#pragma unroll
    for (int j = 0; j < NBK; ++j) {
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float v[4] = {quad(i, j, q4, 0), quad(i, j, q4, 1), quad(i, j, q4, 2), quad(i, j, q4, 3)};
        const int at = acc_off + j * 64 + (MR == 32 ? q4 * 16 : (q4 >> 1) * 16 * PITCH_B + (q4 & 1) * 32);
        char* a0 = buf0 + at;
        char* a1 = buf1 + at;
        if (EPI == EPI_STORE) {
          *reinterpret_cast<uint2*>(a0) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        } else if (EPI == EPI_GELU) {
          float a[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) a[e] = gelu_poly(v[e]);
          *reinterpret_cast<uint2*>(a0) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
          *reinterpret_cast<uint2*>(a1) = make_uint2(pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]));
        } else {
          const uint2 zq = *reinterpret_cast<const uint2*>(a0);
          const float z[4] = {__uint_as_float(zq.x << 16), __uint_as_float(zq.x & 0xFFFF0000u),
                              __uint_as_float(zq.y << 16), __uint_as_float(zq.y & 0xFFFF0000u)};
          float d[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) d[e] = v[e] * gelu_grad_poly(z[e]);
          *reinterpret_cast<uint2*>(a0) = make_uint2(pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3]));
        }
      }
    }
    // row-wise read-back and store (LDS operations of one wave complete in program order)
#pragma unroll
    for (int t = 0; t < NT_; ++t) {
      const bool zero = KIND != KIND_TN && (off[i][t] & 1u);
      const uint4 none = make_uint4(0, 0, 0, 0);
      const uint4 v = *reinterpret_cast<const uint4*>(buf0 + (RPI * t + rl) * PITCH_B + cc * 16);
      stb16<(EPI == EPI_GELU || KIND == KIND_TN)>(rC, off[i][t] & ~1u, zero ? none : v);
      if (EPI == EPI_GELU) {
        const uint4 v2 = *reinterpret_cast<const uint4*>(buf1 + (RPI * t + rl) * PITCH_B + cc * 16);
        stb16(rC2, off[i][t] & ~1u, zero ? none : v2);
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// bf16 MFMA tile with an LDS-DMA pipeline.
//
// TM x TN output tile, k tile 64, WM x WN waves over the tile times WK waves over the MFMA steps of a k tile (two
// of 32 k or four of 16 k; WK = 2: two of the four per group, whose sums are added through LDS at the end).  Global memory
// goes straight to LDS (buffer_load ... lds, 16 bytes per lane, no VGPR staging, no ds_write) into two rings of whole k
// tiles, SA tiles of the A operand and SB of the B operand.  A k tile is 64 wide so that every request of a k-contiguous
// operand covers whole 128-byte lines.  A wave instruction fills 1 KiB of consecutive 16-byte slots in lane
// order, so a tile is stored unpadded and bank conflicts are avoided by permuting WHICH 16-byte chunk of a row
// each lane fetches (an XOR swizzle that the fragment reads undo).  Every lane of a request fetches from inside the
// tensor: the zero fill of an out-of-range request can reach LDS after the wait for it is over, and would then
// destroy what the slot was refilled with.  Rows and columns outside the problem and padding rows are fetched
// from another row / column (what they yield is not stored, or stored as zeros), k indexes behind the end of a k tile
// from its first one (the fragments of both operands are masked).
//   operand with k contiguous in memory : [row][64 k] (128-byte rows, 8 chunks), chunk c of row r in slot
//       c ^ ((r >> 1) & 7); fragments are read with ds_read_b128.
//   operand with k as the slow index    : [64 k][T cols], chunk c of k-row k in slot c ^ 4 (k & 3) (T = 64:
//       c ^ 4 ((k >> 1) & 1); 16 x 16 MFMAs: also ^ 2 ((k >> 3) & 1), because the 16-lane groups then differ in k);
//       fragments are read with the transposing LDS load ds_read_b64_tr_b16: a
//       16-lane group reads a 4(k) x 16(col) patch (lane s: k-row s/4, 8-byte piece s%4) and lane i receives
//       the 4 k-values of column i.
// Pipeline: the fragments of MFMA step s+1 are read under step s, each between two MFMAs (Reads).  Once per k tile, inside its
// last step (when the fragments of that step are in registers, so nobody needs the tile's LDS any more), each wave waits until
// its own requests for the next tile have landed, all waves meet at a barrier, the fragments of the next tile's
// first step are read, and the freed slots are refilled: tile t+SB of B, then tile t+SA of A, one request
// between MFMA rows.  The last SA tiles have nothing to request behind them; they are a loop of their own, in which a
// wave waits for all of its requests instead of for the older ones by count.
// What bounds it: with every compute unit busy, the power limit (the clock falls to 1.7 - 1.8 GHz) and the delivery
// of tiles from L2; with few tiles, the latency of a k tile.  k tiles of 64 instead of 32 (64-byte pieces of
// k-contiguous rows fetch half a cache line and look every line up twice): 8 experts of 16384 x 4096 x 7168, per
// GEMM, 6.83 / 6.44 (forward) and 6.90 / 7.59 (backward) -> 6.3 / 5.9 and 6.1 / 6.1 ms, 1.1 - 1.2 -> 1.2 - 1.35
// PFLOP/s.  Four waves of 128 x 128 and rows padded off a power of two measured no better.
// Which MFMA: under the power limit 16x16x32 costs less energy per flop than 32x32x16 (on random operands in registers 2.05
// against 1.81 PFLOP/s, operands from LDS 1.80 against 1.55).  In this kernel it buys clock, 1.74 against 1.51 GHz, and
// pays only with the reads spread between the MFMAs: reads behind every fourth MFMA, 65 % of the cycles busy and no
// gain; spread, 69 %: the three launches of the GEMMs above and the merged backward launch 6.74 / 6.27 / 6.45 / 18.99 ->
// 6.57 / 6.11 / 6.25 / 18.39 ms.  The tiles with two wave groups over k keep 32x32x16, which gives each group two steps
// per k tile, and so do weight gradients with few k tiles (Tile256Brief), which are not under the power limit.  Tried
// without gain: rows of the last step in front of the barrier 2 -> 3 or 4 (to 4 % slower at 12 k tiles), s_setprio for half
// of the waves, a second barrier that frees B's slot in the first step (-1 to +3 % in single launches).
// ------------------------------------------------------------------------------------------
#define LDS_AS __attribute__((address_space(3)))
constexpr int DK = 64;   // k tile
// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding (gfx9 encoding)
constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }
constexpr int lgkmcnt_imm(int n) { return 0xC07F | (n << 8); }   // LDS operations of a wave end in order

template <int TM_, int TN_, int WM_, int WN_, int WK_, int SA_, int SB_, int MR_ = WK_ == 1 ? 16 : 32>
struct TileCfg {
  static constexpr int TM = TM_, TN = TN_, WM = WM_, WN = WN_, WK = WK_, SA = SA_, SB = SB_;
  static constexpr int NW = WM * WN * WK;             // waves
  static constexpr int MR = MR_;                      // MFMA: MR x MR x KS
  static constexpr int KS = 512 / MR;
  static constexpr int MB = TM / WM / MR, NB = TN / WN / MR;   // MFMA blocks per wave
  static constexpr int RA = TM / 8 / NW, RB = TN / 8 / NW;     // requests (1 KiB) per wave and k tile
  static constexpr int SPT = DK / KS / WK;            // MFMA steps per wave and k tile
  static constexpr int A_UNIT = TM * DK * 2, B_UNIT = TN * DK * 2;
  static constexpr int LDS = SA * A_UNIT + SB * B_UNIT;
  static_assert(SPT % 2 == 0, "the steps take turns with the two register sets of B fragments");
  static_assert(TM / 8 % NW == 0 && TN / 8 % NW == 0, "requests are dealt evenly");
  static_assert(SA == SB || SA == SB + 1, "ring depths");
};

__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t r, char* lds_wave_base, uint32_t byte_off) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (LDS_AS void*)lds_wave_base, 16, (int)byte_off, 0, 0, 0);
}
// Fragment reads are issued as volatile asm: the compiler then neither reorders them nor guards
// them with conservative waits against the LDS-DMA requests in flight.  The kernel waits for them
// itself (s_waitcnt lgkmcnt(0)) and passes the registers through ready() before the MFMAs use them.  Every read is
// waited for like that, also one that is not used: the compiler takes the registers as written at the read.
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
union Frag {
  bf16x8_t v;
  u32x4_t q;
  u32x2_t h[2];
};
template <int OFF>
__device__ __forceinline__ void lds_read_kc(Frag& f, uint32_t addr) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.q) : "v"(addr), "n"(OFF));
}
template <int OFF, int HOFF>   // HOFF: distance of the second half's k-rows
__device__ __forceinline__ void lds_read_nc(Frag& f, uint32_t addr) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.h[0]) : "v"(addr), "n"(OFF));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(f.h[1]) : "v"(addr), "n"(OFF + HOFF));
}
__device__ __forceinline__ void ready(Frag& f) { asm volatile("" : "+v"(f.q)); }

__device__ __forceinline__ int clamp_count(int c, int Cc) { return min(max(c, 0), Cc); }

template <int I, int N, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<I + 1, N>(f);
  }
}

// Workgroup -> output tile.  Workgroup ids are dealt round-robin to the 8 XCDs, so id % 8 names the XCD (problems
// of a merged launch start at multiples of 8).  Linear tile order: expert by expert, blocks of 16 row tiles, in a block
// strips of 4 tile columns, in a strip row by row.  32 consecutive tiles (what an XCD's 32 CUs run at the same time) then
// form an 8 x 4 patch, which shares 8 + 4 operand slices per k step in that XCD's L2 instead of 1 + 32, and the XCDs take
// consecutive patches: the whole chip is in one 16 x 16 block, whose operands the last-level cache can hold until the
// block is done (what misses L2 stays the same).  (With a contiguous range of the order per XCD the eight XCDs were in
// eight experts, whose strips together do not fit that cache: 8 experts of 16384 x 4096 x 7168, two forward GEMMs,
// dZ, merged backward: 6.57 / 6.11 / 6.25 / 18.39 -> 6.12 / 5.50 / 5.91 / 17.11 ms on one card.)
// Where an expert's operands fit in an XCD's L2 (tile_runs) a row-tiled GEMM keeps the contiguous ranges: an XCD then reads
// those of few experts, and every strip but the first finds them in its L2.
// t = index within an expert of tm_n row tiles.
__device__ __forceinline__ void patch_order(int t, int tm_n, int tiles_n, int& tm, int& tn) {
  constexpr int SW = 4, RB = 16;
  int m0 = 0;                           // first row tile of the block
  if (tm_n > RB) {                      // (a division that few rows do without)
    m0 = t / (RB * tiles_n) * RB;
    t -= m0 * tiles_n;
    tm_n = min(RB, tm_n - m0);
  }
  const int full = tiles_n / SW, strip = tm_n * SW;
  if (t < full * strip) {
    const int sn = t / strip, r = t - sn * strip;
    tm = r / SW;
    tn = sn * SW + (r - tm * SW);
  } else {
    const int w = tiles_n - full * SW, r = t - full * strip;
    tm = r / w;
    tn = full * SW + (r - tm * w);
  }
  tm += m0;
}
// the i-th of n tiles (n = 8 per_xcd, rounded up) that XCD x takes: runs of 32 in turn, or one range
__device__ __forceinline__ int xcd_tile(const GemmArgs& p, int x, int i, int per_xcd) {
  const int full = per_xcd & p.run_mask;
  return i < full ? ((i & ~31) * 8 + x * 32) + (i & 31) : full * 8 + x * (per_xcd - full) + (i - full);
}
// With row counts the order holds the row tiles that have occupied rows only (compacted: an expert with n occupied rows
// has ceil(n / TM) of them).  Where padding has to be stored as zeros the workgroups behind them do that: with one chunk
// per expert a workgroup for every tile of padding (fill_tile; padding rows inside a multiplied tile are stored by that
// tile); with several, whose padding is spread over the buffer, a workgroup for an equal share of all padding rows
// (fill_shares), about one for a tile's worth, or for four with very many.  The grid has a workgroup for every tile of the
// capacity, and MORE_SHARES (grid_of); the rest leave at once.
// How many shares there are matters little.  One for each tile's worth of padding, and one for four, forward and backward call:
// 8 experts of 3500 occupied in 20480 rows x 2048 x 2048, 32 chunks, 713 / 961 and 700 / 942 us; 4 of 8 chunks of
// 512 x 1024 x 2048, half full, 114.1 / 171.4 and 110.7 / 171.6; 16 chunks of 300 x 1024 x 1024, a third full, 50.2 / 78.5 and
// 51.7 / 75.6.  (place() counts 256 compute units with one workgroup each; with small tiles there is room for more.)
// Fewer and larger shares between the tiles, to store beside the matrix work, measured slower: a compute unit stores no more
// than some 20 GB/s while the others load the memory system, and the whole chip 4.5 to 5 TB/s.
// With a workgroup that walked the rows of every tile of zeros the first of these shapes took 471 / 391 / 380 us (the forward
// GEMMs and dZ, which stores no zeros), with shares 427 / 296 / 238.
// Returns 0: nothing to do, 1: a tile to multiply, 2: padding to fill (one chunk: tile g, tm, tn; several: share g of tm).
constexpr int MORE_SHARES = 64;
template <int TM, bool ZEROS>
__device__ __forceinline__ int map_tile(const GemmArgs& p, int vb, bool counted, int& g, int& tm, int& tn) {
  const int x = vb & 7, i = vb >> 3;
  if (!counted) {
    const int per_xcd = (p.total_tiles + 7) / 8;
    const int tile = xcd_tile(p, x, i, per_xcd);
    if (i >= per_xcd || tile >= p.total_tiles) return 0;
    const int tiles_per_g = p.tiles_m * p.tiles_n;
    g = tile / tiles_per_g;
    patch_order(tile - g * tiles_per_g, p.tiles_m, p.tiles_n, tm, tn);
    return 1;
  }
  // tile: index among the T tiles to multiply, or -1 (g and tm are set if a share of the padding is to be filled)
  auto place = [&](int T, int& what) {
    const int Z = p.total_tiles - T;      // tiles' worth of padding behind the multiplied tiles
    const int idle = -T & 255;            // compute units without a tile in the last round
    const int nz = !ZEROS ? 0 : p.n_src == 1 ? Z : idle > 0 && Z <= 2 * idle ? min(2 * idle, Z + MORE_SHARES)
                              : Z <= 1024 ? Z + MORE_SHARES : max(1024, Z / 4);
    const int per_t = (T + 7) / 8, per_z = (nz + 7) / 8, n = per_t + per_z;
    what = 0;
    if (i >= n) return -1;
    if (i >= per_t) {
      g = (i - per_t) * 8 + x;
      tm = nz;
      what = g < nz ? 2 : 0;
      return -1;
    }
    const int tile = xcd_tile(p, x, i, per_t);
    if (tile >= T) return -1;
    what = 1;
    return tile;
  };
  int what;
  if (p.n_src == 1 && p.G <= 16) {   // few counts: scalar loads, in the scalar cache from a compute unit's second tile on
    int o[16], occ_all = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) o[e] = p.cnt[min(e, p.G - 1)];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      o[e] = e < p.G ? (clamp_count(o[e], p.Cc) + TM - 1) / TM : 0;
      occ_all += o[e];
    }
    int tile = place(occ_all * p.tiles_n, what);
    if (what == 0) return what;
    const bool zero = what == 2;
    if (zero) tile = g;
    int first = 0, mine = 0, og = 0, run = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = e < p.G ? (zero ? p.tiles_m - o[e] : o[e]) : 0;
      if (run * p.tiles_n <= tile && m > 0) { g = e; first = run; mine = m; og = o[e]; }
      run += m;
    }
    patch_order(tile - first * p.tiles_n, mine, p.tiles_n, tm, tn);
    if (zero) tm += og;
    return what;
  }
  // 64 experts at a time, a lane each; with fewer the lanes share the chunks of an expert
  const int lane = threadIdx.x & 63;
  const int width = p.G >= 64 ? 64 : p.G <= 1 ? 1 : 1 << (32 - __builtin_clz(p.G - 1));   // a power of two
  auto occupied = [&](int e0) {      // row tiles of expert e0 + lane % width that hold occupied rows
    const int e = e0 + (lane & (width - 1)), step = 64 / width;
    int n = 0;
    if (e < p.G) {
#pragma unroll 4
      for (int s = lane / width; s < p.n_src; s += step) n += clamp_count(p.cnt[s * p.G + e], p.Cc);
    }
    for (int d = width; d < 64; d <<= 1) n += __shfl_xor(n, d, 64);
    return lane < width ? (n + TM - 1) / TM : 0;
  };
  const int o0 = occupied(0);
  int occ_all = 0;
  for (int e0 = 0; e0 < p.G; e0 += 64) {
    int o = e0 == 0 ? o0 : occupied(e0);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) o += __shfl_xor(o, d, 64);
    occ_all += o;
  }
  int tile = place(__builtin_amdgcn_readfirstlane(occ_all) * p.tiles_n, what);
  if (what == 0 || (what == 2 && p.n_src > 1)) return what;
  const bool zero = what == 2;
  if (zero) tile = g;
  int run = 0;   // row tiles of the experts before e0
  for (int e0 = 0; e0 < p.G; e0 += 64) {
    const int o = e0 == 0 ? o0 : occupied(e0);
    const int m = zero ? (lane < width && e0 + lane < p.G ? p.tiles_m - o : 0) : o;
    int incl = m;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(incl, d, 64);
      if (lane >= d) incl += v;
    }
    const unsigned long long hit = __ballot((run + incl) * p.tiles_n > tile);
    if (hit) {
      const int l = __ffsll((long long)hit) - 1;
      const int before = __builtin_amdgcn_readlane(incl - m, l), mine = __builtin_amdgcn_readlane(m, l);
      g = e0 + l;
      patch_order(tile - (run + before) * p.tiles_n, mine, p.tiles_n, tm, tn);
      if (zero) tm += __builtin_amdgcn_readlane(o, l);
      return what;
    }
    run += __builtin_amdgcn_readlane(incl, 63);
  }
  return 0;
}

// Stores the rows of row tile tm of expert g in n0 .. n0 + TN - 1 as zeros (one chunk per expert).  ESZ = bytes per element;
// TWO = the second output as well.
template <int ESZ, int TM, int TN, bool TWO>
__device__ __forceinline__ void fill_tile(const GemmArgs& p, int g, int tm, int tn) {
  constexpr int CPR = TN * ESZ / 16;       // 16-byte pieces per row
  const int col = tn * TN + (threadIdx.x % CPR) * (16 / ESZ);
  if (col >= p.Ndim) return;
  const u32x4_t z = {0u, 0u, 0u, 0u};
  const int step = blockDim.x / CPR, end = min((tm + 1) * TM, p.Cc);
  for (int r = tm * TM + threadIdx.x / CPR; r < end; r += step) {
    const int64_t at = ((int64_t)g * p.Cc + r) * p.ldc + col;
    *reinterpret_cast<u32x4_t*>(reinterpret_cast<char*>(p.C) + at * ESZ) = z;
    if (TWO) *reinterpret_cast<u32x4_t*>(reinterpret_cast<char*>(p.C2) + at * ESZ) = z;
  }
}

// Stores share `at` of `shares` of the padding rows of all chunks as zeros: a chunk's padding is one run of memory up to its
// end.
template <int ESZ, bool TWO>
__device__ __forceinline__ void fill_shares(const GemmArgs& p, int at, int shares) {
  const int lane = threadIdx.x & 63, chunks = p.n_src * p.G;     // n_src G Cc < 2^31 (checked on the host)
  const int row_units = (int)(p.ldc * ESZ / 16);                 // 16-byte pieces per row
  auto padding = [&](int c) { return c < chunks ? p.Cc - clamp_count(p.cnt[c], p.Cc) : 0; };
  int rows = 0;
  for (int c0 = 0; c0 < chunks; c0 += 64) rows += padding(c0 + lane);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) rows += __shfl_xor(rows, d, 64);
  rows = __builtin_amdgcn_readfirstlane(rows);
  const int per = (int)(((unsigned)rows + shares - 1) / (unsigned)shares);
  const int r0 = min((int64_t)per * at, (int64_t)rows), r1 = min(r0 + (int64_t)per, (int64_t)rows);
  int run = 0;                                                   // padding rows in front of c0
  for (int c0 = 0; c0 < chunks && run < r1; c0 += 64) {
    const int n = padding(c0 + lane);
    int incl = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(incl, d, 64);
      if (lane >= d) incl += v;
    }
    const int first = run + incl - n;
    unsigned long long hit = __ballot(n > 0 && first < r1 && first + n > r0);
    while (hit) {
      const int l = __ffsll((long long)hit) - 1;
      hit &= hit - 1;
      const int nl = __builtin_amdgcn_readlane(n, l), f = __builtin_amdgcn_readlane(first, l);
      const int lo = max(r0 - f, 0), hi = min(r1 - f, nl);
      const int64_t base = ((int64_t)(c0 + l + 1) * p.Cc - nl + lo) * row_units, units = (int64_t)(hi - lo) * row_units;
      const u32x4_t z = {0u, 0u, 0u, 0u};
      u32x4_t* c = reinterpret_cast<u32x4_t*>(p.C) + base;
      u32x4_t* c2 = reinterpret_cast<u32x4_t*>(TWO ? p.C2 : p.C) + base;
#pragma unroll 4
      for (int64_t u = threadIdx.x; u < units; u += blockDim.x) {
        __builtin_nontemporal_store(z, c + u);
        if (TWO) __builtin_nontemporal_store(z, c2 + u);
      }
    }
    run += __builtin_amdgcn_readlane(incl, 63);
  }
}

// Compacted row order of an expert that receives several chunks with row counts: its occupied rows, chunk by chunk.  Finds
// the physical rows of N positions in [m0, m0 + span); occ = there is one.  A span touches few of the chunks.
template <int N>
__device__ __forceinline__ void compact_rows(const GemmArgs& p, int g, int m0, int span, const int (&r)[N], int (&row)[N],
                                             bool (&occ)[N]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int n = 0; n < N; ++n) { row[n] = 0; occ[n] = false; }
  int run = 0;   // positions of the chunks before s0
  for (int s0 = 0; s0 < p.n_src && run < m0 + span; s0 += 64) {
    const int c = s0 + lane < p.n_src ? clamp_count(p.cnt[(s0 + lane) * p.G + g], p.Cc) : 0;
    int incl = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int v = __shfl_up(incl, d, 64);
      if (lane >= d) incl += v;
    }
    unsigned long long hit = __ballot(c > 0 && run + incl > m0 && run + incl - c < m0 + span);
    while (hit) {
      const int l = __ffsll((long long)hit) - 1;
      hit &= hit - 1;
      const int cl = __builtin_amdgcn_readlane(c, l), first = run + __builtin_amdgcn_readlane(incl, l) - cl;
      const int base = ((s0 + l) * p.G + g) * p.Cc;
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const int d = r[n] - first;
        if ((uint32_t)d < (uint32_t)cl) { row[n] = base + d; occ[n] = true; }
      }
    }
    run += __builtin_amdgcn_readlane(incl, 63);
  }
}

struct KTile {
  int row0, lim;   // first row of the k tile in the operand (row-tiled GEMMs: first k), rows (k values) that exist
};
// The reduction of a weight gradient runs over the expert's rows chunk by chunk, up to each chunk's row count; empty
// chunks are passed over.  With few chunks a k tile never crosses a chunk, so that its grouping is the same with and without
// row counts; with PACK_CHUNKS of them or more (half a k tile lost in each) the rows are packed: a k tile is made of
// pieces of several chunks.  32 chunks of 110 rows on average, 8 experts x 2048 x 2048, merged backward launch: 991 -> 851 us,
// a part of it from the padding; 4 chunks of 180 rows: 41.9 -> 39.1 us.  Two or three chunks would gain 0 to 5 % (backward
// call, 8 experts x 1024 x 2048, 60 % full: 3 chunks of 100 rows 63.1 -> 60.1 us, 3 of 200 83.8 -> 81.1, 2 of 700 151.5 ->
// 150.9); they stay whole for the same bits with and without counts.
constexpr int PACK_CHUNKS = 4;
// Of a reduction cut into parts, whole k tiles of one chunk are dealt to the parts in turn, by their index in the capacity: the
// parts are equally long whatever the counts, and the sums are grouped the same with and without them (PARTS).  Packed k
// tiles, which only exist with counts, are cut into consecutive runs (skip).
template <bool PARTS = false>
struct ChunkWalk {
  const GemmArgs& p;
  int g, part, cnt = 0, s0 = 0, row = 0, left = 0;   // cnt: rows of chunk s0 + lane
  unsigned long long mask = 0;
  __device__ __forceinline__ ChunkWalk(const GemmArgs& p_, int g_, int part_ = 0) : p(p_), g(g_), part(part_) {}
  __device__ __forceinline__ void load() {     // counts of chunks s0 .. s0 + 63, one per lane
    const int s = s0 + (threadIdx.x & 63);
    cnt = s < p.n_src ? (p.cnt != nullptr ? clamp_count(p.cnt[s * p.G + g], p.Cc) : p.Cc) : 0;
    mask = __ballot(cnt > 0);
  }
  __device__ __forceinline__ int first_tile(int s, int step) const {   // of this part in chunk s
    const int at = (part - s * ((p.Cc + step - 1) / step)) % p.splits;
    return at < 0 ? at + p.splits : at;
  }
  __device__ __forceinline__ int start(int step, bool packed) {   // returns the number of k tiles
    int nk = 0;
    for (s0 = 0; s0 < p.n_src; s0 += 64) {
      load();
      int n = packed ? cnt : (cnt + step - 1) / step;
      if (PARTS) {
        const int at = first_tile(s0 + (threadIdx.x & 63), step);
        n = n > at ? (n - at - 1) / p.splits + 1 : 0;
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) n += __shfl_xor(n, d, 64);
      nk += __builtin_amdgcn_readfirstlane(n);
    }
    s0 = 0;
    if (p.n_src > 64) load();
    return packed ? (nk + step - 1) / step : nk;
  }
  __device__ __forceinline__ void skip(int n) {   // passes over the first n rows
    while (n > 0) {
      if (mask == 0) { if (s0 + 64 >= p.n_src) return; s0 += 64; load(); continue; }
      const int l = __ffsll((long long)mask) - 1, c = __builtin_amdgcn_readlane(cnt, l);
      mask &= mask - 1;
      if (c > n) {
        left = c - n;
        row = ((s0 + l) * p.G + g) * p.Cc + n;
      }
      n -= c;
    }
  }
  __device__ __forceinline__ bool enter(int step) {   // the next chunk that has rows; false: past the end
    if (__builtin_expect(mask == 0, 0)) {              // (out of the k loop's way)
      while (mask == 0 && s0 + 64 < p.n_src) { s0 += 64; load(); }
      if (mask == 0) return false;
    }
    const int l = __ffsll((long long)mask) - 1, at = PARTS ? first_tile(s0 + l, step) * step : 0;
    mask &= mask - 1;
    left = __builtin_amdgcn_readlane(cnt, l) - at;
    row = ((s0 + l) * p.G + g) * p.Cc + at;
    return true;
  }
  __device__ __forceinline__ KTile next(int step) {   // the next rows of one chunk, at most `step`; past the end: no rows
    if constexpr (PARTS) {                             // (a chunk may have no k tile of this part)
      while (left <= 0) { if (!enter(step)) return KTile{0, 0}; }
    } else {
      if (left <= 0 && !enter(step)) return KTile{0, 0};
    }
    const KTile t{row, min(left, step)};
    const int on = PARTS ? step * p.splits : step;
    row += on;
    left -= on;
    return t;
  }
};

// The fragment reads of a tile's k loop.  A row's A fragment is replaced by the next step's once the row has been
// multiplied, the B fragments, which every row uses, have two register sets.  The next step's reads are taken in
// the order B0 A0 B1 A1 ... and spread between the MFMAs (place: behind which MFMA of the step), so that
// they do not queue up in front of the multiplications.  A row waits for its own fragments by count: the LDS reads of a
// wave return in order.
template <int KIND, typename CF>
struct Reads {
  static constexpr int MB = CF::MB, NB = CF::NB, N = MB + NB;
  static constexpr int BR = MB > 4 ? 2 : 1;          // rows of a k tile's last step in front of the barrier
  static_assert(MB >= NB, "the order of the reads");
  static constexpr bool is_b(int op) { return op < 2 * NB && op % 2 == 0; }
  static constexpr int of(int op) { return op < 2 * NB ? op / 2 : op - NB; }     // which fragment
  static constexpr int ins(int op) { return (is_b(op) ? KIND != KIND_NT : KIND == KIND_TN) ? 2 : 1; }   // LDS instructions
  static constexpr int place(int st, int op) {
    if (st == CF::SPT - 1) return BR * NB - 1 + op * (MB * NB - BR * NB) / (N - 1);   // behind the barrier
    return is_b(op) ? of(op) * NB + NB / 2 : of(op) + 1 < MB ? (of(op) + 1) * NB : MB * NB - 1;
  }
  static constexpr bool in_place() {                 // no A fragment is replaced before its row has been multiplied
    for (int op = 0; op < N; ++op)
      if (!is_b(op) && (place(0, op) < of(op) * NB + NB - 1 || place(CF::SPT - 1, op) < of(op) * NB + NB - 1)) return false;
    return true;
  }
  static_assert(in_place(), "the order of the reads");
  // LDS instructions that may still be in flight when row `row` of step st is about to be multiplied
  static constexpr int newer(int st, int row) {
    int n = 0;
    const int need = row == 0 ? (NB > 1 ? 2 * NB - 2 : 1) : row < NB ? 2 * row + 1 : row + NB;   // row 0: every B fragment
    for (int op = need + 1; op < N; ++op) n += ins(op);
    for (int op = 0; op < N; ++op) n += place(st, op) < row * NB ? ins(op) : 0;
    return n < 15 ? n : 15;
  }
};

// How a weight-gradient GEMM finds its k-rows.  GATHER: the k-slow A operand (X^T dZ) is the token matrix read through the
// inverse slot map (row r of the chunk is token gather[g C + r] / gather_k); n_src = 1.  PACKED: k tiles of pieces of
// several chunks (ChunkWalk).
enum { ROWS_PLAIN = 0, ROWS_GATHER = 1, ROWS_PACKED = 2 };
template <int KIND, int EPI, typename CF, int ROWS = ROWS_PLAIN>
__device__ __forceinline__ void gemm_dma_tile(const GemmArgs& p, char* smem, int vb) {
  constexpr bool GATHER = ROWS == ROWS_GATHER, PIECES = ROWS == ROWS_PACKED;
  constexpr bool A_NC = (KIND == KIND_TN);                     // A has k as the slow index
  constexpr bool B_NC = (KIND == KIND_NN || KIND == KIND_TN);  // B has k as the slow index
  constexpr int TM = CF::TM, TN = CF::TN, WM = CF::WM, WN = CF::WN, WK = CF::WK, SA = CF::SA, SB = CF::SB;
  constexpr int MB = CF::MB, NB = CF::NB, RA = CF::RA, RB = CF::RB, SPT = CF::SPT, MR = CF::MR, KS = CF::KS;
  constexpr int WTM = TM / WM, WTN = TN / WN;   // wave tile
  static_assert(!A_NC || TM == 64 || TM == 128 || TM == 256, "k-slow tiles are a power of two wide");
  static_assert(ROWS == ROWS_PLAIN || KIND == KIND_TN, "rows of a reduction");
  static_assert(!GATHER || (KIND == KIND_TN && CF::NW == 8), "row gather in the reduction: eight k-rows per wave");

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps LDS bases in SGPRs
  const int wk = WK == 1 ? 0 : wave / (WM * WN);
  const int wm = (wave / WN) % WM, wn = wave % WN;

  int g, tm, tn;
  const bool counted = KIND != KIND_TN && p.cnt != nullptr;
  int part = 0;   // EPI_PART: which part of the reduction; the parts of a tile are total_tiles apart
  if (EPI == EPI_PART) {
    const int per = (p.total_tiles + 7) / 8 * 8;
    part = vb / per;
    vb -= part * per;
  }
  const int what = map_tile<TM, EPI != EPI_DGELU>(p, vb, counted, g, tm, tn);   // (dZ of a padding row is never read)
  if (what == 0) return;
  if (KIND != KIND_TN && __builtin_expect(what == 2, 0))
    return p.n_src == 1 ? fill_tile<2, TM, TN, EPI == EPI_GELU>(p, g, tm, tn) : fill_shares<2, EPI == EPI_GELU>(p, g, tm);
  const int m0 = tm * TM, n0 = tn * TN;
  const bool compact = counted && p.n_src > 1;

  const int64_t b_base = (int64_t)g * p.b_goff + p.b_off;
  const __amdgpu_buffer_rsrc_t rA = make_rsrc(p.A, (uint32_t)p.a_bytes);
  const uint64_t b_rem = p.b_bytes - (uint64_t)b_base * 2;
  const __amdgpu_buffer_rsrc_t rB =
      (KIND == KIND_TN) ? make_rsrc(p.B, (uint32_t)p.b_bytes)
                        : make_rsrc(reinterpret_cast<const bf16_t*>(p.B) + b_base, b_rem > OOB ? OOB : (uint32_t)b_rem);

  // physical rows of the requests' A rows (row-tiled GEMMs) and of rows lane, lane + 64 of the wave tile
  int q_row[RA];
  uint32_t out_off[2] = {OOB, OOB};   // byte offset of the row in the output (+ 1: a row of zeros), or OOB
  if (KIND != KIND_TN) {
    int r[RA + 2], row[RA + 2];
    bool occ[RA + 2], here[2];   // there is a row to multiply; there is a row to store (zeros if not occ)
#pragma unroll
    for (int j = 0; j < RA; ++j) r[j] = m0 + (wave * RA + j) * 8 + (lane >> 3);
#pragma unroll
    for (int j = 0; j < 2; ++j) r[RA + j] = m0 + wm * WTM + 64 * j + lane;
    if (compact) {
      compact_rows<RA + 2>(p, g, m0, TM, r, row, occ);
#pragma unroll
      for (int j = 0; j < 2; ++j) here[j] = occ[RA + j];
    } else {
      const int cnt_g = counted ? clamp_count(p.cnt[g], p.Cc) : p.Mdim;
#pragma unroll
      for (int j = 0; j < RA + 2; ++j) {
        occ[j] = r[j] < cnt_g;
        if (j >= RA) here[j - RA] = r[j] < p.Mdim;
        row[j] = p.n_src == 1 ? g * p.Cc + r[j] : (int)phys_row(min(r[j], p.Mdim - 1), g, p.G, p.Cc);
      }
      if (p.gather != nullptr) {   // rows are the tokens that the slots hold; an empty slot is a row of zeros
        int iv[RA + 2];
#pragma unroll
        for (int j = 0; j < RA + 2; ++j) iv[j] = p.gather[(int64_t)g * p.Cc + min(r[j], p.Mdim - 1)];
#pragma unroll
        for (int j = 0; j < RA + 2; ++j) {
          const uint32_t tok = p.gather_k == 1 ? (uint32_t)iv[j] : __umulhi((uint32_t)iv[j], p.gather_magic);
          occ[j] = occ[j] && iv[j] >= 0 && (int64_t)tok < p.gather_rows;
          if (j < RA) row[j] = (int)tok;
        }
      }
    }
#pragma unroll
    for (int j = 0; j < RA; ++j) q_row[j] = occ[j] ? row[j] : 0;   // no row: any row of the tensor
#pragma unroll
    for (int j = 0; j < 2; ++j)
      if (here[j]) out_off[j] = (uint32_t)row[RA + j] * (uint32_t)p.ldc * 2u + (occ[RA + j] ? 0u : 1u);
  }
  // 32 x 32 pieces a wave finishes (WK = 2: MR = 32, a piece is an MFMA block)
  constexpr int EMB = (WK == 2 && MB >= 2) ? MB / 2 : WTM / 32;
  constexpr int ENB = (WK == 2 && MB < 2 && NB >= 2) ? NB / 2 : WTN / 32;
  constexpr bool ONE = WK == 2 && MB < 2 && NB < 2;            // a single block: the second group's waves finish nothing
  const int e_i = (WK == 2 && MB >= 2) ? wk * EMB : 0, e_j = (WK == 2 && MB < 2 && NB >= 2) ? wk * ENB : 0;
  const int e_n = n0 + wn * WTN + 32 * e_j;
  char* e_lds = smem + wave * (CF::LDS / CF::NW / 64 * 64);

  // ---- k tiles: Kdim / 64 of a row-tiled GEMM, the walk over the expert's chunks for a weight gradient ----
  ChunkWalk<EPI == EPI_PART && !PIECES> walk(p, g, part);
  int nk = KIND == KIND_TN ? walk.start(DK, PIECES) : (p.Kdim + DK - 1) / DK;
  int k_left = nk;               // packed parts: k tiles that the walk has not been asked for
  if (EPI == EPI_PART && PIECES) {
    const int t0 = (int)((int64_t)nk * part / p.splits), t1 = (int)((int64_t)nk * (part + 1) / p.splits);
    walk.skip(t0 * DK);
    k_left = nk = t1 - t0;
  }

  // ---- per-lane request coordinates: byte offset of the lane's row / column, the k index within the tile that the
  // request covers (k-slow) or starts at (k-contiguous), and the byte offset of that k index ----
  uint32_t a_req[RA], b_req[RB], a_ko[RA], b_ko[RB];
  int a_k[RA], b_k[RB];
  constexpr int ACPR = TM / 8, BCPR = TN / 8;   // k-slow: 16-byte chunks per k-row
  const uint32_t lda2 = (uint32_t)p.lda * 2u, ldb2 = (uint32_t)p.ldb * 2u;
  auto swz_nc = [](int k, int cpr) {
    return cpr >= 16 ? 4 * (k & 3) + (MR == 16 ? 2 * ((k >> 3) & 1) : 0) : 4 * ((k >> 1) & 1);
  };
#pragma unroll
  for (int j = 0; j < RA; ++j) {
    const int q = wave * RA + j;
    if (!A_NC) {
      a_k[j] = ((lane & 7) ^ ((4 * q + (lane >> 4)) & 7)) * 8;
      a_req[j] = (uint32_t)q_row[j] * lda2;
      a_ko[j] = (uint32_t)a_k[j] * 2u;
    } else {
      a_k[j] = q * (64 / ACPR) + lane / ACPR;
      const int col = m0 + (((lane % ACPR) ^ swz_nc(a_k[j], ACPR)) * 8);
      a_req[j] = (uint32_t)(col < p.Mdim ? col : m0) * 2u;
      a_ko[j] = GATHER ? 0u : (uint32_t)a_k[j] * lda2;
    }
  }
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    const int q = wave * RB + j;
    if (!B_NC) {
      b_k[j] = ((lane & 7) ^ ((4 * q + (lane >> 4)) & 7)) * 8;
      b_req[j] = (uint32_t)min(n0 + q * 8 + (lane >> 3), p.Ndim - 1) * ldb2;
      b_ko[j] = (uint32_t)b_k[j] * 2u;
    } else {
      b_k[j] = q * (64 / BCPR) + lane / BCPR;
      const int col = n0 + (((lane % BCPR) ^ swz_nc(b_k[j], BCPR)) * 8);
      b_req[j] = (uint32_t)(col < p.Ndim ? col : n0) * 2u;
      b_ko[j] = (uint32_t)b_k[j] * ldb2;
    }
  }

  // GATHER: the k-rows of a k tile are token rows.  Lane l loads the slot-map entry of k-row l, one request set ahead of
  // the A requests that use it and before that set's own requests: the wait for tile t+1 at the next barrier then covers
  // the entries as well, and nothing waits for them by itself.  The eight rows a wave requests are the same for all
  // its lanes.  An empty slot is fetched as token 0 and masked.
  uint32_t g_now[RA];   // byte offset of the token row behind this lane's k-row of the next A request
  const __amdgpu_buffer_rsrc_t rG = make_rsrc(p.gather, GATHER ? (uint32_t)((int64_t)p.G * p.Cc * 4) : 0u);
  auto gather_fetch = [&](int row0) -> int {   // entries past the map read as zero; rows past the row count are masked
    return (int)__builtin_amdgcn_raw_buffer_load_b32(rG, (row0 + lane) * 4, 0, 0);
  };
  auto gather_rows = [&](int entry) -> uint64_t {   // returns which of the 64 slots are occupied
    constexpr int RPR = A_NC ? 64 / ACPR : 1;   // k-rows per request
    const uint32_t tok = p.gather_k == 1 ? (uint32_t)entry : __umulhi((uint32_t)entry, p.gather_magic);
    const bool full = entry >= 0 && (int64_t)tok < p.gather_rows;
    const uint32_t off = full ? tok * (uint32_t)(p.lda * 2) : 0u;
#pragma unroll
    for (int j = 0; j < RA; ++j) {
      uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)off, (wave * RA + j) * RPR);
#pragma unroll
      for (int u = 1; u < RPR; ++u) {
        const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)off, (wave * RA + j) * RPR + u);
        o = lane / ACPR == u ? v : o;
      }
      g_now[j] = o;
    }
    return __ballot(full);
  };
  // PIECES: byte offsets of this lane's k-rows in the newest k tile (A's next requests) and the one before it (B's)
  uint32_t ka_off[PIECES ? RA : 1], kb_off[PIECES ? RB : 1], kb_new[PIECES ? RB : 1];
  static_assert(!PIECES || SA == SB + 1, "B's requests are a k tile behind A's");
  auto next_ktile = [&]() -> KTile {
    KTile t{0, 0};                                   // past the end: no rows
    if (EPI != EPI_PART || !PIECES || k_left-- > 0) t = walk.next(DK);
    if constexpr (PIECES) {
#pragma unroll
      for (int j = 0; j < RB; ++j) { kb_off[j] = kb_new[j]; kb_new[j] = (uint32_t)t.row0 * ldb2 + b_ko[j]; }
#pragma unroll
      for (int j = 0; j < RA; ++j) ka_off[j] = (uint32_t)t.row0 * lda2 + a_ko[j];
      {
        while (t.lim > 0 && t.lim < DK) {
          const KTile piece = walk.next(DK - t.lim);
          if (piece.lim == 0) break;
          const uint32_t d = (uint32_t)(piece.row0 - t.lim);
#pragma unroll
          for (int j = 0; j < RA; ++j) ka_off[j] = a_k[j] >= t.lim ? d * lda2 + a_ko[j] : ka_off[j];
#pragma unroll
          for (int j = 0; j < RB; ++j) kb_new[j] = b_k[j] >= t.lim ? d * ldb2 + b_ko[j] : kb_new[j];
          t.lim += piece.lim;
        }
      }
      if (t.lim < DK) {   // missing k rows are fetched from the tile's first one
#pragma unroll
        for (int j = 0; j < RA; ++j) ka_off[j] = a_k[j] < t.lim ? ka_off[j] : (uint32_t)t.row0 * lda2;
#pragma unroll
        for (int j = 0; j < RB; ++j) kb_new[j] = b_k[j] < t.lim ? kb_new[j] : (uint32_t)t.row0 * ldb2;
      }
    }
    return t;
  };
  // One request (1 KiB) of k tile kt into ring slot `slot`.
  auto request_a = [&](const KTile& kt, int slot, int j) {
    const uint32_t in = a_k[j] < kt.lim ? a_ko[j] : 0u;   // missing k rows are fetched from the tile's first one
    const uint32_t add = GATHER ? g_now[j] : PIECES ? ka_off[PIECES ? j : 0] : (uint32_t)kt.row0 * (A_NC ? lda2 : 2u) + in;
    dma16(rA, smem + slot * CF::A_UNIT + (wave * RA + j) * 1024, a_req[j] + add);
  };
  auto request_b = [&](const KTile& kt, int slot, int j) {
    const uint32_t in = b_k[j] < kt.lim ? b_ko[j] : 0u;
    const uint32_t add = PIECES ? kb_off[PIECES ? j : 0] : (B_NC ? (uint32_t)kt.row0 * ldb2 : (uint32_t)kt.row0 * 2u) + in;
    dma16(rB, smem + SA * CF::A_UNIT + slot * CF::B_UNIT + (wave * RB + j) * 1024, b_req[j] + add);
  };
  auto ktile_at = [&](int t) -> KTile { return KTile{t * DK, p.Kdim - t * DK}; };   // row-tiled GEMMs

  // ---- per-lane fragment addresses (bytes); see the layout above ----
  const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_AS char*)smem;
  uint32_t a_fr[A_NC ? MB : 1], b_fr[B_NC ? NB : 1];
  {
    const int b = lane >> 4, s = lane & 15;
    const int chunk = ((wk * SPT * (KS / 8) + lane / MR) ^ ((lane >> 1) & 7)) * 16;
    const int oct = MR == 32 ? b >> 1 : b, half = MR == 32 ? 16 * (b & 1) : 0;   // k-slow: the 16-lane group's patch
    const int knc = KS * wk * SPT + 8 * oct + (s >> 2);
    if (!A_NC) {
      a_fr[0] = lds0 + (wm * WTM + (lane & (MR - 1))) * 128 + chunk;
    } else {
#pragma unroll
      for (int i = 0; i < (A_NC ? MB : 1); ++i) {
        const int col = wm * WTM + MR * i + half + 4 * (s & 3);
        a_fr[i] = lds0 + knc * (2 * TM) + (((col >> 3) ^ swz_nc(knc, ACPR)) * 16) + ((s & 1) * 8);
      }
    }
    if (!B_NC) {
      b_fr[0] = lds0 + SA * CF::A_UNIT + (wn * WTN + (lane & (MR - 1))) * 128 + chunk;
    } else {
#pragma unroll
      for (int j = 0; j < (B_NC ? NB : 1); ++j) {
        const int col = wn * WTN + MR * j + half + 4 * (s & 3);
        b_fr[j] = lds0 + SA * CF::A_UNIT + knc * (2 * TN) + (((col >> 3) ^ swz_nc(knc, BCPR)) * 16) + ((s & 1) * 8);
      }
    }
  }
  // a row's A fragment is replaced by the next step's once the row has been multiplied; B has two register sets
  Frag fa[MB], fb[2][NB];
  using RD = Reads<KIND, CF>;
  constexpr int BR = RD::BR;
  auto read_op = [&](int slot_a, int slot_b, auto st_tag, auto op_tag) {   // read `op` of step ST
    constexpr int ST = decltype(st_tag)::value, OP = decltype(op_tag)::value, I = RD::of(OP);
    if constexpr (RD::is_b(OP)) {
      const uint32_t so = (uint32_t)slot_b * CF::B_UNIT;
      if constexpr (!B_NC) lds_read_kc<I * MR * 128>(fb[ST & 1][I], (b_fr[0] + so) ^ (2u * KS * ST));
      else lds_read_nc<ST * KS * 2 * TN, 8 * TN>(fb[ST & 1][I], b_fr[B_NC ? I : 0] + so);
    } else {
      const uint32_t so = (uint32_t)slot_a * CF::A_UNIT;
      if constexpr (!A_NC) lds_read_kc<I * MR * 128>(fa[I], (a_fr[0] + so) ^ (2u * KS * ST));
      else lds_read_nc<ST * KS * 2 * TM, 8 * TM>(fa[I], a_fr[A_NC ? I : 0] + so);
    }
  };
  auto frags_ready = [&](int set) {
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
#pragma unroll
    for (int i = 0; i < MB; ++i) ready(fa[i]);
#pragma unroll
    for (int j = 0; j < NB; ++j) ready(fb[set][j]);
  };

  typename AccBlock<MR>::type acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < MR * MR / 64; ++q) acc[i][j][q] = 0.f;

  // Refill set t (issued after the barrier of tile t): tile t+SB of B, then tile t+SA of A.  kb, ka: its tiles.
  constexpr int NREQ = RA + RB;
  // The requests of a set are spread evenly over the MFMAs up to the next barrier: issued together they stall the waves (all
  // behind the barrier, 128 x 128 tiles over 860 k tiles: 604 -> 724 us; two at a time, the merged launch of 256 x 256
  // tiles: 17.1 -> 18.1 ms).
  constexpr int SL_LAST = (MB - BR) * NB + 1, SL = SL_LAST + (SPT - 1) * MB * NB;   // slots: in the last step, in all
  constexpr auto slot_of = [](int r) constexpr { return r * SL / NREQ; };
  constexpr auto before = [](int slot) constexpr {
    int n = 0;
    for (int r = 0; r < NREQ; ++r) n += r * SL / NREQ < slot;
    return n;
  };
  constexpr int N_LAST = before(SL_LAST);                            // requests issued in the last step
  // newer requests than those of tile t+1, at barrier t
  constexpr int IN_FLIGHT = (SA > SB ? RA : 0) + (SB - 2) * (NREQ + (GATHER ? 1 : 0));
  KTile ka{0, 0}, kb{0, 0};
  int g_entry = 0;        // GATHER: slot-map entries of g_next, the tile after ka
  KTile g_next{0, 0};
  uint64_t k_mask[SA];    // TN: which k-rows of tiles t .. t + SA - 1 exist (GATHER: and are occupied)
  int k_lim[SA];          // GATHER: their numbers of rows
  auto mask_of = [&](const KTile& kt, uint64_t full) -> uint64_t {
    return kt.lim >= DK ? full : kt.lim <= 0 ? 0ull : full & ((1ull << kt.lim) - 1ull);
  };
  // prologue: the refills that would have gone before the first tile, and the last-step part of set -1
  {
    KTile pro[SA];
#pragma unroll
    for (int t = 0; t < SA; ++t)
      if (!PIECES) pro[t] = KIND == KIND_TN ? next_ktile() : ktile_at(t);
    int g_pro[SA];
    if (GATHER) {
#pragma unroll
      for (int t = 0; t < SA; ++t) g_pro[t] = gather_fetch(pro[t].row0);
      g_next = next_ktile();
      g_entry = gather_fetch(g_next.row0);
    }
    auto pro_a = [&](int t) {
      const uint64_t full = GATHER ? gather_rows(g_pro[t]) : ~0ull;
      k_mask[t] = mask_of(pro[t], full);
      k_lim[t] = pro[t].lim;
    };
#pragma unroll
    for (int st = -SA; st <= -2; ++st) {
      if (PIECES) pro[st + SA] = next_ktile();
      if (st + SB >= 0) {
#pragma unroll
        for (int j = 0; j < RB; ++j)
          if (pro[st + SB].lim > 0) request_b(pro[st + SB], st + SB, j);
      }
      pro_a(st + SA);
#pragma unroll
      for (int j = 0; j < RA; ++j)
        if (pro[st + SA].lim > 0) request_a(pro[st + SA], st + SA, j);
    }
    if (PIECES) pro[SA - 1] = next_ktile();
    ka = pro[SA - 1];
    kb = pro[SB - 1];
    pro_a(SA - 1);
    unrolled<0, N_LAST>([&](auto r) {
      constexpr int R = decltype(r)::value;
      if constexpr (R < RB) { if (kb.lim > 0) request_b(kb, SB - 1, R); }
      else { if (ka.lim > 0) request_a(ka, SA - 1, R - RB); }
    });
    // this wave's requests for tile 0 have landed
    if (nk >= SA) __builtin_amdgcn_s_waitcnt(vmcnt_imm(IN_FLIGHT + N_LAST));
    else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __builtin_amdgcn_s_barrier();
  }
  using K0 = std::integral_constant<int, 0>;
  unrolled<0, RD::N>([&](auto op) { read_op(0, 0, K0{}, op); });

  auto mfma = [&](int set, int i, int j) {
    if constexpr (MR == 32) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[set][j].v, fa[i].v, acc[i][j], 0, 0, 0);
    else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[set][j].v, fa[i].v, acc[i][j], 0, 0, 0);
  };
  int sa = 0, sb = 0;                 // ring slots of the current tile
  int wa = SA - 1, wb = SB - 1;       // ring slots that the refill set in progress goes to
  auto issue = [&](auto slot_tag, auto last_tag) {    // the requests of a slot; LAST: the tile may be past the end
    constexpr bool LAST = decltype(last_tag)::value;
    unrolled<0, NREQ>([&](auto r) {
      constexpr int R = decltype(r)::value;
      if constexpr (slot_of(R) == decltype(slot_tag)::value) {
        if constexpr (R < RB) { if (!LAST || kb.lim > 0) request_b(kb, wb, R); }
        else { if (!LAST || ka.lim > 0) request_a(ka, wa, R - RB); }
      }
    });
  };
  // zeroes the k-rows of set `set` (step ST of a tile) that do not exist, in both operands: what was fetched in their
  // place may be an infinity.  (GATHER: an empty slot is a row of zeros in A only, as in the dispatched buffer.)
  auto mask_frags = [&](uint64_t mask_a, uint64_t mask_b, auto st_tag) {
    constexpr int ST = decltype(st_tag)::value;
    auto lanes = [&](uint64_t mask) {
      const uint32_t bits = (uint32_t)(mask >> (KS * (wk * SPT + ST))) >> (8 * (lane / MR));
      u32x4_t m;
      if (KIND != KIND_TN) {   // K % 8 == 0: a lane's 8 values exist together
        const uint32_t all = (bits & 1u) ? ~0u : 0u;
        m = u32x4_t{all, all, all, all};
        return m;
      }
#pragma unroll
      for (int d = 0; d < 4; ++d) m[d] = ((bits >> (2 * d)) & 1u) * 0x0000FFFFu + ((bits >> (2 * d + 1)) & 1u) * 0xFFFF0000u;
      return m;
    };
    const u32x4_t ma = lanes(mask_a), mb = GATHER ? lanes(mask_b) : ma;
#pragma unroll
    for (int i = 0; i < MB; ++i) fa[i].q &= ma;
#pragma unroll
    for (int j = 0; j < NB; ++j) fb[ST & 1][j].q &= mb;
  };
  // one k tile; LAST: one of the last SA tiles, whose refills may be past the end
  auto k_tile = [&](int t, auto last_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    const int na = sa + 1 == SA ? 0 : sa + 1, nb = sb + 1 == SB ? 0 : sb + 1;   // slots of tile t+1
    const uint64_t mask = KIND == KIND_TN ? k_mask[0] : LAST ? mask_of(ktile_at(t), ~0ull) : ~0ull;
    const uint64_t mask_b = GATHER ? mask_of(KTile{0, k_lim[0]}, ~0ull) : mask;
    unrolled<0, SPT>([&](auto st) {
      constexpr int ST = decltype(st)::value;
      using NEXT = std::integral_constant<int, (ST + 1) % SPT>;
      // row 0 needs its own A fragment and all B fragments; a step with missing k rows waits for everything and masks it
      __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(RD::newer(ST, 0)));
#pragma unroll
      for (int j = 0; j < NB; ++j) ready(fb[ST & 1][j]);
      ready(fa[0]);
      if constexpr (KIND == KIND_TN || LAST) {
        if (__builtin_expect(mask != ~0ull, 0)) {   // (its code stays out of the k loop's way)
          frags_ready(ST & 1);
          mask_frags(mask, mask_b, st);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      unrolled<0, MB>([&](auto i) {
        constexpr int I = decltype(i)::value;
        if constexpr (I > 0) {
          if constexpr (ST < SPT - 1 || I < BR) __builtin_amdgcn_s_waitcnt(lgkmcnt_imm(RD::newer(ST, I)));
          ready(fa[I]);
        }
        unrolled<0, NB>([&](auto j) {
          constexpr int J = decltype(j)::value, AT = I * NB + J;
          __builtin_amdgcn_sched_barrier(0);
          mfma(ST & 1, I, J);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (ST == SPT - 1 && AT == BR * NB - 1) {
            // this wave's requests for tile t+1 have landed; so have its reads of tile t
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(LAST ? 0 : IN_FLIGHT) & 0xF0FF);
            __builtin_amdgcn_s_barrier();                        // everyone is done with tile t, and tile t+1 is complete
            __builtin_amdgcn_sched_barrier(0);
            wa = sa; wb = sb;
            if (KIND == KIND_TN) {
              const KTile nx = GATHER ? g_next : next_ktile();
              if constexpr (SA > SB) kb = ka; else kb = nx;
              ka = nx;
              uint64_t full = ~0ull;
              if (GATHER) {
                full = gather_rows(g_entry);
                g_next = next_ktile();
                g_entry = gather_fetch(g_next.row0);
              }
#pragma unroll
              for (int u = 0; u + 1 < SA; ++u) { k_mask[u] = k_mask[u + 1]; k_lim[u] = k_lim[u + 1]; }
              k_mask[SA - 1] = mask_of(ka, full);
              k_lim[SA - 1] = ka.lim;
            } else {
              ka = ktile_at(t + SA);
              kb = ktile_at(t + SB);
            }
          }
          unrolled<0, RD::N>([&](auto op) {
            if constexpr (RD::place(ST, decltype(op)::value) == AT) {
              if constexpr (ST < SPT - 1) read_op(sa, sb, NEXT{}, op);
              else read_op(na, nb, NEXT{}, op);
            }
          });
          if constexpr (ST < SPT - 1) issue(std::integral_constant<int, SL_LAST + ST * MB * NB + AT>{}, last_tag);
          else if constexpr (AT >= BR * NB - 1) issue(std::integral_constant<int, AT - BR * NB + 1>{}, last_tag);
          __builtin_amdgcn_sched_barrier(0);
        });
      });
    });
    sa = na; sb = nb;
  };
  const int n_main = nk - SA;    // every refill of these tiles exists
  int t = 0;
  for (; t < n_main; ++t) k_tile(t, std::false_type{});
  for (; t < nk; ++t) k_tile(t, std::true_type{});
  // The last tile (or, without k tiles, the prologue) has read a first step that nobody multiplies: its registers stay
  // taken until the reads have landed, or they would overwrite what the compiler puts there.
  frags_ready(0);
  __builtin_amdgcn_s_waitcnt(0x0070);  // every request is done before LDS is reused
  __syncthreads();

  if constexpr (WK == 2) {   // each of the two wave groups finishes half of the blocks: exchange the other halves
    f32x16_t mine[EMB][ENB];
    float4* xch = reinterpret_cast<float4*>(smem) + (size_t)wave * (EMB * ENB * 4 * 64);
    const float4* oth = reinterpret_cast<const float4*>(smem) + (size_t)(wave ^ (WM * WN)) * (EMB * ENB * 4 * 64);
#pragma unroll
    for (int i = 0; i < EMB; ++i)
#pragma unroll
      for (int j = 0; j < ENB; ++j)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          float own[4], snd[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float lo = acc[i][j][q4 * 4 + e];
            const float hi = ONE ? lo : acc[MB >= 2 ? EMB + i : i][MB >= 2 ? j : (ONE ? 0 : ENB) + j][q4 * 4 + e];
            own[e] = wk ? hi : lo;
            snd[e] = wk ? lo : hi;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) mine[i][j][q4 * 4 + e] = own[e];
          xch[((i * ENB + j) * 4 + q4) * 64 + lane] = make_float4(snd[0], snd[1], snd[2], snd[3]);
        }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < EMB; ++i)
#pragma unroll
      for (int j = 0; j < ENB; ++j)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const float4 v = oth[((i * ENB + j) * 4 + q4) * 64 + lane];
          mine[i][j][q4 * 4 + 0] += v.x; mine[i][j][q4 * 4 + 1] += v.y;
          mine[i][j][q4 * 4 + 2] += v.z; mine[i][j][q4 * 4 + 3] += v.w;
        }
    __syncthreads();
    if (ONE && wk != 0) return;
    if constexpr (EPI == EPI_PART) {   // straight from the registers: 4 columns of a row per lane and group
      float* dst = p.part + ((int64_t)part * p.G + g) * p.Mdim * p.Ndim;
#pragma unroll
      for (int i = 0; i < EMB; ++i)
#pragma unroll
        for (int j = 0; j < ENB; ++j)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int m = m0 + wm * WTM + 32 * (e_i + i) + (lane & 31), n = e_n + 32 * j + 8 * q4 + 4 * (lane >> 5);
            if (m < p.Mdim && n < p.Ndim)
              *reinterpret_cast<float4*>(dst + (int64_t)m * p.Ndim + n) =
                  make_float4(mine[i][j][q4 * 4], mine[i][j][q4 * 4 + 1], mine[i][j][q4 * 4 + 2], mine[i][j][q4 * 4 + 3]);
          }
      return;
    }
    store_tile_lds<KIND, EPI, 32, EMB, ENB>(p, mine, e_lds, g, m0 + wm * WTM, 32 * e_i, e_n, out_off, lane);
  } else {
    store_tile_lds<KIND, EPI, MR, EMB, ENB>(p, acc, e_lds, g, m0 + wm * WTM, 0, e_n, out_off, lane);
  }
}

template <int KIND, int EPI, typename CF, int ROWS = ROWS_PLAIN>
__global__ __launch_bounds__(64 * CF::NW) void ffn_gemm_dma(const GemmArgs p) {
  __shared__ __attribute__((aligned(1024))) char smem[CF::LDS];
  gemm_dma_tile<KIND, EPI, CF, ROWS>(p, smem, (int)blockIdx.x);
}

using Tile256 = TileCfg<256, 256, 2, 4, 1, 3, 2>;
// Weight gradients over at most 8 k tiles of rows, k tiles of one chunk.  There the launch is bound by what a tile does
// outside its k loop and by the writes, and the shorter steps of 32x32x16 start and drain faster.  Backward call, 16x16x32 and
// this, in turn: 16 experts of 64 / 256 / 512 x 2048 x 4096 267 / 430 / 582 and 264 / 421 / 578 us; 24 of 200 x 1024 x 2048 133.2
// and 131.1; 2 of 512 x 1024 x 3584 49.5 and 48.7; beyond, 16 of 900 x 1024 x 1024 130.7 and 132.4, 4 of 700 x 2048 x 4096 191.9
// and 194.5.
constexpr int BRIEF_ROWS = 8 * DK;
using Tile256Brief = TileCfg<256, 256, 2, 4, 1, 3, 2, 32>;
using Tile192 = TileCfg<192, 256, 2, 4, 1, 3, 2>;
using Tile128 = TileCfg<128, 128, 2, 2, 2, 3, 2>;
using Tile64x128 = TileCfg<64, 128, 1, 4, 2, 3, 3>;
using Tile64 = TileCfg<64, 64, 1, 2, 2, 5, 5>;
using Tile32x64 = TileCfg<32, 64, 1, 2, 2, 6, 6>;

// The three GEMMs of the backward pass that only depend on dZ, in one launch: dX = dZ W1^T (row-tiled,
// the long tiles, first in the grid) and the two weight gradients.  nbx and nbw are the (multiple-of-8)
// workgroup counts of the first two problems.  EPI: of the weight gradients.
template <typename CFX, typename CFW, int EPI, int ROWS>   // ROWS_GATHER: the third problem only
__global__ __launch_bounds__(512) void ffn_bwd_trio(const GemmArgs px, const GemmArgs pw2, const GemmArgs pw1, int nbx,
                                                    int nbw) {
  static_assert(CFX::NW == 8 && CFW::NW == 8, "one block size");
  __shared__ __attribute__((aligned(1024))) char smem[CFX::LDS > CFW::LDS ? CFX::LDS : CFW::LDS];
  const int b = (int)blockIdx.x;
  if (b < nbx) gemm_dma_tile<KIND_NT, EPI_STORE, CFX>(px, smem, b);
  else if (b < nbx + nbw) gemm_dma_tile<KIND_TN, EPI, CFW, ROWS == ROWS_GATHER ? ROWS_PLAIN : ROWS>(pw2, smem, b - nbx);
  else gemm_dma_tile<KIND_TN, EPI, CFW, ROWS>(pw1, smem, b - nbx - nbw);
}

// Adds the parts of the two split weight gradients in order and stores them in bf16: a thread owns 4 columns of a row.
__global__ __launch_bounds__(256) void ffn_add_parts(const GemmArgs pw2, const GemmArgs pw1, int64_t n2, int64_t n) {
  int64_t u = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (u >= n) return;
  const GemmArgs& p = u < n2 ? pw2 : pw1;
  if (u >= n2) u -= n2;
  const int64_t size = (int64_t)p.G * p.Mdim * p.Ndim, at = u * 4;
  const float* src = p.part + at;
  float4 v = *reinterpret_cast<const float4*>(src);
#pragma unroll 8
  for (int q = 1; q < p.splits; ++q) {
    const float4 w = *reinterpret_cast<const float4*>(src + q * size);
    v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
  }
  const int64_t row = at / p.Ndim, g = row / p.Mdim;
  bf16_t* dst = reinterpret_cast<bf16_t*>(p.C) + g * p.c_goff + p.c_off + (row - g * p.Mdim) * p.ldc + (at - row * p.Ndim);
  *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(v.x, v.y), pack_bf16x2(v.z, v.w));
}

// ------------------------------------------------------------------------------------------
// fp32 kernel: fp64 matrix cores (v_mfma_f64_16x16x4_f64: lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16] and
// receives D[4 r + l / 16][l % 16], r = 0..3), fp64 accumulation.
//
// TM x TN tile, four waves: TM / 16 of them own 16 rows each, with two row waves the other two take the other half of every k
// chunk, and the halves' sums meet in LDS.  k chunks of 32.  Which k a quarter of the lanes feeds in which step is free as
// long as both operands agree: it takes SPL consecutive ones, one a step.  So A needs no LDS: a lane's values are 16-byte pieces
// of its row (weight gradients: single values, 16 lanes to 64 bytes).  B is converted to fp64 once per workgroup on its way into
// LDS ([k][column], pitch TN + 2 doubles: the k rows of a 32-lane read fall into different halves of the banks), in two buffers:
// the next chunk is converted and stored between the current one's products, and the one after it requested.  No fetch
// stands in a branch, so that the compiler can wait for them by count: what does not exist is fetched from somewhere else in the
// tensor and, along k, zeroed.
// Bound by the fp64 matrix rate (77 TFLOP/s measured for the bare instruction) less the vector instructions between, of which
// a conversion costs a tenth of a matrix instruction.  8192 rows x 2048 x 2048, forward and backward call, with both operands staged
// and two barriers per chunk 2.31 and 4.63 ms (59 TFLOP/s) -> 2.06 and 4.07 ms (67); 8 experts of 256 x 512 x 2048 180 and
// 324 -> 158 and 284 us; 8 of 51 x 1024 x 4096 204 and 409 -> 178 and 338; 4 of 62 x 64 x 128 8.5 and 9.9 -> 8.4 and 9.5; but one chunk
// alone is latency and code that is fetched for the first time, 4 of 62 x 32 x 32 6.3 and 8.3 -> 6.6 and 8.5.
// ------------------------------------------------------------------------------------------
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int FK = 32;   // k chunk
template <int TM, int TN>
constexpr int f32_lds() { return 2 * FK * (TN + 2) * 8; }
template <int KIND, int EPI, int TM, int TN, bool WIDE>   // WIDE: leading dimensions that 32-bit offsets do not reach
__device__ __forceinline__ void gemm_f32_tile(const GemmArgs& p, double* Bs, int vb) {
  constexpr bool A_NC = KIND == KIND_TN, B_NC = KIND != KIND_NT;   // k is the slow index in memory
  constexpr int RW = TM / 16, KW = 4 / RW, NJ = TN / 16;            // row waves, k halves, blocks of 16 columns
  constexpr int SPL = 8 / KW;                                       // steps of a wave per chunk
  constexpr int PB = TN + 2, BUF = FK * PB, UB = TN * FK / 4 / 256; // 16-byte pieces of B per thread and chunk
  static_assert(RW * KW == 4 && NJ % KW == 0 && (KW == 1 || RW * 64 * (4 * NJ + 1) <= 2 * BUF), "the halves' sums fit in the buffers");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rw = wave % RW, kw = wave / RW;
  const int kb = kw * (FK / KW) + SPL * (lane >> 4);                // this lane's first k of a chunk
  int g, tm, tn;
  const bool counted = KIND != KIND_TN && p.cnt != nullptr;
  const int what = map_tile<TM, EPI != EPI_DGELU>(p, vb, counted, g, tm, tn);   // (dZ of a padding row is never read)
  if (what == 0) return;
  if (KIND != KIND_TN && __builtin_expect(what == 2, 0))
    return p.n_src == 1 ? fill_tile<4, TM, TN, EPI == EPI_GELU>(p, g, tm, tn) : fill_shares<4, EPI == EPI_GELU>(p, g, tm);
  const int m0 = tm * TM, n0 = tn * TN;
  const float* __restrict__ A = reinterpret_cast<const float*>(p.A);
  const float* __restrict__ B = reinterpret_cast<const float*>(p.B) + (KIND == KIND_TN ? 0 : (int64_t)g * p.b_goff + p.b_off);

  // rows (row-tiled GEMMs): of this lane's A values and, lane l, of output row l of the tile
  int a_row = 0, o_row = 0;
  bool o_zero = false;
  if (KIND != KIND_TN) {
    int r[2] = {m0 + rw * 16 + (lane & 15), m0 + lane}, row[2];
    bool occ[2], here = false;   // there is a row to multiply; there is a row to store (zeros if not occ)
    if (counted && p.n_src > 1) {
      compact_rows<2>(p, g, m0, TM, r, row, occ);
      here = occ[1];
    } else {
      const int cnt_g = counted ? clamp_count(p.cnt[g], p.Cc) : p.Mdim;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        occ[u] = r[u] < cnt_g;
        if (u == 1) here = r[u] < p.Mdim;
        row[u] = (int)phys_row(min(r[u], p.Mdim - 1), g, p.G, p.Cc);
        if (p.gather != nullptr) {
          const int64_t tok = a_src_row(p, min(r[u], p.Mdim - 1), g);
          occ[u] = occ[u] && tok >= 0;
          if (u == 0) row[u] = (int)tok;
        }
      }
    }
    a_row = occ[0] ? row[0] : 0;   // no row: any row, its results are not stored
    o_row = here ? row[1] : -1;
    o_zero = !occ[1];
  }
  ChunkWalk<> walk(p, g);
  const int nk = KIND == KIND_TN ? walk.start(FK, false) : (p.Kdim + FK - 1) / FK;
  auto ktile = [&](int t) -> KTile {      // behind the last one: no k, and row 0
    if (KIND == KIND_TN) return walk.next(FK);
    return t < nk ? KTile{t * FK, p.Kdim - t * FK} : KTile{0, 0};
  };

  // ---- A: this lane's SPL values of a chunk.  Weight gradients: column m of rows kb .. kb + SPL - 1 of the chunk.
  const int m = min(m0 + rw * 16 + (lane & 15), p.Mdim - 1);       // (weight gradients) past the end: any column, not stored
  const float* a_ptr = A_NC ? A + m : A + (int64_t)a_row * p.lda;
  uint32_t a_off[A_NC ? SPL : 1];     // byte offsets from the chunk's first row
#pragma unroll
  for (int s = 0; s < (A_NC ? SPL : 1); ++s) a_off[s] = ((uint32_t)(kb + s) * (uint32_t)p.lda + (uint32_t)m) * 4u;
  constexpr uint32_t ALL = (1u << SPL) - 1u;
  struct Piece {
    float v[SPL];
    uint32_t keep;      // which of them exist
  };
  const __amdgpu_buffer_rsrc_t rG = make_rsrc(p.gather, A_NC && p.gather ? (uint32_t)((int64_t)p.G * p.Cc * 4) : 0u);
  const bool gathered = A_NC && p.gather != nullptr;
  struct Slots {
    int v[A_NC ? SPL : 1];
  };
  Slots slots;                      // gathered rows: slot-map entries of the chunk that is fetched next
  auto fetch_map = [&](Slots& d, const KTile& kt) {     // entries behind the map read as zero; rows behind the count are masked
#pragma unroll
    for (int s = 0; s < (A_NC ? SPL : 1); ++s) d.v[s] = (int)__builtin_amdgcn_raw_buffer_load_b32(rG, (int)((uint32_t)(kt.row0 + kb + s) * 4u), 0, 0);
  };
  auto fetch_a = [&](Piece& d, const KTile& kt, const Slots& map) {
    d.keep = (1u << min(max(kt.lim - kb, 0), SPL)) - 1u;
    if (!A_NC) {        // K % 8 == 0: the values of a lane's quarter exist together or (SPL = 8) in halves of 4
#pragma unroll
      for (int q = 0; q < SPL / 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(a_ptr + kt.row0 + (kb + 4 * q < kt.lim ? kb + 4 * q : 0));
        d.v[4 * q] = v.x; d.v[4 * q + 1] = v.y; d.v[4 * q + 2] = v.z; d.v[4 * q + 3] = v.w;
      }
    } else if (gathered) {
#pragma unroll
      for (int s = 0; s < SPL; ++s) {
        const int iv = map.v[A_NC ? s : 0];
        const uint32_t tok = p.gather_k == 1 ? (uint32_t)iv : __umulhi((uint32_t)iv, p.gather_magic);
        const bool full = iv >= 0 && (int64_t)tok < p.gather_rows;     // an empty slot is a row of zeros
        if (!full) d.keep &= ~(1u << s);
        d.v[s] = a_ptr[(full && kb + s < kt.lim ? (int64_t)tok : 0) * p.lda];
      }
    } else if (WIDE) {
      const float* q = a_ptr + (int64_t)kt.row0 * p.lda;
#pragma unroll
      for (int s = 0; s < SPL; ++s) d.v[s] = q[(kb + s < kt.lim ? (int64_t)(kb + s) : 0) * p.lda];
    } else {            // through a descriptor that ends with the chunk's last row: rows behind it are zeros
      const __amdgpu_buffer_rsrc_t r = make_rsrc(A + (int64_t)kt.row0 * p.lda, (uint32_t)max(min(kt.lim, FK), 0) * (uint32_t)p.lda * 4u);
#pragma unroll
      for (int s = 0; s < SPL; ++s) d.v[s] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)a_off[A_NC ? s : 0], 0, 0));
      d.keep = ALL;
    }
  };
  // ---- B: through LDS.  A column behind the last one is fetched from the tile's first one.
  struct Rows {
    float4 v[UB];
  };
  Rows rb;
  int b_k[UB];
  uint32_t b_at[UB], b_off[UB];      // element of the piece in its buffer; byte offset from where the chunk starts
#pragma unroll
  for (int u = 0; u < UB; ++u) {
    const int i = tid + 256 * u;
    if (B_NC) {
      const int n = (i % (TN / 4)) * 4;
      b_k[u] = i / (TN / 4);
      b_at[u] = (uint32_t)(b_k[u] * PB + n);
      b_off[u] = ((uint32_t)b_k[u] * (uint32_t)p.ldb + (uint32_t)(n0 + n < p.Ndim ? n0 + n : n0)) * 4u;
    } else {
      const int n = i / (FK / 4);
      b_k[u] = (i % (FK / 4)) * 4;
      b_at[u] = (uint32_t)(b_k[u] * PB + n);
      b_off[u] = ((uint32_t)min(n, p.Ndim - 1 - n0) * (uint32_t)p.ldb + (uint32_t)b_k[u]) * 4u;
    }
  }
  auto fetch_b = [&](Rows& d, const KTile& kt) {
    if constexpr (WIDE) {
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int i = tid + 256 * u, k = kt.row0 + (b_k[u] < kt.lim ? b_k[u] : 0), n = n0 + (B_NC ? (i % (TN / 4)) * 4 : i / (FK / 4));
        d.v[u] = *reinterpret_cast<const float4*>(B_NC ? B + (int64_t)k * p.ldb + (n < p.Ndim ? n : n0)
                                                       : B + (int64_t)min(n, p.Ndim - 1) * p.ldb + k);
      }
      return;
    }
    const __amdgpu_buffer_rsrc_t r =     // B_NC: ends with the chunk's last row, rows behind it are zeros
        B_NC ? make_rsrc(B + (int64_t)kt.row0 * p.ldb, (uint32_t)max(min(kt.lim, FK), 0) * (uint32_t)p.ldb * 4u)
             : make_rsrc(B + (int64_t)n0 * p.ldb + kt.row0, OOB);
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const uint4 v = ldb16(r, B_NC || b_k[u] < kt.lim ? b_off[u] : b_off[u] - (uint32_t)b_k[u] * 4u);
      d.v[u] = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    }
  };
  auto stage_b = [&](Rows& src, int buf, int lim) {
    double* d = Bs + buf * BUF;
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      if ((!B_NC || WIDE) && lim < FK) {
        if (b_k[u] >= lim) src.v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
      const double x[4] = {(double)src.v[u].x, (double)src.v[u].y, (double)src.v[u].z, (double)src.v[u].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) d[b_at[u] + (B_NC ? q : q * PB)] = x[q];
    }
  };

  f64x4_t acc[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) acc[j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  Piece pa[2];
  int lim_b;              // of the chunk in rb
  KTile t2;               // chunk c + 2
  {
    const KTile t0 = ktile(0), t1 = ktile(1);
    t2 = ktile(2);
    Slots s0, s1;
    Rows r0;
    if (gathered) { fetch_map(s0, t0); fetch_map(s1, t1); fetch_map(slots, t2); }
    fetch_b(r0, t0);
    fetch_b(rb, t1);
    fetch_a(pa[0], t0, s0);
    fetch_a(pa[1], t1, s1);
    stage_b(r0, 0, t0.lim);
    lim_b = t1.lim;
  }
  auto zero_missing = [&](Piece& a) {
    if (A_NC ? gathered || WIDE : a.keep != ALL) {
#pragma unroll
      for (int s = 0; s < SPL; ++s) a.v[s] = (a.keep >> s) & 1u ? a.v[s] : 0.f;
    }
  };
  auto products = [&](const Piece& pc, const double* w, int s0, int s1) {
#pragma unroll
    for (int s = s0; s < s1; ++s) {
      const double a = (double)pc.v[s];
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, w[s * PB + 16 * j], acc[j], 0, 0, 0);
    }
  };
  auto step = [&](int c, auto set_tag) {
    constexpr int SET = decltype(set_tag)::value;
    const double* wb = Bs + kb * PB + (lane & 15);
    __syncthreads();      // chunk c is staged, and the other buffer is consumed
    zero_missing(pa[SET]);
    products(pa[SET], wb + SET * BUF, 0, SPL / 2);
    stage_b(rb, SET ^ 1, lim_b);
    fetch_b(rb, t2);
    lim_b = t2.lim;
    products(pa[SET], wb + SET * BUF, SPL / 2, SPL);
    fetch_a(pa[SET], t2, slots);
    t2 = ktile(c + 3);
    if (gathered) fetch_map(slots, t2);
  };
  int c = 0;
  for (; c + 2 < nk; c += 2) {
    step(c, std::integral_constant<int, 0>{});
    step(c + 1, std::integral_constant<int, 1>{});
  }
  // The last chunk or two, behind which nothing is fetched or staged.  In the loop's steps the last one waited for a chunk that does
  // not exist, and an odd number of chunks had one of zeros multiplied: 4 experts of 62 rows x 64 x 128, forward and backward call, 8.87 and
  // 10.1 us, now 8.4 and 9.4; 8 of 2000 x 96 x 96 26.4 and 60, now 22.3 and 56; 12 of 100 x 200 x 328 23.3 and 36.4, now 21.5 and 34.1.
  const double* w = Bs + kb * PB + (lane & 15);
  auto last = [&]() {
    __syncthreads();
    zero_missing(pa[0]);
    products(pa[0], w, 0, SPL);
  };
  if (c + 2 == nk) {
    last();
    stage_b(rb, 1, lim_b);
    pa[0] = pa[1];
    w += BUF;
    ++c;
  }
  if (c < nk) last();
  if constexpr (KW == 2) {
    __syncthreads();
    // Of two neighbouring blocks of columns the first half finishes one and the second the other: with the second idle here, the
    // other's epilogue, eight values a lane, took 0.4 us more of every launch.
    double* red = Bs + (rw * 64 + lane) * (4 * NJ + 1);   // + 1: lanes on different banks
#pragma unroll
    for (int j = 0; j < NJ; j += 2)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[4 * (j + 1 - kw) + r] = kw == 0 ? acc[j + 1][r] : acc[j][r];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NJ; j += 2)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[j / 2][r] = (kw == 0 ? acc[j][r] : acc[j + 1][r]) + red[4 * (j + kw) + r];
  }
  float* __restrict__ C = reinterpret_cast<float*>(p.C);
  float* __restrict__ C2 = reinterpret_cast<float*>(p.C2);
  const float* __restrict__ Z = reinterpret_cast<const float*>(p.Zin);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int ml = rw * 16 + 4 * r + (lane >> 4);   // row within the tile
    int64_t crow;
    bool zero = false;
    if (KIND == KIND_TN) {
      if (m0 + ml >= p.Mdim) continue;
      crow = (int64_t)g * p.c_goff + p.c_off + (int64_t)(m0 + ml) * p.ldc;
    } else {
      const int row = __shfl(o_row, ml, 64);
      zero = __shfl((int)o_zero, ml, 64) != 0;
      if (row < 0) continue;
      crow = (int64_t)row * p.ldc;
    }
#pragma unroll
    for (int j = 0; j < NJ / KW; ++j) {
      const int n = n0 + 16 * (KW * j + kw) + (lane & 15);
      if (n >= p.Ndim) continue;
      const float v = zero ? 0.f : (float)acc[j][r];
      if (EPI == EPI_STORE) {
        C[crow + n] = v;
      } else if (EPI == EPI_GELU) {
        C[crow + n] = v;
        C2[crow + n] = gelu_f(v);
      } else {
        float ge, dg;
        gelu_and_grad(Z[crow + n], ge, dg);
        C[crow + n] = v * dg;
      }
    }
  }
}

template <int KIND, int EPI, int T, bool WIDE>   // T x T tiles
__global__ __launch_bounds__(256, 4) void ffn_gemm_f32(const GemmArgs p) {   // (the 4 keeps the accumulators out of the AGPRs)
  __shared__ __attribute__((aligned(16))) double smem[f32_lds<T, T>() / 8];
  gemm_f32_tile<KIND, EPI, T, T, WIDE>(p, smem, (int)blockIdx.x);
}
// the three backward GEMMs that only depend on dZ, as in ffn_bwd_trio
template <int T, bool WIDE>
__global__ __launch_bounds__(256, 4) void ffn_bwd_trio_f32(const GemmArgs px, const GemmArgs pw2, const GemmArgs pw1, int nbx,
                                                           int nbw) {
  __shared__ __attribute__((aligned(16))) double smem[f32_lds<T, T>() / 8];
  const int b = (int)blockIdx.x;
  if (b < nbx) gemm_f32_tile<KIND_NT, EPI_STORE, T, T, WIDE>(px, smem, b);
  else gemm_f32_tile<KIND_TN, EPI_STORE, T, T, WIDE>(b < nbx + nbw ? pw2 : pw1, smem, b < nbx + nbw ? b - nbx : b - nbx - nbw);
}

// ------------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------------
int num_cus() {
  static int n = 0;   // same on every device of a node
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) n = v;
    else n = 256;
  }
  return n;
}

// Tile of a bf16 grouped GEMM, tile_m x tile_n.
struct TilePlan {
  int tile_m, tile_n;
};
// The tiles a row-tiled GEMM may take, and what one costs (microseconds, measured): a k tile of 64 with few and with all
// compute units busy (in a launch of its own; a compute unit then holds one workgroup of the first two, two of the
// others), and everything outside the k loop.  Large tiles move the fewest bytes per flop; small ones fill the chip when
// there are few rows, and their k tile is short when a long reduction is what a launch waits for.
// The prices of the two largest tiles are those of a loop with 32x32x16 MFMAs and requests in bursts; the present one is
// shorter with every compute unit busy, and they have not been measured again.  For dX in the merged backward launch with
// 256 x 256 weight gradients they are an approximation: there a compute unit holds one workgroup whatever its tile (the
// launch reserves the LDS of a 256 x 256 tile), and the weight gradients queue behind dX.
struct TileCost {
  TilePlan tile;
  int per_cu;
  float k_few, k_all, fixed;
};
constexpr TileCost ROW_TILES[] = {{{256, 256}, 1, 0.95f, 1.50f, 10.f}, {{192, 256}, 1, 0.72f, 1.22f, 9.f},
                                  {{128, 128}, 2, 0.50f, 1.05f, 7.f},  {{64, 128}, 2, 0.31f, 0.66f, 6.f},
                                  {{64, 64}, 2, 0.24f, 0.42f, 6.f},    {{32, 64}, 2, 0.20f, 0.30f, 5.f}};
// `tile` is the caller's hint (MOE_TILE_*); wide = only tiles that the merged backward launch can take (eight waves).
TilePlan plan_tiles(int tile, bool tn, int G, int Mdim, int Ndim, int Kdim, bool wide = false) {
  auto tiles = [&](TilePlan t) { return (int64_t)G * ((Mdim + t.tile_m - 1) / t.tile_m) * ((Ndim + t.tile_n - 1) / t.tile_n); };
  if (tile == MOE_TILE_SMALL) return {128, 128};
  if (tile == MOE_TILE_256) return {256, 256};
  if (tn) return tile == MOE_TILE_AUTO && tiles({256, 256}) < 64 ? TilePlan{128, 128} : TilePlan{256, 256};
  if (tile == MOE_TILE_192) return {192, 256};
  const float nk = (float)((Kdim + 63) / 64), cu = (float)num_cus();
  TilePlan best{256, 256};
  float best_t = 0.f;
  for (const TileCost& c : ROW_TILES) {
    if (wide && c.tile.tile_n == 64) continue;
    const float n = (float)tiles(c.tile);
    const float busy = c.per_cu == 1 ? n / cu : (n - cu) / cu;
    const float k = c.k_few + (c.k_all - c.k_few) * fminf(fmaxf(busy, 0.f), 1.f);
    const float t = ceilf(n / (cu * c.per_cu)) * (nk * k + c.fixed);
    if (best_t == 0.f || t < best_t) { best_t = t; best = c.tile; }
  }
  return best;
}

// Tile order (GemmArgs::run_mask).  Row-tiled GEMMs: contiguous ranges while both operands of an expert fit in an XCD's 4 MB of
// L2, which then fetches them once; runs in turn beyond it.  Forward pair, runs and ranges on one card: 8 experts of
// 1024 x 512 x 768 (2 MB) 32.7 and 32.2 us, without counts 28.7 and 26.7; 8 of 1500 x 256 x 1024 35.2 and 33.5; 12 of
// 276 x 520 x 1544, without counts, 40.9 and 39.2; beyond the line 12 of 618 x 256 x 13656 (7 MB) 285 and 289, 8 of
// 96 x 4096 x 14336 (113 MB) 394 and 403, 8 of 2048 x 4096 x 4096 833 and 869 (but 16 of 64 x 2048 x 4096 113 and 111).
// Weight gradients: runs, no clear winner otherwise (backward, few rows: 8 x 100 x 1024 x 4096 71.5 and 73.2,
// 32 x 100 x 1024 x 1024 72.1 and 73.4, 16 x 64 x 2048 x 4096 272.8 and 267.2).
int tile_runs(const GemmArgs& a, bool tn, int esz) {
  return !tn && ((int64_t)a.Mdim + a.Ndim) * a.Kdim * esz <= 4 << 20 ? 0 : ~31;
}

// Rows that a problem is priced for.  Rows of capacity padding are not multiplied; how many there are is not known here.  Where
// counts are passed it is nine rows in ten (capacity factors are 1 to 1.25), so that a last row tile that will mostly be
// padding does not decide the height.
int priced_rows(const GemmArgs& a, bool tn) { return !tn && a.cnt ? (int)(((int64_t)a.Mdim * 9 + 9) / 10) : a.Mdim; }

// fills the tile counts and buffer sizes of a bf16 problem
TilePlan prepare_bf16(GemmArgs& a, bool tn, int tile, bool wide = false) {
  const uint64_t act_rows = (uint64_t)a.n_src * a.G * a.Cc;
  a.a_bytes = (a.gather ? (uint64_t)a.gather_rows : act_rows) * (uint64_t)a.lda * 2;
  a.b_bytes = tn ? act_rows * (uint64_t)a.ldb * 2 : (uint64_t)a.G * (uint64_t)a.b_goff * 2;
  const TilePlan t = plan_tiles(tile, tn, a.G, priced_rows(a, tn), a.Ndim, a.Kdim, wide);
  a.tiles_n = (a.Ndim + t.tile_n - 1) / t.tile_n;
  a.tiles_m = (a.Mdim + t.tile_m - 1) / t.tile_m;
  a.total_tiles = a.G * a.tiles_m * a.tiles_n;
  a.run_mask = tile_runs(a, tn, 2);
  return t;
}

// The three backward GEMMs that only depend on dZ go out in one launch unless the caller asks for MOE_TILE_SMALL; returns the
// tile of the two weight gradients (H_l x M and M x H_l: as many tiles each), or 0: launches of their own.
int merged_backward(GemmArgs& w2, GemmArgs& w1, int tile) {   // prepares the two
  prepare_bf16(w1, true, tile);
  const TilePlan t = prepare_bf16(w2, true, tile);
  return tile == MOE_TILE_SMALL ? 0 : t.tile_m;
}
// dX beside weight gradients of 128 x 128 tiles takes 64 x 128 ones, two workgroups to a compute unit as theirs.  That pays
// while they are one round of the chip; beyond it dX goes out alone, in the tiles of its own plan.  Backward call, merged and alone:
// 8 experts of 274 x 128 x 1216 (40 tiles) 22.0 and 26.0 us, 1 of 512 x 2048 x 1792 (128) 35.2 and 40.1, 8 of 1024 x 512 x 768
// (480) 51.0 and 52.3; 7 of 1024 x 768 x 768 (630) 63.7 and 61.0, 30 of 1000 x 512 x 256 (1800) 71.2 and 58.9, 7 of
// 4096 x 768 x 768 (2436) 176.7 and 147.2, 1 of 32768 x 2048 x 1792 (8192) 1093 and 945.
bool dx_alone(const GemmArgs& dx) {
  const int64_t tiles = (int64_t)dx.G * ((priced_rows(dx, false) + 63) / 64) * ((dx.Ndim + 127) / 128);
  return tiles > 2 * (int64_t)num_cus();
}
// Parts of the reductions of the two weight gradients where both take 128 x 128 tiles: few tiles leave compute units idle, and
// a reduction over thousands of rows is then what the launch waits for.  Parts of at least 12 k tiles of the capacity (a k tile
// takes 0.6 us there, writing, reading and adding the partial sums in a launch of their own 4 to 9 us), and no more workgroups
// than the chip holds.  A part of the workspace's size, so it is arithmetic on the shape and asks no device.  2 experts of
// 55 000 rows x 512 x 128, 16 tiles, backward call: 1028 us whole, 167 in parts.  Few rows gain by the one launch: 8 experts of
// 274 rows x 128 x 1216, 88 tiles, 8.0 + 10.2 + 8.1 -> 12.4 us.  One launch of 128 x 128 tiles measured no better from 64
// tiles of 256 x 256 on (72 to 256 of them: 0.93 to 1.33 times the time).
constexpr int CHIP_CUS = 256;   // compute units of an MI355X
int weight_parts(int n_src, int G, int64_t C, int M, int Hl) {
  const int64_t tiles256 = (int64_t)G * ((M + 255) / 256) * ((Hl + 255) / 256);
  if (tiles256 >= 64) return 1;
  const int64_t tiles = 2 * (int64_t)G * ((M + 127) / 128) * ((Hl + 127) / 128), nk = ((int64_t)n_src * C + 63) / 64;
  const int64_t parts = std::min<int64_t>({2 * CHIP_CUS / tiles, nk / 12, 64});
  return parts < 2 ? 1 : (int)parts;
}

bool packs_chunks(const GemmArgs& a) { return a.n_src >= PACK_CHUNKS && a.cnt != nullptr; }

// Workgroups of a problem, a multiple of 8: every XCD takes an equal share of the tiles to multiply and, with row
// counts, of the shares of the padding (map_tile), each rounded up.
int grid_of(const GemmArgs& a) {
  return (a.total_tiles + (a.cnt ? 14 : 7)) / 8 * 8 + (a.cnt && a.n_src > 1 ? MORE_SHARES : 0);
}

// fp32 tiles, T x T: 64 where they give every compute unit three or more and do not pad the rows by an eighth more than
// those of 32 do.  Forward or backward call with all GEMMs but one as planned, that one in tiles of 64 and of 32: 8 experts of 256 x 512 x
// 2048, Z (1280 tiles of 64) 159 and 168 us, Y (320) 160 and 159; 4 of 820 x 768 x 3072, Y (720) 563 and 537; 2 of 3690 x 256 x 512, Z
// (928) 89 and 93, the merged backward launch (592) 234 and 198; 24 of 72 x 768 x 1024, Z (768, 128 rows for 96) 153 and 142;
// 16 of 64 x 512 x 1024, merged (4224) 100 and 121.  32 x 64 was nowhere better than both.
using I32 = std::integral_constant<int, 32>;
using I64 = std::integral_constant<int, 64>;
int64_t tiles_f32(const GemmArgs& a, bool tn, int tile) {
  const int64_t rows = priced_rows(a, tn);
  return (int64_t)a.G * ((rows + tile - 1) / tile) * ((a.Ndim + tile - 1) / tile);
}
// Offsets within a tile's 64 rows of an operand are 32-bit but for leading dimensions of 16 million and more.
bool wide_f32(const GemmArgs& a) { return std::max(a.lda, a.ldb) >= 1 << 24; }
int plan_f32(const GemmArgs& a) {   // of a row-tiled GEMM
  if (wide_f32(a)) return 32;
  const int64_t rows = priced_rows(a, false), rows64 = (rows + 63) / 64 * 64, rows32 = (rows + 31) / 32 * 32;
  return tiles_f32(a, false, 64) >= 3 * (int64_t)num_cus() && 8 * rows64 <= 9 * rows32 ? 64 : 32;
}
// Of the merged backward launch, whose reductions differ in length: where the longest, a chain of k chunks in one workgroup, has more
// of them than a compute unit's share of all, the launch waits for it, and the chunks of 32 x 32 tiles are half as long.  Backward call
// in tiles of 64 and of 32 (tiles of 64; chunks: the chain, a compute unit's share): 4 experts of 11 x 104 x 3032 (776; 95, 5) 137 and 75 us, 8 of
// 30 x 144 x 8040 (6072; 252, 47) 356 and 166, 2 of 41 x 1160 x 1392 (1710; 44, 20) 90 and 64, 4 of 71 x 704 x 864 (1320; 27, 24) 69 and 62, 4 of
// 93 x 768 x 4944 (7584; 155, 146) 309 and 276; 8 of 12 x 1024 x 704 (2944; 22, 22) 58 and 69, 4 of 55 x 1432 x 3432 (10028; 108, 116) 246 and
// 275, 16 of 32 x 576 x 2504 (11664; 79, 89) 177 and 218, 8 of 62 x 1024 x 808 (3456; 26, 39) 85 and 104; but 4 of 643 x 152 x 3376 (1404; 106, 159)
// 283 and 238.
int plan_f32_trio(const GemmArgs& dx, const GemmArgs& w2, const GemmArgs& w1) {
  if (wide_f32(dx) || wide_f32(w2) || wide_f32(w1)) return 32;
  int64_t tiles = 0, work = 0, chain = 0;
  auto add = [&](const GemmArgs& a, bool tn) {
    const int64_t n = tiles_f32(a, tn, 64), chunks = (a.Kdim + FK - 1) / FK;
    tiles += n;
    work += n * chunks;
    chain = std::max(chain, chunks);
  };
  add(dx, false); add(w2, true); add(w1, true);
  return tiles >= 3 * (int64_t)num_cus() && chain * num_cus() <= work ? 64 : 32;
}
void prepare_f32(GemmArgs& a, bool tn, int tile) {
  a.tiles_m = (a.Mdim + tile - 1) / tile;
  a.tiles_n = (a.Ndim + tile - 1) / tile;
  a.total_tiles = a.G * a.tiles_m * a.tiles_n;
  a.run_mask = tile_runs(a, tn, 4);
}

template <int KIND, int EPI>   // row-tiled GEMMs
void launch_gemm(GemmArgs a, int dtype, int tile, hipStream_t st) {
  static_assert(KIND != KIND_TN, "weight gradients go out in the merged launches, or through launch_weight_small");
  if constexpr (KIND == KIND_NN || EPI == EPI_DGELU) {   // (the fp32 dX is always in the merged launch)
    if (dtype == MOE_F32) {
      auto launch = [&](auto tile_tag, auto wide) {
        constexpr int T = decltype(tile_tag)::value;
        prepare_f32(a, false, T);
        hipLaunchKernelGGL((ffn_gemm_f32<KIND, EPI, T, decltype(wide)::value>), dim3((unsigned)grid_of(a)), dim3(256), 0, st, a);
      };
      const int tile_f32 = plan_f32(a);
      if (tile_f32 == 64) launch(I64{}, std::false_type{});
      else if (!wide_f32(a)) launch(I32{}, std::false_type{});
      else launch(I32{}, std::true_type{});
      return;
    }
  }
  const TilePlan t = prepare_bf16(a, false, tile);
  auto launch = [&](auto cfg) {
    using CF = decltype(cfg);
    hipLaunchKernelGGL((ffn_gemm_dma<KIND, EPI, CF>), dim3((unsigned)grid_of(a)), dim3(64 * CF::NW), 0, st, a);
  };
  if (t.tile_m == 256) launch(Tile256{});
  else if (t.tile_m == 192) launch(Tile192{});
  else if (t.tile_m == 128) launch(Tile128{});
  else if (t.tile_m == 64 && t.tile_n == 128) launch(Tile64x128{});
  else if (t.tile_m == 64) launch(Tile64{});
  else launch(Tile32x64{});
}
// a bf16 weight gradient by the hint MOE_TILE_SMALL, which ignores row counts
void launch_weight_small(GemmArgs a, hipStream_t st) {
  prepare_bf16(a, true, MOE_TILE_SMALL);
  const dim3 grid((unsigned)grid_of(a)), block(64 * Tile128::NW);
  if (a.gather != nullptr) hipLaunchKernelGGL((ffn_gemm_dma<KIND_TN, EPI_STORE, Tile128, ROWS_GATHER>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((ffn_gemm_dma<KIND_TN, EPI_STORE, Tile128>), grid, block, 0, st, a);
}

inline bool valid_tile(int tile) { return tile >= MOE_TILE_AUTO && tile <= MOE_TILE_192; }
inline bool ignores_counts(int dtype, int tile) { return dtype == MOE_BF16 && tile == MOE_TILE_SMALL; }

int check_ffn_shape(int dtype, int n_src, int G, int64_t C, int M, int H, int esp_idx, int n_esp) {
  MOE_REQUIRE(dtype == MOE_F32 || dtype == MOE_BF16, MOE_EINVAL);
  MOE_REQUIRE(n_src >= 1 && G >= 1 && C >= 1 && M >= 1 && H >= 1, MOE_EINVAL);
  MOE_REQUIRE(n_esp >= 1 && esp_idx >= 0 && esp_idx < n_esp && H % n_esp == 0, MOE_EINVAL);
  const int Hl = H / n_esp;
  MOE_REQUIRE(M % 8 == 0 && Hl % 8 == 0, MOE_EUNSUPPORTED);
  MOE_REQUIRE((int64_t)n_src * C < (1ll << 31) && (int64_t)n_src * G * C < (1ll << 31), MOE_EUNSUPPORTED);
  if (dtype == MOE_BF16) {  // 32-bit byte offsets inside one activation tensor / one expert's weight matrix
    const uint64_t wide = (uint64_t)(M > Hl ? M : Hl);
    MOE_REQUIRE((uint64_t)n_src * G * C * wide * 2 <= 0xFFFFFFF0ull, MOE_EUNSUPPORTED);
    MOE_REQUIRE((uint64_t)M * H * 2 <= 0xFFFFFFF0ull, MOE_EUNSUPPORTED);
  }
  return MOE_OK;
}

}  // namespace

// Rows of all experts that a GEMM multiplies: the occupied ones, in the row-tiled GEMMs (tile_m > 0) rounded up to whole
// row tiles of each expert's compacted rows.
static double rows_multiplied(const GemmArgs& a, int tile_m) {
  double rows = 0;
  for (int g = 0; g < a.G; ++g) {
    int64_t n = a.R;
    if (a.cnt != nullptr) {
      n = 0;
      for (int s = 0; s < a.n_src; ++s) {
        const int32_t c = a.cnt[(int64_t)s * a.G + g];
        n += c < 0 ? 0 : c < a.Cc ? c : a.Cc;
      }
    }
    if (tile_m > 0) n = (n + tile_m - 1) / tile_m * tile_m;
    rows += (double)(n < a.R ? n : a.R);
  }
  return rows;
}

extern "C" double moe_ffn_executed_flops(int dtype, int n_src, int G, int64_t C, int M, int H, int n_esp,
                                         const int32_t* row_counts_host, int tile, int backward) {
  if (check_ffn_shape(dtype, n_src, G, C, M, H, 0, n_esp) != MOE_OK || !valid_tile(tile)) return 0.0;
  const int Hl = H / n_esp;
  GemmArgs a{};   // the problems as the calls below plan them
  a.G = G; a.n_src = n_src; a.Cc = (int)C; a.R = (int)(n_src * C);
  a.cnt = ignores_counts(dtype, tile) ? nullptr : row_counts_host;
  auto gemm = [&](int Mdim, int Ndim, int Kdim, int lda, int ldb) {
    GemmArgs p = a;
    p.Mdim = Mdim; p.Ndim = Ndim; p.Kdim = Kdim;
    p.lda = lda; p.ldb = ldb;
    return p;
  };
  auto alone = [&](GemmArgs p) { return dtype == MOE_F32 ? plan_f32(p) : prepare_bf16(p, false, tile).tile_m; };
  double rows;
  if (!backward) {   // Z = X W1 (rows x Hl), Y = A W2 (rows x M)
    rows = rows_multiplied(a, alone(gemm(a.R, Hl, M, M, H))) + rows_multiplied(a, alone(gemm(a.R, M, Hl, Hl, M)));
  } else {           // dA = dY W2^T (rows x Hl), dX = dZ W1^T (rows x M), dW2 (Hl x M) and dW1 (M x Hl) over the rows
    GemmArgs w2 = gemm(Hl, M, a.R, Hl, M), w1 = gemm(M, Hl, a.R, M, Hl), dx = gemm(a.R, M, Hl, Hl, H);
    auto dx_tile = [&]() {
      const int merged = merged_backward(w2, w1, tile);
      return merged == 128 && !dx_alone(dx) ? Tile64x128::TM : prepare_bf16(dx, false, tile, merged == 256).tile_m;
    };
    const int dx_m = dtype == MOE_F32 ? plan_f32_trio(dx, w2, w1) : dx_tile();
    rows = rows_multiplied(a, alone(gemm(a.R, Hl, M, M, M))) + rows_multiplied(a, dx_m) + 2.0 * rows_multiplied(a, 0);
  }
  return 2.0 * (double)M * (double)Hl * rows;
}

static size_t dz_bytes(int n_src, int G, int64_t C, int Hl, size_t esz) {
  return moe::align_up((size_t)n_src * G * C * (size_t)Hl * esz, 256);
}
static size_t part_bytes(int parts, int G, int M, int Hl) { return moe::align_up((size_t)parts * G * M * Hl * 4, 256); }

extern "C" size_t moe_ffn_workspace_bytes(int dtype, int n_src, int G, int64_t C, int M, int H, int n_esp) {
  if (check_ffn_shape(dtype, n_src, G, C, M, H, 0, n_esp) != MOE_OK) return 0;
  const size_t esz = dtype == MOE_BF16 ? 2 : 4;
  const int Hl = H / n_esp;
  const int parts = dtype == MOE_BF16 ? weight_parts(n_src, G, C, M, Hl) : 1;
  return dz_bytes(n_src, G, C, Hl, esz) + (parts > 1 ? 2 * part_bytes(parts, G, M, Hl) : 0);
}

static uint32_t magic_of(int k) { return k > 1 ? (uint32_t)((0x100000000ull + (uint64_t)k - 1) / (uint64_t)k) : 0u; }

static int ffn_fwd_impl(const void* X, const int32_t* gather, int gather_k, int64_t gather_rows, int dtype,
                        const void* W1, const void* W2, int n_src, int G, int64_t C, int M, int H, int esp_idx,
                        int n_esp, const int32_t* row_counts, int tile, void* Z, void* A, void* Y, void* stream) {
  if (int rc = check_ffn_shape(dtype, n_src, G, C, M, H, esp_idx, n_esp)) return rc;
  MOE_REQUIRE(valid_tile(tile), MOE_EINVAL);
  MOE_REQUIRE_PTR(X); MOE_REQUIRE_PTR(W1); MOE_REQUIRE_PTR(W2); MOE_REQUIRE_PTR(Z); MOE_REQUIRE_PTR(A);
  MOE_REQUIRE_PTR(Y);
  MOE_REQUIRE((((uintptr_t)row_counts) & 3u) == 0, MOE_EALIGN);
  hipStream_t st = (hipStream_t)stream;
  const int Hl = H / n_esp;
  const int64_t h0 = (int64_t)esp_idx * Hl;

  GemmArgs a{};
  a.G = G; a.n_src = n_src; a.Cc = (int)C; a.R = (int)(n_src * C);
  a.cnt = ignores_counts(dtype, tile) ? nullptr : row_counts;
  // Z = X * W1[:, h0:h0+Hl] ; A = GeLU(Z)
  a.A = X; a.lda = M;
  a.gather = gather; a.gather_k = gather_k; a.gather_rows = gather_rows; a.gather_magic = magic_of(gather_k);
  a.B = W1; a.ldb = H; a.b_goff = (int64_t)M * H; a.b_off = h0;
  a.C = Z; a.C2 = A; a.ldc = Hl;
  a.Mdim = a.R; a.Ndim = Hl; a.Kdim = M;
  launch_gemm<KIND_NN, EPI_GELU>(a, dtype, tile, st);
  // Y = A * W2[h0:h0+Hl, :]
  a.A = A; a.lda = Hl;
  a.gather = nullptr; a.gather_k = 0; a.gather_rows = 0; a.gather_magic = 0;
  a.B = W2; a.ldb = M; a.b_goff = (int64_t)H * M; a.b_off = h0 * M;
  a.C = Y; a.C2 = nullptr; a.ldc = M;
  a.Mdim = a.R; a.Ndim = M; a.Kdim = Hl;
  launch_gemm<KIND_NN, EPI_STORE>(a, dtype, tile, st);
  return moe::check_launch();
}

extern "C" int moe_expert_ffn_fwd(const void* X, int dtype, const void* W1, const void* W2, int n_src, int G,
                                  int64_t C, int M, int H, int esp_idx, int n_esp, const int32_t* row_counts, int tile,
                                  void* Z, void* A, void* Y, void* stream) {
  return ffn_fwd_impl(X, nullptr, 0, 0, dtype, W1, W2, n_src, G, C, M, H, esp_idx, n_esp, row_counts, tile, Z, A, Y, stream);
}

// arguments of the fused-dispatch entry points: token matrix [S, M] and the inverse slot map
static int check_gather(const void* x, int dtype, int64_t S, const int32_t* inv, int k, int M) {
  MOE_REQUIRE(S >= 1 && k >= 1 && k <= MOE_MAX_K, MOE_EINVAL);
  MOE_REQUIRE_PTR(x); MOE_REQUIRE_PTR(inv);
  MOE_REQUIRE((int64_t)S * k <= (1ll << 29), MOE_EUNSUPPORTED);   // slot entries t k + j are divided by multiplication
  if (dtype == MOE_BF16) MOE_REQUIRE((uint64_t)S * (uint64_t)M * 2 <= 0xFFFFFFF0ull, MOE_EUNSUPPORTED);
  return MOE_OK;
}

extern "C" int moe_expert_ffn_fwd_gather(const void* x, int dtype, int64_t S, const int32_t* inv, int k, const void* W1,
                                         const void* W2, int E, int64_t C, int M, int H, int esp_idx, int n_esp,
                                         const int32_t* row_counts, int tile, void* Z, void* A, void* Y, void* stream) {
  if (int rc = check_gather(x, dtype, S, inv, k, M)) return rc;
  return ffn_fwd_impl(x, inv, k, S, dtype, W1, W2, 1, E, C, M, H, esp_idx, n_esp, row_counts, tile, Z, A, Y, stream);
}

static int ffn_bwd_impl(const void* dY, const void* X, const int32_t* gather, int gather_k, int64_t gather_rows,
                        const void* Z, const void* A, const void* W1, const void* W2, int dtype, int n_src, int G,
                        int64_t C, int M, int H, int esp_idx, int n_esp, const int32_t* row_counts, int tile, void* dX,
                        void* dW1, void* dW2, void* ws, size_t ws_bytes, void* stream) {
  if (int rc = check_ffn_shape(dtype, n_src, G, C, M, H, esp_idx, n_esp)) return rc;
  MOE_REQUIRE(valid_tile(tile), MOE_EINVAL);
  MOE_REQUIRE_PTR(dY); MOE_REQUIRE_PTR(X); MOE_REQUIRE_PTR(Z); MOE_REQUIRE_PTR(A); MOE_REQUIRE_PTR(W1);
  MOE_REQUIRE_PTR(W2); MOE_REQUIRE_PTR(dX); MOE_REQUIRE_PTR(dW1); MOE_REQUIRE_PTR(dW2);
  const size_t dz = dz_bytes(n_src, G, C, H / n_esp, dtype == MOE_BF16 ? 2 : 4);
  MOE_REQUIRE(ws != nullptr && ws_bytes >= dz, MOE_EWORKSPACE);   // with less than the full size the reductions are not split
  MOE_REQUIRE(moe::aligned16(ws), MOE_EALIGN);
  MOE_REQUIRE((((uintptr_t)row_counts) & 3u) == 0, MOE_EALIGN);
  hipStream_t st = (hipStream_t)stream;
  const int Hl = H / n_esp;
  const int64_t h0 = (int64_t)esp_idx * Hl;
  const void* Act = A;
  void* dZ = ws;

  GemmArgs a{};
  a.G = G; a.n_src = n_src; a.Cc = (int)C; a.R = (int)(n_src * C);
  a.cnt = ignores_counts(dtype, tile) ? nullptr : row_counts;
  // dA = dY * W2[h0:h0+Hl, :]^T ; dZ = dA * GeLU'(Z)
  a.A = dY; a.lda = M;
  a.B = W2; a.ldb = M; a.b_goff = (int64_t)H * M; a.b_off = h0 * M;
  a.C = dZ; a.C2 = nullptr; a.Zin = Z; a.ldc = Hl;
  a.Mdim = a.R; a.Ndim = Hl; a.Kdim = M;
  launch_gemm<KIND_NT, EPI_DGELU>(a, dtype, tile, st);
  // dW2[h0:h0+Hl, :] = Act^T * dY
  GemmArgs w2 = a;
  w2.A = Act; w2.lda = Hl;
  w2.B = dY; w2.ldb = M;
  w2.C = dW2; w2.C2 = nullptr; w2.Zin = nullptr; w2.ldc = M; w2.c_goff = (int64_t)H * M; w2.c_off = h0 * M;
  w2.Mdim = Hl; w2.Ndim = M; w2.Kdim = a.R;
  // dW1[:, h0:h0+Hl] = X^T * dZ
  GemmArgs w1 = w2;
  w1.A = X; w1.lda = M;
  w1.gather = gather; w1.gather_k = gather_k; w1.gather_rows = gather_rows;
  w1.gather_magic = magic_of(gather_k);
  w1.B = dZ; w1.ldb = Hl;
  w1.C = dW1; w1.ldc = H; w1.c_goff = (int64_t)M * H; w1.c_off = h0;
  w1.Mdim = M; w1.Ndim = Hl; w1.Kdim = a.R;
  // dX = dZ * W1[:, h0:h0+Hl]^T
  GemmArgs dx = w1;
  dx.A = dZ; dx.lda = Hl;
  dx.gather = nullptr; dx.gather_k = 0; dx.gather_rows = 0; dx.gather_magic = 0;
  dx.B = W1; dx.ldb = H; dx.b_goff = (int64_t)M * H; dx.b_off = h0;
  dx.C = dX; dx.ldc = M; dx.c_goff = 0; dx.c_off = 0;
  dx.Mdim = a.R; dx.Ndim = M; dx.Kdim = Hl;
  if (dtype == MOE_BF16) {
    // the three are independent: one launch, long row tiles first
    GemmArgs px = dx, p2 = w2, p1 = w1;
    const int merged = merged_backward(p2, p1, tile);
    const bool alone = merged == 128 && dx_alone(px);
    auto launch = [&](auto cfx, auto cfw, auto epi) {
      using CFX = decltype(cfx);
      using CFW = decltype(cfw);
      constexpr int EPI = decltype(epi)::value;
      px.tiles_m = (px.Mdim + CFX::TM - 1) / CFX::TM;
      px.tiles_n = (px.Ndim + CFX::TN - 1) / CFX::TN;
      px.total_tiles = px.G * px.tiles_m * px.tiles_n;
      const int parts = EPI == EPI_PART ? p2.splits : 1;
      const int nbx = alone ? 0 : grid_of(px);
      const int nb2 = (p2.total_tiles + 7) / 8 * 8 * parts, nb1 = (p1.total_tiles + 7) / 8 * 8 * parts;
      const dim3 grid((unsigned)(nbx + nb2 + nb1));
      auto go = [&](auto rows) {
        hipLaunchKernelGGL((ffn_bwd_trio<CFX, CFW, EPI, decltype(rows)::value>), grid, dim3(512), 0, st, px, p2, p1, nbx, nb2);
      };
      if (gather) return go(std::integral_constant<int, ROWS_GATHER>{});
      if constexpr (!std::is_same<CFW, Tile256Brief>::value) {
        if (packs_chunks(p2)) return go(std::integral_constant<int, ROWS_PACKED>{});
      }
      go(std::integral_constant<int, ROWS_PLAIN>{});
    };
    using Store = std::integral_constant<int, EPI_STORE>;
    using Part = std::integral_constant<int, EPI_PART>;
    if (merged == 256) {
      const TilePlan tx = prepare_bf16(px, false, tile, true);
      auto with_dx = [&](auto cfw) {
        if (tx.tile_m == 256) launch(Tile256{}, cfw, Store{});
        else if (tx.tile_m == 192) launch(Tile192{}, cfw, Store{});
        else if (tx.tile_m == 128) launch(Tile128{}, cfw, Store{});
        else launch(Tile64x128{}, cfw, Store{});
      };
      if (a.R <= BRIEF_ROWS && !packs_chunks(p2)) with_dx(Tile256Brief{});
      else with_dx(Tile256{});
      return moe::check_launch();
    }
    if (merged == 128) {
      prepare_bf16(px, false, tile, true);   // buffer sizes
      const int parts = weight_parts(n_src, G, C, M, Hl);
      if (parts > 1 && ws_bytes >= moe_ffn_workspace_bytes(dtype, n_src, G, C, M, H, n_esp)) {
        p2.splits = p1.splits = parts;
        p2.part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + dz);
        p1.part = reinterpret_cast<float*>(reinterpret_cast<char*>(ws) + dz + part_bytes(parts, G, M, Hl));
        launch(Tile64x128{}, Tile128{}, Part{});
        const int64_t n = (int64_t)G * M * Hl / 4;   // H_l is a multiple of 8
        hipLaunchKernelGGL(ffn_add_parts, dim3((unsigned)((2 * n + 255) / 256)), dim3(256), 0, st, p2, p1, n, 2 * n);
      } else {
        launch(Tile64x128{}, Tile128{}, Store{});
      }
      if (alone) launch_gemm<KIND_NT, EPI_STORE>(dx, dtype, tile, st);
      return moe::check_launch();
    }
  }
  if (dtype == MOE_F32) {   // one launch here too
    auto launch = [&](auto tile_tag, auto wide) {
      constexpr int T = decltype(tile_tag)::value;
      prepare_f32(dx, false, T); prepare_f32(w2, true, T); prepare_f32(w1, true, T);
      const int nbx = grid_of(dx), nb2 = grid_of(w2), nb1 = grid_of(w1);
      hipLaunchKernelGGL((ffn_bwd_trio_f32<T, decltype(wide)::value>), dim3((unsigned)(nbx + nb2 + nb1)), dim3(256), 0, st, dx, w2, w1, nbx, nb2);
    };
    if (plan_f32_trio(dx, w2, w1) == 64) launch(I64{}, std::false_type{});
    else if (!wide_f32(dx) && !wide_f32(w2) && !wide_f32(w1)) launch(I32{}, std::false_type{});
    else launch(I32{}, std::true_type{});
    return moe::check_launch();
  }
  launch_weight_small(w2, st);
  launch_weight_small(w1, st);
  launch_gemm<KIND_NT, EPI_STORE>(dx, dtype, tile, st);
  return moe::check_launch();
}

extern "C" int moe_expert_ffn_bwd(const void* dY, const void* X, const void* Z, const void* A, const void* W1,
                                  const void* W2, int dtype, int n_src, int G, int64_t C, int M, int H, int esp_idx,
                                  int n_esp, const int32_t* row_counts, int tile, void* dX, void* dW1, void* dW2,
                                  void* ws, size_t ws_bytes, void* stream) {
  return ffn_bwd_impl(dY, X, nullptr, 0, 0, Z, A, W1, W2, dtype, n_src, G, C, M, H, esp_idx, n_esp, row_counts, tile, dX,
                      dW1, dW2, ws, ws_bytes, stream);
}

extern "C" int moe_expert_ffn_bwd_gather(const void* dY, const void* x, int64_t S, const int32_t* inv, int k,
                                         const void* Z, const void* A, const void* W1, const void* W2, int dtype, int E,
                                         int64_t C, int M, int H, int esp_idx, int n_esp, const int32_t* row_counts,
                                         int tile, void* dX, void* dW1, void* dW2, void* ws, size_t ws_bytes,
                                         void* stream) {
  if (int rc = check_gather(x, dtype, S, inv, k, M)) return rc;
  MOE_REQUIRE((int64_t)E * C <= (1ll << 29), MOE_EUNSUPPORTED);   // 32-bit byte offsets into the slot map
  return ffn_bwd_impl(dY, x, inv, k, S, Z, A, W1, W2, dtype, 1, E, C, M, H, esp_idx, n_esp, row_counts, tile, dX, dW1, dW2,
                      ws, ws_bytes, stream);
}
