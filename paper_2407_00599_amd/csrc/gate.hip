// Gate of the MoE layer (Section II-A "Gating Function") on the rank's MP token slice
// (Section III-B): logits = x Wg (+bias), top-k, combine weights, capacity slots.
//
// Kernels (wave64 throughout):
//   gate_logits_split   : E <= 16, few tokens for their M.  A block owns 2 to 8 tokens, its waves split M.
//   gate_logits_few     : 16 tokens x 16 experts per block on the fp64 matrix cores (v_mfma_f64_16x16x4_f64), the waves split M.
//   gate_logits_mfma4   : E <= 8, many bf16 tokens: the matrix cores' form with four 4 x 4 blocks.
//   gate_logits_mfma    : E > 16, many tokens.  64 tokens x 64 experts per block.
//   gate_topk           : W lanes per token, k arg-max rounds (ties -> lower expert index); softmax weights;
//                         per-block (choice, expert) histogram for the slot scan.  With a single token block it
//                         assigns the slots as well.  (The logits kernels for up to 16 experts select them
//                         themselves, up to three choices of a few hundred to a few thousand tokens.)
//   gate_scan           : one wave per expert; exclusive scan of the histograms over token blocks and
//                         over choices (choice-major priority), per-expert demand counts.
//   gate_slots          : rank of each (token, choice) inside its block via wave ballots,
//                         slot = base + rank if < C; inverse map; -1 tails of inv.
// The logits are accumulated in fp64 and rounded once to fp32, so the routing decision is
// taken on the same fp32 numbers a double-precision reference produces.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"

// Scratch of moe_gate_topk_static: the per-block histograms and their scan, which moe_gate_topk keeps in
// the caller's workspace.  One copy per GPU, held until the process ends.  In host code this name is only a
// handle for hipGetSymbolAddress; kernels are given the address that call returns for the current device.
static __device__ __align__(256) unsigned char scratch[MOE_GATE_STATIC_SCRATCH_BYTES];

namespace {

using namespace moe;

constexpr int GATE_TB = 64;   // tokens per block in gate_topk / gate_slots (one per thread)

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl_xor(lo, mask, 64);
  hi = __shfl_xor(hi, mask, 64);
  return __hiloint2double(hi, lo);
}

constexpr int TOPK_MAX = 3;
struct TopK {      // what a logits kernel that also selects the experts writes (k = 0: it does not)
  int k, norm;
  int32_t* idx;
  float* w;
};
// Top-k of one token by one thread, whose logits it holds: v[0 .. E - 1], E <= EPL.  The same steps as in gate_topk, where a lane holds
// all of a token's experts: the k rounds are a loop, so that there is little code to fetch.  sel takes the chosen logits, `stride` apart,
// in LDS.
template <int EPL>
__device__ __forceinline__ void pick_experts(const float (&v)[EPL], int E, int k, int norm_topk, float* sel, int stride,
                                             int32_t* __restrict__ idx, float* __restrict__ w) {
  unsigned taken = E < 32 ? ~0u << E : 0u;
  float mx = 0.f, den = 0.f;
  for (int j = 0; j < k; ++j) {
    float cv = 0.f;
    int ce = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (!(taken & (1u << i)) && (ce == 0x7fffffff || v[i] > cv)) { cv = v[i]; ce = i; }
    taken |= 1u << (ce & 31);
    if (j == 0) mx = cv;
    den += expf(cv - mx);
    sel[j * stride] = cv;
    idx[j] = min(ce, E - 1);
  }
  if (!norm_topk) {   // weights over all experts instead of the selected ones
    den = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (i < E) den += expf(v[i] - mx);
  }
  for (int j = 0; j < k; ++j) w[j] = expf(sel[j * stride] - mx) / den;
}

// E <= 16 and few tokens, where the latency of one block's walk along M is the time of the call: a block owns T
// tokens and its waves split M (pieces of 128, 2 consecutive m per lane).  A lane's weights are 2 E consecutive floats,
// read from L2 (with E = EC as 16-byte pieces) and converted once for the T tokens; the waves' sums are added through
// LDS.  Pieces of 4 m per lane need fewer requests, but a request then touches twice the lines, which several waves'
// requests push out of L1 before their other halves are read.  256 tokens x 4096, 8 experts: 13 us, where a walk in
// chunks staged through LDS with a barrier each took 49.  The 16 x 16 tiles took over many products that this kernel
// had; against them, the call: 2000 x 4096, 8 experts 13.7 and 21.0 us; 700 x 4096, 9 experts 15.5 and 19.8.
constexpr int LS_MAXW = 8;
template <int EC, bool BF16, int T, bool FULL>   // FULL: E = EC
__global__ __launch_bounds__(64 * LS_MAXW) void gate_logits_split(const void* __restrict__ x, const float* __restrict__ Wg,
                                                                  const float* __restrict__ bias, float* __restrict__ logits,
                                                                  int64_t S, int M, int E, const TopK tk) {
  constexpr int NOUT = T * EC;
  static_assert(NOUT == 32 || NOUT == 64, "the reduction below leaves an output in every lane or every second one");
  __shared__ double red[LS_MAXW][NOUT];
  __shared__ float lg[T][EC + 1], sel[TOPK_MAX * T];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const int64_t t0 = (int64_t)blockIdx.x * T;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Wg), 0, (uint32_t)((uint64_t)M * E * 4), 0x00020000);
  double acc[NOUT];
#pragma unroll
  for (int i = 0; i < NOUT; ++i) acc[i] = 0.0;
#pragma unroll 2
  for (int m = (wave * 64 + lane) * 2; m < M; m += nw * 128) {   // M % 8 == 0: both elements are in or out
    float xv[T][2];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const int64_t off = (t0 + t < S ? t0 + t : S - 1) * (int64_t)M + m;   // a token past the end: any row, not stored
      if (BF16) {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const bf16_t*>(x) + off);
        xv[t][0] = __uint_as_float(v << 16); xv[t][1] = __uint_as_float(v & 0xFFFF0000u);
      } else {
        const float2 v = *reinterpret_cast<const float2*>(reinterpret_cast<const float*>(x) + off);
        xv[t][0] = v.x; xv[t][1] = v.y;
      }
    }
    float wv[2][EC];
    if (FULL) {
      const float4* wp = reinterpret_cast<const float4*>(Wg + (int64_t)m * EC);
#pragma unroll
      for (int i = 0; i < EC / 2; ++i) {
        const float4 v = wp[i];
        float* d = &wv[4 * i / EC][(4 * i) % EC];
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
      }
    } else {   // an expert past the end: the next row's weights (behind the last row: zeros, from the descriptor), not stored
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int e = 0; e < EC; ++e)
          wv[q][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, (m + q) * E * 4 + e * 4, 0, 0));
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double wd[EC];
#pragma unroll
      for (int e = 0; e < EC; ++e) wd[e] = (double)wv[q][e];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const double xd = (double)xv[t][q];
#pragma unroll
        for (int e = 0; e < EC; ++e) acc[t * EC + e] = fma(xd, wd[e], acc[t * EC + e]);
      }
    }
  }
  // halving reduction over the lanes: after the step with lane mask lm a lane whose bit lm is set holds
  // the upper half of its value list, summed with its partner's; once a single value is left the
  // remaining lane bits are plain butterfly sums.  At the end lane l holds value l >> log2(64 / NOUT).
#pragma unroll
  for (int st = 0; st < 6; ++st) {
    const int lm = 32 >> st;
    if ((NOUT >> st) > 1) {
      const int h = NOUT >> (st + 1);
      const bool up = (lane & lm) != 0;
#pragma unroll
      for (int i = 0; i < h; ++i) {
        const double keep = up ? acc[i + h] : acc[i];
        const double send = up ? acc[i] : acc[i + h];
        acc[i] = keep + shfl_xor_f64(send, lm);
      }
    } else {
      acc[0] += shfl_xor_f64(acc[0], lm);
    }
  }
  constexpr int REP = 64 / NOUT;
  if (lane % REP == 0) red[wave][lane / REP] = acc[0];
  __syncthreads();
  if (threadIdx.x < NOUT) {
    const int64_t t = t0 + threadIdx.x / EC;
    const int e = threadIdx.x % EC;
    double v = 0.0;
    for (int q = 0; q < nw; ++q) v += red[q][threadIdx.x];
    const float l = (float)(bias && e < E ? v + (double)bias[e] : v);
    if (t < S && e < E) logits[t * E + e] = l;
    lg[threadIdx.x / EC][e] = l;
  }
  if (tk.k == 0) return;
  __syncthreads();
  if (threadIdx.x < T && t0 + threadIdx.x < S) {
    float v[EC];
#pragma unroll
    for (int e = 0; e < EC; ++e) v[e] = lg[threadIdx.x][e];
    const int64_t at = (t0 + threadIdx.x) * tk.k;
    pick_experts<EC>(v, E, tk.k, tk.norm, sel + threadIdx.x, T, tk.idx + at, tk.w + at);
  }
}

// E > 16: fp64 matrix cores.  v_mfma_f64_16x16x4_f64 multiplies a 16 x 4 by a 4 x 16 tile of doubles (lane l
// supplies A[l % 16][l / 16] and B[l / 16][l % 16], and receives D[4 r + l / 16][l % 16], r = 0..3).  Which k a quarter of the
// lanes feeds in which step is free as long as both operands agree: of a chunk of 32 it takes 8 consecutive ones, one a
// step, so that a token's operand is what lies in memory and needs no LDS.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int LM_KC = 32;
// 8 consecutive values of a token, as stored
template <bool BF16>
struct TokenPiece {
  uint4 r[BF16 ? 1 : 2];
  __device__ __forceinline__ void load(const void* row, int k, int M) {   // zeros behind the last one
    const uint4* p = reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(row) + (int64_t)(k < M ? k : 0) * (BF16 ? 2 : 4));
#pragma unroll
    for (int i = 0; i < (BF16 ? 1 : 2); ++i) {
      const uint4 v = p[i];
      r[i] = k < M ? v : make_uint4(0u, 0u, 0u, 0u);
    }
  }
  __device__ __forceinline__ double get(int i) const {
    if (BF16) {
      const uint32_t v = (&r[0].x)[i >> 1];
      return (double)__uint_as_float((i & 1) ? (v & 0xFFFF0000u) : (v << 16));
    }
    return (double)__uint_as_float((&r[BF16 ? 0 : i >> 2].x)[i & 3]);
  }
};

// Many tokens.  A block owns 64 tokens x 64 experts (grid.y walks the expert blocks); KW = 1, 2 or 4 groups of four waves take alternate
// chunks of M and add their sums through LDS at the end; a wave owns 16 tokens x 64 experts (four accumulator tiles).  The
// weights are converted once per group on their way into LDS ([k][expert], pitch 66 doubles: the two k rows of a 32-lane read
// fall into different halves of the banks), in two buffers: the next chunk is converted and stored between the current
// one's products, and the one after it requested.
// Bound by the fp64 matrix rate (77 TFLOP/s for the bare instruction) less the vector instructions between (a conversion costs
// a tenth of a matrix instruction): one per matrix instruction here, and four waves per SIMD, so that they, the barriers and the
// fetches hide behind other waves' products.  The fetches stand in no branch, so that the compiler can wait for them by count.
// 16384 x 2048 x 64: 91 us with both operands staged, two waves per SIMD and guarded fetches -> 68 us (63 TFLOP/s).
constexpr int LM_PITCH = 66;
template <bool BF16, int KW>
__global__ __launch_bounds__(256 * KW, 4) void gate_logits_mfma(const void* __restrict__ x, const float* __restrict__ Wg,
                                                                const float* __restrict__ bias, float* __restrict__ logits,
                                                                int64_t S, int M, int E) {
  constexpr int BUF = LM_KC * LM_PITCH, RED = (KW - 1) * 256 * 17;
  __shared__ double smem[KW * 2 * BUF > RED ? KW * 2 * BUF : RED];
  const int tid = threadIdx.x & 255, lane = tid & 63;
  const int kw = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t tb = (int64_t)blockIdx.x * 64;
  const int e0 = blockIdx.y * 64, kq = 8 * (lane >> 4);
  double* ws = smem + kw * 2 * BUF;
  constexpr uint32_t ESZ = BF16 ? 2 : 4;
  // Fetches go through descriptors that start at the chunk: a lane's offset (bytes) stays, the rest is uniform.  What does not
  // exist is fetched from somewhere else inside the tensor: tokens and experts past the end are not stored, values of k
  // past the end are zeroed in both operands (only the last chunk can have some).
  const int t = (int)min((int64_t)(wave * 16 + (lane & 15)), S - 1 - tb);
  const uint32_t xo = (uint32_t)t * (uint32_t)M * ESZ, xk = (uint32_t)kq * ESZ;   // 64 M ESZ < 2^32 (the host's check)
  const int k_last = (M - 1) / LM_KC * LM_KC;      // a chunk behind it is fetched from there, and counts as zeros
  auto fetch_x = [&](TokenPiece<BF16>& d, int k0) {
    k0 = min(k0, k_last);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(reinterpret_cast<const char*>(x)) + (tb * M + k0) * ESZ, 0, 0xFFFFFFF0u, 0x00020000);
    const uint32_t off = xo + (k0 + LM_KC <= M ? xk : k0 + kq < M ? xk : 0u);
#pragma unroll
    for (int i = 0; i < (BF16 ? 1 : 2); ++i) {
      typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
      const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 16 * i, 0);
      d.r[i] = make_uint4(v.x, v.y, v.z, v.w);
    }
  };
  // staging: expert tid % 64, k rows tid / 64 + 4 u
  const uint32_t we = (uint32_t)min(e0 + (tid & 63), E - 1) * 4u;
  float wraw[8];
  auto fetch_w = [&](int k0) {
    k0 = min(k0, k_last);
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Wg) + (int64_t)k0 * E, 0, 0xFFFFFFF0u, 0x00020000);
#pragma unroll
    for (int u = 0; u < 8; ++u)
      wraw[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)we, min(wave + 4 * u, M - 1 - k0) * E * 4, 0));
  };
  auto stage_w = [&](int buf, int k0) {
    if (k0 + LM_KC > M) {
#pragma unroll
      for (int u = 0; u < 8; ++u) wraw[u] = k0 + wave + 4 * u < M ? wraw[u] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) ws[buf * BUF + (wave + 4 * u) * LM_PITCH + (tid & 63)] = (double)wraw[u];
  };
  f64x4_t acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) acc[j] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  const int nch = (M + LM_KC * KW - 1) / (LM_KC * KW);
  auto chunk = [&](int c) { return (c * KW + kw) * LM_KC; };   // a group's last one may lie behind the end
  TokenPiece<BF16> piece[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    fetch_x(piece[c], chunk(c));
    fetch_w(chunk(c));
    if (c == 0) stage_w(0, chunk(0));
  }
  auto step = [&](int c, auto set) {
    constexpr int SET = decltype(set)::value;
    __syncthreads();   // chunk c is staged, and the other buffer is consumed
    const int k0 = chunk(c), k1 = chunk(c + 1), k2 = chunk(c + 2);
    if (k0 + LM_KC > M && k0 + kq >= M) {
#pragma unroll
      for (int i = 0; i < (BF16 ? 1 : 2); ++i) piece[SET].r[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    const double* w = ws + SET * BUF + kq * LM_PITCH + (lane & 15);
    auto products = [&](int s0) {
#pragma unroll
      for (int s = s0; s < s0 + 4; ++s) {
        const double a = piece[SET].get(s);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, w[s * LM_PITCH + j * 16], acc[j], 0, 0, 0);
      }
    };
    products(0);
    stage_w(SET ^ 1, k1);
    fetch_w(k2);
    products(4);
    fetch_x(piece[SET], k2);
  };
  int c = 0;
  for (; c + 1 < nch; c += 2) {
    step(c, std::integral_constant<int, 0>{});
    step(c + 1, std::integral_constant<int, 1>{});
  }
  if (c < nch) step(c, std::integral_constant<int, 0>{});
  if constexpr (KW > 1) {
    __syncthreads();
    double* red = smem + (wave * 64 + lane) * 17;   // 17: lanes on different banks
    if (kw > 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(kw - 1) * 256 * 17 + 4 * j + r] = acc[j][r];
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll 1
    for (int g = 0; g < KW - 1; ++g)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][r] += red[g * 256 * 17 + 4 * j + r];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int e = e0 + j * 16 + (lane & 15);
    if (e >= E) continue;
    const double bj = bias ? (double)bias[e] : 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t to = tb + wave * 16 + 4 * r + (lane >> 4);
      if (to < S) logits[to * E + e] = (float)(acc[j][r] + bj);
    }
  }
}

// Few tokens: a block owns 16 tokens x 16 experts, and its waves split M; both operands come from memory, whose values the
// lanes convert.  The time is the walk of one wave along M, so that the more compute units take part the better; with every one
// busy it is the fp64 matrix rate.  The gate's call: 512 x 4096, 64 experts, 189 us with 64 x 64 tiles (8 compute units) -> 23;
// 4096 x 2048, 64 experts, 100 -> 37; 16384 x 4096, 16 experts, 198 us with the 4-block form and 399 in fp32 with vector FMAs -> 61
// and 70.  Requests of four chunks at a time measured no better (4096 x 2048, 128 experts, 70 -> 82 us), nor did 32 experts per wave.
constexpr int LF_NW = 16;
template <bool BF16>
__global__ __launch_bounds__(64 * LF_NW, 4) void gate_logits_few(const void* __restrict__ x, const float* __restrict__ Wg,
                                                                 const float* __restrict__ bias, float* __restrict__ logits,
                                                                 int64_t S, int M, int E, const TopK tk) {
  __shared__ double red[LF_NW][4][64];
  __shared__ float lg[16][17], sel[TOPK_MAX * 16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nw = blockDim.x >> 6;
  const int64_t tb = (int64_t)blockIdx.x * 16;
  const int e0 = blockIdx.y * 16, kq = 8 * (lane >> 4);
  const int64_t t = min(tb + (lane & 15), S - 1);     // past the end: any row and any expert, not stored
  const void* row = reinterpret_cast<const char*>(x) + t * (int64_t)M * (BF16 ? 2 : 4);
  const float* wcol = Wg + min(e0 + (lane & 15), E - 1);
  f64x4_t acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) acc[i] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  for (int k0 = wave * LM_KC; k0 < M; k0 += nw * LM_KC) {
    const int k = k0 + kq;      // M % 8 == 0: a lane's 8 values are in or out together
    TokenPiece<BF16> a;
    a.load(row, k, M);
    float w[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const float v = wcol[(int64_t)((k < M ? k : 0) + s) * E];
      w[s] = k < M ? v : 0.f;
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) acc[s & 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a.get(s), (double)w[s], acc[s & 1], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[0][r] + acc[1][r];
  __syncthreads();
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    const int r = i >> 6, l = i & 63, e = e0 + (l & 15);
    double v = 0.0;
    for (int q = 0; q < nw; ++q) v += red[q][r][l];
    const int64_t to = tb + 4 * r + (l >> 4);
    const float f = (float)(bias && e < E ? v + (double)bias[e] : v);
    if (to < S && e < E) logits[to * E + e] = f;
    lg[4 * r + (l >> 4)][l & 15] = f;
  }
  if (tk.k == 0) return;      // (up to 16 experts: the block has all of a token's logits)
  __syncthreads();
  if (threadIdx.x < 16 && tb + threadIdx.x < S) {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) v[e] = lg[threadIdx.x][e];
    const int64_t at = (tb + threadIdx.x) * tk.k;
    pick_experts<16>(v, E, tk.k, tk.norm, sel + threadIdx.x, 16, tk.idx + at, tk.w + at);
  }
}

// E <= 8 and many tokens: the fp64 matrix cores in their 4-block form.  v_mfma_f64_4x4x4_4b_f64 multiplies
// four independent 4 x 4 tiles by 4 x 4 tiles (k = 4) per instruction: lane l = 16 kk + 4 blk + i supplies
// A_blk[i][kk] and B_blk[kk][i], and receives D_blk[l / 16][l % 4] for blk = (l / 4) % 4 (layout confirmed with
// a one-wave probe).  On this chip the instruction runs on the fp64 vector units at their FMA rate (16
// cycles, during which the SIMD issues no other vector instruction), so what it buys is not arithmetic
// rate but structure: no cross-lane reduction, and every converted x value feeds 4 experts per
// instruction.  The conversion bf16 -> fp64 costs 20 cycles per 64 values (v_cvt_f64_f32 is quarter rate),
// as much as 1.25 matrix instructions, so each value is converted exactly once per wave: the four blocks are
// four token groups (16 tokens per instruction) and the experts are taken in NP passes of 4 that share the
// converted A operand (NP = 1, 2 for E <= 4, 8).
//   x:  fetched with whole-line requests (a lane takes 16 bytes, eight consecutive lanes one 128-byte piece
//       of a token row = 64 m, one instruction 8 rows) three steps ahead into registers, then passed through
//       a wave-private LDS region to reach the operand layout, in which neighbouring lanes hold DIFFERENT
//       tokens.  A lane of the operand layout reads 16 bytes = 8 consecutive m of its token, which feed 8
//       instructions per pass (the k index of instruction s is m = base + 8 kk + s: any bijection between
//       lanes and m serves, as long as A and B agree); a 64-m step is two such groups.  Row r stores piece p at
//       slot p ^ r, which makes both the row-wise writes and the operand-layout reads conflict-free.
//   Wg: converted to fp64 once per block and 512-m super-chunk on its way into LDS (double-buffered, one
//       barrier per super-chunk), in the order the lanes read it (16 bytes per lane; the four blocks read the
//       same addresses).
//   A block is TW x 2 waves: TW token waves (32 tokens each, two accumulator sets per pass), times 2 waves
//   that split the steps of a super-chunk and add their sums through LDS at the end.
//   Token rows and weights are fetched through buffer descriptors: an index outside the problem becomes an
//   out-of-range offset, which the hardware answers with zeros, so the loop body has no branches and the
//   compiler is free to interleave fetches, conversions and matrix instructions.
typedef unsigned int g4_u32x4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t G4_OOB = 0xFFFFFFF0u;
constexpr int G4_KW = 2, G4_NS = 2, G4_SB = 4, G4_TS = 16;
constexpr int G4_SC = 64 * G4_SB * G4_KW;    // m per super-chunk
template <int NP, int TW>
__global__ __launch_bounds__(64 * TW * G4_KW) void gate_logits_mfma4(const bf16_t* __restrict__ x, const float* __restrict__ Wg,
                                                                      const float* __restrict__ bias, float* __restrict__ logits,
                                                                      int64_t S, int M, int E) {
  constexpr int KW = G4_KW, NS = G4_NS, SB = G4_SB, SC = G4_SC, TS = G4_TS;
  constexpr int NT = 64 * TW * KW;
  constexpr int ROWS = NS * TS;        // tokens per wave
  constexpr int NLD = ROWS / 8;        // fetches per step (8 rows each)
  constexpr int EP = 4 * NP;           // experts, padded
  constexpr int STEP_D = 64 * EP;      // doubles per 64-m step: [u 2][pass NP][p 4][kk 4][j 4][2]
  constexpr int BUF_D = SB * KW * STEP_D;
  constexpr int NST = SC * EP / NT;    // staged weights per thread and super-chunk
  static_assert(SC * EP % NT == 0, "staging layout");
  constexpr int RED_D = TW * KW * NS * NP * 64;
  __shared__ __attribute__((aligned(16))) double Bs[(2 * BUF_D > RED_D ? 2 * BUF_D : RED_D)];
  __shared__ __attribute__((aligned(16))) char Xs[TW * KW * ROWS * 128];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int tw = wave / KW, kw = wave % KW;
  const int kk = lane >> 4, blk = (lane >> 2) & 3, li = lane & 3;
  const int tok_in_set = 4 * blk + li;
  const int64_t tset0 = ((int64_t)blockIdx.x * TW + tw) * ROWS;   // first token of this wave
  const int nsc = (M + SC - 1) / SC;

  // descriptors over the rank's token rows [S, M] and over Wg [M, E] (the host checks both are below 4 GiB)
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(x), 0, (uint32_t)((uint64_t)S * M * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Wg), 0, (uint32_t)((uint64_t)M * E * 4), 0x00020000);

  // ---- weights: global -> registers -> fp64 in LDS, in the lanes' read order ----
  // thread tid stages expert e = tid % EP of the rows ml0 + n (NT / EP), n = 0 .. NST - 1, of a super-chunk
  float wreg[NST];
  const int w_e = tid % EP, w_ml0 = tid / EP;
  const uint32_t w_step = (uint32_t)(NT / EP) * (uint32_t)E * 4u;
  auto fetch_w = [&](int sc) {
    const int m_first = sc * SC + w_ml0;
    const uint32_t base = ((uint32_t)m_first * (uint32_t)E + (uint32_t)w_e) * 4u;
#pragma unroll
    for (int n = 0; n < NST; ++n) {
      const bool ok = (m_first + n * (NT / EP) < M) & (w_e < E);
      const uint32_t off = ok ? base + (uint32_t)n * w_step : G4_OOB;
      wreg[n] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, (int)off, 0, 0));
    }
  };
  auto stage_w = [&](int buf) {
    double* dst = Bs + buf * BUF_D;
#pragma unroll
    for (int n = 0; n < NST; ++n) {
      const int idx = tid + n * NT, ml = idx / EP, e = idx % EP;
      const int st = ml >> 6, r = ml & 63, u = r >> 5, k4 = (r & 31) >> 3, sx = r & 7;   // group u = the 32-m half
      const int ps = e >> 2, j = e & 3;
      dst[st * STEP_D + ((((u * NP + ps) * 4 + (sx >> 1)) * 4 + k4) * 4 + j) * 2 + (sx & 1)] = (double)wreg[n];
    }
  };

  // ---- token rows: ring of SB register sets in the fetch layout (row = lane / 8, 16-byte piece = lane % 8) ----
  uint4 raw[SB][NLD];
  uint32_t row_off[NLD];                     // byte offset of this lane's piece at m = 0, or out of range
#pragma unroll
  for (int ld = 0; ld < NLD; ++ld) {
    const int64_t t = tset0 + 8 * ld + (lane >> 3);
    row_off[ld] = t < S ? (uint32_t)(((uint64_t)t * M + 8 * (lane & 7)) * 2) : G4_OOB;
  }
  auto fetch_x = [&](int n, int slot) {      // n = this wave's step number: super-chunk n / SB, step kw SB + n % SB
    const int m0 = (n / SB) * SC + (kw * SB + n % SB) * 64;
    const bool in = m0 + 8 * (lane & 7) < M;
#pragma unroll
    for (int ld = 0; ld < NLD; ++ld) {
      const uint32_t off = (row_off[ld] != G4_OOB && in) ? row_off[ld] + (uint32_t)m0 * 2u : G4_OOB;
      const g4_u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)off, 0, 0);
      raw[slot][ld] = make_uint4(v.x, v.y, v.z, v.w);
    }
  };
  // wave-private LDS region [ROWS][8 pieces of 16 bytes], piece p of row r at slot p ^ (r % 8)
  char* xw = Xs + wave * (ROWS * 128);
  const int wr_off = (lane >> 3) * 128 + (((lane & 7) ^ (lane >> 3)) * 16);        // + ld * 1024
  int rd_off[NS][2];                                                              // set q, group u
#pragma unroll
  for (int q = 0; q < NS; ++q)
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int r = q * TS + tok_in_set;
      rd_off[q][u] = r * 128 + (((4 * u + kk) ^ (r & 7)) * 16);
    }
  const int b_off = (kk * 4 + li) * 2;       // this lane's place among the 16 B lanes of a pass (doubles)

  double acc[NS][NP];
#pragma unroll
  for (int q = 0; q < NS; ++q)
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) acc[q][ps] = 0.0;

  fetch_w(0);
  const int nsteps = nsc * SB;
#pragma unroll
  for (int n = 0; n < SB - 1; ++n) fetch_x(n, n);
  stage_w(0);
  __syncthreads();

  for (int sc = 0; sc < nsc; ++sc) {
    if (sc + 1 < nsc) fetch_w(sc + 1);
    const double* bbuf = Bs + (sc & 1) * BUF_D + kw * SB * STEP_D + b_off;
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) {
      const int n = sc * SB + sb;
      if (n + SB - 1 < nsteps) fetch_x(n + SB - 1, (sb + SB - 1) % SB);
      // fetch layout -> operand layout through the wave's LDS region (LDS operations of a wave complete in order)
#pragma unroll
      for (int ld = 0; ld < NLD; ++ld) *reinterpret_cast<uint4*>(xw + ld * 1024 + wr_off) = raw[sb][ld];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        double da[NS][8];                    // the 8 values of this lane's piece, converted once
#pragma unroll
        for (int q = 0; q < NS; ++q) {
          const uint4 v = *reinterpret_cast<const uint4*>(xw + rd_off[q][u]);
#pragma unroll
          for (int sx = 0; sx < 8; ++sx) {
            const uint32_t wd = (&v.x)[sx >> 1];
            da[q][sx] = (double)__uint_as_float((sx & 1) ? (wd & 0xFFFF0000u) : (wd << 16));
          }
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          double2 b2[NP];
#pragma unroll
          for (int ps = 0; ps < NP; ++ps)
            b2[ps] = *reinterpret_cast<const double2*>(bbuf + sb * STEP_D + ((u * NP + ps) * 4 + p) * 32);
#pragma unroll
          for (int ps = 0; ps < NP; ++ps)
#pragma unroll
            for (int q = 0; q < NS; ++q) acc[q][ps] = __builtin_amdgcn_mfma_f64_4x4x4f64(da[q][2 * p], b2[ps].x, acc[q][ps], 0, 0, 0);
#pragma unroll
          for (int ps = 0; ps < NP; ++ps)
#pragma unroll
            for (int q = 0; q < NS; ++q) acc[q][ps] = __builtin_amdgcn_mfma_f64_4x4x4f64(da[q][2 * p + 1], b2[ps].y, acc[q][ps], 0, 0, 0);
        }
      }
    }
    if (sc + 1 < nsc) stage_w((sc + 1) & 1);
    __syncthreads();
  }

  // ---- add the KW partial sums through LDS (the weight buffers are free now) and store ----
  double* red = Bs;
  if (kw != 0) {
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
      for (int ps = 0; ps < NP; ++ps) red[(((tw * KW + kw) * NS + q) * NP + ps) * 64 + lane] = acc[q][ps];
  }
  __syncthreads();
  if (kw == 0) {
    const int i = lane >> 4, j = lane & 3;
#pragma unroll
    for (int ps = 0; ps < NP; ++ps) {
      const int e = 4 * ps + j;
      const double bj = (bias != nullptr && e < E) ? (double)bias[e] : 0.0;
#pragma unroll
      for (int q = 0; q < NS; ++q) {
        double v = acc[q][ps];
#pragma unroll
        for (int w2 = 1; w2 < KW; ++w2) v += red[(((tw * KW + w2) * NS + q) * NP + ps) * 64 + lane];
        const int64_t t = tset0 + q * TS + 4 * blk + i;
        if (t < S && e < E) logits[t * E + e] = (float)(v + bj);
      }
    }
  }
}

struct Cand {
  float v;
  int e;  // INT_MAX = no candidate
};
__device__ __forceinline__ Cand better(Cand a, Cand b) {
  if (b.e == 0x7fffffff) return a;
  if (a.e == 0x7fffffff) return b;
  if (b.v > a.v || (b.v == a.v && b.e < a.e)) return b;
  return a;
}

// Rank of each lane's expert among the lanes before it with the same expert (live lanes only).
__device__ __forceinline__ int match_rank(int e, bool live, int E, int lane) {
  unsigned long long same = __ballot(live);
  for (int bit = 1; bit < E; bit <<= 1) {
    const unsigned long long has = __ballot((e & bit) != 0);
    same &= (e & bit) ? has : ~has;
  }
  return __popcll(same & ((1ull << lane) - 1ull));
}

// Top-k of TB tokens.  W lanes hold a token's logits (lane r of a group the experts r, r + W, ...; W EPL >= E): the
// arg-max rounds compare within a lane first and need log2(W) cross-lane steps, none up to 16 experts.  The rounds are
// a loop and the code is small: every launch fetches its instructions anew, and at a few hundred tokens that fetch is
// a good part of its time.
// ONE (all tokens fit in one block): the slots are assigned here, and neither histograms nor a second launch are
// needed.  32 tokens, 8 experts: 4 + 9 us in two launches -> 4 us.
constexpr int topk_tokens(int W, bool one) { return !one ? GATE_TB : 1024 / W < 256 ? 1024 / W : 256; }
template <int W, int EPL, bool ONE>
__global__ __launch_bounds__(topk_tokens(W, ONE) * W) void gate_topk(const float* __restrict__ logits, int64_t S, int E, int k,
                                                                     int norm_topk, int32_t* __restrict__ idx, float* __restrict__ w,
                                                                     int32_t* __restrict__ blockhist, int pair_major, int64_t C,
                                                                     int32_t* __restrict__ slot, int32_t* __restrict__ inv,
                                                                     int32_t* __restrict__ counts) {
  constexpr int TB = topk_tokens(W, ONE), NT = TB * W, NSUB = TB / 64;   // ONE: demand is counted per 64 tokens
  constexpr int EP = W * EPL;
  __shared__ int hist[(ONE ? NSUB : 1) * MOE_MAX_K * EP];
  __shared__ float selv[MOE_MAX_K * TB];
  __shared__ int sele[ONE ? MOE_MAX_K * TB : 1];
  __shared__ int count_s[ONE ? EP : 1];
  const int tid = threadIdx.x, lane = tid & 63, r = tid % W, tl = tid / W;
  const int npair = k * E;
  for (int i = tid; i < (ONE ? NSUB : 1) * npair; i += NT) hist[i] = 0;
  const int64_t t = (int64_t)blockIdx.x * TB + tl;
  const bool live = t < S;
  float v[EPL];
  unsigned taken = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = r + i * W;
    v[i] = logits[min(t, S - 1) * E + min(e, E - 1)];
    if (!(live && e < E)) taken |= 1u << i;
  }
  const unsigned absent = taken;
  __syncthreads();
  float mx = 0.f, den = 0.f;
  for (int j = 0; j < k; ++j) {
    Cand c{0.f, 0x7fffffff};
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (!(taken & (1u << i)) && (c.e == 0x7fffffff || v[i] > c.v)) c = Cand{v[i], r + i * W};
#pragma unroll
    for (int m = 1; m < W; m <<= 1) {
      Cand o;
      o.v = __shfl_xor(c.v, m, 64);
      o.e = __shfl_xor(c.e, m, 64);
      c = better(c, o);
    }
    if (c.e % W == r) taken |= 1u << (c.e / W & 31);
    if (j == 0) mx = c.v;
    den += expf(c.v - mx);
    if (live && r == 0) {
      const int e = min(c.e, E - 1);   // (logits that are not numbers can leave a group's lanes of different minds)
      selv[j * TB + tl] = c.v;
      if (ONE) sele[j * TB + tl] = e;
      idx[t * k + j] = e;
      atomicAdd(&hist[(ONE ? (tl >> 6) * npair : 0) + j * E + e], 1);
    }
  }
  if (!norm_topk) {   // weights over all experts instead of the selected ones
    den = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i)
      if (!(absent & (1u << i))) den += expf(v[i] - mx);
#pragma unroll
    for (int m = 1; m < W; m <<= 1) den += __shfl_xor(den, m, 64);
  }
  if (live) {   // a group's lanes are in one wave, whose LDS operations complete in order
    for (int j = r; j < k; j += W) w[t * k + j] = expf(selv[j * TB + tl] - mx) / den;
  }
  __syncthreads();
  if constexpr (!ONE) {
    // [choice][expert][block] for gate_scan, which reads a (choice, expert) row, or bytes [block][choice][expert]
    for (int i = tid; i < npair; i += NT) {
      if (pair_major) blockhist[(int64_t)i * gridDim.x + blockIdx.x] = hist[i];
      else reinterpret_cast<uint8_t*>(blockhist)[(int64_t)blockIdx.x * npair + i] = (uint8_t)hist[i];   // at most 64
    }
  } else {
    // choice-major queues: positions of the first token of every (64 tokens, choice, expert)
    for (int e = tid; e < E; e += NT) {
      int run = 0;
      for (int j = 0; j < k; ++j)
        for (int q = 0; q < NSUB; ++q) {
          const int h = hist[q * npair + j * E + e];
          hist[q * npair + j * E + e] = run;
          run += h;
        }
      count_s[e] = run;
      counts[e] = run;
    }
    __syncthreads();
    for (int u = tid >> 6; u < NSUB * k; u += NT / 64) {   // one wave per (choice, 64 tokens)
      const int j = u / NSUB, q = u - j * NSUB, tq = q * 64 + lane;
      const bool ok = tq < S;
      const int e = ok ? sele[j * TB + tq] : 0;
      const int rank = match_rank(e, ok, E, lane);
      if (ok) {
        const int pos = hist[q * npair + j * E + e] + rank;
        const bool keep = pos < C;
        slot[(int64_t)tq * k + j] = keep ? pos : -1;
        if (keep) inv[(int64_t)e * C + pos] = tq * k + j;
      }
    }
    const uint32_t total = (uint32_t)((int64_t)E * C);   // below 2^31
    for (uint32_t i = tid; i < total; i += NT) {
      const uint32_t e = i / (uint32_t)C;
      if (i - e * (uint32_t)C >= (uint32_t)count_s[e]) inv[i] = -1;
    }
  }
}

// blockhist[j][e][b] -> blockbase[j][e][b] = queue position of the first (token, choice j) of
// token block b at expert e.  Choice-major: all choice-0 demand of e precedes choice 1, ...
// One wave per expert; 64 blocks are scanned per step with a shuffle prefix sum.
__global__ __launch_bounds__(256) void gate_scan(const int32_t* __restrict__ blockhist, int nblk, int E, int k,
                                                 int32_t* __restrict__ blockbase, int32_t* __restrict__ counts) {
  const int lane = threadIdx.x & 63;
  const int e = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (e >= E) return;
  int run = 0;
  for (int j = 0; j < k; ++j) {
    const int64_t row = ((int64_t)j * E + e) * nblk;
    for (int b0 = 0; b0 < nblk; b0 += 64) {
      const int b = b0 + lane;
      const int h = b < nblk ? blockhist[row + b] : 0;
      int incl = h;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
      }
      if (b < nblk) blockbase[row + b] = run + incl - h;
      run += __shfl(incl, 63, 64);
    }
  }
  if (lane == 0) counts[e] = run;
}

// One block per GATE_TB tokens, wave j ranks choice j.
// SLOTS_SCAN: queue positions of the block's first tokens come from gate_scan (base, counts).
// SLOTS_HIST: every block works them out itself from the histograms [block][choice][expert] -- for each
// (choice j, expert e) the demand of the earlier blocks, plus all demand of the earlier choices -- which saves the
// scan launch; block 0 also writes counts.  Same integers either way.  A count of 64 tokens fits in a byte: rows of bytes are read
// four pairs at a time by groups of threads that share the blocks between them, and the groups' sums meet in LDS.  The rows come from
// the other XCDs' writes, and a thread's up to 16 requests at a time are in flight together: with a loop of strided int32 rows,
// which the compiler left one request deep, the gate of 8192 tokens x 2048, top-4 of 128, took 87.5 us, now 81.2; 4096 x 256, top-8 of
// 64, 21.8 and 19.1; 24000 x 64, top-3 of 32, 24.1 and 19.2.
// SLOTS_IDX: the same from the choices themselves, which every block counts (integer sums in LDS: the order does not matter); the
// logits kernel has then selected the experts, and there are no histograms.
constexpr int SLOT_NT = 512;
enum { SLOTS_SCAN, SLOTS_HIST, SLOTS_IDX };
template <int FROM>
__global__ __launch_bounds__(SLOT_NT) void gate_slots(const int32_t* __restrict__ idx, const int32_t* __restrict__ base,
                                                      int32_t* __restrict__ counts, int64_t S, int E, int k,
                                                      int64_t C, int32_t* __restrict__ slot, int32_t* __restrict__ inv) {
  static_assert(GATE_TB == 64 && SLOT_NT / 64 >= MOE_MAX_K, "a wave per choice, a lane per token");
  constexpr bool SELF = FROM != SLOTS_SCAN;
  __shared__ __attribute__((aligned(16))) int base_s[SELF ? MOE_MAX_K * MOE_MAX_E : 1];   // queue position of this block's first (j, e) token
  __shared__ __attribute__((aligned(16))) int tot_s[SELF ? MOE_MAX_K * MOE_MAX_E : 1];    // demand of (j, e) over all blocks
  __shared__ int count_s[SELF ? MOE_MAX_E : 1];              // total demand of expert e
  __shared__ int copies_s[FROM == SLOTS_IDX ? 2 * TOPK_MAX * 16 * 8 : 1];   // (up to 16 experts)
  const int tid = threadIdx.x, lane = tid & 63, j = tid >> 6;
  const int64_t t = (int64_t)blockIdx.x * GATE_TB + lane;
  const bool live = t < S && j < k;
  const int e = live ? idx[t * k + j] : 0;
  if (SELF) {
    const int nblk = (int)gridDim.x, me = (int)blockIdx.x, npair = k * E;
    if constexpr (FROM == SLOTS_HIST) {
      for (int i = tid; i < npair; i += SLOT_NT) base_s[i] = tot_s[i] = 0;
      __syncthreads();
    }
    if constexpr (FROM == SLOTS_IDX) {
      // [in front of this block's tokens, behind][pair][copy]: eight copies, or the lanes of a wave queue up at a few counters
      int* cnt = copies_s;
      for (int i = tid; i < 2 * npair * 8; i += SLOT_NT) cnt[i] = 0;
      __syncthreads();
      const int n = (int)(S * k), before = me * GATE_TB * k;      // S k < 2^31
      auto count = [&](int i, int ee) { atomicAdd(&cnt[((i < before ? 0 : npair) + i % k * E + ee) * 8 + (lane & 7)], 1); };
#pragma unroll 4
      for (int i = tid * 4; i < (n & ~3); i += SLOT_NT * 4) {
        const int4 v = *reinterpret_cast<const int4*>(idx + i);
        count(i, v.x); count(i + 1, v.y); count(i + 2, v.z); count(i + 3, v.w);
      }
      if (tid < (n & 3)) count((n & ~3) + tid, idx[(n & ~3) + tid]);
      __syncthreads();
      for (int i = tid; i < npair; i += SLOT_NT) {
        int pre = 0, post = 0;
#pragma unroll
        for (int c = 0; c < 8; ++c) { pre += cnt[i * 8 + c]; post += cnt[(npair + i) * 8 + c]; }
        base_s[i] = pre;
        tot_s[i] = pre + post;
      }
    }
    auto sum_rows = [&](auto vec_tag) {   // V pairs per thread and row
      typedef decltype(vec_tag) vec_t;
      constexpr int V = sizeof(vec_t);
      const vec_t* hist = reinterpret_cast<const vec_t*>(base);
      const int nu = npair / V;
      int lanes = 1;
      while (lanes < nu && lanes < SLOT_NT) lanes <<= 1;
      const int groups = SLOT_NT / lanes, gr = tid / lanes;
      auto add_up = [&](int u, auto u_tag) {
        constexpr int U = decltype(u_tag)::value;   // rows requested together
        uint32_t tot[2] = {}, pre[2] = {};   // two 16-bit sums each, of up to 512 rows (see the rule) of up to 64
        for (int b = gr; b < nblk; b += U * groups) {
          uint32_t h[U];
#pragma unroll
          for (int q = 0; q < U; ++q) h[q] = hist[(uint32_t)(min(b + q * groups, nblk - 1) * nu + u)];
#pragma unroll
          for (int q = 0; q < U; ++q) {
            const int bq = b + q * groups;
            const uint32_t v = bq < nblk ? h[q] : 0u, ev = v & 0x00FF00FFu, od = (v >> 8) & 0x00FF00FFu;
            tot[0] += ev; tot[1] += od;
            pre[0] += bq < me ? ev : 0u; pre[1] += bq < me ? od : 0u;
          }
        }
        int t[V], p[V];
#pragma unroll
        for (int q = 0; q < V; ++q) {
          t[q] = (int)(tot[q & 1] >> (8 * (q & 2)) & 0xFFFFu);
          p[q] = (int)(pre[q & 1] >> (8 * (q & 2)) & 0xFFFFu);
        }
        // Where a wave's lanes would queue up at few counters (lanes with the same pairs are `lanes` apart) they add up first: 100000 x
        // 64, top-1 of 4, 46.5 -> 29.8 us; x 256, top-2 of 4, 45.2 -> 38.5; but 200000 x 64, top-1 of 2 (V = 1, lanes = 2) 47.7 and 49.0, 70000 x
        // 64, top-2 of 16 (8 lanes) 30.9 and 31.5.
        const bool sum_first = lanes <= (V == 4 ? 2 : 1);
        if (sum_first)
          for (int o = lanes; o < 64; o <<= 1)
#pragma unroll
            for (int q = 0; q < V; ++q) { t[q] += __shfl_xor(t[q], o, 64); p[q] += __shfl_xor(p[q], o, 64); }
        if (!sum_first || lane < lanes) {
#pragma unroll
          for (int q = 0; q < V; ++q) { atomicAdd(&tot_s[u * V + q], t[q]); atomicAdd(&base_s[u * V + q], p[q]); }
        }
      };
      for (int u = tid % lanes; u < nu; u += lanes) {
        if (nblk <= 4 * groups) add_up(u, std::integral_constant<int, 4>{});
        else add_up(u, std::integral_constant<int, 16>{});
      }
    };
    if constexpr (FROM == SLOTS_HIST) {
      if (npair % 4 == 0) sum_rows(uint32_t{});
      else sum_rows(uint8_t{});
    }
    __syncthreads();
    // choice-major queues: all demand of the earlier choices at expert e comes first
    for (int ee = tid; ee < E; ee += SLOT_NT) {
      int run = 0;
      for (int c = 0; c < k; ++c) {
        base_s[c * E + ee] += run;
        run += tot_s[c * E + ee];
      }
      count_s[ee] = run;
      if (me == 0) counts[ee] = run;
    }
    __syncthreads();
  }
  if (j < k) {
    const int rank = match_rank(e, live, E, lane);
    if (live) {
      const int pos = (SELF ? base_s[j * E + e] : base[((int64_t)j * E + e) * gridDim.x + blockIdx.x]) + rank;
      const bool keep = pos < C;
      slot[t * k + j] = keep ? pos : -1;
      if (keep) inv[(int64_t)e * C + pos] = (int32_t)(t * k + j);
    }
  }
  // empty tail of every expert's block: slots [min(counts[e], C), C)
  const int64_t total = (int64_t)E * C;   // below 2^31
  for (int64_t i = (int64_t)blockIdx.x * SLOT_NT + tid; i < total; i += (int64_t)gridDim.x * SLOT_NT) {
    const uint32_t ee = (uint32_t)i / (uint32_t)C, c = (uint32_t)i - ee * (uint32_t)C;
    if (c >= (uint32_t)(SELF ? count_s[ee] : counts[ee])) inv[i] = -1;
  }
}

}  // namespace

// Address of the current device's copy of the scratch array, looked up once per device (with that device
// current) and kept; nullptr if the runtime refuses.
static void* static_scratch() {
  constexpr int MAX_DEV = 64;
  static void* ptr[MAX_DEV] = {};
  static std::mutex mu;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEV) return nullptr;
  std::lock_guard<std::mutex> lock(mu);
  if (ptr[dev] == nullptr) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
    ptr[dev] = p;
  }
  return ptr[dev];
}

extern "C" size_t moe_gate_workspace_bytes(int64_t S, int E, int k) {
  if (S < 1 || E < 1 || k < 1) return 0;
  const int64_t nblk = (S + GATE_TB - 1) / GATE_TB;
  return moe::align_up((size_t)nblk * k * E * sizeof(int32_t), 256) * 2;
}

// ws == nullptr: the workspace is this GPU's static scratch array (moe_gate_topk_static)
static int gate_topk_impl(const void* x, int x_dtype, const float* Wg, const float* gate_bias,
                          int64_t S_total, int M, int E, int k, int64_t C, int mp_idx, int n_mp, int norm_topk,
                          float* logits, int32_t* idx, int32_t* slot, float* w, int32_t* inv, int32_t* counts,
                          void* ws, size_t ws_bytes, bool static_ws, void* stream) {
  MOE_REQUIRE(n_mp >= 1 && mp_idx >= 0 && mp_idx < n_mp, MOE_EINVAL);
  MOE_REQUIRE(S_total >= 1 && S_total % n_mp == 0, MOE_EINVAL);
  const int64_t S = S_total / n_mp;
  if (int rc = moe::common_shape_check(S, x ? M : 8, E, k, C)) return rc;
  MOE_REQUIRE(norm_topk >= -1 && norm_topk <= 1, MOE_EINVAL);
  if (x) {
    MOE_REQUIRE(x_dtype == MOE_F32 || x_dtype == MOE_BF16, MOE_EINVAL);
    MOE_REQUIRE_PTR(x);
    MOE_REQUIRE_PTR(Wg);
  }
  MOE_OPTIONAL_PTR(gate_bias);
  MOE_REQUIRE_PTR(logits); MOE_REQUIRE_PTR(idx); MOE_REQUIRE_PTR(slot); MOE_REQUIRE_PTR(w);
  MOE_REQUIRE_PTR(inv); MOE_REQUIRE_PTR(counts);
  const size_t need = moe_gate_workspace_bytes(S, E, k);
  if (static_ws) {
    MOE_REQUIRE(need <= MOE_GATE_STATIC_SCRATCH_BYTES, MOE_ESCRATCH);
    ws = static_scratch();
    MOE_REQUIRE(ws != nullptr, MOE_ELAUNCH);
  } else {
    MOE_REQUIRE(ws != nullptr && ws_bytes >= need, MOE_EWORKSPACE);
    MOE_REQUIRE(moe::aligned16(ws), MOE_EALIGN);
  }
  const int norm = norm_topk < 0 ? (k >= 2 ? 1 : 0) : norm_topk;
  hipStream_t st = (hipStream_t)stream;
  const int nblk = (int)((S + GATE_TB - 1) / GATE_TB);
  int32_t* blockhist = (int32_t*)ws;
  int32_t* blockbase = (int32_t*)((char*)ws + need / 2);

  bool selected = false;   // the logits kernel selects the experts too
  if (x) {
    const bool bf = x_dtype == MOE_BF16;
    const size_t esz = bf ? 2 : 4;
    const void* xs = (const char*)x + (size_t)mp_idx * S * M * esz;
    TopK tk{0, norm, idx, w};
    // Up to 16 experts and three choices the logits kernels select the experts as well (a thread per token, whose rounds are a chain), and
    // gate_slots counts the choices, 2048 of them in a step of each block.  The call, three launches and two: 2048 x 768, 16 experts, top-2, 12.9
    // and 11.3 us; 4096 x 1024, 8, top-2, 13.6 and 12.4; x 256, three steps: 6000 choices, 2, top-1 8.9 and 9.3, 4, top-2 9.2 and 8.1, 8,
    // top-3 9.4 and 9.2, 16, top-1 10.6 and 9.5; four steps: 8000, 2, top-1 9.1 and 10.3, top-2 9.2 and 9.0, 8, top-2 9.3 and 9.3, top-3 9.5
    // and 10.4, 12, top-1 11.0 and 10.6, top-3 10.5 and 10.9, 16, top-2 9.9 and 9.8; 2000 x 512, 12, top-4, 12.0 and 12.6.  Up to 256 tokens
    // gate_topk assigns the slots as well, two launches either way, and its one block is the faster for few tokens of few experts:
    // 256 x 64, 2, top-1 5.8 and 6.4, 4, top-1 6.1 and 6.4, 4, top-3 7.4 and 7.5 (257 x 64, 4, top-1 10.6 and 6.4); 65 x 64, 8, top-1 6.2
    // and 6.4, top-2 6.6 and 6.6; 100 x 64, 8, top-2 6.9 and 6.6; 65 x 64, 16, top-3 8.7 and 9.0; 100 x 64, 12, top-1 7.3 and 7.5, 16,
    // top-2 7.8 and 7.7; 128 x 64, 16, top-2 7.9 and 7.75; 160 x 1024, 12, top-2 10.5 and 10.3.
    const int64_t one_block = E <= 4 ? 256 : E <= 8 ? 64 : 112;
    if (E <= 16 && k <= TOPK_MAX && S > one_block && S * k <= (k == 2 || (k == 1 && E >= 8) ? 8192 : 6144)) tk.k = k;
    auto launch_few = [&]() {
      selected = tk.k != 0;
      const dim3 grid((unsigned)((S + 15) / 16), (unsigned)((E + 15) / 16)), block(64 * std::min(LF_NW, (M + LM_KC - 1) / LM_KC));
      if (bf) hipLaunchKernelGGL(gate_logits_few<true>, grid, block, 0, st, xs, Wg, gate_bias, logits, S, M, E, tk);
      else hipLaunchKernelGGL(gate_logits_few<false>, grid, block, 0, st, xs, Wg, gate_bias, logits, S, M, E, tk);
    };
    // Up to 16 experts.  What the 16 x 16 tiles cost does not depend on how many of the 16 columns are experts: 8192 x 1024 17 us (the
    // call), 16384 x 4096 61, fp32 29 at 16384 x 1024.  The others are faster
    // - with many tokens in bf16, where 8 or 4 columns are not multiplied (mfma4): 8 experts, 8192 x 1024 17.7 and 15.2, 9000 x 1024 18.0 and
    //   19.1, 14000 x 2048 27.8 and 36.1, 32768 x 4096 69 and 114, but 14000 x 256 14.1 and 12.7; 4 experts, 7000 x 2048 19.7 and 22.2, 8192 x 2048
    //   19.8 and 22.4; but 16 experts, 32768 x 4096 126 and 114;
    // - with few tokens for their M, where the walk along M is the time (split): it goes by its blocks per compute unit.
    // Up to 8 experts a block has 4 tokens or, from 1024 on, 8, and 2048 / blocks waves.  Split and 16 x 16 tiles, 8 experts, bf16 where not said:
    //   up to 1024 tokens 512 x 1024 13.5 and 14.0, 1000 x 512 7.7 and 8.1;
    //   one block a compute unit (2048 tokens): 2000 x 1024 11.4 and 9.9, x 1536 12.0 and 11.7, x 2048 11.7 and 13.1, x 4096 13.7 and 21.0;
    //   some one and some two: 2500 x 2048 18.6 and 13.6, x 4096 23.1 and 21.4;
    //   two (4096): 4096 x 1536 12.8 and 12.3, x 2048 13.6 and 14.4, x 4096 17.7 and 21.6, fp32 x 2048 16.5 and 15.3, x 4096 24.2 and 24.6;
    //   two waves a block: 6000 x 1024 13.8 and 14.3, 5000 x 1536 15.4 and 17.3, 8000 x 2048 19.9 and 22.7, x 4096 26.8 and 35.1; fp32 5000 x 2048
    //     26.5 and 22.6, 6000 x 2048 21.9 and 22.8, 8000 x 2048 25.8 and 24.7, 5000 x 4096 35.6 and 36.4.
    // From 9 experts on split's time goes by its blocks, of 2 tokens or, from 1024 on, 4, per compute unit, split and 16 x 16 tiles:
    //   one (512 tokens): 16 experts, 300 x 1024 11.5 and 10.0, 16 x 1536 10.7 and 11.0, 512 x 2048 13.6 and 13.3, 512 x 4096 18.4 and 20.1; 12,
    //     64 x 1024 9.8 and 9.5, 64 x 1536 10.1 and 11.3; 9, 64 x 520 8.7 and 8.2, 64 x 1024 9.5 and 9.5, fp32 9.6 and 10.0, 512 x 2048 11.2
    //     and 13.1;
    //   two (1023 tokens), which the products of 14 or 16 columns fill: 700 x 4096, 16 experts 24.0 and 20.2, 12 18.7 and 20.0, 9 15.5 and
    //     19.8; 1000 x 3072, 10 18.1 and 16.6, 9 16.5 and 16.7; 1000 x 8192, 14 36 and 33, 12 31 and 33;
    //   some one and some two: 1400 x 4096, 9 25.7 and 20.1;
    //   two of four waves, not the more that fewer blocks get (1641 to 2048 tokens): 2000 x 3072, 16 experts 21.9 and 17.4, 14 16.9 and 17.4,
    //     2000 x 4096, 14 18.9 and 21.6; 2000 x 2048, 9 14.3 and 13.6;
    //   more: 3000 x 4096, 9 23.5 and 22.0, 3000 x 8192, 12 40 and 36.
    const bool rows32 = (uint64_t)S * (uint64_t)M * 2 <= 0xFFFFFFF0ull;
    bool split;
    if (E <= 8) {
      const int least = S <= 2048 ? 2048 : S <= 4096 ? (bf ? 2048 : 3072) : bf || (S > 5400 && S <= 7000) ? 1536 : 3072;
      split = S < 1024 || ((S <= 2048 || (S > 3400 && S < 8192)) && M >= least);
    } else {
      split = S <= 512 ? M > 90 * E : S < 1024 ? E <= 12 && M >= 341 * E : S > 1640 && S <= 2048 && E <= 14 && M >= 3072;
    }
    if (bf && E <= 8 && rows32 && (E <= 4 ? S >= 8192 : M >= 512 ? S > 8192 : S >= 16384)) {
      // fp64 matrix cores; TW token waves (32 tokens each) per block so that the grid has about two blocks per
      // compute unit or more
      const int tw = S >= 512 * 4 * 32 ? 4 : S >= 512 * 2 * 32 ? 2 : 1;
      const int64_t tpb = (int64_t)tw * G4_NS * G4_TS;     // tokens per block
      const dim3 grid((unsigned)((S + tpb - 1) / tpb)), block(64 * tw * G4_KW);
      const bf16_t* xb = (const bf16_t*)xs;
#define LAUNCH_M4(np, tw_) hipLaunchKernelGGL((gate_logits_mfma4<np, tw_>), grid, block, 0, st, xb, Wg, gate_bias, logits, S, M, E)
#define LAUNCH_M4_TW(np) do { if (tw == 4) LAUNCH_M4(np, 4); else if (tw == 2) LAUNCH_M4(np, 2); else LAUNCH_M4(np, 1); } while (0)
      if (E <= 4) LAUNCH_M4_TW(1); else LAUNCH_M4_TW(2);
#undef LAUNCH_M4_TW
#undef LAUNCH_M4
    } else if (E <= 16 && split && (uint64_t)M * E * 4 < (1ull << 31)) {   // 32-bit offsets into Wg
      // As many waves over M as it has pieces.  From a thousand tokens on, twice the tokens per block (half the
      // weight traffic and conversions) and waves that walk several pieces, about 2048 of them in all, so that the
      // reduction at a wave's end does not outweigh its products.
      const bool many = S >= 1024;
      const int T = (E <= 8 ? 4 : 2) * (many ? 2 : 1);
      const int64_t blocks = (S + T - 1) / T;
      int nw = (M + 127) / 128 < LS_MAXW ? (M + 127) / 128 : LS_MAXW;
      if (many && nw > 2048 / blocks) nw = (int)(2048 / blocks);
      if (nw < 1) nw = 1;
      const dim3 grid((unsigned)blocks), block(64 * nw);
#define LAUNCH_SPLIT(ec, t, full) do { \
    if (bf) hipLaunchKernelGGL((gate_logits_split<ec, true, t, full>), grid, block, 0, st, xs, Wg, gate_bias, logits, S, M, E, tk); \
    else hipLaunchKernelGGL((gate_logits_split<ec, false, t, full>), grid, block, 0, st, xs, Wg, gate_bias, logits, S, M, E, tk); } while (0)
#define LAUNCH_SPLIT_E(full8, full16) do { \
    if (E <= 8) { if (many) LAUNCH_SPLIT(8, 8, full8); else LAUNCH_SPLIT(8, 4, full8); } \
    else { if (many) LAUNCH_SPLIT(16, 4, full16); else LAUNCH_SPLIT(16, 2, full16); } } while (0)
      if (E == 8 || E == 16) LAUNCH_SPLIT_E(true, true); else LAUNCH_SPLIT_E(false, false);
      selected = tk.k != 0;
#undef LAUNCH_SPLIT_E
#undef LAUNCH_SPLIT
    } else if (E <= 16) {
      launch_few();
    } else {
      // 16 x 16 tiles while 64 x 64 ones are at most 128 (half of the compute units).  The call, 64 x 64 and 16 x 16: 512 x 4096, 64
      // experts (8) 189 and 23 us; 4096 x 2048, 64 (64) 77 and 37; 128 (128) 82 and 71; 6144 x 2048, 128 (192) 80 and 93.
      // With two chunks of M at most a block is start and end only, and more than four 16 x 16 ones a compute unit are dearer: M = 64,
      // 4096 tokens, 64 experts (1024 blocks of 16 x 16) 12.4 and 10.6; 8192, 32 (1024) 11.6 and 10.3; 8192, 64 (2048) 13.0 and 14.4;
      // M = 16 11.3 and 10.7, 10.2 and 10.3, 11.8 and 14.2.
      // Groups over M: a group costs its chunks, rounded up, and the exchange of the sums.  Four while there is one block per
      // compute unit and M is long enough, 16384 x 2048, 64 experts: 81 us, two 86; one, two and four: 16384 tokens, 64 experts
      // (256 blocks), M = 64 13.5, 13.7, 16.8; 128 16.3, 16.3, 16.8; 192 18.8, 18.3, 21.2; 224 19.8, 20.7, 21.1; 256 21.4, 20.7, 21.2; 320
      // 24.1, 22.9, 25.3; 384 26.6, 25.2, 25.0; 1024 53.2, 48.1, 46.2; 9000 tokens, 128 (282) M = 96 19.9, 23.2, 26.9; 224 28.6, 31.0, 35.2;
      // 256 30.8, 31.1, 35.4; 512 47.9, 47.0, 51.4.
      const dim3 grid((unsigned)((S + 63) / 64), (unsigned)((E + 63) / 64));
      const uint64_t tiles = (uint64_t)grid.x * grid.y;
#define LAUNCH_WIDE(bf_, kw_) hipLaunchKernelGGL((gate_logits_mfma<bf_, kw_>), grid, dim3(256 * kw_), 0, st, xs, Wg, gate_bias, logits, S, M, E)
      const bool few = M <= 2 * LM_KC ? ((S + 15) / 16) * ((E + 15) / 16) <= 1024 : tiles <= 128;
      if (few || M >= 1 << 24) {   // (the other kernel has 32-bit offsets within a block's tokens)
        launch_few();
      } else if (M < 8 * LM_KC) {
        if (bf) LAUNCH_WIDE(true, 1); else LAUNCH_WIDE(false, 1);
      } else if (tiles <= 256 && M >= 12 * LM_KC) {
        if (bf) LAUNCH_WIDE(true, 4); else LAUNCH_WIDE(false, 4);
      } else {
        if (bf) LAUNCH_WIDE(true, 2); else LAUNCH_WIDE(false, 2);
      }
#undef LAUNCH_WIDE
    }
  }
  if (selected) {
    hipLaunchKernelGGL(gate_slots<SLOTS_IDX>, dim3(nblk), dim3(SLOT_NT), 0, st, idx, nullptr, counts, S, E, k, C, slot, inv);
    return moe::check_launch();
  }
  // Every block reads all histograms (a byte per block, choice and expert) itself up to 256 KiB of them and 64 MiB over all blocks.
  // The gate with the scan launch and without: 8192 x 256, top-8 of 256 (256 KiB, 32 MiB) 52.1 and 46.4 us; 16384 x 256, top-2 of 256 (128
  // KiB, 32 MiB) 57.6 and 54.0; 70000 x 64, top-2 of 16 (34 KiB, 37 MiB) 41.8 and 29.9; 32768 x 256, top-2 of 64 (64 KiB, 32 MiB) 40.2 and 32.9.
  const int64_t npair = (int64_t)k * E;
  const bool self = nblk * npair <= 1 << 18 && (int64_t)nblk * nblk * npair <= 1 << 26;
  auto route = [&](auto w_tag, auto epl_tag) {   // returns true: the slots are assigned too
    constexpr int W = decltype(w_tag)::value, EPL = decltype(epl_tag)::value;
    if (S <= topk_tokens(W, true)) {
      hipLaunchKernelGGL((gate_topk<W, EPL, true>), dim3(1), dim3(topk_tokens(W, true) * W), 0, st, logits, S, E, k, norm, idx,
                         w, blockhist, 0, C, slot, inv, counts);
      return true;
    }
    hipLaunchKernelGGL((gate_topk<W, EPL, false>), dim3(nblk), dim3(GATE_TB * W), 0, st, logits, S, E, k, norm, idx, w, blockhist,
                       self ? 0 : 1, C, slot, inv, counts);
    return false;
  };
  using std::integral_constant;
  bool done;
  if (E <= 4) done = route(integral_constant<int, 1>{}, integral_constant<int, 4>{});
  else if (E <= 8) done = route(integral_constant<int, 1>{}, integral_constant<int, 8>{});
  else if (E <= 16) done = route(integral_constant<int, 1>{}, integral_constant<int, 16>{});
  else if (E <= 32) done = route(integral_constant<int, 4>{}, integral_constant<int, 8>{});
  else if (E <= 64) done = route(integral_constant<int, 8>{}, integral_constant<int, 8>{});
  else if (E <= 128) done = route(integral_constant<int, 8>{}, integral_constant<int, 16>{});
  else done = route(integral_constant<int, 16>{}, integral_constant<int, 16>{});
  if (done) return moe::check_launch();
  if (self) {
    hipLaunchKernelGGL(gate_slots<SLOTS_HIST>, dim3(nblk), dim3(SLOT_NT), 0, st, idx, blockhist, counts, S, E, k, C, slot, inv);
  } else {
    hipLaunchKernelGGL(gate_scan, dim3((E + 3) / 4), dim3(256), 0, st, blockhist, nblk, E, k, blockbase, counts);
    hipLaunchKernelGGL(gate_slots<SLOTS_SCAN>, dim3(nblk), dim3(SLOT_NT), 0, st, idx, blockbase, counts, S, E, k, C, slot, inv);
  }
  return moe::check_launch();
}

extern "C" int moe_gate_topk(const void* x, int x_dtype, const float* Wg, const float* gate_bias,
                             int64_t S_total, int M, int E, int k, int64_t C, int mp_idx, int n_mp, int norm_topk,
                             float* logits, int32_t* idx, int32_t* slot, float* w, int32_t* inv, int32_t* counts,
                             void* ws, size_t ws_bytes, void* stream) {
  return gate_topk_impl(x, x_dtype, Wg, gate_bias, S_total, M, E, k, C, mp_idx, n_mp, norm_topk, logits, idx, slot, w,
                        inv, counts, ws, ws_bytes, false, stream);
}

extern "C" int moe_gate_topk_static(const void* x, int x_dtype, const float* Wg, const float* gate_bias,
                                    int64_t S_total, int M, int E, int k, int64_t C, int mp_idx, int n_mp,
                                    int norm_topk, float* logits, int32_t* idx, int32_t* slot, float* w,
                                    int32_t* inv, int32_t* counts, void* stream) {
  return gate_topk_impl(x, x_dtype, Wg, gate_bias, S_total, M, E, k, C, mp_idx, n_mp, norm_topk, logits, idx, slot, w,
                        inv, counts, nullptr, 0, true, stream);
}
