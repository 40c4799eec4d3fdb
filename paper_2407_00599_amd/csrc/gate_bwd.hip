// Backward of the gating function of Section II-A (linear layer + softmax + top-k), with the
// top-k selection held fixed.
//
//   E <= 16 : gate_bwd_fused (dlogits, dx and the dWg partial sums in one kernel) + gate_dwg_reduce.
//   E  > 16 : with norm_topk and many experts per selected one, gate_dx_sparse (dlogits and dx) and gate_dwg_sparse, which take
//             the selected experts only, + gate_dwg_reduce; otherwise gate_dlogits (one wave per token), gate_dx_wide (dx[t,m] (+)= sum_e dl[t,e]
//             Wg[m,e]), gate_dwg_wide + gate_dwg_reduce.
//   dl: norm_topk: dl[e_j] = w_j (dw_j - sum_j' w_j' dw_j'), otherwise dl[e] = sum_j dw_j p[e_j] (delta(e,e_j) - p[e]) with
//   p = softmax(l).
//   dWg[m,e] = sum_t x[t,m] dl[t,e] is formed as per-token-chunk fp32 partial sums followed by a
//   fixed-order fp64 reduction (no atomics, so the result is the same on every run); dbias[e] =
//   sum_t dl[t,e] rides along as an extra row m = M of the partials.
#include <algorithm>

#include "common.h"

namespace {

using namespace moe;

// tokens per dWg partial sum: a multiple of 8, at least 8, and at most 256 partial sums
// (more than 16 experts: at most 64 partial sums of at least 64 tokens, the partials being E/8 times larger)
inline int dwg_chunk(int64_t S, int E) {
  const int64_t parts = E <= 16 ? 256 : 64, least = E <= 16 ? 8 : 64;
  const int64_t c = (S + parts - 1) / parts;
  return (int)(c < least ? least : (c + 7) / 8 * 8);
}

// The selected experts' weights and weight gradients of a token, all requested together.
struct Picks {
  float w[MOE_MAX_K], g[MOE_MAX_K];
  int e[MOE_MAX_K];
  float inner;   // sum_j w_j dw_j
  __device__ __forceinline__ Picks(const float* dw, const float* wt, const int32_t* idx, int64_t t, int k) {
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j) {
      const int64_t at = t * k + (j < k ? j : k - 1);
      w[j] = wt[at]; g[j] = dw[at]; e[j] = idx[at];
    }
    inner = 0.f;
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j)
      if (j < k) inner = fmaf(w[j], g[j], inner); else e[j] = -1;
  }
};

// E > 16: one wave per token, a lane per expert (four passes at most), so that rows of logits and dlogits are read and
// written whole.  8192 x 128: 36 us with a thread per token -> 5 us.
__global__ __launch_bounds__(256) void gate_dlogits(const float* __restrict__ dw, const float* __restrict__ w,
                                                    const int32_t* __restrict__ idx, const float* __restrict__ logits,
                                                    int64_t S, int E, int k, int norm_topk, float* __restrict__ dl) {
  constexpr int EPL = MOE_MAX_E / 64;
  const int lane = threadIdx.x & 63;
  const int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= S) return;
  const Picks p(dw, w, idx, t, k);
  float v[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) v[i] = 0.f;
  if (!norm_topk) {
    float l[EPL], mx = -__builtin_inff(), den = 0.f;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      l[i] = logits[t * E + min(lane + 64 * i, E - 1)];
      mx = fmaxf(mx, l[i]);
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      v[i] = expf(l[i] - mx);
      if (lane + 64 * i < E) den += v[i];
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) den += __shfl_xor(den, d, 64);
#pragma unroll
    for (int i = 0; i < EPL; ++i) v[i] = -(v[i] / den) * p.inner;
  }
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane + 64 * i;
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j)
      if (p.e[j] == e) v[i] += norm_topk ? p.w[j] * (p.g[j] - p.inner) : p.w[j] * p.g[j];
    if (e < E) dl[t * E + e] = v[i];
  }
}

template <bool BF16>
__device__ __forceinline__ void st8g(void* base, int64_t off, const float* f) {
  if (BF16) {
    *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(base) + off) = pack_bf16x8(f);
  } else {
    float4* p = reinterpret_cast<float4*>(reinterpret_cast<float*>(base) + off);
    p[0] = make_float4(f[0], f[1], f[2], f[3]);
    p[1] = make_float4(f[4], f[5], f[6], f[7]);
  }
}

// dWg[i] = sum over the chunks of partial[chunk][i], in a fixed order: the four waves of a block take
// every fourth group of four chunks each (four running fp64 sums apiece, so sixteen loads are in flight
// per output), and wave 0 adds the four results.
// BY_EXPERT: the sums lie as [chunk][E][M], the bias rows [chunk][E] behind them all.
template <bool BY_EXPERT>
__global__ __launch_bounds__(256) void gate_dwg_reduce(const float* __restrict__ partial, int nchunk, int M, int E,
                                                       float* __restrict__ dWg, float* __restrict__ dbias) {
  __shared__ double red[4][64];
  const int o = threadIdx.x & 63, gq = threadIdx.x >> 6;
  int64_t i = (int64_t)blockIdx.x * 64 + o;
  int64_t n = (int64_t)(M + 1) * E;
  const int64_t me = (int64_t)M * E, first = i;
  if (BY_EXPERT) {
    if (i < me) n = me;
    else if (i < n) { partial += me * nchunk; i -= me; n = E; }
  }
  double s[4] = {0, 0, 0, 0};
  if (i < n) {
    int c = gq * 4;
    for (; c + 20 <= nchunk; c += 32) {   // two of this wave's groups at a time: eight loads in flight
      float v[8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        v[u] = partial[(int64_t)(c + u) * n + i];
        v[4 + u] = partial[(int64_t)(c + 16 + u) * n + i];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += (double)v[u];
#pragma unroll
      for (int u = 0; u < 4; ++u) s[u] += (double)v[4 + u];
    }
    for (; c < nchunk; c += 16) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c + u < nchunk) s[u] += (double)partial[(int64_t)(c + u) * n + i];
    }
  }
  red[gq][o] = (s[0] + s[1]) + (s[2] + s[3]);
  __syncthreads();
  if (gq == 0 && i < n) {
    const double t = (red[0][o] + red[1][o]) + (red[2][o] + red[3][o]);
    if (first < me) dWg[BY_EXPERT ? i % M * E + i / M : i] = (float)t;
    else if (dbias) dbias[first - me] = (float)t;
  }
}

template <bool BF16>
__device__ __forceinline__ void st4g(void* base, int64_t off, const float* f) {
  if (BF16) {
    *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(base) + off) = make_uint2(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]));
  } else {
    *reinterpret_cast<float4*>(reinterpret_cast<float*>(base) + off) = make_float4(f[0], f[1], f[2], f[3]);
  }
}
template <bool BF16>
__device__ __forceinline__ void st4g(__amdgpu_buffer_rsrc_t row, uint32_t at, const float (&f)[4]) {
  if (BF16) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u32x2{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3])}, row, at, 0, 0);
  } else {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])}, row, at, 0, 0);
  }
}

// raw (unconverted) CPT elements of a row: requested for all tokens of a stage first, converted when used
template <bool BF16, int CPT>
struct RawRow {
  uint32_t r[BF16 ? CPT / 2 : CPT];
  __device__ __forceinline__ void load(const void* base, int64_t off) {
    constexpr int NB = (BF16 ? CPT / 2 : CPT) * 4;   // bytes: 8, 16 or 32
    const char* p = reinterpret_cast<const char*>(base) + off * (BF16 ? 2 : 4);
    if (NB == 8) { const uint2 v = *reinterpret_cast<const uint2*>(p); r[0] = v.x; r[1] = v.y; }
    else {
#pragma unroll
      for (int i = 0; i < NB / 16; ++i) {
        const uint4 v = reinterpret_cast<const uint4*>(p)[i];
        r[4 * i] = v.x; r[4 * i + 1] = v.y; r[4 * i + 2] = v.z; r[4 * i + 3] = v.w;
      }
    }
  }
  __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t row, uint32_t at) {     // at: bytes
    constexpr int ND = BF16 ? CPT / 2 : CPT;
    if constexpr (ND == 2) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b64(row, at, 0, 0);
      r[0] = v[0]; r[1] = v[1];
    } else {
#pragma unroll
      for (int i = 0; i < ND / 4; ++i) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(row, at + 16 * i, 0, 0);
        r[4 * i] = v[0]; r[4 * i + 1] = v[1]; r[4 * i + 2] = v[2]; r[4 * i + 3] = v[3];
      }
    }
  }
  __device__ __forceinline__ void zero() {
#pragma unroll
    for (int i = 0; i < (BF16 ? CPT / 2 : CPT); ++i) r[i] = 0u;
  }
  __device__ __forceinline__ float get(int q) const {
    if (BF16) return __uint_as_float((q & 1) ? (r[q >> 1] & 0xFFFF0000u) : (r[q >> 1] << 16));
    return __uint_as_float(r[q]);
  }
};

// ---------------------------------------------------------------------------------------------
// E <= 16: the whole gate backward except the final reduction in ONE kernel.  A block of four waves owns one
// chunk of tokens (the unit of a dWg partial sum) and 256 columns of M; a thread owns 4 consecutive columns of a quarter
// of the tokens, so that its slice of Wg and its dWg accumulators fit in registers.  The chunk's dlogits rows go to
// LDS first (one thread per token; column block 0 also stores them); then every wave reads the x and old dx pieces of its
// tokens once, FT tokens at a time, and uses them twice:
//     dWg partial[e][q] += x[t, q] dl[t, e]        dx[t, q] (+)= sum_e dl[t, e] Wg[q, e]
// The four waves' sums meet in LDS, half of the columns at a time, are added in fp64 in a fixed order and leave it so that
// [m][e] rows are written contiguously.  A chunk is a multiple of 16 tokens; up to 2048 tokens the workspace has two rows
// per chunk, and the second takes what the rounding of the first left: these sums then lose no more than chains of 8
// tokens would (1003 x 520, 12 experts, relative error of dWg: 5.2e-8 with the waves added in fp32, 3.9e-8 now, 4.2e-8
// with chains of 8).
// Memory-bound at large sizes; at small ones the time is a chain of latencies, the fetch of the instructions among
// them: a version that unrolled 16 tokens was 17 to 34 KB of straight-line code and, with one wave per chunk, wrote
// eight times the partial sums.  Against that version, the call with its reduction: 2048 x 768, 16 experts: 32.8 ->
// 19.6 us; 4096 x 1024, 8 experts: 22.9 -> 20.2 us; 1003 x 520, 12 experts: 24.2 -> 17.2 us; 32768 x 4096, 8 experts: 205 -> 182 us.
// A wave's first stage is requested before the dlogits are formed and every later one while its predecessor is used, token by
// token; a stage without branches keeps the compiler from moving all its sums behind them, which spilled.  The call, with requests
// in the stage itself and with this: 2048 x 768, 16 experts: 19.4 -> 16.9 us; 4096 x 1024, 8: 19.9 -> 18.1; 8192 x 1024, top-1 of 8: 23.4 ->
// 20.2; 32768 x 4096, 8: 182 -> 171; 16384 x 2048, top-4 of 16: 91 -> 69; fp32, 5000 x 1024, 16: 36 -> 29.  The choices' weights requested
// earlier as well: 16.6, 19.1, 23.1, 174, 68, 28 (8 experts spill).
// ---------------------------------------------------------------------------------------------
constexpr int FW = 4;                                    // waves per block
constexpr int FT = 4;                                    // tokens per stage of a wave
constexpr int FUSED_CHUNK = 256;                         // dlogits rows in LDS at a time
// tokens per block: at most 256 partial sums (their number is at most that of dwg_chunk, which sizes the workspace); where a
// chunk has two rows, at most 64 of them, so that the rows do not cost more than the tokens (2048 x 768, 16 experts:
// 128 chunks 24.0 us, 64 chunks 19.6 us)
inline int64_t fused_chunk(int64_t S) {
  const int64_t step = FW * FT, parts = S <= 2048 ? 64 : 256, c = (S + parts - 1) / parts;
  return (c + step - 1) / step * step;
}
template <bool BF16, int EC>
__global__ __launch_bounds__(64 * FW, EC > 8 ? 2 : BF16 ? 4 : 3) void gate_bwd_fused(const float* __restrict__ dw, const float* __restrict__ w,
                                                          const int32_t* __restrict__ idx, const float* __restrict__ logits,
                                                          const void* __restrict__ x, const float* __restrict__ Wg,
                                                          int S, int M, int E, int k, int norm_topk, int chunk,
                                                          float* __restrict__ dl_out, void* __restrict__ dx, int accumulate,
                                                          float* __restrict__ partial, int nrows) {
  constexpr int CPT = 4, MT = 64 * CPT, PITCH = MT + 8, NTHR = 64 * FW;
  constexpr int HC = MT / 2, HPITCH = HC + 8;      // half of the columns
  static_assert(FUSED_CHUNK == NTHR, "a thread per dlogits row");
  __shared__ __attribute__((aligned(16))) float outs[FW * EC * HPITCH];
  static_assert(FW * HPITCH >= PITCH, "holds the slab of Wg too");
  __shared__ __attribute__((aligned(16))) float dls[FUSED_CHUNK * EC];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mb = blockIdx.x * MT;
  const int tb = (int)blockIdx.y * chunk, te = tb + min(chunk, S - tb);   // S k < 2^31
  const int rest_row = (int)(gridDim.y + blockIdx.y);    // row for what rounding leaves, if there is one
  const bool lone = rest_row >= nrows && te - tb <= 2 * FT;   // without it a few tokens are one wave's, one chain of sums

  float acc[EC][CPT];
#pragma unroll
  for (int e = 0; e < EC; ++e)
#pragma unroll
    for (int q = 0; q < CPT; ++q) acc[e][q] = 0.f;
  float colsum = 0.f;   // thread EC q + e of column block 0, q < 4, sums dl[t, e] over the tokens t = q (mod 4) for the bias row

  // a wave's next stage is requested token by token as the current one is used, the first one before the dlogits are formed
  const int n = te - tb, step = lone ? FT : FW * FT;
  int pos = lone && wave > 0 ? n : wave * FT;
  RawRow<BF16, CPT> xr[FT], dr[FT];
  // Rows through descriptors: behind the chunk's end, behind the last column, and dx that is not read, zeros come without a
  // request and stores go nowhere, so that a stage is one piece of code without branches.
  constexpr int ESZ = BF16 ? 2 : 4;
  const uint32_t row_bytes = (uint32_t)min(MT, M - mb) * ESZ, at = (uint32_t)lane * CPT * ESZ;
  auto row_of = [&](const void* base, int tok, bool there) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(base)) + ((tb + min(tok, n - 1)) * (int64_t)M + mb) * ESZ,
                                             0, there && tok < n ? row_bytes : 0u, 0x00020000);
  };
  auto fetch = [&](int u, int tok) {
    xr[u].load(row_of(x, tok, true), at);
    dr[u].load(row_of(dx, tok, accumulate != 0), at);
  };
  const uint32_t inv_e = 65536u / (uint32_t)E + 1u;   // i / E = i inv_e >> 16 for i < 4096, E <= 16
  static_assert(MT * 16 <= 4096 && FUSED_CHUNK * 16 <= 4096, "");

  for (int done = 0; done < n; done += FUSED_CHUNK) {
    const int c0 = tb + done, nc = min(te - c0, FUSED_CHUNK);
    if (done > 0) __syncthreads();   // the previous dl rows are consumed
    if (done == 0) {
      // The block's slab of Wg, contiguous in memory, goes through LDS once for the four waves: read directly, a lane's
      // weights are strided pieces, and every request of a wave is 64 lines.
      const float* slab = Wg + (int64_t)mb * E;
      const int ms = min(MT, M - mb);
      if (E % 4 == 0) {
        float4 v[EC / 4];
#pragma unroll
        for (int u = 0; u < EC / 4; ++u) v[u] = reinterpret_cast<const float4*>(slab)[min(tid + NTHR * u, ms * E / 4 - 1)];
#pragma unroll
        for (int u = 0; u < FT; ++u) fetch(u, pos + u);
#pragma unroll
        for (int u = 0; u < EC / 4; ++u) {
          const int i = (tid + NTHR * u) * 4, m = (int)((uint32_t)i * inv_e >> 16), e = i - m * E;
          if (m < MT) {
            outs[e * PITCH + m] = v[u].x; outs[(e + 1) * PITCH + m] = v[u].y;
            outs[(e + 2) * PITCH + m] = v[u].z; outs[(e + 3) * PITCH + m] = v[u].w;
          }
        }
      } else {
        // NS values requested together (behind the end the last one again): 2000 x 2048, fp32, 6 experts 19.8 -> 19.3 us; 8192 x 4096, 13 118 ->
        // 114, fp32 150 -> 136.  Two in bf16 with up to 8 experts, whose code for whole fours, beside this, takes 1 % longer with three.
        constexpr int NS = BF16 && EC == 8 ? 2 : 3;
#pragma unroll 1
        for (int i0 = tid; i0 < ms * E; i0 += NS * NTHR) {
          float v[NS];
#pragma unroll
          for (int u = 0; u < NS; ++u) v[u] = slab[min(i0 + u * NTHR, ms * E - 1)];
#pragma unroll
          for (int u = 0; u < NS; ++u) {
            const int i = min(i0 + u * NTHR, ms * E - 1), m = (int)((uint32_t)i * inv_e >> 16);
            outs[(i - m * E) * PITCH + m] = v[u];
          }
        }
#pragma unroll
        for (int u = 0; u < FT; ++u) fetch(u, pos + u);
      }
    }
    if (wave * 64 < nc) {
      const int64_t t = c0 + min(tid, nc - 1);
      const Picks p(dw, w, idx, t, k);
      float row[EC];
#pragma unroll
      for (int e = 0; e < EC; ++e) row[e] = 0.f;
      if (!norm_topk) {
        float mx = -__builtin_inff(), den = 0.f;
#pragma unroll
        for (int e = 0; e < EC; ++e) {
          row[e] = logits[t * E + (e < E ? e : E - 1)];
          mx = fmaxf(mx, row[e]);
        }
#pragma unroll
        for (int e = 0; e < EC; ++e) {
          row[e] = expf(row[e] - mx);
          if (e < E) den += row[e];
        }
#pragma unroll
        for (int e = 0; e < EC; ++e) row[e] = e < E ? -(row[e] / den) * p.inner : 0.f;
      }
      // rows behind the chunk's end: zeros, which the last stage multiplies
#pragma unroll
      for (int e = 0; e < EC; ++e) dls[tid * EC + e] = tid < nc ? row[e] : 0.f;
#pragma unroll
      for (int j = 0; j < MOE_MAX_K; ++j)
        if (tid < nc && (unsigned)p.e[j] < (unsigned)E)      // (-1 from k on)
          dls[tid * EC + p.e[j]] += norm_topk ? p.w[j] * (p.g[j] - p.inner) : p.w[j] * p.g[j];
    }
    __syncthreads();
    float wr[CPT][EC];     // (read again for further dlogits rows: not held while these are formed)
#pragma unroll
    for (int e = 0; e < EC; ++e) {
      const float4 v = e < E ? *reinterpret_cast<const float4*>(&outs[e * PITCH + lane * CPT]) : make_float4(0.f, 0.f, 0.f, 0.f);
      wr[0][e] = v.x; wr[1][e] = v.y; wr[2][e] = v.z; wr[3][e] = v.w;
    }
    if (blockIdx.x == 0) {
      // through a descriptor: a 32-bit offset per lane instead of an address, which would not stay in a register
      const __amdgpu_buffer_rsrc_t rl = __builtin_amdgcn_make_buffer_rsrc(dl_out + (int64_t)c0 * E, 0, (uint32_t)(nc * E * 4), 0x00020000);
      for (int i = tid; i < nc * E; i += NTHR) {
        const int t = (int)((uint32_t)i * inv_e >> 16), e = i - t * E;
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(dls[t * EC + e]), rl, i * 4, 0, 0);
      }
      if (tid < 4 * EC) {
#pragma unroll 8
        for (int t = 0; t < nc; t += 4) colsum += dls[t * EC + tid];   // (rows behind the end are zeros)
      }
    }
    for (; pos < done + nc; pos += step) {
      const int u0 = pos - done;
#pragma unroll
      for (int u = 0; u < FT; ++u) {   // a row behind the end: zeros
        float xv[CPT], dv[CPT];
#pragma unroll
        for (int q = 0; q < CPT; ++q) { xv[q] = xr[u].get(q); dv[q] = dr[u].get(q); }
        fetch(u, pos + step + u);
#pragma unroll
        for (int e4 = 0; e4 < EC; e4 += 4) {
          const float4 d4 = *reinterpret_cast<const float4*>(&dls[(u0 + u) * EC + e4]);
          const float d[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int q = 0; q < CPT; ++q) {
              acc[e4 + v][q] = fmaf(xv[q], d[v], acc[e4 + v][q]);
              dv[q] = fmaf(d[v], wr[q][e4 + v], dv[q]);
            }
        }
        st4g<BF16>(row_of(dx, pos + u, true), at, dv);
      }
    }
  }
  __syncthreads();   // every wave has its weights
  float* out = partial + (int64_t)blockIdx.y * (M + 1) * E;
  float* rest = rest_row < nrows ? partial + (int64_t)rest_row * (M + 1) * E : nullptr;
  auto put_sum = [&](double v, int64_t at) {
    const float hi = (float)v;
    out[at] = hi;
    if (rest != nullptr) rest[at] = fabsf(hi) <= 3.402823466e38f ? (float)(v - (double)hi) : 0.f;   // (an infinity leaves nothing)
  };
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    if ((lane >> 5) == h) {
#pragma unroll
      for (int e = 0; e < EC; ++e)
        *reinterpret_cast<float4*>(&outs[(wave * EC + e) * HPITCH + (lane & 31) * CPT]) =
            make_float4(acc[e][0], acc[e][1], acc[e][2], acc[e][3]);
    }
    __syncthreads();
    for (int i = tid; i < HC * EC; i += NTHR) {
      const int m = i / EC, e = i - m * EC, mg = mb + h * HC + m;
      double v[FW];
#pragma unroll
      for (int q = 0; q < FW; ++q) v[q] = (double)outs[(q * EC + e) * HPITCH + m];
      if (mg < M && e < E) put_sum((v[0] + v[1]) + (v[2] + v[3]), (int64_t)mg * E + e);
    }
    __syncthreads();
  }
  if (blockIdx.x == 0 && wave == 0) {
    double v[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = (double)__shfl(colsum, EC * q + lane % EC, 64);
    if (lane < E) put_sum((v[0] + v[1]) + (v[2] + v[3]), (int64_t)M * E + lane);   // E <= EC
  }
}

// ---------------------------------------------------------------------------------------------
// E > 16.  The two products run on the fp32 matrix cores: v_mfma_f32_32x32x2_f32, lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32] and receives D[8 (i / 4) + 4 (l / 32) + i % 4][l % 32], i = 0..15.  Operands are read straight from
// memory in the layout in which they lie: which k a lane's half feeds in which step, and which row or column of the
// output a lane's index names, are free as long as both operands agree, so the lanes take 8 to 16 consecutive bytes and no
// LDS and no barriers are needed; the reuse between waves comes from the caches.  8192 x 2048 x 128 experts (4.3 GFLOP
// each; 27 us at the nominal matrix rate): dx 187 -> 67 us, dWg 132 -> 55 us against vector FMAs on operands
// staged through LDS.
// ---------------------------------------------------------------------------------------------
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// gate_dx_wide: dx^T tiles (rows: columns of M, columns: tokens).  A wave owns 32 tokens, whose dl rows it holds in
// registers (KG groups of 8 experts), and walks WX_COLS columns 32 at a time.  Row 8 q + 4 h + i of a tile stands for column
// 16 h + 4 q + i, so that the lane's 16 results are 16 consecutive columns of its token.  k step i of a group takes experts 8 g + i and 8 g + 4 + i.
constexpr int WX_COLS = 128;
template <bool BF16, int KG>
__global__ __launch_bounds__(256) void gate_dx_wide(const float* __restrict__ dl, const float* __restrict__ Wg,
                                                    void* __restrict__ dx, int64_t S, int M, int E, int accumulate) {
  const int lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
  const int64_t t = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 32 + row;
  if (t - row >= S) return;
  const bool tok = t < S;
  const bool vec = (E & 3) == 0;      // 16-byte loads of four consecutive experts
  auto load4 = [&](const float* base, int e) -> float4 {   // experts e .. e + 3, zeros behind the last one
    if (vec) return e < E ? *reinterpret_cast<const float4*>(base + e) : make_float4(0.f, 0.f, 0.f, 0.f);
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = e + i < E ? base[e + i] : 0.f;
    return make_float4(v[0], v[1], v[2], v[3]);
  };
  float4 d[KG];
  const float* drow = dl + (tok ? t : S - 1) * E;   // a token past the end: any row, not stored
#pragma unroll
  for (int g = 0; g < KG; ++g) d[g] = load4(drow, 8 * g + 4 * half);
  const int cb = blockIdx.y * WX_COLS, ce = min(M, cb + WX_COLS);
  const int wcol = 16 * ((row >> 2) & 1) + 4 * (row >> 3) + (row & 3);   // the column that this lane's row stands for
  for (int c0 = cb; c0 < ce; c0 += 32) {
    const float* wrow = Wg + (int64_t)min(c0 + wcol, M - 1) * E;
    const int c = c0 + 16 * half;    // M is a multiple of 8: runs of 8 columns are in or out together
    RawRow<BF16, 8> old[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (accumulate && tok && c + 8 * q < M) old[q].load(dx, t * (int64_t)M + c + 8 * q); else old[q].zero();
    }
    f32x16_t acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      const float4 wv = load4(wrow, 8 * g + 4 * half);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv.x, d[g].x, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv.y, d[g].y, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv.z, d[g].z, acc, 0, 0, 0);
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wv.w, d[g].w, acc, 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float o[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) o[i] = old[q].get(i) + acc[8 * q + i];
      if (tok && c + 8 * q < M) st8g<BF16>(dx, t * (int64_t)M + c + 8 * q, o);
    }
  }
}

// gate_dwg_wide: a wave owns one token chunk, 128 columns of M and 64 experts: 4 x 2 tiles, in which lane l % 32 stands
// for columns 4 (l % 32) + {0..3} and experts 2 (l % 32) + {0, 1}, so that a token's pieces of x and dl are whole lines; k step:
// two tokens, one per half of the wave.  Four steps are requested while the four before are multiplied, and two waves share a SIMD.
// partial[chunk][m][e] for m < M, plus row m = M (column sums of dl) for the bias gradient.
constexpr int WW_COLS = 128;
template <bool BF16>
__global__ __launch_bounds__(256, 2) void gate_dwg_wide(const void* __restrict__ x, const float* __restrict__ dl,
                                                     float* __restrict__ partial, int64_t S, int M, int E, int chunk) {
  constexpr int U = 4;
  const int lane = threadIdx.x & 63, li = lane & 31, half = lane >> 5;
  const int mb = (blockIdx.x * 4 + (threadIdx.x >> 6)) * WW_COLS;
  if (mb >= M) return;
  const int e0 = blockIdx.z * 64 + 2 * li;
  const int64_t tb = (int64_t)blockIdx.y * chunk;
  const int64_t te = (tb + chunk < S) ? tb + chunk : S;
  const int c0 = min(mb + 4 * li, M - 4);           // a lane behind the last column: any columns, not stored
  const int ea = min(e0, E - 1), eb = min(e0 + 1, E - 1);
  f32x16_t acc[4][2];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[b][f][i] = 0.f;
  float sum[2] = {0.f, 0.f};
  RawRow<BF16, 4> xr[2][U];
  float dr[2][U][2];
  auto fetch = [&](int set, int64_t t0) {   // tokens behind the end: the last one, masked when multiplied
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t t = min(t0 + 2 * u + half, te - 1);
      xr[set][u].load(x, t * (int64_t)M + c0);
      dr[set][u][0] = dl[t * E + ea];
      dr[set][u][1] = dl[t * E + eb];
    }
  };
  auto multiply = [&](int set, int64_t t0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool in = t0 + 2 * u + half < te;
      const float d0 = in ? dr[set][u][0] : 0.f, d1 = in ? dr[set][u][1] : 0.f;
      sum[0] += d0; sum[1] += d1;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const float a = in ? xr[set][u].get(b) : 0.f;
        acc[b][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, d0, acc[b][0], 0, 0, 0);
        acc[b][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, d1, acc[b][1], 0, 0, 0);
      }
    }
  };
  fetch(0, tb);
  for (int64_t t0 = tb; t0 < te; t0 += 4 * U) {   // two sets of 2 U tokens
    if (t0 + 2 * U < te) fetch(1, t0 + 2 * U);
    multiply(0, t0);
    if (t0 + 2 * U < te) {
      if (t0 + 4 * U < te) fetch(0, t0 + 4 * U);
      multiply(1, t0 + 2 * U);
    }
  }
  float* out = partial + (int64_t)blockIdx.y * (M + 1) * E;
#pragma unroll
  for (int i = 0; i < 16; ++i)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      const int m = mb + 4 * (8 * (i >> 2) + 4 * half + (i & 3)) + b;
      if (m < M) {
        if (e0 < E) out[(int64_t)m * E + e0] = acc[b][0][i];
        if (e0 + 1 < E) out[(int64_t)m * E + e0 + 1] = acc[b][1][i];
      }
    }
  if (mb == 0) {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const float s = sum[f] + __shfl_xor(sum[f], 32, 64);
      if (half == 0 && e0 + f < E) out[(int64_t)M * E + e0 + f] = s;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// E > 16 and norm_topk: a token's dl row has its k selected experts' entries and zeros elsewhere, so both products only take
// those.  The dense products multiply the zeros too, so that an infinity or a NaN in x or Wg makes a NaN of them: a slab or a
// tile that holds one is multiplied with all experts.
// ---------------------------------------------------------------------------------------------
constexpr int SG_NT = 512, SG_NW = SG_NT / 64;

// bits of a non-finite value in a 32-bit word as loaded
template <bool BF16>
__device__ __forceinline__ bool not_finite(uint32_t v) {
  if (BF16) return (v & 0x7F80u) == 0x7F80u || (v & 0x7F800000u) == 0x7F800000u;
  return (v & 0x7F800000u) == 0x7F800000u;
}

// dx and the dl rows.  A workgroup owns 64 columns of a run of tokens.  The columns' slab of Wg goes through LDS transposed
// ([expert][column]); 16 lanes take a token's piece, 4 columns each, and add k rows of the slab.  The dl rows are stored on the
// way, a part of them by each column block.  Bound by memory once the slab is there: 8192 x 2048, top-4 of 128, 23 us (71 MB),
// against 65 us with all experts on the matrix cores and 5 for the dl rows; 16384 x 2048, top-2 of 64, 31 against 85 and 8.
constexpr int SX_C = 64, SX_PITCH = SX_C + 4, SX_TPI = SG_NT / 16;   // columns; of the slab; tokens at a time
constexpr int SX_U = 4;                                             // tokens per thread and step
template <int EP> constexpr int sx_tokens() { return EP > 128 ? 128 : 256; }   // most tokens of a workgroup
template <bool BF16, int EP>   // E <= EP
__global__ __launch_bounds__(SG_NT, 4) void gate_dx_sparse(const float* __restrict__ dw, const float* __restrict__ w,
                                                           const int32_t* __restrict__ idx, const float* __restrict__ Wg, int S,
                                                           int M, int E, int k, float* __restrict__ dl_out,
                                                           void* __restrict__ dx, int accumulate, int chunk, int ncb) {
  __shared__ __attribute__((aligned(16))) float wt[EP * SX_PITCH];
  __shared__ __attribute__((aligned(16))) uint2 ent[sx_tokens<EP>() * MOE_MAX_K];   // (expert, dl); what is missing is (0, 0)
  __shared__ int odd_s;
  const int tid = threadIdx.x, k2 = (k + 1) & ~1;
  const int run = (int)blockIdx.x / ncb, cx = (int)blockIdx.x - run * ncb, mb = cx * SX_C;   // the column blocks of a run are neighbours
  const int tb = run * chunk, nt = min(chunk, S - tb);
  const int c0 = 4 * (tid & 15), col = mb + c0, tq = tid >> 4;
  const bool cok = col < M;
  RawRow<BF16, 4> old[2][SX_U];
  auto fetch = [&](int set, int t0) {
#pragma unroll
    for (int u = 0; u < SX_U; ++u) {
      const int t = t0 + tq + u * SX_TPI;
      if (accumulate && cok && t < nt) old[set][u].load(dx, (int64_t)(tb + t) * M + col); else old[set][u].zero();
    }
  };
  if (tid == 0) odd_s = 0;
  const bool vec = (E & 3) == 0;
  constexpr int NV = SX_C * EP / 4 / SG_NT;        // pieces of 4 experts per thread: 8 lanes take 8 of a row, 8 rows to a wave
  float4 wv[NV];
  if (vec) {
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      const int i = tid + n * SG_NT, m = (i >> 3) % SX_C, c = (i >> 3) / SX_C * 8 + (i & 7);
      wv[n] = mb + m < M && 4 * c < E ? *reinterpret_cast<const float4*>(Wg + (int64_t)(mb + m) * E + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  }
  fetch(0, 0);
  if (tid < nt) {
    const Picks p(dw, w, idx, tb + tid, k);
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j)
      if (j < k2) ent[tid * k2 + j] = (unsigned)p.e[j] < (unsigned)E ? make_uint2((uint32_t)p.e[j], __float_as_uint(p.w[j] * (p.g[j] - p.inner)))
                                                                   : make_uint2(0u, 0u);
  }
  __syncthreads();
  bool odd = false;
  if (vec) {
#pragma unroll
    for (int n = 0; n < NV; ++n) {
      const int i = tid + n * SG_NT, m = (i >> 3) % SX_C, c = (i >> 3) / SX_C * 8 + (i & 7);
      const float f[4] = {wv[n].x, wv[n].y, wv[n].z, wv[n].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        wt[(4 * c + q) * SX_PITCH + m] = f[q];
        odd |= not_finite<false>(__float_as_uint(f[q]));
      }
    }
  } else {
    for (int i = tid; i < SX_C * E; i += SG_NT) {
      const int m = i / E, e = i - m * E;
      const float v = mb + m < M ? Wg[(int64_t)mb * E + i] : 0.f;
      wt[e * SX_PITCH + m] = v;
      odd |= not_finite<false>(__float_as_uint(v));
    }
  }
  if (odd) odd_s = 1;
  {   // this column block's share of the dl rows
    const int r0 = (int)((int64_t)nt * cx / ncb), n = ((int)((int64_t)nt * (cx + 1) / ncb) - r0) * E;
    for (int i = tid; i < n; i += SG_NT) {
      const int r = r0 + i / E, e = i % E;
      float v = 0.f;
      for (int j = 0; j < k2; ++j) {
        const uint2 q = ent[r * k2 + j];
        v += (int)q.x == e ? __uint_as_float(q.y) : 0.f;
      }
      dl_out[(int64_t)(tb + r0) * E + i] = v;
    }
  }
  __syncthreads();
  const bool dense = odd_s != 0;
  auto step = [&](int set, int t0) {
    float acc[SX_U][4];
#pragma unroll
    for (int u = 0; u < SX_U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[u][q] = 0.f;
    auto add = [&](int u, int e, float d) {
      const float4 v = *reinterpret_cast<const float4*>(wt + e * SX_PITCH + c0);
      acc[u][0] = fmaf(d, v.x, acc[u][0]); acc[u][1] = fmaf(d, v.y, acc[u][1]);
      acc[u][2] = fmaf(d, v.z, acc[u][2]); acc[u][3] = fmaf(d, v.w, acc[u][3]);
    };
    const uint2* my[SX_U];
#pragma unroll
    for (int u = 0; u < SX_U; ++u) my[u] = ent + min(t0 + tq + u * SX_TPI, nt - 1) * k2;
    if (__builtin_expect(!dense, 1)) {
      for (int j = 0; j < k2; j += 2) {
        uint4 q[SX_U];
#pragma unroll
        for (int u = 0; u < SX_U; ++u) q[u] = *reinterpret_cast<const uint4*>(my[u] + j);
#pragma unroll
        for (int u = 0; u < SX_U; ++u) {
          add(u, (int)q[u].x, __uint_as_float(q[u].y));
          add(u, (int)q[u].z, __uint_as_float(q[u].w));
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < SX_U; ++u)
        for (int e = 0; e < E; ++e) {
          float d = 0.f;
          for (int j = 0; j < k2; ++j) d += (int)my[u][j].x == e ? __uint_as_float(my[u][j].y) : 0.f;
          add(u, e, d);
        }
    }
#pragma unroll
    for (int u = 0; u < SX_U; ++u) {
      const int t = t0 + tq + u * SX_TPI;
      float o[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) o[q] = old[set][u].get(q) + acc[u][q];
      if (cok && t < nt) st4g<BF16>(dx, (int64_t)(tb + t) * M + col, o);
    }
  };
  constexpr int STEP = SX_U * SX_TPI;
  for (int t0 = 0; t0 < nt; t0 += 2 * STEP) {
    if (t0 + STEP < nt) fetch(1, t0 + STEP);
    step(0, t0);
    if (t0 + STEP < nt) {
      if (t0 + 2 * STEP < nt) fetch(0, t0 + 2 * STEP);
      step(1, t0 + STEP);
    }
  }
}

// dWg, as partial sums: [chunk][E][M], the bias rows [chunk][E] behind them all.  A workgroup owns 128 columns, 2 to a lane, of
// a chunk of tokens.  It takes the chunk in tiles, whose rows of x go to LDS and whose entries are sorted by expert (a stable
// counting sort: ranks by ballots, no atomics); a wave adds the rows of every eighth expert (neighbours may be popular together).
// Rounding.  The entries of a tile are added in two fp32 chains of at most four, these in fp64, the chunk's sum is rounded.  In
// units of the last place of one entry, the variance that an entry adds is then (n + 1) / 2 for chains of n, and 1; for the one
// chain per expert and dwg_chunk tokens that all experts are summed in, with n entries in it, (n + 1) / 2 alone.  So these sums are
// no farther off from n = 4 there, or from 6 where the tile is longer than that chunk; n is the average expert's, and columns of
// the rarest ones under skewed routing are up to 1.3 times as far off (4e-8 and 3.5e-8).  Below that (EXACT) the products are added in
// fp64, which costs a fifth of the kernel.  Relative error of dWg, all experts and this: 8192 x 2048, top-4 of 128 (n = 4) 5.1e-8
// and 4.9e-8, top-4 of 24 9.1e-8 and 5.3e-8; 4096 x 512, top-2 of 160 3.9e-8 and, EXACT, 3.6e-8 (4.5e-8 in fp32 chains).
// 8192 x 2048, top-4 of 128, 31 us where reading x takes 6, against 54 us on the fp32 matrix cores; 16384 x 2048, top-2 of 64, 35
// against 61.  What the 31 us go into was not taken apart; in question are the chain of LDS reads (entry, row of x) per four entries,
// the sort, which every column block does again with six barriers a tile, and the fetch of the code: the sums of all of a wave's
// experts are in registers, so the loop over them is unrolled, 14 to 18 KB of it at EP = 64, 25 to 33 at 128, 46 to 59 at 256, walked
// once a tile.  EP = 128 spills 8 to 14 loop invariants, reloaded once a tile.
constexpr int SW_C = 128;
template <bool BF16> constexpr int sw_tile() { return BF16 ? 128 : 64; }   // tokens
template <bool BF16, int EP, bool EXACT>   // E <= EP
__global__ __launch_bounds__(SG_NT, EP > 128 ? 2 : 4) void gate_dwg_sparse(const float* __restrict__ dw, const float* __restrict__ w,
                                                                           const int32_t* __restrict__ idx,
                                                                           const void* __restrict__ x, int S, int M, int E, int k,
                                                                           float* __restrict__ partial, int chunk) {
  constexpr int ESZ = BF16 ? 2 : 4, TT = sw_tile<BF16>(), NG = TT * MOE_MAX_K / 64, EPW = EP / SG_NW;
  __shared__ __attribute__((aligned(16))) char xs[TT * SW_C * ESZ];
  __shared__ __attribute__((aligned(16))) uint2 list[TT * MOE_MAX_K + 3 * EP];   // (row's place, dl) by expert, in runs of whole fours
  __shared__ float2 raw[TT * MOE_MAX_K];                                     // (w, dw) in token order
  __shared__ int hist[NG * EP], first[EP], total[EP], odd_s;
  constexpr int ROW = SW_C * ESZ;    // bytes
  struct XV {                        // a lane's two columns of a row, as stored
    uint32_t r[ESZ / 2];
    __device__ __forceinline__ float lo() const { return __uint_as_float(BF16 ? r[0] << 16 : r[0]); }
    __device__ __forceinline__ float hi() const { return __uint_as_float(BF16 ? r[0] & 0xFFFF0000u : r[ESZ / 2 - 1]); }
  };
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto xval = [&](uint32_t at) -> XV {
    XV v;
    if (BF16) {
      v.r[0] = *reinterpret_cast<const uint32_t*>(xs + at + lane * 4);
    } else {
      const uint2 q = *reinterpret_cast<const uint2*>(xs + at + lane * 8);
      v.r[0] = q.x; v.r[ESZ / 2 - 1] = q.y;
    }
    return v;
  };
  const int cw = (int)blockIdx.x, mb = cw * SW_C, part = (int)blockIdx.y, tb = part * chunk, te = tb + min(chunk, S - tb);
  constexpr int PPR = SW_C * ESZ / 16, UX = TT * PPR / SG_NT;         // 16-byte pieces per row; per thread
  constexpr int GW = NG / SG_NW;                                      // groups of 64 entries per wave
  static_assert(NG % SG_NW == 0, "groups are dealt evenly");
  const int xc = mb + (tid % PPR) * (16 / ESZ);                       // M is a multiple of 8: a piece is in or out
  uint4 xr[UX];
  float pw[GW], pg[GW];
  int pe[GW];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int q = 0; q < GW; ++q) {
      const int i = (q * SG_NW + wave) * 64 + lane;
      const bool in = i < min(TT, te - t0) * k;
      const int64_t at = (int64_t)t0 * k + (in ? i : 0);
      pw[q] = w[at]; pg[q] = dw[at]; pe[q] = in ? idx[at] : -1;
    }
#pragma unroll
    for (int u = 0; u < UX; ++u) {
      const int t = t0 + tid / PPR + u * (SG_NT / PPR);
      xr[u] = t < te && xc < M ? *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(x) + ((int64_t)t * M + xc) * ESZ)
                               : make_uint4(0u, 0u, 0u, 0u);
    }
  };
  double acc[EPW][2];
#pragma unroll
  for (int i = 0; i < EPW; ++i) acc[i][0] = acc[i][1] = 0.0;
  double bias = 0.0;     // lane i: sum of dl of expert SG_NW i + wave
  fetch(tb);
  for (int t0 = tb; t0 < te; t0 += TT) {
    const int nt = min(TT, te - t0);
    __syncthreads();   // the previous tile is consumed
    if (tid == 0) odd_s = 0;
    for (int i = tid; i < NG * EP; i += SG_NT) hist[i] = 0;
    int e[GW];
    float wj[GW], gj[GW];
#pragma unroll
    for (int q = 0; q < GW; ++q) {
      raw[(q * SG_NW + wave) * 64 + lane] = make_float2(pw[q], pg[q]);
      e[q] = (unsigned)pe[q] < (unsigned)E ? pe[q] : -1;
      wj[q] = pw[q]; gj[q] = pg[q];
    }
    bool odd = false;
#pragma unroll
    for (int u = 0; u < UX; ++u) {
      *reinterpret_cast<uint4*>(xs + (tid + u * SG_NT) * 16) = xr[u];
      odd |= not_finite<BF16>(xr[u].x) | not_finite<BF16>(xr[u].y) | not_finite<BF16>(xr[u].z) | not_finite<BF16>(xr[u].w);
    }
    __syncthreads();
    if (odd) odd_s = 1;
    if (t0 + TT < te) fetch(t0 + TT);
    int rank[GW], row[GW];
    float d[GW];
#pragma unroll
    for (int q = 0; q < GW; ++q) {
      const int i = (q * SG_NW + wave) * 64 + lane;
      unsigned long long same = __ballot(e[q] >= 0);
      rank[q] = 0; row[q] = 0; d[q] = 0.f;
      if (same == 0) continue;
      for (int bit = 1; bit < E; bit <<= 1) {
        const unsigned long long has = __ballot((e[q] & bit) != 0);
        same &= (e[q] & bit) ? has : ~has;
      }
      rank[q] = __popcll(same & ((1ull << lane) - 1ull));
      if (e[q] >= 0) {
        if (rank[q] == 0) hist[(q * SG_NW + wave) * EP + e[q]] = __popcll(same);
        row[q] = i / k;
        float inner = 0.f;
        for (int j = 0; j < k; ++j) inner = fmaf(raw[row[q] * k + j].x, raw[row[q] * k + j].y, inner);
        d[q] = wj[q] * (gj[q] - inner);
      }
    }
    __syncthreads();
    if (tid < EP) {
      int h[NG], run = 0;
#pragma unroll
      for (int q = 0; q < NG; ++q) h[q] = hist[q * EP + tid];
#pragma unroll
      for (int q = 0; q < NG; ++q) {
        hist[q * EP + tid] = run;
        run += h[q];
      }
      total[tid] = run;
    }
    __syncthreads();
    if (wave == 0) {
      constexpr int PL = EP / 64;     // experts per lane
      int v[PL], sum = 0;
#pragma unroll
      for (int q = 0; q < PL; ++q) { v[q] = (total[lane * PL + q] + 3) & ~3; sum += v[q]; }
      int incl = sum;
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) {
        const int o = __shfl_up(incl, s, 64);
        if (lane >= s) incl += o;
      }
      int run = incl - sum;
#pragma unroll
      for (int q = 0; q < PL; ++q) { first[lane * PL + q] = run; run += v[q]; }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < GW; ++q)
      if (e[q] >= 0) list[first[e[q]] + hist[(q * SG_NW + wave) * EP + e[q]] + rank[q]] = make_uint2((uint32_t)(row[q] * ROW), __float_as_uint(d[q]));
    if (tid < EP)
      for (int u = total[tid]; u & 3; ++u) list[first[tid] + u] = make_uint2(0u, 0u);
    __syncthreads();
    const int my_e = SG_NW * (lane < EPW ? lane : 0) + wave;
    int my_first = first[my_e], my_total = total[my_e];
    const bool dense = odd_s != 0;
#pragma unroll
    for (int i = 0; i < EPW; ++i) {
      asm volatile("" : "+v"(my_first), "+v"(my_total));   // (the reads of the lanes stay where they are)
      const int m = __builtin_amdgcn_readlane(my_total, i);
      if (m == 0 && !dense) continue;
      const uint2* run = list + __builtin_amdgcn_readlane(my_first, i);
      if (__builtin_expect(!dense, 1)) {
        for (int u = 0; u < m; u += 8) {
          float s[2][2] = {{0.f, 0.f}, {0.f, 0.f}}, sb[2] = {0.f, 0.f};   // !EXACT: two chains of at most four
          auto four = [&](int o) {
            const uint4 q0 = *reinterpret_cast<const uint4*>(run + o), q1 = *reinterpret_cast<const uint4*>(run + o + 2);
            const XV v[4] = {xval(q0.x), xval(q0.z), xval(q1.x), xval(q1.z)};
            const float d[4] = {__uint_as_float(q0.y), __uint_as_float(q0.w), __uint_as_float(q1.y), __uint_as_float(q1.w)};
#pragma unroll
            for (int n = 0; n < 4; ++n) {
              if (EXACT) {
                acc[i][0] = fma((double)v[n].lo(), (double)d[n], acc[i][0]);
                acc[i][1] = fma((double)v[n].hi(), (double)d[n], acc[i][1]);
                if (cw == 0) bias += lane == i ? (double)d[n] : 0.0;
              } else {
                s[n & 1][0] = fmaf(v[n].lo(), d[n], s[n & 1][0]);
                s[n & 1][1] = fmaf(v[n].hi(), d[n], s[n & 1][1]);
                sb[n & 1] += d[n];
              }
            }
          };
          four(u);
          if (u + 4 < m) four(u + 4);
          if (!EXACT) {
#pragma unroll
            for (int c = 0; c < 2; ++c) acc[i][c] += (double)s[0][c] + (double)s[1][c];
            if (cw == 0) bias += lane == i ? (double)sb[0] + (double)sb[1] : 0.0;
          }
        }
      } else {
        int u = 0;
        for (int t = 0; t < nt; ++t) {   // the run is in token order
          float d = 0.f;
          for (; u < m && run[u].x == (uint32_t)(t * ROW); ++u) d += __uint_as_float(run[u].y);
          const XV v = xval((uint32_t)(t * ROW));
          acc[i][0] = fma((double)v.lo(), (double)d, acc[i][0]);
          acc[i][1] = fma((double)v.hi(), (double)d, acc[i][1]);
          bias += lane == i ? (double)d : 0.0;
        }
      }
    }
  }
  const int m = mb + 2 * lane;
  float* out = partial + ((int64_t)part * E + wave) * M + m;
#pragma unroll
  for (int i = 0; i < EPW; ++i)
    if (SG_NW * i + wave < E && m < M)
      *reinterpret_cast<float2*>(out + (int64_t)(SG_NW * i) * M) = make_float2((float)acc[i][0], (float)acc[i][1]);
  if (cw == 0 && lane < EPW && SG_NW * lane + wave < E)
    partial[(int64_t)gridDim.y * M * E + (int64_t)part * E + SG_NW * lane + wave] = (float)bias;
}

}  // namespace

extern "C" size_t moe_gate_bwd_workspace_bytes(int64_t S, int M, int E) {
  if (S < 1 || M < 1 || E < 1) return 0;
  const int chunk = dwg_chunk(S, E);
  const int64_t nchunk = (S + chunk - 1) / chunk;
  return moe::align_up((size_t)nchunk * (size_t)(M + 1) * E * sizeof(float), 256);
}

extern "C" int moe_gate_bwd(const float* dw, const float* w, const int32_t* idx, const float* logits, const void* x,
                            int x_dtype, const float* Wg, int64_t S, int M, int E, int k, int norm_topk,
                            float* dlogits, float* dWg, float* dgate_bias, void* dx, int dx_accumulate, void* ws,
                            size_t ws_bytes, void* stream) {
  if (int rc = moe::common_shape_check(S, M, E, k, 1)) return rc;
  MOE_REQUIRE(x_dtype == MOE_F32 || x_dtype == MOE_BF16, MOE_EINVAL);
  MOE_REQUIRE(norm_topk >= -1 && norm_topk <= 1, MOE_EINVAL);
  MOE_REQUIRE(dx_accumulate == 0 || dx_accumulate == 1, MOE_EINVAL);
  MOE_REQUIRE_PTR(dw); MOE_REQUIRE_PTR(w); MOE_REQUIRE_PTR(idx); MOE_REQUIRE_PTR(logits); MOE_REQUIRE_PTR(x);
  MOE_REQUIRE_PTR(Wg); MOE_REQUIRE_PTR(dlogits); MOE_REQUIRE_PTR(dWg); MOE_REQUIRE_PTR(dx);
  MOE_OPTIONAL_PTR(dgate_bias);
  const size_t need = moe_gate_bwd_workspace_bytes(S, M, E);
  MOE_REQUIRE(ws != nullptr && ws_bytes >= need, MOE_EWORKSPACE);
  MOE_REQUIRE(moe::aligned16(ws), MOE_EALIGN);
  const int norm = norm_topk < 0 ? (k >= 2 ? 1 : 0) : norm_topk;
  hipStream_t st = (hipStream_t)stream;
  const bool bf = x_dtype == MOE_BF16;
  const int64_t n = (int64_t)(M + 1) * E;
  if (E <= 16) {   // one fused kernel, then the reduction of the partial sums
    const int EC = E <= 8 ? 8 : 16;
    const int64_t chunk = fused_chunk(S);
    const int nchunk = (int)((S + chunk - 1) / chunk);
    const int ws_rows = (int)((S + dwg_chunk(S, E) - 1) / dwg_chunk(S, E));
    // a second row per chunk where the workspace has them; the last chunk, if of 8 tokens at most, may go without
    const int nrows = ws_rows >= 2 * nchunk - 1 ? (ws_rows < 2 * nchunk ? ws_rows : 2 * nchunk) : nchunk;
    float* partial = (float*)ws;
    const dim3 grid((unsigned)((M + 255) / 256), (unsigned)nchunk);
#define MOE_FUSED(BF, EC_) hipLaunchKernelGGL((gate_bwd_fused<BF, EC_>), grid, dim3(64 * FW), 0, st, dw, w, idx, logits, x, \
                                              Wg, (int)S, M, E, k, norm, (int)chunk, dlogits, dx, dx_accumulate, partial, nrows)
    if (bf) { if (EC == 8) MOE_FUSED(true, 8); else MOE_FUSED(true, 16); }
    else { if (EC == 8) MOE_FUSED(false, 8); else MOE_FUSED(false, 16); }
#undef MOE_FUSED
    hipLaunchKernelGGL(gate_dwg_reduce<false>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, partial, nrows, M, E, dWg,
                       dgate_bias);
    return moe::check_launch();
  }
  const int chunk = dwg_chunk(S, E);
  const int nchunk = (int)((S + chunk - 1) / chunk);   // the partial sums that the workspace holds
  float* partial = (float*)ws;
  // Only the selected experts where they are few.  The call, all experts and this, 8192 x 2048: top-4 of 128 126 and 60 us, top-4
  // of 17 62 and 54, top-6 of 17 62 and 63, top-8 of 24 63 and 70, top-8 of 32 64 and 65; 16384 x 2048, top-2 of 64 145 and 62;
  // 300 x 512, top-2 of 24 29 and 16.
  if (norm && E > 4 * k) {
    const int64_t tile_w = bf ? sw_tile<true>() : sw_tile<false>(), ncw = (M + SW_C - 1) / SW_C, ncx = (M + SX_C - 1) / SX_C;
    auto chunks = [&](int64_t blocks, int64_t columns, int64_t most, int64_t tile) {   // tokens of a workgroup
      const int64_t want = std::max<int64_t>(1, std::min(most, blocks / columns)), c = (S + want - 1) / want;
      return (c + tile - 1) / tile * tile;
    };
    // dWg: two workgroups to a compute unit.  8192 x 2048, top-4 of 128, kernel and reduction: 256 of them 42 + 7 us, 512 32 + 8,
    // 1024 40 + 12.
    const int64_t chunk_w = chunks(512, ncw, nchunk, tile_w), chunk_x = std::min<int64_t>(chunks(1024, ncx, S, SX_TPI), E > 128 ? 128 : 256);
    const int parts = (int)((S + chunk_w - 1) / chunk_w);
    const dim3 gx((unsigned)(ncx * ((S + chunk_x - 1) / chunk_x))), gw((unsigned)ncw, (unsigned)parts);   // (runs of 256 tokens may be more than y holds)
    const bool exact = (int64_t)chunk * k < (tile_w > chunk ? 6 : 4) * E;   // see gate_dwg_sparse
#define MOE_SPARSE(BF, EP) do { \
    hipLaunchKernelGGL((gate_dx_sparse<BF, EP>), gx, dim3(SG_NT), 0, st, dw, w, idx, Wg, (int)S, M, E, k, dlogits, dx, dx_accumulate, \
                       (int)chunk_x, (int)ncx); \
    if (exact) hipLaunchKernelGGL((gate_dwg_sparse<BF, EP, true>), gw, dim3(SG_NT), 0, st, dw, w, idx, x, (int)S, M, E, k, partial, \
                                  (int)chunk_w); \
    else hipLaunchKernelGGL((gate_dwg_sparse<BF, EP, false>), gw, dim3(SG_NT), 0, st, dw, w, idx, x, (int)S, M, E, k, partial, \
                            (int)chunk_w); } while (0)
    if (bf) { if (E <= 64) MOE_SPARSE(true, 64); else if (E <= 128) MOE_SPARSE(true, 128); else MOE_SPARSE(true, 256); }
    else { if (E <= 64) MOE_SPARSE(false, 64); else if (E <= 128) MOE_SPARSE(false, 128); else MOE_SPARSE(false, 256); }
#undef MOE_SPARSE
    hipLaunchKernelGGL(gate_dwg_reduce<true>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, partial, parts, M, E, dWg,
                       dgate_bias);
    return moe::check_launch();
  }
  hipLaunchKernelGGL(gate_dlogits, dim3((unsigned)((S + 3) / 4)), dim3(256), 0, st, dw, w, idx, logits, S, E, k,
                     norm, dlogits);
  const dim3 grid_dx((unsigned)((S + 127) / 128), (unsigned)((M + WX_COLS - 1) / WX_COLS));
#define MOE_DX(kg) do { \
    if (bf) hipLaunchKernelGGL((gate_dx_wide<true, kg>), grid_dx, dim3(256), 0, st, dlogits, Wg, dx, S, M, E, dx_accumulate); \
    else hipLaunchKernelGGL((gate_dx_wide<false, kg>), grid_dx, dim3(256), 0, st, dlogits, Wg, dx, S, M, E, dx_accumulate); } while (0)
  if (E <= 32) MOE_DX(4); else if (E <= 64) MOE_DX(8); else if (E <= 128) MOE_DX(16); else MOE_DX(32);
#undef MOE_DX
  const dim3 grid_w((unsigned)((M + 4 * WW_COLS - 1) / (4 * WW_COLS)), (unsigned)nchunk, (unsigned)((E + 63) / 64));
  if (bf) hipLaunchKernelGGL(gate_dwg_wide<true>, grid_w, dim3(256), 0, st, x, dlogits, partial, S, M, E, chunk);
  else hipLaunchKernelGGL(gate_dwg_wide<false>, grid_w, dim3(256), 0, st, x, dlogits, partial, S, M, E, chunk);
  hipLaunchKernelGGL(gate_dwg_reduce<false>, dim3((unsigned)((n + 63) / 64)), dim3(256), 0, st, partial, nchunk, M, E, dWg,
                     dgate_bias);
  return moe::check_launch();
}
