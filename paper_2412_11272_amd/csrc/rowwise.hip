// Bandwidth-bound kernels: ragged pack + hush append (with the row maps the convolutions need) and
// LayerNorm.  Both read and write every byte exactly once with 16-byte accesses.
#include <cstring>

#include "device_utils.h"
#include "kernels.h"

namespace wf {

namespace {

// ---------------------------------------------------------------------------------------------
// prep: (1) packed[r, :] = frame t of stream i  (t < T_i: the caller's frame; else hush[t - T_i]),
//           the concatenation x (+) h of every stream laid back to back without padding;
//       (2) conv1 row map: window of packed row r starts at row r-1; the first frame of a stream has
//           no left neighbour and the last no right neighbour (zero padding is per stream);
//       (3) conv2 row map: token j of stream i reads frames 2j-1, 2j, 2j+1 of that stream.
// One thread per 8 mel bins (threads [0, total_frames * n_mels/8)), then one thread per token.
// The index arrays are read from cu_frames .. n_frames, wherever those lie (device memory or LDS).
template <typename TIN, typename TOUT, typename TID>
__device__ __forceinline__ void prep_thread(const PrepArgs &p, const int32_t *cu_frames, const int32_t *cu_seqlens,
                                            const int32_t *frame_offset, const int32_t *n_frames) {
  const int cpr = p.n_mels >> 3;                       // 8-element chunks per frame
  const TID n_pack = (TID)p.total_frames * cpr;
  const TID gid = (TID)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid < n_pack) {
    const int r = (int)(gid / cpr), c = (int)(gid - (TID)r * cpr);
    const int i = find_stream(cu_frames, p.B, r);
    const int t = r - cu_frames[i];
    const int T = n_frames[i];
    const int Tp = cu_frames[i + 1] - cu_frames[i];
    TOUT *dst = (TOUT *)p.packed + (size_t)r * p.n_mels + c * 8;
    if (t < T) {
      const TIN *src = (const TIN *)p.mel + ((size_t)frame_offset[i] + t) * p.n_mels + c * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[e] = (TOUT)(float)src[e];
    } else {
      const TOUT *src = (const TOUT *)p.hush + (size_t)(t - T) * p.n_mels + c * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) dst[e] = src[e];
    }
    if (c == 0) {
      p.frame_src[r] = r - 1;
      p.frame_flags[r] = (t == 0 ? 1 : 0) | (t == Tp - 1 ? 2 : 0);
    }
    return;
  }
  const TID m = gid - n_pack;
  if (m < (TID)p.M) {
    const int i = find_stream(cu_seqlens, p.B, (int)m);
    const int j = (int)m - cu_seqlens[i];
    const int Tp = cu_frames[i + 1] - cu_frames[i];
    p.tok_src[m] = cu_frames[i] + 2 * j - 1;
    p.tok_flags[m] = (j == 0 ? 1 : 0) | (2 * j + 1 >= Tp ? 2 : 0);
    p.tok_pos[m] = j;
  }
}

template <typename TIN, typename TOUT>
__global__ void __launch_bounds__(256) prep_kernel(PrepArgs p) {
  prep_thread<TIN, TOUT, long>(p, p.cu_frames, p.cu_seqlens, p.frame_offset, p.n_frames);
}

// The index arrays come along in the arguments; block 0 also leaves them on the device for the kernels that follow.
struct IntsArg { int32_t n; int32_t v[kInlineInts]; };
static_assert(sizeof(PrepArgs) + sizeof(int32_t *) + sizeof(IntsArg) <= kLaunchBytes, "arguments of prep_inline_kernel");
static_assert(4 * sizeof(void *) + 2 * sizeof(int) + sizeof(IntsArg) <= kLaunchBytes, "arguments of embed_inline_kernel");

__device__ __forceinline__ void stage_ints(int32_t *lds, const IntsArg &a, int n, int32_t *dst) {
  for (int i = threadIdx.x; i < n; i += 256) lds[i] = a.v[i];
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.n; i += 256) dst[i] = a.v[i];
  __syncthreads();
}

template <typename TIN, typename TOUT>
__global__ void __launch_bounds__(256) prep_inline_kernel(PrepArgs p, int32_t *dst, IntsArg a) {
  __shared__ int32_t s[kInlineInts];
  const int S1 = p.B + 1;
  stage_ints(s, a, 4 * S1, dst);
  prep_thread<TIN, TOUT, unsigned>(p, s, s + S1, s + 2 * S1, s + 3 * S1);
}

// ---------------------------------------------------------------------------------------------
// LayerNorm: one wave per row, the row lives in registers between the two statistics passes
// (mean, then centred variance -- the biased one), fp32 statistics.  rows: out[i] = LayerNorm(x[rows[i]]) (NULL: x[i]).
// EARLY: gain and shift are requested together with the row.  For a few hundred rows a call is one chain of latencies, and
// loading them after the statistics puts a second memory latency into it (425 x 1280: 6.2 -> 5.4 us); once the chip is full
// the registers they occupy cost more (6361 x 1280: 12.6 us late, 17.3 early; both with the sums over a wave by shuffles).
// (ADD: the late form of wide rows adds a piece up as it arrives.  With the additions after all loads the compiler's other order of
// copies costs large calls 13 %, 31 694 x 1280 52.6 -> 59.6 us; rows of up to 512 values gain 5 % by it, 31 694 x 384 15.3 -> 14.5.)
// NP > 0: the residual product in front left its result as NP partial sums; they and its bias are added to the row first
// (part after part: deterministic) and the new row is stored.
template <typename TOUT, int MAXV, bool EARLY, int NP = 0>   // MAXV float4 per lane: d <= 256 * MAXV
__global__ void __launch_bounds__(256) layernorm_kernel(float *__restrict__ x, const int32_t *__restrict__ rows,
                                                        const float *__restrict__ g, const float *__restrict__ b,
                                                        TOUT *__restrict__ out, int M, int d, float eps, Partials pt, Prefetch pf) {
  __shared__ __attribute__((aligned(16))) unsigned char unread[4096];
  if (blockIdx.x >= (unsigned)(M + 3) / 4) {
    prefetch_block(pf, blockIdx.x - (M + 3) / 4, unread);
    return;
  }
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= M) return;
  const int lane = threadIdx.x & 63;
  const int nv = d >> 2;                               // float4 per row
  int xrow = row;
  if constexpr (EARLY) xrow = rows ? rows[row] : row;
  const f32x4 *xr = (const f32x4 *)(x + (size_t)xrow * d);
  const f32x4 *gr = (const f32x4 *)g, *br = (const f32x4 *)b;
  f32x4 v[MAXV], gg[EARLY ? MAXV : 1], bb[EARLY ? MAXV : 1];
  constexpr bool ADD = !EARLY && NP == 0 && MAXV > 2;
  float sum = 0.0f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int idx = lane + i * 64;
    if (idx < nv) {
      v[i] = xr[idx];
      if constexpr (EARLY) { gg[i] = gr[idx]; bb[i] = br[idx]; }
      if constexpr (ADD) sum += v[i][0] + v[i][1] + v[i][2] + v[i][3];
    }
  }
  if constexpr (NP > 0) {
    f32x4 w[NP][MAXV], wb[MAXV];
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = lane + i * 64;
      if (idx < nv) {
#pragma unroll
        for (int k = 0; k < NP; ++k) w[k][i] = ((const f32x4 *)(pt.part + ((size_t)k * pt.M + xrow) * d))[idx];
        wb[i] = ((const f32x4 *)pt.bias)[idx];
      }
    }
#pragma unroll
    for (int i = 0; i < MAXV; ++i) {
      const int idx = lane + i * 64;
      if (idx < nv) {
        f32x4 t = wb[i];
#pragma unroll
        for (int k = 0; k < NP; ++k)
#pragma unroll
          for (int e = 0; e < 4; ++e) t[e] += w[k][i][e];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[i][e] += t[e];
        if (!rows) ((f32x4 *)(x + (size_t)xrow * d))[idx] = v[i];
      }
    }
  }
  if constexpr (!ADD) {
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
      if (lane + i * 64 < nv) sum += v[i][0] + v[i][1] + v[i][2] + v[i][3];
  }
  sum = wave_sum(sum);
  const float mu = sum / (float)d;
  float sq = 0.0f;
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int idx = lane + i * 64;
    if (idx < nv) {
#pragma unroll
      for (int e = 0; e < 4; ++e) { const float t = v[i][e] - mu; sq += t * t; }
    }
  }
  sq = wave_sum(sq);
  const float rstd = rsqrtf(sq / (float)d + eps);
#pragma unroll
  for (int i = 0; i < MAXV; ++i) {
    const int idx = lane + i * 64;
    if (idx < nv) {
      f32x4 gi, bi, y;
      if constexpr (EARLY) { gi = gg[i]; bi = bb[i]; }
      else { gi = gr[idx]; bi = br[idx]; }
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = (v[i][e] - mu) * rstd * gi[e] + bi[e];
      if constexpr (sizeof(TOUT) == 2) {
        *(bf16x4 *)((__bf16 *)out + (size_t)row * d + idx * 4) = to_bf16x4(y);
      } else {
        *(f32x4 *)((float *)out + (size_t)row * d + idx * 4) = y;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Decoder input: x[r, :] = table[tok[r], :] + pos[pos_idx[r], :], one thread per 4 features.
template <typename TTAB, typename TID>
__device__ __forceinline__ void embed_thread(const TTAB *__restrict__ table, const float *__restrict__ pos, const int32_t *tok,
                                             const int32_t *pos_idx, float *__restrict__ x, int rows, int d) {
  const int cpr = d >> 2;
  const TID gid = (TID)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (TID)rows * cpr) return;
  const int r = (int)(gid / cpr), c = (int)(gid - (TID)r * cpr) * 4;
  const TTAB *t = table + (size_t)tok[r] * d + c;
  const f32x4 pe = *(const f32x4 *)(pos + (size_t)pos_idx[r] * d + c);
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = (float)t[e] + pe[e];
  *(f32x4 *)(x + (size_t)r * d + c) = v;
}

template <typename TTAB>
__global__ void __launch_bounds__(256) embed_kernel(const TTAB *__restrict__ table, const float *__restrict__ pos,
                                                    const int32_t *__restrict__ tok, const int32_t *__restrict__ pos_idx,
                                                    float *__restrict__ x, int rows, int d) {
  embed_thread<TTAB, long>(table, pos, tok, pos_idx, x, rows, d);
}

template <typename TTAB>
__global__ void __launch_bounds__(256) embed_inline_kernel(const TTAB *__restrict__ table, const float *__restrict__ pos,
                                                           float *__restrict__ x, int rows, int d, int32_t *dst, IntsArg a) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < a.n; i += 256) dst[i] = a.v[i];
  embed_thread<TTAB, unsigned>(table, pos, a.v, a.v + rows, x, rows, d);
}

// The caller's ints as a kernel argument.
hipError_t take_ints(const InlineInts &in, int need, IntsArg *a) {
  if (!in.dst || !in.src || in.n < need || in.n > kInlineInts) return hipErrorInvalidValue;
  a->n = in.n;
  memcpy(a->v, in.src, (size_t)in.n * 4);
  return hipSuccess;
}

}  // namespace

hipError_t launch_embed(const void *table, int table_bf16, const float *pos, const int32_t *tok, const int32_t *pos_idx,
                        float *x, int32_t rows, int32_t d, hipStream_t s, InlineInts in) {
  if (rows <= 0) return hipSuccess;
  if (d % 4 != 0) return hipErrorInvalidValue;
  const long n = (long)rows * (d / 4);
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  if (in.n > 0) {
    IntsArg a;
    const hipError_t err = take_ints(in, 2 * rows, &a);
    if (err != hipSuccess) return err;
    if (table_bf16) hipLaunchKernelGGL(embed_inline_kernel<__bf16>, grid, block, 0, s, (const __bf16 *)table, pos, x, rows, d, in.dst, a);
    else hipLaunchKernelGGL(embed_inline_kernel<float>, grid, block, 0, s, (const float *)table, pos, x, rows, d, in.dst, a);
    return hipGetLastError();
  }
  if (table_bf16) hipLaunchKernelGGL(embed_kernel<__bf16>, grid, block, 0, s, (const __bf16 *)table, pos, tok, pos_idx, x, rows, d);
  else hipLaunchKernelGGL(embed_kernel<float>, grid, block, 0, s, (const float *)table, pos, tok, pos_idx, x, rows, d);
  return hipGetLastError();
}

hipError_t launch_layernorm(float *x, const int32_t *rows, const float *g, const float *b, void *out, int out_bf16,
                            int32_t M, int32_t d, float eps, hipStream_t s, Partials pt, Prefetch pf) {
  if (M <= 0) return hipSuccess;
  if (pt.n == 1 || pt.n < 0 || pt.n > 4 || (pt.n && (!pt.part || !pt.bias || pt.M < M))) return hipErrorInvalidValue;
  if (d % 4 != 0 || d > 256 * 8) return hipErrorInvalidValue;
  if (pf.bytes && (!pf.p || pf.bytes % 16 || pf.bytes >= 1u << 31)) return hipErrorInvalidValue;
  const dim3 grid((M + 3) / 4 + (pf.bytes ? pf.blocks : 0)), block(256);
  const bool early = M <= 2048 || rows;        // two workgroups per compute unit; rows by index exist in that form only
#define WF_LN2(T, V, E, P) hipLaunchKernelGGL((layernorm_kernel<T, V, E, P>), grid, block, 0, s, x, rows, g, b, (T *)out, M, d, eps, pt, pf)
#define WF_LN1(T, V, E)                    \
  do {                                     \
    if (pt.n == 2) WF_LN2(T, V, true, 2);  \
    else if (pt.n == 3) WF_LN2(T, V, true, 3); \
    else if (pt.n == 4) WF_LN2(T, V, true, 4); \
    else WF_LN2(T, V, E, 0);               \
  } while (0)
#define WF_LN(V)                                                                           \
  do {                                                                                     \
    if (out_bf16) { if (early) { WF_LN1(__bf16, V, true); } else { WF_LN1(__bf16, V, false); } }   \
    else { if (early) { WF_LN1(float, V, true); } else { WF_LN1(float, V, false); } }              \
  } while (0)
  if (d <= 256 * 2) WF_LN(2);
  else if (d <= 256 * 5) WF_LN(5);
  else WF_LN(8);
#undef WF_LN
#undef WF_LN1
#undef WF_LN2
  return hipGetLastError();
}

hipError_t launch_prep(const PrepArgs &a, int packed_bf16, hipStream_t s, InlineInts in) {
  const long n = prep_threads(a.total_frames, a.n_mels, a.M);
  if (n <= 0) return hipSuccess;
  const dim3 grid((unsigned)((n + 255) / 256)), block(256);
  if (in.n > 0) {
    IntsArg ints;
    const hipError_t err = prep_takes_ints(in.n, n) ? take_ints(in, 4 * (a.B + 1), &ints) : hipErrorInvalidValue;
    if (err != hipSuccess) return err;
#define WF_PREP(TI, TO) hipLaunchKernelGGL((prep_inline_kernel<TI, TO>), grid, block, 0, s, a, in.dst, ints)
    if (packed_bf16) { if (a.mel_is_bf16) WF_PREP(__bf16, __bf16); else WF_PREP(float, __bf16); }
    else { if (a.mel_is_bf16) WF_PREP(__bf16, float); else WF_PREP(float, float); }
#undef WF_PREP
    return hipGetLastError();
  }
  if (packed_bf16) {
    if (a.mel_is_bf16) hipLaunchKernelGGL((prep_kernel<__bf16, __bf16>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((prep_kernel<float, __bf16>), grid, block, 0, s, a);
  } else {
    if (a.mel_is_bf16) hipLaunchKernelGGL((prep_kernel<__bf16, float>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((prep_kernel<float, float>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace wf
