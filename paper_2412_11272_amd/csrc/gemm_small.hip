// bf16 MFMA GEMMs for SMALL row counts (a single stream's buffer, a few hundred tokens: the case the paper's
// method itself runs, Section "Operations"), where nothing is bound by the matrix pipe and everything by how long
// the chain of dependent steps of one workgroup is and by how many workgroups share the work.
//
//   out = epilogue(A . W^T),  A [M, K], W [N, K], fp32 accumulation, M up to about a thousand rows of a narrow model, or few
//   enough rows of any product (gemm_small_few_rows, gemm_slice_applies).
//
//   gemm_slice_kernel   the operand is in memory as it is needed: plain rows or the windows of a convolution, eight waves share K
//   gemm_ln_kernel      the operand is LayerNorm(x) of an fp32 matrix x with rows of at most 512 values (every model narrow enough
//                       for this file), normalised on the way in.  This removes two kernels per transformer block; with a few
//                       hundred tokens each kernel in the chain costs 3-5 us whatever it does.
//   gemm_small_kernel   four waves share K: short reductions and weights of 4 GiB and more (takes_four_waves), LayerNorm(x) of longer rows
//                       (wf_op_ln_linear only)

#include <algorithm>
#include <mutex>

#include "gemm_epilogue.h"

namespace wf {

namespace {

constexpr int SBM = 32, SBN = 32, SBK = 64;
constexpr int kMaxLnK = 2048;     // gemm_small_kernel keeps the LayerNorm gain and shift of the whole row in LDS (A_LN)
constexpr unsigned kOutside = 0xFFFFFFF0u;         // a byte offset no buffer reaches: the load returns zeros

typedef __attribute__((address_space(3))) void lds_void;

// Plain rows and windows of a short reduction, and LayerNorm(x) operands of up to kMaxLnK values.  32-row tiles, 32, 64 or 128 columns
// wide (NB column blocks of 32): the launcher takes the widest that still leaves about 160 workgroups, because every column tile
// re-reads (and re-normalises) the same 32 rows.  The four waves split the reduction: in every 64-deep K step wave w multiplies the
// k slice [16 w, 16 w + 16) with one 32x32x16 MFMA, and the four partial tiles are added in a fixed order through LDS at the end
// (deterministic).  Chunks are requested eight (widest tile: four) K steps ahead into registers, two K steps are staged in LDS per
// barrier.  A_LN: the workgroup first computes mean and 1/sqrt(var + eps) of its 32 rows (one pass, sums shifted by the row's
// first element so that the variance does not cancel), then every chunk is (x - mean) * rstd * gamma + beta rounded to bf16 --
// exactly what the LayerNorm kernel would have stored.
template <int AMODE, int EPI, int NB>
__global__ void __launch_bounds__(256) gemm_small_kernel(GemmArgs p) {
  constexpr int TN = NB * SBN;                                               // tile width in columns
  constexpr int DEPTH = NB >= 4 ? 4 : 8;                                     // K steps in flight (register ring)
  // SPB K steps are staged in LDS per barrier, double-buffered (NS = 2 SPB stages per operand); the four waves'
  // partial tiles reuse the same memory after the K loop.
  constexpr int SPB = 2, NS = 2 * SPB;               // (four per barrier measured the same as two)
  constexpr int STAGE_BYTES = NS * (SBM + TN) * 128, PART_BYTES = 4 * SBM * (TN + 4) * 4;
  __shared__ __attribute__((aligned(16))) unsigned char sMem[STAGE_BYTES > PART_BYTES ? STAGE_BYTES : PART_BYTES];
  unsigned char(*sA)[SBM * 128] = (unsigned char(*)[SBM * 128])sMem;                     // [stage][row][64 bf16]
  unsigned char(*sW)[TN * 128] = (unsigned char(*)[TN * 128])(sMem + NS * SBM * 128);
  float(*sPart)[SBM][TN + 4] = (float(*)[SBM][TN + 4])sMem;
  __shared__ __attribute__((aligned(16))) float sGain[AMODE == A_LN ? kMaxLnK : 4], sShift[AMODE == A_LN ? kMaxLnK : 4];

  const int tiles_n = p.N / TN;
  const int m0 = (blockIdx.x / tiles_n) * SBM, n0 = (blockIdx.x % tiles_n) * TN;
  if constexpr (AMODE == A_PLAIN && EPI == EPI_BIAS) p.out = group_out(p, n0);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lg = lane >> 5;

  // ---- load descriptors: thread -> (row r, 16-byte chunk ch) of both operand tiles, fixed over the K loop
  const int r = tid >> 3, ch = tid & 7;
  int row = m0 + r;
  row = row < p.M ? row : p.M - 1;               // rows past M are computed but never stored
  const int lds_off = r * 128 + ((ch ^ ((r >> 1) & 7)) << 4);
  const __bf16 *W = (const __bf16 *)p.W;
  const __bf16 *wptr[NB];                        // weight rows n0 + 32 j + r
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = n0 + j * SBN + r;
    wptr[j] = p.w_panels ? W + ((size_t)(n >> 8) * (p.K >> 6) << 14) + ((n & 255) << 6) + ch * 8 : W + (size_t)n * p.K + ch * 8;
  }
  const int wstep = p.w_panels ? 1 << 14 : SBK;
  const __bf16 *aptr = nullptr;
  const float *xptr = nullptr;
  int flags = 0;
  if constexpr (AMODE == A_PLAIN) aptr = (const __bf16 *)p.A + (size_t)row * p.lda + ch * 8;
  else if constexpr (AMODE == A_CONV3) {
    aptr = (const __bf16 *)p.A + (long)p.row_src[row] * p.C + ch * 8;
    flags = p.row_flags[row];
  } else xptr = (const float *)p.A + (size_t)row * p.lda + ch * 8;

  [[maybe_unused]] float mu = 0.0f, rstd = 0.0f;     // A_LN: statistics of this thread's row
  // ---- operand pipeline: chunks of K step kt + DEPTH - 1 are requested while step kt is multiplied
  u32x4 wreg[DEPTH][NB];
  [[maybe_unused]] u32x4 areg[DEPTH];
  [[maybe_unused]] f32x4 xreg[DEPTH][2];
  const int nk = p.K / SBK;
  auto request = [&](int kt, int slot) {
#pragma unroll
    for (int j = 0; j < NB; ++j) wreg[slot][j] = *(const u32x4 *)(wptr[j] + (size_t)kt * wstep);
    if constexpr (AMODE == A_PLAIN) {
      areg[slot] = *(const u32x4 *)(aptr + kt * SBK);
    } else if constexpr (AMODE == A_CONV3) {
      const int kk = kt * SBK + ch * 8;          // chunks never straddle taps: C % 8 == 0
      const int tap = kk / p.C;
      const bool ok = (kk < 3 * p.C) && !((tap == 0) && (flags & 1)) && !((tap == 2) && (flags & 2));
      u32x4 v = {0u, 0u, 0u, 0u};
      if (ok) v = *(const u32x4 *)(aptr + kt * SBK);
      areg[slot] = v;
    } else {
      xreg[slot][0] = *(const f32x4 *)(xptr + kt * SBK);
      xreg[slot][1] = *(const f32x4 *)(xptr + kt * SBK + 4);
    }
  };
  auto commit = [&](int kt, int slot) {          // registers -> LDS stage kt % NS
    unsigned char *dA = sA[kt & (NS - 1)] + lds_off, *dW = sW[kt & (NS - 1)] + lds_off;
#pragma unroll
    for (int j = 0; j < NB; ++j) *(u32x4 *)(dW + j * SBN * 128) = wreg[slot][j];
    if constexpr (AMODE == A_LN) {
      const int k = kt * SBK + ch * 8;
      const f32x4 g0 = *(const f32x4 *)&sGain[k], g1 = *(const f32x4 *)&sGain[k + 4];
      const f32x4 b0 = *(const f32x4 *)&sShift[k], b1 = *(const f32x4 *)&sShift[k + 4];
      f32x4 y0, y1;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y0[e] = (xreg[slot][0][e] - mu) * rstd * g0[e] + b0[e];
        y1[e] = (xreg[slot][1][e] - mu) * rstd * g1[e] + b1[e];
      }
      const bf16x4 c0 = to_bf16x4(y0), c1 = to_bf16x4(y1);
      *(bf16x8 *)dA = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
    } else {
      *(u32x4 *)dA = areg[slot];
    }
  };

  f32x16 acc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.0f;
#pragma unroll
  for (int d = 0; d < DEPTH; ++d)
    if (d < nk) request(d, d);
  // ---- A_LN: statistics of the tile's 32 rows (after the first operand requests, so that their latencies overlap).
  // Eight threads per row, each over every eighth 32-byte piece, eight pieces requested at a time.
  if constexpr (AMODE == A_LN) {
    for (int k = tid * 4; k < p.K; k += 1024) {   // gain and shift of the whole row -> LDS (a load per K step would sit
      *(f32x4 *)&sGain[k] = *(const f32x4 *)(p.ln_g + k);   // on the critical path of every step)
      *(f32x4 *)&sShift[k] = *(const f32x4 *)(p.ln_b + k);
    }
    const float *xr = (const float *)p.A + (size_t)row * p.lda;
    const float pivot = xr[0];
    float s1 = 0.0f, s2 = 0.0f;
    for (int k0 = ch * 8; k0 < p.K; k0 += 512) {
      f32x4 a[8], b[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = min(k0 + i * 64, p.K - 8);         // past the end: a valid address, the values are not used
        a[i] = *(const f32x4 *)(xr + k);
        b[i] = *(const f32x4 *)(xr + k + 4);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (k0 + i * 64 < p.K) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float da = a[i][e] - pivot, db = b[i][e] - pivot;
            s1 += da + db;
            s2 += da * da + db * db;
          }
        }
      }
    }
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) {     // the eight threads of a row are neighbouring lanes
      s1 += __shfl_xor(s1, off);
      s2 += __shfl_xor(s2, off);
    }
    const float inv_k = 1.0f / (float)p.K;
    const float ms = s1 * inv_k;                 // mean - pivot
    const float var = fmaxf(s2 * inv_k - ms * ms, 0.0f);
    mu = pivot + ms;
    rstd = rsqrtf(var + p.ln_eps);
    __syncthreads();                             // gain / shift are in LDS
  }
  // fragment of wave `wave`: row l32, k slice 16 * wave + 8 * lg .. + 7 = chunk 2 * wave + lg
  const int frag_off = l32 * 128 + (((2 * wave + lg) ^ ((l32 >> 1) & 7)) << 4);
  // SPB K steps per barrier: they are written to their stages, their register slots are refilled with the steps
  // DEPTH further on, and after one barrier all of them are multiplied.  The group after the next one reuses these
  // stages; a wave gets there only through the next barrier, which every wave reaches after its reads of this group.
  auto multiply = [&](int kt) {
    const bf16x8 xf = *(const bf16x8 *)(sA[kt & (NS - 1)] + frag_off);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bf16x8 wf = *(const bf16x8 *)(sW[kt & (NS - 1)] + j * SBN * 128 + frag_off);
      acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, acc[j], 0, 0, 0);
    }
  };
  static_assert(DEPTH % SPB == 0, "the ring is walked SPB slots at a time");
  for (int kt0 = 0; kt0 < nk; kt0 += DEPTH) {
#pragma unroll
    for (int d = 0; d < DEPTH; d += SPB) {       // unrolled by the ring depth: register slots are compile-time
      const int kt = kt0 + d;
      if (kt < nk) {
#pragma unroll
        for (int q = 0; q < SPB; ++q)
          if (kt + q < nk) commit(kt + q, d + q);
#pragma unroll
        for (int q = 0; q < SPB; ++q)
          if (kt + q + DEPTH < nk) request(kt + q + DEPTH, d + q);
        __syncthreads();                         // the stages of steps kt .. kt + SPB - 1 are complete
#pragma unroll
        for (int q = 0; q < SPB; ++q)
          if (kt + q < nk) multiply(kt + q);
      }
    }
  }
  __syncthreads();                               // every wave is done with the stages: the partial tiles may overwrite them

  // ---- the four k slices are added in wave order; lane holds token l32, features 8 (i / 4) + 4 lg + i % 4 of block j
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) sPart[wave][l32][j * SBN + 8 * (i >> 2) + 4 * lg + (i & 3)] = acc[j][i];
  __syncthreads();
  // thread -> row er, 4 consecutive features from ec in each of the NB column blocks
  const int er = tid >> 3, m = m0 + er;
  if (m >= p.M) return;
  [[maybe_unused]] int prow = 0;
  if constexpr (EPI == EPI_BIAS_GELU_POS) prow = p.row_pos[m];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int ec = j * SBN + (tid & 7) * 4;
    f32x4 v = *(const f32x4 *)&sPart[0][er][ec];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const f32x4 t = *(const f32x4 *)&sPart[w][er][ec];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += t[e];
    }
    const int nn = n0 + ec;
    const f32x4 b = *(const f32x4 *)(p.bias + nn);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += b[e];
    if constexpr (EPI == EPI_BIAS) {
      __bf16 *dst = (p.out2 && nn >= p.n_split) ? (__bf16 *)p.out2 + (size_t)m * p.ldo2 + (nn - p.n_split)
                                                 : (__bf16 *)p.out + (size_t)m * p.ldo + nn;
      *(bf16x4 *)dst = to_bf16x4(v);
    } else if constexpr (EPI == EPI_BIAS_GELU) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
      *(bf16x4 *)((__bf16 *)p.out + (size_t)m * p.ldo + nn) = to_bf16x4(v);
    } else if constexpr (EPI == EPI_BIAS_RESID) {
      f32x4 *o = (f32x4 *)((float *)p.out + (size_t)m * p.ldo + nn);
      const f32x4 x = *o;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] += x[e];
      *o = v;
    } else {
      const f32x4 pe = *(const f32x4 *)(p.pos + (size_t)prow * p.N + nn);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]) + pe[e];
      *(f32x4 *)((float *)p.out + (size_t)m * p.ldo + nn) = v;
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// out = epilogue(LayerNorm(x) . W^T) for rows of at most 512 values.  A call is one chain of latencies, so everything it
// reads is requested at once: the weight tile [64, K], gain and shift go global -> LDS as a whole, a workgroup's TM rows into
// registers, where they are normalised (mean, then centred variance) and left in LDS as the bf16 operand.  Two barriers, then the waves
// multiply the whole of K in order, each a 16-column strip of its own, and store without a reduction.
// A workgroup keeps its weight tile for the row tiles g, g + row_groups, ...
// What bounds it: the L1 takes 16 clocks an instruction of 1 KB, whether lanes ask for the same lines or not, so gain and shift go to
// the LDS once instead of to every wave's registers (a third of all load instructions); then the additions of the statistics, which every
// column tile repeats for its rows, and the LDS reads of the K loop.
// Before and after gain and shift in the LDS, statistics under the weights' arrival and the choice of 16 to 64 rows (us a launch): 75 x 1152 x
// 384 3.9 -> 3.4, 100 x 1536 x 512 4.6 -> 3.7, 244 x 2048 x 512 5.7 -> 5.0, 425 x 1536 x 512 8.1 -> 5.8, 925 x 1152 x 384 8.0 -> 6.6.
// Encoder calls: 75 tokens, d = 384 90.3 -> 84.5; 243 tokens, d = 512 162 -> 157; prefill of 100 tokens, d = 512 250 -> 231 us.
// (With K known only at run time the exposed LDS latency of every K step took a third of the gain over the unfused kernels back.)
constexpr int kLnRowK = 512, kLnTN = 64;

// NK: K / 64 where it is known when compiled (the loads and the K loop are then straight-line code), else 0.
template <int TM, int EPI, int NK>
__global__ void __launch_bounds__(256) gemm_ln_kernel(GemmArgs p, int row_groups) {
#ifdef __HIP_DEVICE_COMPILE__       // buffer resources are a device type: the host only needs the kernel's name
  constexpr int TN = kLnTN, TB = TM / 16, RI = TM / 16;           // row blocks of the product; turns of four rows a wave
  constexpr int JV = NK ? NK : kLnRowK / 64;                      // 64-column pieces of a row
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_ln[];
  const int K = NK ? NK * 64 : p.K, nk = K >> 6;
  unsigned char *sW = smem_ln, *sA = smem_ln + nk * TN * 128;      // [K step][row][64 bf16], chunk c of row r at c ^ ((r >> 1) & 7)
  float *sGain = (float *)(sA + nk * TM * 128), *sShift = sGain + kLnRowK;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int tiles_n = p.N / TN, tiles_m = (p.M + TM - 1) / TM;
  const int n0 = blockIdx.x % tiles_n * TN;

  // ---- gain and shift: one load instruction a wave.  (Loads to the LDS in the buffer form: behind the global form the compiler waits
  // for every load at the first use of any, and the statistics would not run while the weights arrive.)
  {
    // The place of a wave's half is part of the vector offset, which the bounds check against K values covers by definition.
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)(wave < 2 ? p.ln_g : p.ln_b), 0, K * 4, 0x00027000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void *)((wave < 2 ? sGain : sShift) + (wave & 1) * 256), 16, (wave & 1) * 1024 + lane * 16, 0, 0, 0);
  }
  // A wave's loads complete in order, so this one has landed once the rows are in registers, if it was issued before them: the fence sees
  // to that.  The first barrier below publishes gain and shift on the strength of it, without a wait for the weights.
  __builtin_amdgcn_sched_barrier(0x1);             // (arithmetic may cross: held back as well, the rows leave 0.1 .. 0.2 us later)
  // ---- rows: 16 lanes a row, four columns of every 64; this lane's rows of a tile are RI * 4 * wave + 4 i + lq
  f32x4 x[RI][JV];
  auto request = [&](int tile) {
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      const float *xr = (const float *)p.A + (size_t)min(tile * TM + (wave * RI + i) * 4 + lq, p.M - 1) * p.lda + l16 * 4;
#pragma unroll
      for (int j = 0; j < JV; ++j)
        if (j < nk) x[i][j] = *(const f32x4 *)(xr + j * 64);
    }
  };
  int tile = blockIdx.x / tiles_n;
  request(tile);
  const f32x4 bias = *(const f32x4 *)(p.bias + n0 + wave * 16 + lq * 4);
  {
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W, 0, (int)((size_t)(p.w_panels ? (p.N + 255) & ~255 : p.N) * K * 2), 0x00027000);
    const int rr = lane >> 3, wrow = p.w_panels ? 128 : K * 2, wstep = p.w_panels ? 32768 : 128;
    const int base = (p.w_panels ? (((n0 >> 8) * nk) << 15) + ((n0 & 255) << 7) : n0 * K * 2) + wave * 8 * wrow;      // (a tile lies in one panel)
    const int off = rr * wrow + (((lane & 7) ^ ((wave * 4 + (rr >> 1)) & 7)) << 4);
#pragma unroll NK ? NK : 1
    for (int kt = 0; kt < nk; ++kt)
#pragma unroll
      for (int i = 0; i < TN / 32; ++i)            // eight rows of 128 bytes per instruction
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(sW + (kt * TN + (i * 4 + wave) * 8) * 128), 16, off, base + i * 32 * wrow + kt * wstep, 0, 0);
  }
  const float inv_k = 1.0f / (float)K;
  auto process = [&](int tile, bool first) {
    float mu[RI], rstd[RI];
#pragma unroll
    for (int i = 0; i < RI; ++i) {
      float sum = 0.0f, sq = 0.0f;
#pragma unroll
      for (int j = 0; j < JV; ++j)
        if (j < nk) sum += (x[i][j][0] + x[i][j][1]) + (x[i][j][2] + x[i][j][3]);
      mu[i] = row_sum(sum) * inv_k;
#pragma unroll
      for (int j = 0; j < JV; ++j)
        if (j < nk)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            x[i][j][e] -= mu[i];
            sq += x[i][j][e] * x[i][j][e];
          }
      rstd[i] = rsqrtf(row_sum(sq) * inv_k + p.ln_eps);
    }
    if (first) {          // gain and shift were requested before the rows: this wave's part of them is in the LDS by now
#pragma unroll
      for (int i = 0; i < RI; ++i) asm volatile("" : "+v"(rstd[i]));        // (the rows have been read: not an instruction, but no way round it)
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < JV; ++j)
      if (j < nk) {
        const f32x4 g = *(const f32x4 *)(sGain + j * 64 + l16 * 4), b = *(const f32x4 *)(sShift + j * 64 + l16 * 4);
#pragma unroll
        for (int i = 0; i < RI; ++i) {
          const int r = (wave * RI + i) * 4 + lq;
          f32x4 y;
#pragma unroll
          for (int e = 0; e < 4; ++e) y[e] = x[i][j][e] * rstd[i] * g[e] + b[e];
          *(bf16x4 *)(sA + (j * TM + r) * 128 + (((l16 >> 1) ^ ((r >> 1) & 7)) << 4) + (l16 & 1) * 8) = to_bf16x4(y);
        }
      }
    __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0) lgkmcnt(0): this wave's rows are in LDS, its weights too
    __syncthreads();
    if (tile + row_groups < tiles_m) request(tile + row_groups);
    f32x4 acc[TB];
#pragma unroll
    for (int i = 0; i < TB; ++i) acc[i] = bias;
    const int sw = (l16 >> 1) & 7;
    const unsigned char *cw = sW + (wave * 16 + l16) * 128, *cx = sA + l16 * 128;
#pragma unroll NK ? NK : 1
    for (int kt = 0; kt < nk; ++kt)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int off = ((4 * t + lq) ^ sw) << 4;
        const bf16x8 wf = *(const bf16x8 *)(cw + kt * TN * 128 + off);
#pragma unroll
        for (int i = 0; i < TB; ++i) {
          const bf16x8 xf = *(const bf16x8 *)(cx + (kt * TM + i * 16) * 128 + off);
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf, xf, acc[i], 0, 0, 0);
        }
      }
    // lane holds, of token l16 of a row block, features 16 wave + 4 lq .. + 3
#pragma unroll
    for (int i = 0; i < TB; ++i) {
      const int m = tile * TM + i * 16 + l16, nn = n0 + wave * 16 + lq * 4;
      f32x4 v = acc[i];
      if constexpr (EPI == EPI_BIAS_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
      }
      if (m < p.M) {
        __bf16 *dst = (EPI == EPI_BIAS && p.out2 && nn >= p.n_split) ? (__bf16 *)p.out2 + (size_t)m * p.ldo2 + (nn - p.n_split)
                                                                     : (__bf16 *)p.out + (size_t)m * p.ldo + nn;
        *(bf16x4 *)dst = to_bf16x4(v);
      }
    }
  };
  process(tile, true);    // by itself: its first wait is for the rows only, the weights arrive under the statistics
  for (tile += row_groups; tile < tiles_m; tile += row_groups) {
    __syncthreads();      // the operand has been read; the next rows may take its place
    process(tile, false);
  }
#endif
}

constexpr int ln_smem(int tm, int k) { return (kLnTN + tm) * k * 2 + 2 * kLnRowK * 4; }

template <int TM, int EPI, int NK>
hipError_t launch_ln_tile(const GemmArgs &a, hipStream_t s) {
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute((const void *)gemm_ln_kernel<TM, EPI, NK>, hipFuncAttributeMaxDynamicSharedMemorySize, ln_smem(TM, kLnRowK));
  });
  if (attr_err != hipSuccess) return attr_err;
  const int smem = ln_smem(TM, a.K), tiles_n = a.N / kLnTN, tiles_m = (a.M + TM - 1) / TM;
  const int slots = 256 * std::min(4, 163840 / smem);               // workgroups the chip holds at a time
  const int groups = std::min(tiles_m, std::max(1, slots / tiles_n));
  hipLaunchKernelGGL((gemm_ln_kernel<TM, EPI, NK>), dim3((unsigned)(groups * tiles_n)), dim3(256), smem, s, a, groups);
  return hipGetLastError();
}

// Rows of a tile.  Up to 384 values two workgroups share a CU: 16 rows (3.4 us with one a CU, 4.1 .. 4.4 with two) while two a CU are
// enough, then 32 (5.2 .. 5.5 us), beyond that 16 again (700 x 1536 6.6 and 7.1 us).  Longer rows, one workgroup a CU: the least
// of start + further rounds, fitted to 13 .. 1020 rows of 512 (us: 16 rows 3.7 + 1.45 a round, 32 4.75 + 2.8, 48 5.55 + 4.1, 64
// 6.7 + 4.8); the taken size is the fastest or within 3 % of it.
int pick_ln_rows(int M, int N, int K) {
  const int tiles_n = N / kLnTN;
  auto units = [&](int tm) { return (long)((M + tm - 1) / tm) * tiles_n; };
  if (K <= 384) return units(16) > 512 && units(32) <= 512 ? 32 : 16;
  constexpr struct { int rows; double first, more; } kCost[] = {{16, 3.7, 1.45}, {32, 4.75, 2.8}, {48, 5.55, 4.1}, {64, 6.7, 4.8}};
  int best = 0;
  double cost = 0.0;
  for (const auto &c : kCost) {
    const int tiles_m = (M + c.rows - 1) / c.rows, groups = std::max(1, 256 / tiles_n);
    const double us = c.first + c.more * ((tiles_m + groups - 1) / groups - 1);
    if (!best || us < cost) { best = c.rows; cost = us; }
  }
  return best;
}

template <int EPI, int NK>
hipError_t launch_ln_rows(const GemmArgs &a, hipStream_t s) {
  const int rows = pick_ln_rows(a.M, a.N, a.K);
  if (rows == 16) return launch_ln_tile<16, EPI, NK>(a, s);
  if (rows == 32) return launch_ln_tile<32, EPI, NK>(a, s);
  if constexpr (NK != 6) return rows == 48 ? launch_ln_tile<48, EPI, NK>(a, s) : launch_ln_tile<64, EPI, NK>(a, s);
  return hipErrorInvalidValue;
}

template <int EPI>
hipError_t launch_ln(const GemmArgs &a, hipStream_t s) {
  if (a.N % kLnTN) return hipErrorInvalidValue;
  switch (a.K) {
    case 512: return launch_ln_rows<EPI, 8>(a, s);
    case 384: return launch_ln_rows<EPI, 6>(a, s);
    default: return launch_ln_rows<EPI, 0>(a, s);
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// Products whose operand is in memory as it is needed (plain rows, windows of a convolution).  A workgroup's chain of latencies is
// all there is to such a call, so nothing in it waits for anything but its own operands: the eight waves share the reduction
// (wave w takes the 64-deep K steps w, w + 8, ..), each fetches its steps into an LDS ring of its own, all of them requested at
// the start where they fit, and multiplies them without a barrier.  One barrier later the eight partial tiles are added up
// in wave order.  Which steps a wave takes and in which order does not depend on the tile, so a row's bits do not either.
//
// What bounds it: a launch (1.8 us for a kernel that reads and stores one value), one memory latency, then the operand bytes of a
// tile at 64 bytes a clock, the rate of one L1, or of all tiles at about 19 TB/s over the chip.
// Against the kernel it replaced (four waves walking K together with a barrier every two steps; us a launch in a chain of launches):
// 75 x 384 x 384 2.9 -> 2.6, 75 x 384 x 1536 5.1 -> 3.2, 244 x 512 x 2048 6.7 -> 4.3, 1000 x 512 x 2048 10.6 -> 7.5, 100 x 1280 x 5120
// 13.6 -> 8.1.  Encoder calls: 75 tokens, d = 384 109.6 -> 93, 243 tokens, d = 512 192.7 -> 171; 50 tokens, d = 1024 1046 -> 880.
template <int TM, int TN, int SLOTS>
constexpr int slice_smem() {
  constexpr int stages = 8 * SLOTS * (TM + TN) * 128, parts = 8 * TM * (TN + 4) * 4;
  return stages > parts ? stages : parts;
}

// Wait until at most V of this wave's loads are outstanding.
template <int V>
__device__ __forceinline__ void wait_loads() {
  static_assert(V >= 0 && V < 64, "more loads in flight than the counter holds");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (V & 15) | ((V >> 4) << 14));
}

template <int TM, int TN, int SLOTS, int AMODE, int EPI>
__global__ void __launch_bounds__(512) gemm_slice_kernel(GemmArgs p) {
#ifdef __HIP_DEVICE_COMPILE__       // buffer resources are a device type: the host only needs the kernel's name
  constexpr int NW = 8, TB = TM / 16, FB = TN / 16, XL = TM / 8, WL = TN / 8, LPS = XL + WL;
  constexpr int SLOT = (TM + TN) * 128, PITCH = TN + 4;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_slice[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, lq = lane >> 4, rr = lane >> 3;
  const int tiles_n = p.N / TN;
  const int m0 = blockIdx.x / tiles_n * TM, n0 = blockIdx.x % tiles_n * TN;      // a column of tiles keeps to an XCD or two
  if constexpr (EPI == EPI_BIAS) p.out = group_out(p, n0);
  unsigned char *ring = smem_slice + wave * SLOTS * SLOT;

  // ---- this thread's outputs, and what the epilogue adds to them (requested first: nothing later waits for them)
  constexpr int VEC = TM * TN >= 2048 ? 4 : 2, PER = TM * TN / VEC > 512 ? TM * TN / VEC / 512 : 1, COLS = TN / VEC;
  const bool has = PER > 1 || TM * TN / VEC == 512 || tid < TM * TN / VEC;
  typedef float vec __attribute__((ext_vector_type(VEC)));
  const int ec = tid % COLS * VEC, er = tid / COLS % TM;           // (threads without an output repeat another's)
  const vec bias = *(const vec *)(p.bias + n0 + ec);
  vec add[PER];
  [[maybe_unused]] int prow[PER];
  if constexpr (EPI == EPI_BIAS_RESID) {
#pragma unroll
    for (int u = 0; u < PER; ++u) add[u] = *(const vec *)((const float *)p.out + (size_t)min(m0 + er + u * (512 / COLS), p.M - 1) * p.ldo + n0 + ec);
  } else if constexpr (EPI == EPI_BIAS_GELU_POS) {
#pragma unroll
    for (int u = 0; u < PER; ++u) prow[u] = p.row_pos[min(m0 + er + u * (512 / COLS), p.M - 1)];
  }

  // ---- loads: eight rows of 128 bytes per instruction, 16-byte chunk c of row r at c ^ ((r >> 1) & 7); K steps past the end
  // load from outside the buffer (zeros), so that every wave makes the same number of turns
  const int nk = p.K >> 6, ns = (nk + NW - 1) / NW;
  const size_t a_bytes = p.a_panels ? (size_t)((p.M + 255) >> 8) * 256 * p.K * 2 : ((size_t)(p.M - 1) * p.lda + p.K) * 2;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void *)p.A, 0, AMODE == A_CONV3 ? (int)kOutside : (int)a_bytes, 0x00027000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void *)p.W, 0, (int)((size_t)(p.w_panels ? (p.N + 255) & ~255 : p.N) * p.K * 2), 0x00027000);
  const int astep = p.a_panels ? 32768 : 128, wstep = p.w_panels ? 32768 : 128, wrow = p.w_panels ? 128 : p.K * 2;
  const int wbase = p.w_panels ? (((n0 >> 8) * nk) << 15) + ((n0 & 255) << 7) : (int)((unsigned)n0 * (unsigned)p.K * 2u);        // (a tile lies in one panel)
  const int piece = ((lane & 7) ^ (rr >> 1)) << 4;                 // of the even groups of eight rows; the odd ones have it at ^ 64
  const int woff[2] = {rr * wrow + piece, rr * wrow + (piece ^ 64)};
  int aoff[XL];
  [[maybe_unused]] int aflags[AMODE == A_CONV3 ? XL : 1];
#pragma unroll
  for (int i = 0; i < XL; ++i) {
    const int row = min(m0 + i * 8 + rr, p.M - 1);                 // rows past M are computed but never stored
    if constexpr (AMODE == A_CONV3) { aoff[i] = p.row_src[row]; aflags[i] = p.row_flags[row]; }      // (gemm_slice_reaches)
    else aoff[i] = (p.a_panels ? (((row >> 8) * nk) << 15) + ((row & 255) << 7) : (int)((unsigned)row * (unsigned)p.lda * 2u)) + (piece ^ ((i & 1) << 6));
  }
  auto load_w = [&](int i, int slot) {
    const int kt = wave + i * NW, off = kt < nk ? wbase + kt * wstep : 0;
    const int v[2] = {kt < nk ? woff[0] : (int)kOutside, kt < nk ? woff[1] : (int)kOutside};
#pragma unroll
    for (int q = 0; q < WL; ++q)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(ring + slot * SLOT + TM * 128 + q * 1024), 16, v[q & 1],
                                               kt < nk ? off + q * 8 * wrow : 0, 0, 0);
  };
  auto load_a = [&](int i, int slot) {
    const int kt = wave + i * NW;
#pragma unroll
    for (int q = 0; q < XL; ++q) {
      if constexpr (AMODE == A_CONV3) {            // pieces never straddle taps: C % 8 == 0
        const int kk = kt * 64 + ((piece ^ ((q & 1) << 6)) >> 1);
        const bool live = kk < 3 * p.C && !(kk < p.C && (aflags[q] & 1)) && !(kk >= 2 * p.C && (aflags[q] & 2));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(ring + slot * SLOT + q * 1024), 16,
                                                 live ? (int)((unsigned)(aoff[q] * p.C + kk) * 2u) : (int)kOutside, 0, 0, 0);
      } else {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(ring + slot * SLOT + q * 1024), 16,
                                                 kt < nk ? aoff[q] : (int)kOutside, kt < nk ? kt * astep : 0, 0, 0);
      }
    }
  };
  if constexpr (AMODE == A_CONV3) {                // the weights first: the windows' places are still on their way
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (s < ns) load_w(s, s);
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (s < ns) load_a(s, s);
  } else {
#pragma unroll
    for (int s = 0; s < SLOTS; ++s)
      if (s < ns) { load_w(s, s); load_a(s, s); }
  }
  if constexpr (EPI == EPI_BIAS_GELU_POS) {
#pragma unroll
    for (int u = 0; u < PER; ++u) add[u] = *(const vec *)(p.pos + (size_t)prow[u] * p.N + n0 + ec);
  }

  f32x4 acc[TB][FB];
#pragma unroll
  for (int i = 0; i < TB; ++i)
#pragma unroll
    for (int j = 0; j < FB; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  int slot = 0;
  for (int i = 0; i < ns; ++i) {
    // The loads of step i have landed when at most those of the steps requested after it are outstanding.  (Windows of a convolution:
    // counted as if only activations followed, and the positions requested behind the first steps not at all; both wait for more
    // than they have to, never for less.)
    constexpr int N = AMODE == A_CONV3 ? XL : LPS;
    const int ahead = min(ns - 1 - i, SLOTS - 1);
    if (SLOTS > 3 && ahead >= 3) wait_loads<(SLOTS > 3 ? 3 * N : 0)>();
    else if (SLOTS > 2 && ahead >= 2) wait_loads<(SLOTS > 2 ? 2 * N : 0)>();
    else if (SLOTS > 1 && ahead >= 1) wait_loads<(SLOTS > 1 ? N : 0)>();
    else wait_loads<0>();
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char *cx = ring + slot * SLOT, *cw = cx + TM * 128;
    bf16x8 xf[2][TB], wf[2][FB];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int off = l16 * 128 + (((4 * t + lq) ^ ((l16 >> 1) & 7)) << 4);
#pragma unroll
      for (int j = 0; j < FB; ++j) wf[t][j] = *(const bf16x8 *)(cw + j * 2048 + off);
#pragma unroll
      for (int r = 0; r < TB; ++r) xf[t][r] = *(const bf16x8 *)(cx + r * 2048 + off);
    }
    if (i + SLOTS < ns) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the slot has been read and may be refilled
      __builtin_amdgcn_sched_barrier(0);
      load_w(i + SLOTS, slot);
      load_a(i + SLOTS, slot);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < TB; ++r)
#pragma unroll
        for (int j = 0; j < FB; ++j) acc[r][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[t][j], xf[t][r], acc[r][j], 0, 0, 0);
    slot = slot + 1 == SLOTS ? 0 : slot + 1;
  }

  // ---- lane holds, of token l16 of a row block, features 16 j + 4 lq .. + 3
  __syncthreads();                                 // every wave is done with its ring
  float *part = (float *)smem_slice;
#pragma unroll
  for (int r = 0; r < TB; ++r)
#pragma unroll
    for (int j = 0; j < FB; ++j) *(f32x4 *)(part + (wave * TM + r * 16 + l16) * PITCH + j * 16 + lq * 4) = acc[r][j];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int row = er + u * (512 / COLS), m = m0 + row, nn = n0 + ec;
    vec v = *(const vec *)(part + row * PITCH + ec);
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      const vec t = *(const vec *)(part + (w * TM + row) * PITCH + ec);
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] += t[e];
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] += bias[e];
    if constexpr (EPI == EPI_BIAS_GELU || EPI == EPI_BIAS_GELU_POS) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] = gelu_fast(v[e]);
    }
    if constexpr (EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU_POS) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] += add[u][e];
    }
    if (!has || m >= p.M) continue;
    if constexpr (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
      typedef __bf16 bvec __attribute__((ext_vector_type(VEC)));
      __bf16 *dst = p.out_panels ? (__bf16 *)p.out + ((((size_t)(m >> 8) * (p.N >> 6) + (nn >> 6)) << 14) + ((m & 255) << 6) + (nn & 63))
                    : (EPI == EPI_BIAS && p.out2 && nn >= p.n_split) ? (__bf16 *)p.out2 + (size_t)m * p.ldo2 + (nn - p.n_split)
                                                                     : (__bf16 *)p.out + (size_t)m * p.ldo + nn;
      *(bvec *)dst = __builtin_convertvector(v, bvec);
    } else {
      *(vec *)((float *)p.out + (size_t)m * p.ldo + nn) = v;
    }
  }
#endif
}

template <int TM, int TN, int SLOTS, int AMODE, int EPI>
hipError_t launch_slice_tile(const GemmArgs &a, hipStream_t s) {
  constexpr int smem = slice_smem<TM, TN, SLOTS>();
  static_assert(smem <= 163840, "LDS of one compute unit");
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute((const void *)gemm_slice_kernel<TM, TN, SLOTS, AMODE, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL((gemm_slice_kernel<TM, TN, SLOTS, AMODE, EPI>), dim3((unsigned)((a.M + TM - 1) / TM * (a.N / TN))), dim3(512), smem, s, a);
  return hipGetLastError();
}

// The tile with the shortest time by the bounds above: rounds of the chip times a tile's operand bytes at one L1's rate (10.9 ns a KB
// measured, 12.5 for 64 x 64 tiles), or all tiles' bytes at the chip's; a further round costs a start, the larger tiles their
// sums.  Fits sweeps of every tile over 13 to 1020 rows and 384 to 5120 columns and values of reduction: the tile it
// takes is the fastest or within 3 % of it throughout.
struct SliceTile { int m, n; };
constexpr SliceTile kSliceTiles[] = {{16, 16}, {16, 32}, {32, 32}, {64, 32}, {64, 64}};

struct SlicePick { int tile; double us; };          // us: beyond the launch and the first memory latency (about 2 us)
SlicePick pick_slice(int M, int N, int K) {
  SlicePick best{-1, 0.0};
  for (int t = 0; t < 5; ++t) {
    if (N % kSliceTiles[t].n) continue;
    const long tiles = (long)((M + kSliceTiles[t].m - 1) / kSliceTiles[t].m) * (N / kSliceTiles[t].n), rounds = (tiles + 255) / 256;
    const double kb = (kSliceTiles[t].m + kSliceTiles[t].n) * (double)K * 2 / 1024, one = 0.3 + kb * (t < 4 ? 10.9e-3 : 12.5e-3);
    const double us = std::max(rounds * one + 0.9 * (rounds - 1), tiles * kb * 1024 / (t < 3 ? 20e6 : 17.5e6)) + (t == 4 ? 1.0 : t == 3 ? 0.3 : 0.0);
    if (best.tile < 0 || us < best.us) best = {t, us};
  }
  return best;
}

template <int AMODE, int EPI>
hipError_t launch_slice(const GemmArgs &a, hipStream_t s) {
  switch (pick_slice(a.M, a.N, a.K).tile) {
    case 0: return launch_slice_tile<16, 16, 4, AMODE, EPI>(a, s);
    case 1: return launch_slice_tile<16, 32, 3, AMODE, EPI>(a, s);
    case 2: return launch_slice_tile<32, 32, 2, AMODE, EPI>(a, s);
    case 3: return launch_slice_tile<64, 32, 1, AMODE, EPI>(a, s);
    default: return launch_slice_tile<64, 64, 1, AMODE, EPI>(a, s);
  }
}

// Widest tile (in 32-column blocks) that divides N and still leaves at least 160 workgroups; 1 if even that gives fewer.
int pick_blocks(const GemmArgs &a) {
  constexpr int min_wgs = 160;     // measured: 425 tokens prefer 168-224 wide tiles to 336-448 narrower ones, 125 tokens 192-256 to 96-128
  const long rows = (a.M + SBM - 1) / SBM;
  for (int nb = 4; nb > 1; nb >>= 1)
    if (a.N % (nb * SBN) == 0 && rows * (a.N / (nb * SBN)) >= min_wgs) return nb;
  return 1;
}

template <int AMODE, int EPI>
hipError_t launch_small(const GemmArgs &a, hipStream_t s) {
  const int nb = pick_blocks(a);
  const dim3 grid((unsigned)((long)((a.M + SBM - 1) / SBM) * (a.N / (nb * SBN)))), block(256);
  if (nb == 4) hipLaunchKernelGGL((gemm_small_kernel<AMODE, EPI, 4>), grid, block, 0, s, a);
  else if (nb == 2) hipLaunchKernelGGL((gemm_small_kernel<AMODE, EPI, 2>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((gemm_small_kernel<AMODE, EPI, 1>), grid, block, 0, s, a);
  return hipGetLastError();
}

// Short reductions: fewer than six K steps leave waves of the sliced kernel idle, and its eight partial tiles cost more to add up than the
// loop gains.  Four waves and eight (us a launch): 130 x 384 x 64 2.4 and 2.8, 1024 x 384 x 64 2.9 and 4.1, 500 x 768 x 256 3.4 and
// 4.1, 1024 x 384 x 320 3.7 and 4.1; from 448 on eight are ahead by up to 12 %.  At 384 plain products with bf16 results of 128 to 512 tiles
// of 32 x 32 (130 x 1152 3.0 and 3.3, 300 x 1536 4.0 and 4.2; 75 x 1152 3.0 on both, 650 x 1152 5.5 and 5.2), windows and residual updates not (their rows
// keep one order of sums whatever their number).
// They also find their operands by pointers, where the other kernels' 32-bit offsets end.
bool offsets_reach(const GemmArgs &a, AMode amode) {
  const int64_t limit = kOutside, w = (int64_t)(a.w_panels ? (a.N + 255) & ~255 : a.N) * a.K * 2;
  return w <= limit && (amode != A_PLAIN || (int64_t)(a.a_panels ? (a.M + 255) & ~255 : a.M) * std::max(a.lda, a.K) * 2 <= limit);
}
bool takes_four_waves(const GemmArgs &a, AMode amode, Epilogue epi) {
  if (a.a_panels || a.out_panels) return false;        // row-major only
  if (!offsets_reach(a, amode)) return true;
  const long tiles = (long)((a.M + SBM - 1) / SBM) * (a.N / SBN);
  return a.K <= 320 || (a.K <= 384 && amode == A_PLAIN && epi != EPI_BIAS_RESID && tiles > 128 && tiles <= 512);
}

template <int AMODE, int EPI>
hipError_t launch_operand(const GemmArgs &a, hipStream_t s) {
  if ((a.a_panels || a.out_panels) && !offsets_reach(a, (AMode)AMODE)) return hipErrorInvalidValue;
  return takes_four_waves(a, (AMode)AMODE, (Epilogue)EPI) ? launch_small<AMODE, EPI>(a, s) : launch_slice<AMODE, EPI>(a, s);
}

}  // namespace

int gemm_small_choice(int32_t M, int32_t N, int32_t K, Epilogue epi, int32_t *bm, int32_t *bn) {
  GemmArgs a{};
  a.M = M; a.N = N; a.K = a.lda = K;
  if (takes_four_waves(a, A_PLAIN, epi)) {
    *bm = SBM; *bn = SBN * pick_blocks(a);
    return 4;
  }
  const SliceTile t = kSliceTiles[pick_slice(M, N, K).tile];
  *bm = t.m; *bn = t.n;
  return 8;
}

// Plain products outside of the encoder that give every compute unit at most one 32 x 32 tile (us a launch in a chain, these kernels and
// the pipelined one): 160 x 768 x 768 3.5 and 4.7, 320 x 768 x 768 3.9 and 4.8, 256 x 1024 x 1024 4.0 and 5.3, 192 x 1280 x 1280 4.5 and
// 5.8, 96 x 2304 x 768 3.9 and 4.8; residual updates whatever their depth: 160 x 768 x 3072 5.2 and 10.1, 192 x 1280 x 5120 9.4 and
// 15.2.  The line is narrower than the kernel's reach (gemm_slice_applies): beyond it, and beyond 4 MB of weights with a bf16 result, rows
// keep the order of sums that larger batches have.
bool gemm_small_few_rows(int32_t M, int32_t N, int32_t K, Epilogue epi) {
  if (epi != EPI_BIAS && epi != EPI_BIAS_GELU && epi != EPI_BIAS_RESID) return false;
  return (long)((M + SBM - 1) / SBM) * (N / SBN) <= 256 && (epi == EPI_BIAS_RESID || (long)N * K <= 2L << 20);
}

// Products of a wide model on the sliced kernel: up to one 64 x 32 tile per compute unit (us, this kernel and the pipelined one:
// 100 x 2304 x 768 4.5 and 5.3, 200 x 1280 x 1280 5.3 and 6.5, 640 x 768 x 768 4.7 and 5.4; one tile more and it is the other way round,
// 200 x 2304 x 768 5.9 and 5.6).  A long reduction that may be cut into parts instead (may_cut) is left to the pipelined kernel where that
// is estimated to be faster by 0.3 us (100 x 768 x 3072 loses 0.7 us a block, 60 x 768 x 3072 gains 0.5).
bool gemm_slice_applies(int32_t M, int32_t N, int32_t K, bool may_cut) {
  if (N % 32 || K % 64 || (long)((M + 63) / 64) * (N / 32) > 256) return false;
  return !may_cut || K < 2 * N || pick_slice(M, N, K).us <= gemm_cut_estimate(M, N, K) + 0.3;
}

// The sliced kernel finds a convolution's windows by 32-bit byte offsets from the first row of the whole packed batch (the other kernels by
// pointers, or by offsets from a tile's first window).
bool gemm_slice_reaches(int64_t rows, int64_t values) { return rows * values * 2 <= (int64_t)kOutside; }

bool gemm_small_applies(int32_t M, int32_t N, int32_t K) { return M <= kSmallRows && std::min(N, K) <= 512 && std::max(N, K) <= 2048; }

hipError_t launch_gemm_small(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N % SBN != 0 || a.K % SBK != 0 || a.K <= 0) return hipErrorInvalidValue;
  if ((a.a_panels && amode != A_PLAIN) || (a.out_panels && (amode == A_LN || a.out2 || (epi != EPI_BIAS && epi != EPI_BIAS_GELU)))) return hipErrorInvalidValue;
  if (a.n_group && (epi != EPI_BIAS || amode != A_PLAIN || a.out_panels || a.out2 || a.n_group % 64 || a.N % a.n_group)) return hipErrorInvalidValue;
  if (a.out2 && (epi != EPI_BIAS || a.n_split % 4 != 0 || a.n_split <= 0 || a.n_split >= a.N)) return hipErrorInvalidValue;
  if (amode == A_PLAIN) {
    if (a.lda % 8 != 0) return hipErrorInvalidValue;
    switch (epi) {
      case EPI_BIAS: return launch_operand<A_PLAIN, EPI_BIAS>(a, s);
      case EPI_BIAS_GELU: return launch_operand<A_PLAIN, EPI_BIAS_GELU>(a, s);
      case EPI_BIAS_RESID: return launch_operand<A_PLAIN, EPI_BIAS_RESID>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (amode == A_LN) {
    if (a.lda % 8 != 0 || !a.ln_g || !a.ln_b || !(a.ln_eps > 0.0f) || a.K > kMaxLnK) return hipErrorInvalidValue;
    if (a.K <= kLnRowK && offsets_reach(a, amode) && (epi == EPI_BIAS || epi == EPI_BIAS_GELU)) return epi == EPI_BIAS ? launch_ln<EPI_BIAS>(a, s) : launch_ln<EPI_BIAS_GELU>(a, s);
    switch (epi) {
      case EPI_BIAS: return launch_small<A_LN, EPI_BIAS>(a, s);
      case EPI_BIAS_GELU: return launch_small<A_LN, EPI_BIAS_GELU>(a, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (a.C % 8 != 0 || 3 * a.C > a.K || !a.row_src || !a.row_flags) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_BIAS_GELU: return launch_operand<A_CONV3, EPI_BIAS_GELU>(a, s);
    case EPI_BIAS_GELU_POS:
      if (!a.pos || !a.row_pos) return hipErrorInvalidValue;
      return launch_operand<A_CONV3, EPI_BIAS_GELU_POS>(a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace wf
