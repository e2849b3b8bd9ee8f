// Bidirectional multi-head attention over a ragged batch (head size 64) for gfx950, bf16 MFMA with
// fp32 accumulation and an online (running max / running sum) softmax in fp32.
//
// Tokens of all streams are packed back to back; cu_seqlens gives each stream's row range, and a
// query only ever sees the keys of its own stream.  One workgroup (4 waves) handles one work item
// = (stream, head, 128 consecutive queries); each wave owns 32 queries.  Keys/values are walked in
// tiles of 64, double-buffered in LDS.
//
// Both products are computed transposed: S^T = K Q^T and O^T = V^T P^T.  With
// v_mfma_f32_32x32x16_bf16 a lane then owns ONE query (column lane%32) in the S^T and O^T
// accumulators, so the row max, the rescale factor and the row sum are per-lane scalars, and the
// S^T accumulator registers are, as they stand, the second operand of the P.V MFMA: lane group
// g = lane/32 holds keys {8a + 4g + b}, and the V^T fragment is read with the same key order.
#include <algorithm>
#include <mutex>

#include "device_utils.h"
#include "kernels.h"

namespace wf {

namespace {

constexpr int BQ = 128;    // queries per work item
constexpr int BKV = 64;    // keys per tile
// Where the keys are shared out, a wave's first tile need not be the stream's first, and its logits may be -inf or so far
// below the others that the rounding of reference x scale alone, 2^-25 of it, overflows the exponential.  The reference
// (in powers of two) therefore stops at -2^31, where that rounding is still a factor of 2^64: such a tile weighs 0, not NaN.
constexpr float kMinReference = -0x1p31f;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void glb_void;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// K and V tiles are both kept row-major in LDS, [key][64 features] = 128-byte rows, 16-byte chunk c of
// row r stored at chunk position c ^ swizzle(r) (K: (r >> 1) & 7; V: v_swizzle(r), see there), and are
// filled straight from global memory by
// global_load_lds_dwordx4 (lane l of a wave lands at LDS base + 16 l, so a wave fills 8 rows per
// instruction and applies the swizzle by choosing which chunk it fetches).
//
// The V^T fragment of the P.V product is read with ds_read_b64_tr_b16, which transposes a 16 x 4 block
// of 16-bit elements across a group of 16 lanes: lane r of the group supplies the address of 4
// consecutive elements, and lane i receives element i % 4 of the segments addressed by lanes
// i/4, i/4 + 4, i/4 + 8, i/4 + 12.  Pointing lane r = a + 4e at (key K0 + e, features F0 + 4a ..) gives lane i
// the four keys K0..K0+3 of feature F0 + i: four consecutive reduction indices of one V^T row.
//
// CAUSAL (self-attention among the prompt tokens of a decoder): query r sees keys 0..r.  Tiles that lie
// wholly in the future of a work item are never loaded, a wave skips the tiles that lie wholly in the
// future of its 32 queries (tile starts and wave starts are multiples of 32, so every tile a wave does
// process holds at least one visible key for each of its queries).
// Chunk swizzle of a V row.  A transposing read touches 4 consecutive keys x 64 bytes (4 chunks), so rows r and
// r + 2 -- same half of the 256-byte bank line -- must land in different groups of 4 chunks: the low bit of
// (r >> 1) goes to bit 2 of the XOR mask.  (K rows keep (r >> 1) & 7, which suits 16-row b128 reads.)
__device__ __forceinline__ int v_swizzle(int r) {
  const int q = (r >> 1) & 7;
  return ((q & 1) << 2) | (q >> 1);
}

// KS: number of four-wave groups that share the keys of a work item (group g walks the tiles g, g + KS, ...; the partial
// results meet in LDS at the end).  launch_attention_bf16 says when it is 2.
template <bool CAUSAL, int KS>
__global__ void __launch_bounds__(256 * KS) attention_bf16_kernel(AttnArgs p) {
  // per key group: K[2][8 KB], V[2][8 KB].  One group alone fits the static limit, and its tile addresses are then constants.
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_groups[];
  __shared__ __attribute__((aligned(1024))) unsigned char smem_one[KS == 1 ? 32768 : 16];
  unsigned char *const smem_att = KS == 1 ? smem_one : smem_groups;

  // The grid has the head count rounded up to a multiple of 8.  Consecutive workgroups go to the 8 XCDs in
  // turn, so slot s of every work item lands on XCD s % 8; slot s holds head (s - rot) mod heads8, with rot
  // fixed per stream: every query block of one (stream, head) then finds its K and V in the same L2.  rot
  // advances by n_heads % 8 from one stream to the next in the (cost-sorted) work list, so the XCDs that get
  // one head more than the others change from stream to stream.  Slots without a head leave at once.
  const int heads8 = (p.n_heads + 7) & ~7;
  if (blockIdx.x >= (unsigned)(p.n_work * heads8)) {
    prefetch_block(p.pf, blockIdx.x - p.n_work * heads8, smem_att);
    return;
  }
  const int item = blockIdx.x / heads8;
  const int w1 = p.work[2 * item + 1];
  const int rot = (((w1 >> 20) & 7) * (p.n_heads & 7)) & 7;
  const int head = (blockIdx.x % heads8 + heads8 - rot) % heads8;
  if (head >= p.n_heads) return;
  const int stream = p.work[2 * item];
  const int q0 = w1 & 0xFFFFF;
  const int tok0 = p.cu_q[stream];
  const int Lq = p.cu_q[stream + 1] - tok0;
  const int ktok0 = p.cu_kv[stream];
  const int L = p.cu_kv[stream + 1] - ktok0;     // keys of this stream

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int gwave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wave = gwave & 3, kg = KS > 1 ? gwave >> 2 : 0;    // wave inside its key group, key group
  unsigned char *const sK = smem_att + kg * 32768, *const sV = sK + 16384;
  const int l32 = lane & 31, lg = lane >> 5;
  const int ldq = p.ldq, ld = p.ldkv;
  const __bf16 *Qb = (const __bf16 *)p.q + (size_t)tok0 * ldq + head * 64;
  const __bf16 *Kb = (const __bf16 *)p.k + (size_t)ktok0 * ld + head * 64;
  const __bf16 *Vb = (const __bf16 *)p.v + (size_t)ktok0 * ld + head * 64;

  const int qw0 = q0 + wave * 32;              // first query of this wave
  const bool wave_active = qw0 < Lq;           // waves past the end still help with the loads
  int qrow = qw0 + l32;
  const bool q_valid = qrow < Lq;
  qrow = q_valid ? qrow : Lq - 1;

  // Q fragments for the whole loop: features 16*ks + 8*lg + (0..7) of this lane's query.
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const bf16x8 *)(Qb + (size_t)qrow * ldq + ks * 16 + lg * 8);

  f32x16 o[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  float m_run = -INFINITY;     // running max of the raw logits of this lane's query
  float l_run = 0.0f;          // this lane's share of the running sum (the lane^32 partner has the rest)
  const float c = p.scale * 1.4426950408889634f;   // exp(s*scale) = exp2(s*c)
  const float lazy = 8.0f / c;

  // Tile loads: 16 instructions of 8 rows per tile (8 for K, 8 for V), 4 per wave.
  const int lrow = lane >> 3;
  auto issue = [&](int kt, int buf) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int g = i * 4 + wave;                       // 0..7: K row group, 8..15: V row group
      const int rt = (g & 7) * 8 + lrow;                // row inside the tile
      int key = kt * BKV + rt;
      key = key < L ? key : L - 1;                      // clamped rows are masked out of the softmax below
      const int lch = (lane & 7) ^ (g < 8 ? (rt >> 1) & 7 : v_swizzle(rt));
      const __bf16 *src = (g < 8 ? Kb : Vb) + (size_t)key * ld + lch * 8;
      unsigned char *dst = (g < 8 ? sK : sV) + buf * 8192 + (g & 7) * 1024;
      __builtin_amdgcn_global_load_lds((const glb_void *)src, (lds_void *)dst, 16, 0, 0);
    }
  };

  // V^T fragment addressing (see above): inside its 16-lane group lane r = a + 4e addresses key e, features 4a..4a+3
  const int r16 = lane & 15;
  const int tr_key = r16 >> 2;                           // e
  const int tr_feat = ((lane >> 4) & 1) * 16 + (r16 & 3) * 4;   // feature offset inside a 32-feature block

  const int k_end = CAUSAL ? min(L, q0 + BQ) : L;          // keys this work item can see at all
  const int n_tiles = (k_end + BKV - 1) / BKV;
  if (KS == 1 || kg < n_tiles) issue(kg, 0);
  for (int it = 0; it * KS < n_tiles; ++it) {   // every group makes the same number of turns (they share the barriers)
    const int kt = it * KS + kg;
    const int key0 = kt * BKV;
    __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): my share of tile kt has landed
    __builtin_amdgcn_s_barrier();               // everyone's has; the other buffer is no longer being read
    if (kt + KS < n_tiles) issue(kt + KS, (it + 1) & 1);
    if (!wave_active) continue;
    if (KS > 1 && kt >= n_tiles) continue;
    if (CAUSAL && key0 > qw0 + 31) continue;
    const unsigned char *cK = sK + (it & 1) * 8192, *cV = sV + (it & 1) * 8192;

    // ---- S^T = K Q^T : two 32-key blocks, reduction over the 64 features in 4 steps
    f32x16 s[2];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb2][r] = 0.0f;
      const int row = kb2 * 32 + l32;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 kf = *(const bf16x8 *)(cK + row * 128 + (((2 * ks + lg) ^ ((row >> 1) & 7)) << 4));
        s[kb2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[kb2], 0, 0, 0);
      }
    }
    // lane holds logits of query l32 against keys key0 + 32*kb2 + 8*(r/4) + 4*lg + r%4
    if (key0 + BKV > L) {
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key0 + kb2 * 32 + 8 * (r >> 2) + 4 * lg + (r & 3);
          if (key >= L) s[kb2][r] = -INFINITY;
        }
    }
    if (CAUSAL && key0 + BKV - 1 > qw0) {
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key0 + kb2 * 32 + 8 * (r >> 2) + 4 * lg + (r & 3);
          if (key > qrow) s[kb2][r] = -INFINITY;
        }
    }
    float tmax = s[0][0];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kb2][r]);
    tmax = half_max(tmax);
    const float m_new = fmaxf(m_run, tmax);       // finite: every tile has at least one valid key
    // The softmax reference m_run only has to bound the logits from below by a known margin: it follows the running
    // maximum when some query's maximum has moved up by more than 8 / c (weights up to 2^8 until then; fp32 sums and
    // bf16 weights have the range), which spares most rescales of the accumulators.
    if (__any(m_new > m_run + lazy)) {
      // (a later group's first tile may hold nothing but -inf logits for some queries of the wave: nothing to rescale yet)
      const float alpha = KS > 1 && m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
      m_run = m_new;
    }
    const float mc = KS > 1 ? fmaxf(m_run * c, kMinReference) : m_run * c;
    float psum = 0.0f;
    bf16x8 pf[2][2];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 e0, e1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          e0[e] = __builtin_amdgcn_exp2f(s[kb2][8 * h + e] * c - mc);
          e1[e] = __builtin_amdgcn_exp2f(s[kb2][8 * h + 4 + e] * c - mc);
          psum += e0[e] + e1[e];
        }
        const bf16x4 b0 = to_bf16x4(e0), b1 = to_bf16x4(e1);
        pf[kb2][h] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    l_run += psum;

    // ---- O^T += V^T P^T.  Reduction step (kb2, h) covers the 16 keys the lane pair holds in
    // pf[kb2][h]: group lg has keys 32*kb2 + 16*h + 4*lg + (0..3) and the same + 8.
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int fchunk = (t * 32 + tr_feat) >> 3;           // 16-byte chunk of the features this lane addresses
      const int fin = ((t * 32 + tr_feat) & 7) * 2;         // byte offset inside the chunk
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k0 = kb2 * 32 + 16 * h + 4 * lg + tr_key;   // key row this lane addresses (first half)
          const int k1 = k0 + 8;
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4 *)(cV + k0 * 128 + ((fchunk ^ v_swizzle(k0)) << 4) + fin));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_s16x4 *)(cV + k1 * 128 + ((fchunk ^ v_swizzle(k1)) << 4) + fin));
          const bf16x4 w0 = __builtin_bit_cast(bf16x4, v0), w1 = __builtin_bit_cast(bf16x4, v1);
          const bf16x8 vf = __builtin_shufflevector(w0, w1, 0, 1, 2, 3, 4, 5, 6, 7);
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kb2][h], o[t], 0, 0, 0);
        }
    }
  }

  if (KS == 1 && !wave_active) return;
  const float l_tot = half_sum(l_run);
  __bf16 *orow = (__bf16 *)p.out + (size_t)(tok0 + qrow) * p.d_model + head * 64;
  if constexpr (KS == 1) {
    const float inv = 1.0f / l_tot;
    if (q_valid) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = o[t][g * 4 + e] * inv;
          *(bf16x4 *)(orow + t * 32 + g * 8 + lg * 4) = to_bf16x4(v);
        }
    }
  } else {
    // Merge: the partial outputs (8 four-feature pieces a lane) are laid over the tile buffers, reference and sum behind
    // them; group g then rescales and adds the pieces 8 g / KS .. in group order (deterministic) and stores them.
    f32x4 *sO = (f32x4 *)smem_att;                             // [group][wave][piece][lane]
    float *sML = (float *)(smem_att + KS * 32768);             // [group][wave][2][lane]
    __syncthreads();                                           // every wave is done with the tiles
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 v = {o[t][g * 4], o[t][g * 4 + 1], o[t][g * 4 + 2], o[t][g * 4 + 3]};
        sO[(gwave * 8 + t * 4 + g) * 64 + lane] = v;
      }
    sML[gwave * 128 + lane] = m_run;
    sML[gwave * 128 + 64 + lane] = l_tot;
    __syncthreads();
    if (!q_valid) return;
    float M = -INFINITY, sc[KS], l_all = 0.0f;
#pragma unroll
    for (int k = 0; k < KS; ++k) M = fmaxf(M, sML[(k * 4 + wave) * 128 + lane]);
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const float mk = sML[(k * 4 + wave) * 128 + lane];
      sc[k] = mk == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((mk - M) * c);   // 0: a group without a visible key
      l_all += sML[(k * 4 + wave) * 128 + 64 + lane] * sc[k];
    }
    const float inv = 1.0f / l_all;
#pragma unroll
    for (int i = 0; i < 8 / KS; ++i) {
      const int piece = kg * (8 / KS) + i;                     // features 32 (piece / 4) + 8 (piece % 4) + 4 lg
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        const f32x4 w = sO[((k * 4 + wave) * 8 + piece) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] += w[e] * sc[k];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] *= inv;
      *(bf16x4 *)(orow + (piece >> 2) * 32 + (piece & 3) * 8 + lg * 4) = to_bf16x4(v);
    }
  }
}

template <bool CAUSAL, int KS>
hipError_t launch_keys(const AttnArgs &a, hipStream_t s) {
  constexpr int smem = KS > 1 ? KS * (32768 + 2048) : 0;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute((const void *)attention_bf16_kernel<CAUSAL, KS>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL((attention_bf16_kernel<CAUSAL, KS>), dim3(a.n_work * ((a.n_heads + 7) & ~7) + (a.pf.bytes ? a.pf.blocks : 0)), dim3(256 * KS), smem, s, a);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------
// Variant for batches too small to fill the chip with 128-query work items (one stream's buffer: a few hundred
// tokens).  There the kernel's duration is the length of one workgroup's chain of key tiles, so the chain is cut
// four ways: a workgroup takes 32 queries of one (stream, head) and its four waves walk the key tiles w, w + 4,
// w + 8, ... each with its own running maximum, sum and output accumulators, reading tiles it loads itself into
// LDS buffers of its own (no workgroup barrier inside the loop): NB = 2 of them where a workgroup has a compute unit to
// itself, 1 where a second workgroup on the CU covers the loads (20 heads x 350 tokens 11.2 -> 8.8 us, 6 x 1200 19.4 ->
// 15.4, where two buffers would take two rounds; see attention_form).  At the end the four partial results are rescaled
// to the common maximum and added in wave order through LDS (deterministic).  Same arithmetic per tile as
// attention_bf16_kernel; the grouping of the tiles differs, so results agree to fp32 rounding of the sums, not bit
// for bit.
template <int NB>
__global__ void __launch_bounds__(256) attention_bf16_keysplit_kernel(AttnArgs p) {
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem_ks[];   // per wave: K [NB][8 KB], V [NB][8 KB]

  const int heads8 = (p.n_heads + 7) & ~7;
  if (blockIdx.x >= (unsigned)(4 * p.n_work * heads8)) {
    prefetch_block(p.pf, blockIdx.x - 4 * p.n_work * heads8, smem_ks);
    return;
  }
  // All first quarters of the items' 128 queries, then all second ones, ..: prompts shorter than a quarter leave three of
  // four workgroups without queries, and interleaved with the others those would keep three quarters of the CUs empty (the
  // dispatcher deals consecutive workgroups out round robin).
  const int unit = blockIdx.x / heads8;
  const int item = unit % p.n_work, sub = unit / p.n_work;
  const int w1 = p.work[2 * item + 1];
  const int rot = (((w1 >> 20) & 7) * (p.n_heads & 7)) & 7;
  const int head = (blockIdx.x % heads8 + heads8 - rot) % heads8;
  if (head >= p.n_heads) return;
  const int stream = p.work[2 * item];
  const int q0 = (w1 & 0xFFFFF) + 32 * sub;
  const int tok0 = p.cu_q[stream];
  const int Lq = p.cu_q[stream + 1] - tok0;
  if (q0 >= Lq) return;
  const int ktok0 = p.cu_kv[stream];
  const int L = p.cu_kv[stream + 1] - ktok0;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lg = lane >> 5;
  const int ldq = p.ldq, ld = p.ldkv;
  const __bf16 *Qb = (const __bf16 *)p.q + (size_t)tok0 * ldq + head * 64;
  const __bf16 *Kb = (const __bf16 *)p.k + (size_t)ktok0 * ld + head * 64;
  const __bf16 *Vb = (const __bf16 *)p.v + (size_t)ktok0 * ld + head * 64;
  unsigned char *myK = smem_ks + wave * NB * 16384, *myV = myK + NB * 8192;

  int qrow = q0 + l32;
  const bool q_valid = qrow < Lq;
  qrow = q_valid ? qrow : Lq - 1;
  bf16x8 qf[4];
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) qf[ks] = *(const bf16x8 *)(Qb + (size_t)qrow * ldq + ks * 16 + lg * 8);

  f32x16 o[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[t][r] = 0.0f;
  float m_run = -INFINITY, l_run = 0.0f;
  const float c = p.scale * 1.4426950408889634f;

  // one wave loads a whole tile: 8 instructions of 8 rows for K, 8 for V
  const int lrow = lane >> 3;
  auto issue = [&](int kt, int buf) {
#pragma unroll
    for (int g = 0; g < 8; ++g) {
      const int rt = g * 8 + lrow;
      int key = kt * BKV + rt;
      key = key < L ? key : L - 1;
      const __bf16 *srck = Kb + (size_t)key * ld + ((lane & 7) ^ ((rt >> 1) & 7)) * 8;
      const __bf16 *srcv = Vb + (size_t)key * ld + ((lane & 7) ^ v_swizzle(rt)) * 8;
      __builtin_amdgcn_global_load_lds((const glb_void *)srck, (lds_void *)(myK + buf * 8192 + g * 1024), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const glb_void *)srcv, (lds_void *)(myV + buf * 8192 + g * 1024), 16, 0, 0);
    }
  };
  const int r16 = lane & 15;
  const int tr_key = r16 >> 2;
  const int tr_feat = ((lane >> 4) & 1) * 16 + (r16 & 3) * 4;

  const int n_tiles = (L + BKV - 1) / BKV;
  int buf = 0;
  if (wave < n_tiles) issue(wave, 0);
  for (int kt = wave; kt < n_tiles; kt += 4, buf ^= NB - 1) {
    const int key0 = kt * BKV;
    __builtin_amdgcn_s_waitcnt(0x0F70);         // vmcnt(0): this wave's tile kt has landed (nobody else touches these buffers)
    if (NB == 2 && kt + 4 < n_tiles) issue(kt + 4, buf ^ 1);
    const unsigned char *cK = myK + buf * 8192, *cV = myV + buf * 8192;
    f32x16 s[2];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb2][r] = 0.0f;
      const int row = kb2 * 32 + l32;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        const bf16x8 kf = *(const bf16x8 *)(cK + row * 128 + (((2 * ks + lg) ^ ((row >> 1) & 7)) << 4));
        s[kb2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], s[kb2], 0, 0, 0);
      }
    }
    if (key0 + BKV > L) {
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int key = key0 + kb2 * 32 + 8 * (r >> 2) + 4 * lg + (r & 3);
          if (key >= L) s[kb2][r] = -INFINITY;
        }
    }
    float tmax = s[0][0];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kb2][r]);
    tmax = half_max(tmax);
    const float m_new = fmaxf(m_run, tmax);
    if (__any(m_new > m_run)) {
      // a query without a finite logit so far has nothing to rescale, and its m_run - m_new may be inf - inf
      const float alpha = m_run == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[t][r] *= alpha;
      m_run = m_new;
    }
    const float mc = fmaxf(m_run * c, kMinReference);
    float psum = 0.0f;
    bf16x8 pf[2][2];
#pragma unroll
    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 e0, e1;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          e0[e] = __builtin_amdgcn_exp2f(s[kb2][8 * h + e] * c - mc);
          e1[e] = __builtin_amdgcn_exp2f(s[kb2][8 * h + 4 + e] * c - mc);
          psum += e0[e] + e1[e];
        }
        const bf16x4 b0 = to_bf16x4(e0), b1 = to_bf16x4(e1);
        pf[kb2][h] = __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    l_run += psum;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int fchunk = (t * 32 + tr_feat) >> 3;
      const int fin = ((t * 32 + tr_feat) & 7) * 2;
#pragma unroll
      for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int k0 = kb2 * 32 + 16 * h + 4 * lg + tr_key;
          const int k1 = k0 + 8;
          const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(cV + k0 * 128 + ((fchunk ^ v_swizzle(k0)) << 4) + fin));
          const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(cV + k1 * 128 + ((fchunk ^ v_swizzle(k1)) << 4) + fin));
          const bf16x4 w0 = __builtin_bit_cast(bf16x4, v0), w1b = __builtin_bit_cast(bf16x4, v1);
          const bf16x8 vf = __builtin_shufflevector(w0, w1b, 0, 1, 2, 3, 4, 5, 6, 7);
          o[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[kb2][h], o[t], 0, 0, 0);
        }
    }
    if (NB == 1 && kt + 4 < n_tiles) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0): the tile has been read, its buffer may be refilled
      __builtin_amdgcn_sched_barrier(0);
      issue(kt + 4, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  // ---- merge the four waves' partial results, laid over the tile buffers (every wave is past its last tile read once it reaches
  // the barrier): each wave leaves its outputs, references and sums, and a thread that adds four outputs up scales them itself.
  // A row of 68 words puts the 16 queries that a store instruction serves at a time on different banks (with 64 words the merge of 75
  // tokens took 1.2 of the kernel's 4.0 us).
  constexpr int PITCH = 68;
  __syncthreads();
  float *sO = (float *)smem_ks;                   // [wave][query][64 features]
  float *sM = sO + 4 * 32 * PITCH, *sL = sM + 128;     // [wave][query]
  const float l_tot = half_sum(l_run);
  if (lg == 0) {
    sM[wave * 32 + l32] = m_run;
    sL[wave * 32 + l32] = l_tot;
  }
  // lane holds, of query l32, features t*32 + 8*g + 4*lg + e  (o[t][4*g + e])
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *(f32x4 *)(sO + (wave * 32 + l32) * PITCH + t * 32 + g * 8 + lg * 4) = f32x4{o[t][g * 4], o[t][g * 4 + 1], o[t][g * 4 + 2], o[t][g * 4 + 3]};
  __syncthreads();
  // thread -> query tid / 8, features (tid % 8) * 8 .. + 7
  const int qq = tid >> 3, f0 = (tid & 7) * 8;
  if (q0 + qq < Lq) {
#pragma clang fp contract(off)                    // parts are rounded when scaled, as if each wave had scaled its own: no bit depends on who does
    float M = sM[qq], lsum = 0.0f;
#pragma unroll
    for (int w = 1; w < 4; ++w) M = fmaxf(M, sM[w * 32 + qq]);
    f32x4 a0, a1;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float sc = __builtin_amdgcn_exp2f((sM[w * 32 + qq] - M) * c);     // 0 for a wave that saw no tile (its reference is -inf)
      const f32x4 b0 = *(const f32x4 *)(sO + (w * 32 + qq) * PITCH + f0), b1 = *(const f32x4 *)(sO + (w * 32 + qq) * PITCH + f0 + 4);
      lsum += sL[w * 32 + qq] * sc;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        a0[e] = w == 0 ? b0[e] * sc : a0[e] + b0[e] * sc;
        a1[e] = w == 0 ? b1[e] * sc : a1[e] + b1[e] * sc;
      }
    }
    const float inv = 1.0f / lsum;
#pragma unroll
    for (int e = 0; e < 4; ++e) { a0[e] *= inv; a1[e] *= inv; }
    const bf16x4 c0 = to_bf16x4(a0), c1 = to_bf16x4(a1);
    __bf16 *orow = (__bf16 *)p.out + (size_t)(tok0 + q0 + qq) * p.d_model + head * 64 + f0;
    *(bf16x8 *)orow = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
}

template <int NB>
hipError_t launch_keysplit(const AttnArgs &a, hipStream_t s) {
  constexpr int smem = 4 * NB * 16384;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] {
    attr_err = hipFuncSetAttribute((const void *)attention_bf16_keysplit_kernel<NB>, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
  });
  if (attr_err != hipSuccess) return attr_err;
  hipLaunchKernelGGL(attention_bf16_keysplit_kernel<NB>, dim3(4 * a.n_work * ((a.n_heads + 7) & ~7) + (a.pf.bytes ? a.pf.blocks : 0)), dim3(256), smem, s, a);
  return hipGetLastError();
}

}  // namespace

int attention_q_tile() { return BQ; }

// Calls that leave the chip short of waves last as long as one workgroup's walk over the key tiles (1.05 us a tile), so the
// keys are shared out.  Let x be the busy 32-query workgroups of the XCD that gets most of them (32 CUs each):
//   * at most one per CU, however short the keys: 32-query workgroups, keys cut four ways, with two tile buffers a wave (128 KB
//     of LDS) while x <= 32, else one (64 KB), so that two fit a CU and none waits for a second round.  With heads that do not
//     fill the 8 XCDs evenly and last quarters without queries the dispatcher deals two to some CUs from x = 25 on.  (Two
//     buffers against one: 16 heads x 8 prompts of 20 x 1500 keys, x = 26, 17.4 and 27.2 us; 20 x 350, x = 36, 12.1 and 9.9.)
//   * up to two per CU, and at least three tiles (192 keys) to share: one buffer, a second workgroup covers the loads: 1.00 ..
//     1.16 times as fast as unshared at 192 .. 400 keys and x = 32 .. 48, 1.15 .. 1.5 times beyond; x up to 64 only where the
//     XCDs are filled evenly (20 heads x 6 prompts x 1500 keys, x = 60: 30.4 us against 25.4 with two key groups).
//   * else 128-query items with two key groups while there is at most one per CU (20 x 900 19.9 -> 16.4 us, 12 x 1500 28.8 ->
//     22.4; with more the one-group form is as fast, from 16 heads x 8 x 325 on 10 % faster, and so it is with XCDs that are
//     filled unevenly and nearly full while a stream has few tiles: 20 x 3 x 425 14.9 us against 16.4).
// The whole batch's counts decide, never those of one lane: a batch cut into lanes gives the same bits.
AttnForm attention_form(int32_t n_heads, int32_t B, int64_t M, int64_t Mkv, int64_t n_work) {
  constexpr long cus = 256, per_xcd = cus / 8;
  const long heads8 = (n_heads + 7) & ~7, units = std::min<long>(4L * n_work, M / 32 + B);
  // heads of B equal streams on the fullest XCD (the kernels' slot s of a stream of rank r holds head s - rot(r))
  long most = 0;
  for (int x = 0; x < 8; ++x) {
    long n = 0;
    for (int r = 0; r < std::min(B, 8); ++r) {
      const long rot = (r * (n_heads & 7)) & 7;
      for (long slot = x; slot < heads8; slot += 8)
        if ((slot + heads8 - rot) % heads8 < n_heads) n += (B - r + 7) / 8;
    }
    most = std::max(most, n);
  }
  const long busy = most * units;                        // x = busy / B
  const bool even = n_heads % 8 == 0;
  if (units * n_heads <= cus) return busy <= (even || units == 4L * n_work ? per_xcd : per_xcd * 3 / 4) * B ? ATTN_KEYS4_TWO_BUFFERS : ATTN_KEYS4;
  if (Mkv < 192L * B || (M / BQ + B) * n_heads > cus) return ATTN_PLAIN;
  if (!even && Mkv < 512L * B && most * (M / BQ + B) > 30L * B) return ATTN_PLAIN;
  return busy <= (even || B == 1 ? 2 * per_xcd : per_xcd * 3 / 2) * B ? ATTN_KEYS4 : ATTN_KEYS2;
}

hipError_t launch_attention_bf16(const AttnArgs &a, hipStream_t s) {
  if (a.n_work <= 0) return hipSuccess;
  if (a.d_model != a.n_heads * 64) return hipErrorInvalidValue;
  if (a.pf.bytes && (!a.pf.p || a.pf.bytes % 16 || a.pf.bytes >= 1u << 31)) return hipErrorInvalidValue;
  if (a.ldq % 8 != 0 || a.ldkv % 8 != 0 || !a.q || !a.k || !a.v || !a.cu_q || !a.cu_kv) return hipErrorInvalidValue;
  if (a.causal) {
    if (a.cu_q != a.cu_kv) return hipErrorInvalidValue;
    return launch_keys<true, 1>(a, s);
  }
  switch (attention_form(a.n_heads, a.B, a.M, a.Mkv > 0 ? a.Mkv : a.M, a.n_work_batch > 0 ? a.n_work_batch : a.n_work)) {
    case ATTN_KEYS4_TWO_BUFFERS: return launch_keysplit<2>(a, s);
    case ATTN_KEYS4: return launch_keysplit<1>(a, s);
    case ATTN_KEYS2: return launch_keys<false, 2>(a, s);
    default: return launch_keys<false, 1>(a, s);
  }
}

}  // namespace wf
