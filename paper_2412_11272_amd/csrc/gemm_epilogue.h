// Epilogue of the direct-load MFMA GEMMs, shared by the kernels of gemm_bf16.hip and gemm_pipe.hip.
#pragma once
#include "device_utils.h"
#include "kernels.h"

namespace wf {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// n / d by a multiplication with order_mul(d) = floor(2^32 / d) + 1, exact for n, d < 2^16: a tile finds its place before its first
// load, and a division there is a chain of 30 instructions (a tile 3 of them; with the branches per load instruction that the two
// operand layouts used to make, an encoder call of 425 rows of 1280 2211 -> 2184 us).
__host__ __device__ inline uint32_t order_mul(int d) { return d > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint32_t)d + 1) : 0; }
__host__ __device__ inline int order_div(int n, int d, uint32_t mul) {
  if (d == 1) return n;
  return (n | d) < 65536 ? (int)(((uint64_t)(uint32_t)n * mul) >> 32) : n / d;
}

// The result of the matrix that column n0 belongs to (GemmArgs::n_group), as a base for columns of the whole product.
__device__ __forceinline__ void *group_out(const GemmArgs &p, int n0) {
  if (p.n_group == 0) return p.out;
  const int g = n0 / p.n_group;
  return (__bf16 *)p.out + (size_t)g * (p.group_stride - p.n_group);
}

// Byte offset of a row of a bf16 operand, row-major or in panels of 256 rows, without a branch.
struct RowPlace {
  int shift, mask, panel, row;
  __device__ __forceinline__ RowPlace(bool panels, int nk, int ld)
      : shift(panels ? 8 : 31), mask(panels ? 255 : -1), panel(panels ? nk << 15 : 0), row(panels ? 128 : ld * 2) {}
  __device__ __forceinline__ int operator()(int r) const { return (int)((unsigned)(r >> shift) * (unsigned)panel + (unsigned)(r & mask) * (unsigned)row); }
};

// One wave stores its TM x TN sub-tile at (mw0, nw0).  The accumulators (v_mfma_f32_16x16x32_bf16 with the weight
// fragment as first operand) give a lane 4 consecutive features of ONE token, which would make every store instruction
// touch 16 different rows.  The wave therefore transposes its sub-tile through its own slice `stg` of the LDS (TM rows of
// 256 bytes) and writes whole row segments: 16-byte chunk c of row r sits at chunk position c ^ (r & (CPR-1)).
template <int TM, int TN, int EPI, bool NT>
__device__ __forceinline__ void store_subtile(const GemmArgs &p, unsigned char *stg, const f32x4 (&acc)[TM / 16][TN / 16], int mw0,
                                              int nw0, int lane) {
  [[maybe_unused]] constexpr int FB = TN / 16;
  constexpr int RC = TM <= 80 ? TM : TM / 2;       // rows per pass (bounds the registers of the fp32 addend)
  static_assert(RC % 16 == 0 && TM % RC == 0, "whole 16-row blocks per pass");
  const int l16 = lane & 15, lq = lane >> 4;
  if (EPI == EPI_BIAS || EPI == EPI_BIAS_GELU) {
    constexpr int RB = TN * 2;                     // row bytes (bf16)
    constexpr int CPR = RB / 16;                   // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;                  // rows per store instruction
    static_assert((CPR & (CPR - 1)) == 0 && RC % RPI == 0, "whole rows per store instruction");
    const int rr = lane / CPR, c = lane % CPR;
#pragma unroll
    for (int h = 0; h < TM / RC; ++h) {
#pragma unroll
      for (int i = 0; i < RC / 16; ++i) {
        const int r = i * 16 + l16;
#pragma unroll
        for (int j = 0; j < FB; ++j) {
          const int nl = j * 16 + lq * 4;          // feature inside the wave's sub-tile
          f32x4 v = acc[h * (RC / 16) + i][j];
          if (EPI == EPI_BIAS_GELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
          }
          const int u = nl >> 2;                   // 8-byte unit inside the row
          *(bf16x4 *)(stg + r * RB + ((((u >> 1) ^ (r & (CPR - 1))) << 4) | ((u & 1) << 3))) = to_bf16x4(v);
        }
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): the wave's own LDS writes have landed
#pragma unroll
      for (int it = 0; it < RC / RPI; ++it) {
        const int r = it * RPI + rr;
        const u32x4 v = *(const u32x4 *)(stg + r * RB + ((c ^ (r & (CPR - 1))) << 4));
        const int m = mw0 + h * RC + r;
        if (m < p.M) {
          const int n = nw0 + c * 8;
          __bf16 *dst = p.out_panels ? (__bf16 *)p.out + ((((size_t)(m >> 8) * (p.N >> 6) + (n >> 6)) << 14) + ((m & 255) << 6) + (n & 63))
                        : (p.out2 && n >= p.n_split) ? (__bf16 *)p.out2 + (size_t)m * p.ldo2 + (n - p.n_split)
                                                     : (__bf16 *)p.out + (size_t)m * p.ldo + n;
          // Large bf16 results (QKV, the MLP's hidden activations) are written with the non-temporal hint:
          // they are far bigger than what the caches can hand to the consumer, and written plainly they
          // push the residual stream and the operands of the next kernels out of the memory-side cache.
          if constexpr (NT) __builtin_nontemporal_store(v, (u32x4 *)dst);
          else *(u32x4 *)dst = v;
        }
      }
      if (h + 1 < TM / RC) __builtin_amdgcn_s_waitcnt(0xC07F);   // reads done before the next pass overwrites the slice
    }
  } else {
    // fp32 output: residual update in place (EPI_BIAS_RESID), GELU plus position row (EPI_BIAS_GELU_POS) or
    // plain store (EPI_BIAS_F32), PW features (PW * 4 bytes per row) and RC rows per pass
    constexpr int PW = TN >= 64 ? 64 : TN;         // features per pass
    constexpr int RB = PW * 4, CPR = RB / 16, RPI = 64 / CPR;
    static_assert(RC % RPI == 0, "whole rows per store instruction");
    const int rr = lane / CPR, c = lane % CPR;
    // The residual values a lane will update are requested well before they are needed, so that their
    // memory latency runs under the LDS transposition (and under the previous pass) instead of once per
    // row: half of a pass's rows before its staging writes, the other half right after them (when that
    // pass's accumulators are dead), and the first half of the NEXT pass before this pass's stores.
    constexpr int NIT = RC / RPI, NPC = TN / PW, NPS = NPC * (TM / RC);
    f32x4 res[2][NIT];
    auto fetch_res = [&](int ps, int it) {
      int m = mw0 + ps / NPC * RC + it * RPI + rr;
      m = m < p.M ? m : p.M - 1;
      const int n = nw0 + ps % NPC * PW + c * 4;
      if constexpr (EPI == EPI_BIAS_GELU_POS)      // the addend is the token's position row instead of the old output
        res[ps & 1][it] = *(const f32x4 *)(p.pos + (size_t)p.row_pos[m] * p.N + n);
      else
        res[ps & 1][it] = *(const f32x4 *)((const float *)p.out + (size_t)m * p.ldo + n);
    };
    constexpr bool ADDEND = EPI == EPI_BIAS_RESID || EPI == EPI_BIAS_GELU_POS;
    if (ADDEND) {
#pragma unroll
      for (int it = 0; it < NIT / 2; ++it) fetch_res(0, it);
    }
#pragma unroll
    for (int ps = 0; ps < NPS; ++ps) {
#pragma unroll
      for (int i = 0; i < RC / 16; ++i) {
        const int r = i * 16 + l16;
#pragma unroll
        for (int jj = 0; jj < PW / 16; ++jj) {
          const int j = ps % NPC * (PW / 16) + jj;
          const int nl = j * 16 + lq * 4;
          f32x4 v = acc[ps / NPC * (RC / 16) + i][j];
          if (EPI == EPI_BIAS_GELU_POS) {
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
          }
          const int ch = (nl % PW) >> 2;           // 16-byte chunk inside the pass
          *(f32x4 *)(stg + r * RB + ((ch ^ (r & (CPR - 1))) << 4)) = v;
        }
      }
      if (ADDEND) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int it = NIT / 2; it < NIT; ++it) fetch_res(ps, it);
        if (ps + 1 < NPS) {
#pragma unroll
          for (int it = 0; it < NIT / 2; ++it) fetch_res(ps + 1, it);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        const int r = it * RPI + rr;
        f32x4 v = *(const f32x4 *)(stg + r * RB + ((c ^ (r & (CPR - 1))) << 4));
        const int m = mw0 + ps / NPC * RC + r;
        if (ADDEND) {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += res[ps & 1][it][e];
        }
        const int n = nw0 + ps % NPC * PW + c * 4;
        if (EPI == EPI_BIAS_F32 && p.n_valid > 0) {      // rows of odd length: single words
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (m < p.M && n + e < p.n_valid) ((float *)p.out)[(size_t)m * p.ldo + n + e] = v[e];
        } else if (m < p.M) {
          *(f32x4 *)((float *)p.out + (size_t)m * p.ldo + n) = v;
        }
      }
      __builtin_amdgcn_s_waitcnt(0xC07F);          // reads done before the next pass overwrites the slice
    }
  }
}

}  // namespace wf
