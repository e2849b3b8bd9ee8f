// bf16 MFMA GEMM for products that give the chip at most one output tile per compute unit (a single stream of a few
// hundred tokens up to several thousand rows with few columns):  out = epilogue(A . W^T), fp32 accumulation.
//
// One workgroup of four waves (one per SIMD, so a wave may use up to 512 registers) computes a BM x BN tile, each wave a
// (BM / 2) x (BN / 2) quarter with v_mfma_f32_16x16x32_bf16.  K advances 64 at a time through a ring of LDS stages that
// takes all of the LDS (2 to 8 stages), fragments are double-buffered in registers.  The arithmetic is that of the
// large-batch kernels of gemm_bf16.hip (accumulators start from the bias, K in order, the same instruction), so a row's
// bits do not depend on which of these kernels or tiles computes it, as long as its reduction is not cut (EPI_PARTIAL, a choice
// that goes by the rows of the whole batch: a stream alone and beside others may then differ in the last bits of fp32 sums).
//
// What bounds it and why it is built this way (all figures from one card, weights not in the L2):
//   * With one wave per SIMD nothing but the wave's own instruction order keeps the matrix pipe fed.  A global -> LDS load
//     holds the wave up until the memory pipeline takes it, so the loads are spread between the matrix instructions
//     (128 x 128 tile: 474 ns a K step with the loads in a burst after the barrier, 350 spread, 291 without any loads).
//   * The loop has no branches: steps past the end load from outside the buffer (zeros, no memory traffic), so the count
//     of loads in flight is a constant and every wait leaves the newest stages in flight.
//   * A K step takes about 70 ns + 8.75 ns per KB of operand tile (the L1's line rate); two or four K steps per barrier,
//     whole-step or half-step fragment buffers, row-major or panel operands and a fifth wave prefetching into the L2
//     measure the same or worse.
// Against the 128 x 128 kernel with two workgroups per CU it replaced (us, same shapes): 3156 x 768 x 3072 31.8 -> 22,
// 2600 x 1024 x 4096 41 -> 28.5, 6400 x 1280 x 5120 86 -> 74; against the small-batch kernel at 425 rows: 1280 x 5120
// 28.9 -> 20.5, 3840 x 1280 16.9 -> 10.2.
#include <algorithm>
#include <cmath>
#include <mutex>

#include "gemm_epilogue.h"

namespace wf {

namespace {

typedef __attribute__((address_space(3))) void lds_void;

[[maybe_unused]] constexpr unsigned kOutside = 0xFFFFFFF0u;   // a byte offset no buffer reaches: the load returns zeros

constexpr int pipe_smem(int bm, int bn, int xs, int ws) {
  const int stages = (xs * bm + ws * bn) * 128, slices = 4 * (bm / 2) * 256;
  return stages > slices ? stages : slices;
}

// Wait until at most V of this wave's loads are outstanding.
template <int V>
__device__ __forceinline__ void wait_loads() {
  static_assert(V >= 0 && V < 64, "more loads in flight than the counter holds");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (V & 15) | ((V >> 4) << 14));
}

// Order of a stretch of NMM matrix instructions, NRD fragment reads and NLD loads: the reads among the first instructions
// (at most half of them), the loads spread evenly over the rest (SOON: four instructions apart, for loads that are waited
// for at the end of the stretch).
template <int NMM, int NRD, int NLD, bool SOON = false, int Q = 0>
__device__ __forceinline__ void schedule() {
  constexpr int RP = (2 * NRD + NMM - 1) / NMM, RS = (NRD + RP - 1) / RP;     // reads per slot, slots with reads
  if constexpr (Q < NMM) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    if constexpr (Q < RS) {
      __builtin_amdgcn_sched_group_barrier(0x100, Q + 1 < RS ? RP : NRD - RP * (RS - 1), 0);
    } else {
      constexpr int span = SOON && RS + 4 * NLD < NMM ? 4 * NLD : NMM - RS, q = Q - RS < span ? Q - RS : span, q1 = q < span ? q + 1 : span;
      constexpr int a = q * NLD / span, b = q1 * NLD / span;
      if constexpr (b > a) __builtin_amdgcn_sched_group_barrier(0x020, b - a, 0);
    }
    schedule<NMM, NRD, NLD, SOON, Q + 1>();
  } else {
    __builtin_amdgcn_sched_barrier(0);
  }
}

// XS / WS: LDS stages of the activations / weights (XS = WS or WS + 1).  FULL: the fragments of a whole 64-deep K step are
// double-buffered in registers (small tiles, whose half step has too few matrix instructions to cover an LDS read), else
// those of 32-deep half steps.
template <int BM, int BN, int XS, int WS, bool FULL, int EPI, int AMODE>
__global__ void __launch_bounds__(256, 1) gemm_pipe_kernel(GemmArgs p) {
#ifdef __HIP_DEVICE_COMPILE__       // buffer resources are a device type: the host only needs the kernel's name
  constexpr int TM = BM / 2, TN = BN / 2, TB = TM / 16, FB = TN / 16;
  constexpr int XL = BM / 32, WL = BN / 32, LPS = XL + WL;   // load instructions (8 rows of 128 bytes) per wave and K step
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  unsigned char *sX = smem, *sW = smem + XS * BM * 128;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int l16 = lane & 15, lq = lane >> 4, rr = lane >> 3;

  const int tiles_m = (p.M + BM - 1) / BM, tiles_n = p.N / BN;
  const int splits = EPI == EPI_PARTIAL ? p.k_splits : 1;
  const int n_tiles = tiles_m * tiles_n, n_units = n_tiles * splits, per_xcd = (n_units + 7) >> 3;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= n_units || (int)(blockIdx.x >> 3) >= per_xcd) return;
  const int split = EPI == EPI_PARTIAL ? (unit >= n_tiles) + (unit >= 2 * n_tiles) + (unit >= 3 * n_tiles) : 0;    // (at most four)
  const int tile = unit - split * n_tiles;         // a split's tiles share operands
  const int G = min(p.group_n, tiles_n), gs = tiles_m * G;
  const int grp = order_div(tile, gs, p.div_group), rem = tile - grp * gs, gw = min(G, tiles_n - grp * G);
  const int trow = order_div(rem, gw, gw == G ? p.div_row : p.div_last);
  const int m0 = trow * BM, n0 = (grp * G + rem - trow * gw) * BN;

  // ---- loads: instruction i of this wave fetches rows (4 i + wave) * 8 .. + 7 of the tile
  const int nkt = p.K >> 6;                        // K steps of the whole reduction, and [k0, k0 + nk) of this part
  const int k0 = EPI == EPI_PARTIAL ? order_div(nkt * split, splits, p.div_split) : 0;
  const int nk = EPI == EPI_PARTIAL ? order_div(nkt * (split + 1), splits, p.div_split) - k0 : nkt;
  const size_t a_bytes = p.a_panels ? (size_t)((p.M + 255) >> 8) * 256 * p.K * 2 : ((size_t)(p.M - 1) * p.lda + p.K) * 2;
  // The gathered operand may exceed what 32 bits reach (row_src counts rows of the whole packed batch), so its buffer starts at
  // the tile's first window and the offsets are differences (windows come in ascending order, a tile's within a few rows).
  int src0 = 0;
  if constexpr (AMODE == A_CONV3) src0 = __builtin_amdgcn_readfirstlane(p.row_src[m0]);
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
      (char *)p.A + (AMODE == A_CONV3 ? (long)src0 * p.C * 2 : 0L), 0, AMODE == A_CONV3 ? (int)kOutside : (int)a_bytes, 0x00027000);
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      (void *)p.W, 0, (int)((size_t)(p.w_panels ? (p.N + 255) & ~255 : p.N) * p.K * 2), 0x00027000);
  // (The bounds check takes scalar and vector offset together, both unsigned and without wrapping: measured on this part with
  // addresses on both sides of the end, below and above 2 GiB.  It cuts off the rows past the last one of the operand's last group of eight.)
  const int piece = ((lane & 7) ^ ((4 * wave + (rr >> 1)) & 7)) << 4;       // (row >> 1) & 7 of every row this lane fetches
  const int woff = rr * (p.w_panels ? 128 : p.K * 2) + piece;
  const int wstep = p.w_panels ? 32768 : 128, astep = p.a_panels ? 32768 : 128;    // bytes from one K step to the next
  int wbase[WL], abase[AMODE == A_CONV3 ? 1 : XL];                                  // uniform
  const RowPlace wplace(p.w_panels, nkt, p.K), aplace(p.a_panels, nkt, p.lda);
  int aoff[AMODE == A_CONV3 ? XL : 1];
  [[maybe_unused]] int aflags[AMODE == A_CONV3 ? XL : 1];
#pragma unroll
  for (int i = 0; i < WL; ++i) {
    wbase[i] = wplace(n0 + wave * 8) + i * 32 * wplace.row + k0 * wstep;      // (a tile's columns lie in one panel)
  }
  if constexpr (AMODE == A_CONV3) {
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int row = min(m0 + (i * 4 + wave) * 8 + rr, p.M - 1);
      aoff[i] = (p.row_src[row] - src0) * p.C * 2 + piece;
      aflags[i] = p.row_flags[row];
    }
  } else {
    aoff[0] = rr * (p.a_panels ? 128 : p.lda * 2) + piece;
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int r0 = min(m0 + (i * 4 + wave) * 8, (p.M - 1) & ~7);        // a group past the last row repeats the last one
      abase[i] = aplace(r0) + k0 * astep;
    }
  }
  // Loads [first, last) of a refill: the weights of K step kw into ring slot sw_, then the activations of K step kx into
  // slot sx_.  Steps past the end are out of the buffers' range (no memory is read, zeros go to a slot nobody needs), so
  // that the loop below has no branches and a constant number of loads in flight.
  auto load = [&](int first, int last, int kw, int sw_, int kx, int sx_) {
    const int kwc = min(kw, nk - 1), kxc = min(kx, nk - 1);
    unsigned char *dx = sX + sx_ * BM * 128 + wave * 1024, *dw = sW + sw_ * BN * 128 + wave * 1024;
    const int vw = kw >= nk ? (int)kOutside : woff;
    [[maybe_unused]] const int vx = kx >= nk ? (int)kOutside : aoff[0];
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      if (i < first || i >= last) continue;
      if (i < WL) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (lds_void *)(dw + i * 4096), 16, vw, wbase[i] + kwc * wstep, 0, 0);
      } else {
        const int q = i - WL;
        if constexpr (AMODE == A_CONV3) {              // pieces never straddle taps: C % 8 == 0
          const int kk = kx * 64 + (piece >> 1);
          const bool live = kk < 3 * p.C && !(kk < p.C && (aflags[q] & 1)) && !(kk >= 2 * p.C && (aflags[q] & 2));
          __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(dx + q * 4096), 16, live ? aoff[q] + kx * 128 : (int)kOutside, 0, 0, 0);
        } else {
          __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void *)(dx + q * 4096), 16, vx, abase[q] + kxc * astep, 0, 0);
        }
      }
    }
  };
  // Of a refill's loads, those issued in its first half step (FULL: all of them).
  constexpr int L1 = FULL ? LPS : (WS == 2 ? (2 * LPS + 2) / 3 : (LPS + 1) / 2);
  static_assert(XS == WS || XS == WS + 1, "the activations may run one step further ahead");
  if constexpr (XS > WS) load(WL, LPS, 0, 0, 0, 0);
#pragma unroll
  for (int s = 0; s < WS; ++s) load(0, s == WS - 1 ? L1 : LPS, s, s, s + XS - WS, s + XS - WS);

  f32x4 acc[TB][FB];
#pragma unroll
  for (int j = 0; j < FB; ++j) {
    f32x4 b = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (EPI != EPI_PARTIAL) b = *(const f32x4 *)(p.bias + n0 + wn * TN + j * 16 + lq * 4);
#pragma unroll
    for (int i = 0; i < TB; ++i) acc[i][j] = b;
  }

  const int xrow = (wm * TM + l16) * 128, wrow = (wn * TN + l16) * 128;
  const int sw = (l16 >> 1) & 7;
  constexpr int NB = FULL ? 2 : 1;                  // 32-deep halves per fragment batch
  bf16x8 xf[2][NB][TB], wf[2][NB][FB];
  auto rd = [&](int sx_, int sw_, int t, bf16x8 (&x)[TB], bf16x8 (&w)[FB]) {
    const int off = ((4 * t + lq) ^ sw) << 4;
    const unsigned char *cx = sX + sx_ * BM * 128 + xrow + off, *cw = sW + sw_ * BN * 128 + wrow + off;
#pragma unroll
    for (int j = 0; j < FB; ++j) w[j] = *(const bf16x8 *)(cw + j * 16 * 128);
#pragma unroll
    for (int i = 0; i < TB; ++i) x[i] = *(const bf16x8 *)(cx + i * 16 * 128);
  };
  auto mm = [&](const bf16x8 (&x)[TB], const bf16x8 (&w)[FB]) {
#pragma unroll
    for (int i = 0; i < TB; ++i)
#pragma unroll
      for (int j = 0; j < FB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[j], x[i], acc[i][j], 0, 0, 0);
  };
  // Step kt: its fragments (FULL) or those of its first half are in registers or on their way.  The barrier is reached
  // when every wave has read the whole stage of step kt (its slots may be refilled) and has seen its own
  // loads of step kt + 1 land, whose first fragments are then read under the matrix instructions.
  wait_loads<(WS - 2) * LPS + L1>();
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < NB; ++t) rd(0, 0, t, xf[0][t], wf[0][t]);
  int sx = 0, sw2 = 0;                             // ring slots of step kt
  auto step = [&](int kt, int cur) {
    const int nx = sx + 1 == XS ? 0 : sx + 1, px = sx == 0 ? XS - 1 : sx - 1;
    const int nw = sw2 + 1 == WS ? 0 : sw2 + 1, pw = sw2 == 0 ? WS - 1 : sw2 - 1;
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!FULL) {
      __builtin_amdgcn_s_waitcnt(0xC07F);
      __builtin_amdgcn_sched_barrier(0);
      rd(sx, sw2, 1, xf[1][0], wf[1][0]);
      load(L1, LPS, kt + WS - 1, pw, kt + XS - 1, px);   // the rest of the previous step's refill
      mm(xf[0][0], wf[0][0]);
      schedule<TB * FB, TB + FB, LPS - L1, XS == 2>();
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): the stage of step kt has been read
    wait_loads<(WS - 2) * LPS + (XS - WS) * XL>();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    // (after the last step this reads a stage nobody needs)
    if constexpr (FULL) {
#pragma unroll
      for (int t = 0; t < NB; ++t) rd(nx, nw, t, xf[cur ^ 1][t], wf[cur ^ 1][t]);
      load(0, L1, kt + WS, sw2, kt + XS, sx);
#pragma unroll
      for (int t = 0; t < NB; ++t) mm(xf[cur][t], wf[cur][t]);
      schedule<NB * TB * FB, NB * (TB + FB), L1>();
    } else {
      rd(nx, nw, 0, xf[0][0], wf[0][0]);
      load(0, L1, kt + WS, sw2, kt + XS, sx);
      mm(xf[1][0], wf[1][0]);
      schedule<TB * FB, TB + FB, L1>();
    }
    sx = nx;
    sw2 = nw;
  };
  if constexpr (FULL) {
    int kt = 0;
    for (; kt + 1 < nk; kt += 2) {
      step(kt, 0);
      step(kt + 1, 1);
    }
    if (kt < nk) step(kt, 0);
  } else {
    for (int kt = 0; kt < nk; ++kt) step(kt, 0);
  }

  __builtin_amdgcn_s_waitcnt(0x0070);              // vmcnt(0) lgkmcnt(0)
  __builtin_amdgcn_s_barrier();                    // every wave is done with the stages
  if constexpr (EPI == EPI_PARTIAL) p.out = (float *)p.out + (size_t)split * p.M * p.N;
  if constexpr (EPI == EPI_BIAS) p.out = group_out(p, n0);
  store_subtile<TM, TN, EPI == EPI_PARTIAL ? (int)EPI_BIAS_F32 : EPI, false>(p, smem + wave * (TM * 256), acc, m0 + wm * TM, n0 + wn * TN, lane);
#endif
}

template <int BM, int BN, int XS, int WS, bool FULL, int EPI, int AMODE>
hipError_t launch_tile(GemmArgs a, hipStream_t s) {
  constexpr int smem = pipe_smem(BM, BN, XS, WS);
  static_assert(smem <= 163840, "LDS of one compute unit");
  auto kern = gemm_pipe_kernel<BM, BN, XS, WS, FULL, EPI, AMODE>;
  static std::once_flag once;
  static hipError_t attr_err = hipSuccess;
  std::call_once(once, [&] { attr_err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, smem); });
  if (attr_err != hipSuccess) return attr_err;
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = a.N / BN, tiles = tiles_m * tiles_n * (EPI == EPI_PARTIAL ? a.k_splits : 1);
  // Tile columns per group: the 32 tiles an XCD works on at a time should form a block of about 5 x 6 tiles, which needs
  // the fewest operand panels in its L2; few rows of tiles need no grouping.
  a.group_n = tiles_m <= 6 ? 1 : tiles_n <= 6 ? tiles_n : tiles_n % 5 == 0 ? 5 : 4;
  const int G = std::min(a.group_n, tiles_n);
  a.div_group = order_mul(tiles_m * G); a.div_row = order_mul(G); a.div_last = order_mul(tiles_n % G ? tiles_n % G : G); a.div_split = order_mul(a.k_splits);
  hipLaunchKernelGGL(kern, dim3(8 * ((tiles + 7) / 8)), dim3(256), smem, s, a);
  return hipGetLastError();
}

struct Tile { int bm, bn; };
constexpr Tile kTiles[] = {{32, 64}, {64, 64}, {96, 64}, {128, 64}, {96, 128}, {128, 128}, {192, 128}, {128, 256}, {160, 256}, {192, 256}};
constexpr int kTileCount = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr int kTile128 = 5;          // index of 128 x 128

template <int EPI, int AMODE>
hipError_t launch_index(int t, const GemmArgs &a, hipStream_t s) {
  switch (t) {
    case 0: return launch_tile<32, 64, 8, 8, true, EPI, AMODE>(a, s);
    case 1: return launch_tile<64, 64, 8, 8, true, EPI, AMODE>(a, s);
    case 2: return launch_tile<96, 64, 8, 8, true, EPI, AMODE>(a, s);
    case 3: return launch_tile<128, 64, 6, 6, true, EPI, AMODE>(a, s);
    case 4: return launch_tile<96, 128, 5, 5, true, EPI, AMODE>(a, s);
    case 5: return launch_tile<128, 128, 4, 4, false, EPI, AMODE>(a, s);
    default: break;
  }
  if constexpr (EPI == EPI_PARTIAL) return hipErrorInvalidValue;
  else switch (t) {
    case 6: return launch_tile<192, 128, 4, 3, false, EPI, AMODE>(a, s);
    case 7: return launch_tile<128, 256, 3, 3, false, EPI, AMODE>(a, s);
    case 8: return launch_tile<160, 256, 3, 3, false, EPI, AMODE>(a, s);
    default: return launch_tile<192, 256, 3, 2, false, EPI, AMODE>(a, s);
  }
}

// The smallest tile that leaves at most one per compute unit, if that beats the kernels with two smaller workgroups per
// CU, whose epilogues overlap other tiles' K loops: always up to 128 x 128 (1.04 to 1.9 times, 64 .. 5400 rows), with larger
// tiles when the reduction is at least twice as long as the result is wide, so that the K loop dominates (1.03 to 1.47; short
// reductions lose up to 15 %: 6361 x 1280 x 1280 28.6 -> 32.8 us, 2600 x 3072 x 1024 20.5 -> 22.9) and there are at most
// 10 240 rows.  That limit is a compromise: a call that shares the chip with nothing gains beyond it too (an encoder call of
// 11 000 rows of 768 on one lane 4.08 -> 3.74 ms without it, a prefill of 20 000 rows of 512 2.19 -> 2.04), two lanes of 11 000
// rows each gain at 768 (6.62 -> 6.47 ms) and lose at 1024 (17.99 -> 18.10), where the compute units a kernel takes count as well
// as its time.  (Lanes of 4096 to 10 240 rows keep the larger tiles: 9000 x 1280 in two lanes 15.1 ms with, 16.0 without.)
// -1: none.
int pick_tile(int M, int N, int K) {
  for (int t = 0; t < kTileCount; ++t) {
    if (N % kTiles[t].bn) continue;
    const long tiles = (long)((M + kTiles[t].bm - 1) / kTiles[t].bm) * (N / kTiles[t].bn);
    if (tiles > 256) continue;
    if (t <= kTile128 || (K >= 2 * N && M <= 10240)) return t;
  }
  return -1;
}

// A residual product of a few hundred rows is one tile per compute unit at most, on half of them, and lasts as long as a
// tile's walk over K.  Its reduction is then cut into parts (at most one workgroup per CU in all) that the LayerNorm after
// it adds up; nothing is launched for that.  The estimate below (us) fits sweeps of every tile and 2 to 4 parts over 75 to
// 1025 rows of d = 768, 1024, 1280: the K step of the kernel's header, dearer in the two largest tiles, and 1.7 ns per
// thousand result values and part; an uncut product pays for the residual once as well.  It has to promise 0.7 us.
// 425 x 1280 x 5120: 23.4 -> 14.2 us (LayerNorm + 0.5), 425 x 1280 x 1280: 10.0 -> 8.8 us.
struct Split { int tile, parts; double us; };
Split pick_split(int M, int N, int K) {
  const int t1 = pick_tile(M, N, K), nk = K >> 6;
  if (t1 < 0 || t1 > kTile128 || N > 2048) return {t1, 1, INFINITY};      // (the LayerNorm takes rows of up to 2048 values)
  auto step = [](int t) { return (0.07 + 0.00875 * (kTiles[t].bm + kTiles[t].bn) / 8) * (t < 4 ? 1.0 : t == 4 ? 1.15 : 1.35); };
  const double part = 1.7e-6 * M * N;
  Split best{t1, 1, nk * step(t1) + part + 0.25};
  double cost = best.us - 0.7;
  for (int t = 0; t <= kTile128; ++t) {
    if (N % kTiles[t].bn) continue;
    const long tiles = (long)((M + kTiles[t].bm - 1) / kTiles[t].bm) * (N / kTiles[t].bn);
    for (int parts = 2; parts <= 4; ++parts) {
      if (tiles * parts > 256 || nk < 2 * parts || (int64_t)parts * M * N > kPartialFloats) continue;
      const double c = (nk + parts - 1) / parts * step(t) + parts * part;
      if (c < cost) { cost = c; best = {t, parts, c}; }
    }
  }
  return best;
}

}  // namespace

int gemm_split_choice(int32_t M, int32_t N, int32_t K) {
  return M > 0 && N % 64 == 0 && K % 64 == 0 ? pick_split(M, N, K).parts : 1;
}

double gemm_cut_estimate(int32_t M, int32_t N, int32_t K) {
  return M > 0 && N % 64 == 0 && K % 64 == 0 ? pick_split(M, N, K).us : INFINITY;
}

bool gemm_pipe_tile(int32_t M, int32_t N, int32_t K, int32_t *bm, int32_t *bn) {
  const int t = pick_tile(M, N, K);
  if (t < 0) return false;
  if (bm) *bm = kTiles[t].bm;
  if (bn) *bn = kTiles[t].bn;
  return true;
}
bool gemm_pipe_applies(int32_t M, int32_t N, int32_t K) { return gemm_pipe_tile(M, N, K, nullptr, nullptr); }

// The logits of a few rows: the product streams the embedding matrix, so a row tile no taller than the batch and a column tile
// that gives every compute unit one (64 x 51 866 x 1280: 43 -> 33 us, 1 x 51 865 x 512: 16.6 -> 13.7).
bool gemm_pipe_logits_applies(int32_t M, int32_t N) { return M <= 64 && N % 256 == 0 && N / 256 <= 256; }

hipError_t launch_gemm_pipe(const GemmArgs &a, AMode amode, Epilogue epi, hipStream_t s) {
  if (epi == EPI_BIAS_F32) {
    if (amode != A_PLAIN || !gemm_pipe_logits_applies(a.M, a.N) || a.K % 64 || a.K <= 0) return hipErrorInvalidValue;
    return launch_tile<64, 256, 4, 4, false, EPI_BIAS_F32, A_PLAIN>(a, s);
  }
  if (epi == EPI_PARTIAL) {
    const Split c = pick_split(a.M, a.N, a.K);
    if (amode != A_PLAIN || a.k_splits != c.parts || c.parts < 2) return hipErrorInvalidValue;
    return launch_index<EPI_PARTIAL, A_PLAIN>(c.tile, a, s);
  }
  int t = pick_tile(a.M, a.N, a.K);
  // A first convolution of many rows has four K steps or so: two stages per operand, so that two workgroups share a CU and one's
  // epilogue runs beside the other's loads (22 800 x 1024 x 256: 34 us a launch; the kernel that staged its operands in registers
  // took 49).
  if (t < 0 && amode == A_CONV3 && epi == EPI_BIAS_GELU && !a.a_panels && a.N % 128 == 0 && a.K % 64 == 0 && a.K > 0)
    return launch_tile<128, 128, 2, 2, false, EPI_BIAS_GELU, A_CONV3>(a, s);
  if (t < 0) t = amode == A_PLAIN ? kTileCount - 1 : kTile128;      // more than one tile per CU: products that ask for the tallest tile, and
                                     // convolutions whose taps are no whole K steps
  if (a.N % kTiles[t].bn || a.K % 64 || a.K <= 0) return hipErrorInvalidValue;
  if (amode == A_PLAIN) {
    switch (epi) {
      case EPI_BIAS: return launch_index<EPI_BIAS, A_PLAIN>(t, a, s);
      case EPI_BIAS_GELU: return launch_index<EPI_BIAS_GELU, A_PLAIN>(t, a, s);
      case EPI_BIAS_RESID: return launch_index<EPI_BIAS_RESID, A_PLAIN>(t, a, s);
      default: return hipErrorInvalidValue;
    }
  }
  if (amode != A_CONV3 || a.a_panels) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_BIAS_GELU: return launch_index<EPI_BIAS_GELU, A_CONV3>(t, a, s);
    case EPI_BIAS_GELU_POS: return launch_index<EPI_BIAS_GELU_POS, A_CONV3>(t, a, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace wf
