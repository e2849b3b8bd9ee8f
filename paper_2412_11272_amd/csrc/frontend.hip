// Log-mel front end with the hush word appended at the raw-audio level (declared in
// include/wf_encoder.h, which also states the definition).  fp32 throughout: the spectrogram spans
// eight decades.
//
//   logmel_kernel   one workgroup per FPB consecutive frames of one stream.  The reflect-padded samples of
//                   x (+) h are staged in LDS once (consecutive frames share 240 of their 400 samples), the
//                   400-point DFT is a prime-factor transform 16 x 25 (coprime factors: no twiddles between the
//                   two): 25 real 16-point transforms per frame, then 8 complex 25-point ones (rows 1..7, and
//                   rows 0 and 8, which are real, packed into one), each in the registers of one thread.  Bins
//                   k and 400 - k are conjugate, so rows 0..8 hold all 201 bins and no untangling step is left.
//                   The power spectrum goes back to LDS, one thread per (frame, filter) adds up the bins under
//                   its triangle and stores (log10(max(., 1e-10)) + 4) / 4; the block's largest and smallest
//                   value are kept for the clamp.
//   clamp_kernel    the stream's maximum from its blocks' maxima (no atomics, nothing to reset), then the clamp
//                   to 8 decades below it, on the stored values (scaling and rounding are monotone); blocks whose
//                   smallest value needs no clamp leave without touching their rows.
//
// What bounds it: VALU issue, with too few waves to cover all waits.  20 k lane operations a frame (counted, idle lanes
// included); the VALU of a SIMD is busy 71 % of the kernel, the LDS 32 % (a quarter of that bank conflicts), and the ten waves a CU
// holds next to 30 KB of LDS a workgroup spend 45 % of their time at barriers and loads.  (The dense DFT on the fp32
// matrix cores that this replaced took 358 kflop a frame.)  55 625 frames of 128 filters: 333 -> 57 us per call (this kernel 47, the
// clamp 10; 77 while the table of 64 streams came by a copy); one stream of 437 frames: 65 -> 12 us (8.5 + 3 on the GPU,
// two launches, no upload).
#include "../../include/wf_encoder.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "device_utils.h"
#include "kernels.h"

namespace {

constexpr int kHop = 160, kNfft = 400, kBins = 201;
constexpr double kPi = 3.14159265358979323846;
constexpr int kMaxMels = 256;
constexpr int kMaxTaps = 2 * kBins + 2;        // every bin lies under at most two triangles
constexpr int kInline = 64;                    // streams whose metadata ride in the kernel arguments (one per lane in fe_find)
// Frames per workgroup.  16 frames on 128 threads keep both waves busy in every phase and leave room for five workgroups
// per CU (30 KB of LDS); 8 frames on 256 threads halve the chain of a workgroup where the chip is not full anyway.
constexpr int kFramesLarge = 16, kFramesSmall = 8;
constexpr float kLogFloor = -1.5f;             // (log10(1e-10) + 4) / 4
constexpr int kSmallBatch = 4096;              // frames from which on the large blocks give every CU one

int ffail(int code, const char *fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  const int rc = wf::set_error(code, fmt, ap);
  va_end(ap);
  return rc;
}

#define FE_HIP_TRY(expr)                                                                       \
  do {                                                                                         \
    hipError_t e_ = (expr);                                                                    \
    if (e_ != hipSuccess) return ffail(e_ == hipErrorOutOfMemory ? WF_E_OOM : WF_E_HIP,        \
                                       "%s: %s", #expr, hipGetErrorString(e_));                \
  } while (0)

// One stream of the batch; entry B closes the two prefix sums.
struct FeStream {
  int64_t offset;              // first sample in the caller's buffer
  int32_t n;                   // samples (hush word excluded)
  int32_t frame0;              // first packed row
  int32_t block0;              // first block
  int32_t pad;
};

struct FeArgs {
  const float *audio;          // caller's samples
  const float *hush;           // [H]
  const float *window;         // [25][16]: the taps that column n2 of the transform meets, in order
  const float *taps;           // filter weights, packed filter after filter
  const uint32_t *filters;     // [n_mels] first bin | bins << 8 | first tap << 16, then the n_empty filters without bins
  const FeStream *streams;     // [B + 1], or nullptr: the copy below
  const int32_t *block_stream; // [blocks], with `streams`
  float2 *range;               // [blocks] smallest and largest value of a block
  void *out;                   // [F][n_mels]
  int32_t B, H, n_mels, n_taps, n_empty, blocks;
  FeStream local[kInline + 1];
};
static_assert(sizeof(FeArgs) <= wf::kLaunchBytes, "arguments of a launch");

__device__ __forceinline__ FeStream fe_stream(const FeArgs &p, int i) { return p.streams ? p.streams[i] : p.local[i]; }

__device__ __forceinline__ int fe_find(const FeArgs &p, int block) {
  if (p.streams) return p.block_stream[block];
  if (p.B == 1) return 0;
  const int lane = threadIdx.x & 63;           // one stream per lane and one vote instead of a dependent search
  const bool after = lane < p.B && block >= p.local[lane < p.B ? lane : 0].block0;
  return __popcll(__ballot(after)) - 1;
}

// X[0..8] of 16 real values (W = exp(-2 pi i / 16)): re[1..7], im[1..7], and the real X[0] = re[0], X[8] = im[0].
__device__ __forceinline__ void dft16_real(const float (&x)[16], float (&re)[8], float (&im)[8]) {
  constexpr float s = 0.70710678118654752f, c1 = 0.92387953251128676f, c3 = 0.38268343236508977f;
  float a[8], b[8];
#pragma unroll
  for (int n = 0; n < 8; ++n) { a[n] = x[n] + x[n + 8]; b[n] = x[n] - x[n + 8]; }
  const float e0 = a[0] + a[4], e1 = a[1] + a[5], e2 = a[2] + a[6], e3 = a[3] + a[7];
  const float d0 = a[0] - a[4], d1 = a[1] - a[5], d2 = a[2] - a[6], d3 = a[3] - a[7];
  re[0] = (e0 + e2) + (e1 + e3);
  im[0] = (e0 + e2) - (e1 + e3);
  re[4] = e0 - e2;
  im[4] = e3 - e1;
  const float dm = s * (d1 - d3), dp = s * (d1 + d3);
  re[2] = d0 + dm; im[2] = -(d2 + dp);
  re[6] = d0 - dm; im[6] = d2 - dp;
  // odd bins: n and 8 - n share cosines (opposite sign) and sines
  const float p1 = b[1] - b[7], p2 = s * (b[2] - b[6]), p3 = b[3] - b[5];
  const float q1 = b[1] + b[7], q2 = s * (b[2] + b[6]), q3 = b[3] + b[5];
  const float u = b[0] + p2, v = b[0] - p2, w = b[4] + q2, z = q2 - b[4];
  const float r1 = c1 * p1 + c3 * p3, r3 = c3 * p1 - c1 * p3;
  const float t1 = c3 * q1 + c1 * q3, t3 = c1 * q1 - c3 * q3;
  re[1] = u + r1; im[1] = -(w + t1);
  re[7] = u - r1; im[7] = w - t1;              // sin of 7 pi n / 8: b4 and the even term change sign
  re[3] = v + r3; im[3] = -(z + t3);
  re[5] = v - r3; im[5] = z - t3;
}

// Five-point transform of (r, i)[0..4], in place.
__device__ __forceinline__ void dft5(float (&r)[5], float (&i)[5]) {
  constexpr float c1 = 0.30901699437494742f, c2 = -0.80901699437494742f, s1 = 0.95105651629515357f, s2 = 0.58778525229247313f;
  const float ar = r[1] + r[4], ai = i[1] + i[4], br = r[2] + r[3], bi = i[2] + i[3];
  const float dr = r[1] - r[4], di = i[1] - i[4], er = r[2] - r[3], ei = i[2] - i[3];
  const float m1r = r[0] + c1 * ar + c2 * br, m1i = i[0] + c1 * ai + c2 * bi;
  const float m2r = r[0] + c2 * ar + c1 * br, m2i = i[0] + c2 * ai + c1 * bi;
  const float n1r = s1 * dr + s2 * er, n1i = s1 * di + s2 * ei;
  const float n2r = s2 * dr - s1 * er, n2i = s2 * di - s1 * ei;
  r[0] += ar + br;
  i[0] += ai + bi;
  r[1] = m1r + n1i; i[1] = m1i - n1r;
  r[4] = m1r - n1i; i[4] = m1i + n1r;
  r[2] = m2r + n2i; i[2] = m2i - n2r;
  r[3] = m2r - n2i; i[3] = m2i + n2r;
}

struct Tw { float c, s; };
// exp(-2 pi i m / 25) for the products m = a b of the 5 x 5 split
__device__ constexpr Tw kTw25[17] = {
    {1.0f, 0.0f}, {0.96858316112863108f, -0.24868988716485479f}, {0.87630668004386360f, -0.48175367410171532f},
    {0.72896862742141155f, -0.68454710592868862f}, {0.53582679497899666f, -0.84432792550201508f}, {0.0f, 0.0f},
    {0.06279051952931337f, -0.99802672842827156f}, {0.0f, 0.0f}, {-0.42577929156507266f, -0.90482705246601958f},
    {-0.63742398974868970f, -0.77051324277578925f}, {0.0f, 0.0f}, {0.0f, 0.0f}, {-0.99211470131447788f, -0.12533323356430426f},
    {0.0f, 0.0f}, {0.0f, 0.0f}, {0.0f, 0.0f}, {-0.63742398974868952f, 0.77051324277578936f}};

// 25-point transform as 5 x 5: input n = 5 n1 + n2 at [n1][n2] of (r, i), output k = k1 + 5 k2 at [k1][k2].
__device__ __forceinline__ void dft25(float (&r)[5][5], float (&i)[5][5]) {
#pragma unroll
  for (int n2 = 0; n2 < 5; ++n2) {             // over n1, in place: [k1][n2]
    float tr[5], ti[5];
#pragma unroll
    for (int n1 = 0; n1 < 5; ++n1) { tr[n1] = r[n1][n2]; ti[n1] = i[n1][n2]; }
    dft5(tr, ti);
#pragma unroll
    for (int k1 = 0; k1 < 5; ++k1) {
      const Tw w = kTw25[k1 * n2];
      r[k1][n2] = k1 * n2 == 0 ? tr[k1] : tr[k1] * w.c - ti[k1] * w.s;
      i[k1][n2] = k1 * n2 == 0 ? ti[k1] : tr[k1] * w.s + ti[k1] * w.c;
    }
  }
#pragma unroll
  for (int k1 = 0; k1 < 5; ++k1) dft5(r[k1], i[k1]);   // over n2: [k1][k2]
}

// FPB frames per workgroup of NT threads.
template <int FPB, int NT, typename TOUT>
__global__ void __launch_bounds__(NT) logmel_kernel(FeArgs p) {
  constexpr int kHopStride = kHop + kHop / 32;            // staged sample n sits at n + n / 32: frames are an odd stride apart
  constexpr int kStaged = kHop * (FPB - 1) + kNfft;
  constexpr int kSpec = 201;                              // row stride of the half-transformed frames in float2 (odd)
  constexpr int kWork = kStaged + kStaged / 32 + 1 > FPB * kSpec * 2 ? kStaged + kStaged / 32 + 1 : FPB * kSpec * 2;
  __shared__ __attribute__((aligned(16))) float work[kWork];   // staged samples, then half-transformed rows, then the power
  __shared__ __attribute__((aligned(16))) float sWindow[kNfft];
  __shared__ float sTaps[kMaxTaps];
  __shared__ uint32_t sFilters[kMaxMels];
  __shared__ float sMin[NT / 64], sMax[NT / 64];
  const int tid = threadIdx.x;
  const int stream = fe_find(p, blockIdx.x);
  const FeStream st = fe_stream(p, stream), nx = fe_stream(p, stream + 1);
  const int t0 = ((int)blockIdx.x - st.block0) * FPB;
  const int T = nx.frame0 - st.frame0;
  const int nf = min(FPB, T - t0);                        // frames of this block (at least one)
  const int Np = st.n + p.H;

  // ---- samples 160 t0 - 200 ... of the reflect-padded x (+) h: all of a thread's loads are issued before the first
  // is used (an address select instead of a branch between x and h keeps them independent)
  const float *x = p.audio + st.offset;
  constexpr int kLoads = (kStaged + NT - 1) / NT;
  const int s0 = kHop * t0 - kNfft / 2;
  float v[kLoads];
  if (s0 >= 0 && s0 + kLoads * NT <= st.n) {              // wholly inside x: no index arithmetic
    const float *xs = x + s0 + tid;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) v[q] = xs[q * NT];
  } else {
    const int n_staged = kHop * (nf - 1) + kNfft;
#pragma unroll
    for (int q = 0; q < kLoads; ++q) {
      int s = s0 + min(q * NT + tid, n_staged - 1);       // past the last frame: a valid sample, never used
      s = s < 0 ? -s : s;
      s = s >= Np ? 2 * (Np - 1) - s : s;
      const float *src = s < st.n ? x + s : p.hush + (s - st.n);
      v[q] = *src;
    }
  }
  for (int k = tid; k < kNfft; k += NT) sWindow[k] = p.window[k];
  for (int k = tid; k < p.n_taps; k += NT) sTaps[k] = p.taps[k];
  for (int k = tid; k < p.n_mels; k += NT) sFilters[k] = p.filters[k];
#pragma unroll
  for (int q = 0; q < kLoads; ++q) {
    const int e = q * NT + tid;
    if (e < kStaged) work[e + (e >> 5)] = v[q];
  }
  __syncthreads();

  // ---- 16-point transforms: task (frame f, column n2) takes samples 25 n1 + 16 n2 mod 400
  constexpr int kTasks = FPB * 25, kRounds = (kTasks + NT - 1) / NT;
  float re[kRounds][8], im[kRounds][8];
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    const int task = q * NT + tid;
    if (task < kTasks) {
      const int f = task % FPB, n2 = task / FPB;
      float v[16];
      int n = 16 * n2;
#pragma unroll
      for (int n1 = 0; n1 < 16; ++n1) {
        v[n1] = work[kHopStride * f + n + (n >> 5)] * sWindow[n2 * 16 + n1];
        n += 25;
        n = n >= kNfft ? n - kNfft : n;
      }
      dft16_real(v, re[q], im[q]);
    }
  }
  __syncthreads();                                        // the samples are consumed: their memory takes the rows
  float2 *rows = (float2 *)work;                          // [FPB][8 rows][25]
#pragma unroll
  for (int q = 0; q < kRounds; ++q) {
    const int task = q * NT + tid;
    if (task < kTasks) {
      const int f = task % FPB, n2 = task / FPB;
#pragma unroll
      for (int k1 = 0; k1 < 8; ++k1) rows[f * kSpec + k1 * 25 + n2] = make_float2(re[q][k1], im[q][k1]);
    }
  }
  __syncthreads();

  // ---- 25-point transforms: task (frame f, row r); bin k has k mod 16 = its row and k mod 25 = its output, so
  // output k2 of row r is bin 225 r + 176 k2 mod 400
  constexpr int kRowTasks = FPB * 8;
  static_assert(kRowTasks <= NT, "one 25-point transform per thread");
  float zr[5][5], zi[5][5];
  const int f = tid % FPB, r = tid / FPB;
  if (tid < kRowTasks) {
#pragma unroll
    for (int n = 0; n < 25; ++n) {
      const float2 v = rows[f * kSpec + r * 25 + n];
      zr[n / 5][n % 5] = v.x;
      zi[n / 5][n % 5] = v.y;
    }
    dft25(zr, zi);
  }
  __syncthreads();                                        // rows are consumed: their memory takes the power, [FPB][201]
  float *power = work;
  if (tid < kRowTasks) {
    float *dst = power + f * kSpec;
    if (r > 0) {
      int base = 225 * r % 400;
#pragma unroll
      for (int k2 = 0; k2 < 25; ++k2) {
        int k = base + 176 * k2 % 400;
        k = k >= 400 ? k - 400 : k;
        const float a = zr[k2 % 5][k2 / 5], b = zi[k2 % 5][k2 / 5];
        dst[min(k, 400 - k)] = a * a + b * b;
      }
    } else {                                              // rows 0 and 8, both real: their spectra are Z + Z* and Z - Z*
#pragma unroll
      for (int k2 = 0; k2 < 13; ++k2) {
        const int m = (25 - k2) % 25;
        const float a = zr[k2 % 5][k2 / 5], b = zi[k2 % 5][k2 / 5], c = zr[m % 5][m / 5], d = zi[m % 5][m / 5];
        const int k = 176 * k2 % 400, k8 = (200 + 176 * k2) % 400;
        dst[k <= 200 ? k : 400 - k] = 0.25f * ((a + c) * (a + c) + (b - d) * (b - d));
        dst[k8 <= 200 ? k8 : 400 - k8] = 0.25f * ((a - c) * (a - c) + (b + d) * (b + d));
      }
    }
  }
  __syncthreads();

  // ---- mel filters and log, neighbouring threads on neighbouring filters; a thread takes its filter over G frames at
  // once, so that the taps are read once and the G sums and logarithms are independent
  constexpr int G = 4;
  static_assert(FPB % G == 0, "whole groups of frames");
  float lo = INFINITY, hi = -INFINITY;
  TOUT *out = (TOUT *)p.out + (size_t)(st.frame0 + t0) * p.n_mels;
  for (int e = tid; e < FPB / G * p.n_mels; e += NT) {
    const int g = e / p.n_mels, j = e - g * p.n_mels;
    const uint32_t d = sFilters[j];
    const float *pw = power + g * G * kSpec + (d & 255), *w = sTaps + (d >> 16);
    const int n = (d >> 8) & 255;
    float m[G];
#pragma unroll
    for (int q = 0; q < G; ++q) m[q] = 0.0f;
#pragma unroll 2
    for (int k = 0; k < n; ++k) {
      const float t = w[k];
#pragma unroll
      for (int q = 0; q < G; ++q) m[q] = fmaf(t, pw[q * kSpec + k], m[q]);
    }
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const float y = (log10f(fmaxf(m[q], 1e-10f)) + 4.0f) * 0.25f;
      if (g * G + q < nf) {
        out[(size_t)(g * G + q) * p.n_mels + j] = (TOUT)y;
        lo = fminf(lo, n > 0 ? y : INFINITY);      // the others are clamp_kernel's own business
        hi = fmaxf(hi, y);
      }
    }
  }
  lo = wf::wave_min(lo);
  hi = wf::wave_max(hi);
  if ((tid & 63) == 0) { sMin[tid >> 6] = lo; sMax[tid >> 6] = hi; }
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) { lo = fminf(lo, sMin[w]); hi = fmaxf(hi, sMax[w]); }
    p.range[blockIdx.x] = make_float2(lo, hi);
  }
}

// The clamp of the stored values, one wave per block: 8 decades below the stream's largest value are 2 units of the
// stored scale.  The filters no bin lies under (the lowest ones of 128: they are narrower than the 40 Hz between bins)
// sit at the floor of the logarithm and would force every row to be read again; their few columns are written directly.
template <int FPB, typename TOUT>
__global__ void __launch_bounds__(256) clamp_kernel(FeArgs p) {
  const int lane = threadIdx.x & 63;
  const int b = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (b >= p.blocks) return;
  const int stream = fe_find(p, b);
  const float low = p.range[b].x;
  const FeStream st = fe_stream(p, stream), nx = fe_stream(p, stream + 1);
  float top = -INFINITY;
  for (int k = st.block0 + lane; k < nx.block0; k += 64) top = fmaxf(top, p.range[k].y);
  top = wf::wave_max(top);
  const float floor_v = top - 2.0f;
  const TOUT fl = (TOUT)floor_v;
  const int r0 = st.frame0 + (b - st.block0) * FPB, rows = min(FPB, nx.frame0 - r0);
  TOUT *o = (TOUT *)p.out + (size_t)r0 * p.n_mels;
  if (low < floor_v) {
    for (int e = lane; e < rows * p.n_mels; e += 64)
      if ((float)o[e] < (float)fl) o[e] = fl;
  } else if (kLogFloor < floor_v) {
    for (int e = lane; e < rows * p.n_empty; e += 64) {
      const int r = e / p.n_empty;
      o[(size_t)r * p.n_mels + p.filters[p.n_mels + e - r * p.n_empty]] = fl;
    }
  }
}

template <int FPB, int NT, typename TOUT>
void launch_logmel(const FeArgs &a, hipStream_t s) {
  hipLaunchKernelGGL((logmel_kernel<FPB, NT, TOUT>), dim3(a.blocks), dim3(NT), 0, s, a);
  hipLaunchKernelGGL((clamp_kernel<FPB, TOUT>), dim3((a.blocks + 3) / 4), dim3(256), 0, s, a);
}

}  // namespace

// Pinned staging slots for the per-call index arrays.  A slot is reused only after its copy has left it; the
// ring is deep enough that a caller who enqueues short calls back to back blocks on work issued many calls
// ago (waking from such a wait costs more than several of these calls take on the GPU).
constexpr int kIdxSlots = 32;

struct wf_frontend {
  wf_frontend_config cfg{};
  int64_t max_frames = 0, max_blocks = 0;
  int n_taps = 0, n_empty = 0;
  std::vector<void *> allocs;
  float *hush = nullptr, *window = nullptr, *taps = nullptr;
  uint32_t *filters = nullptr;
  float2 *range = nullptr;
  unsigned char *idx_dev = nullptr;      // FeStream[max_streams + 1] | int32 block_stream[max_blocks]
  unsigned char *idx_host[kIdxSlots] = {};
  hipEvent_t idx_evt[kIdxSlots] = {};
  bool idx_used[kIdxSlots] = {};
  int idx_next = 0;
};

namespace {

int fe_alloc(wf_frontend *fe, void **p, size_t bytes) {
  *p = nullptr;
  hipError_t err = hipMalloc(p, bytes ? bytes : 256);
  if (err != hipSuccess) {
    (void)hipGetLastError();
    return ffail(WF_E_OOM, "hipMalloc(%zu bytes): %s", bytes, hipGetErrorString(err));
  }
  fe->allocs.push_back(*p);
  return WF_OK;
}

template <typename T>
int fe_upload(wf_frontend *fe, T **dst, const std::vector<T> &src) {
  int rc = fe_alloc(fe, (void **)dst, src.size() * sizeof(T));
  if (rc) return rc;
  FE_HIP_TRY(hipMemcpy(*dst, src.data(), src.size() * sizeof(T), hipMemcpyHostToDevice));
  return WF_OK;
}

double hz_to_mel(double f) { return 2595.0 * std::log10(1.0 + f / 700.0); }
double mel_to_hz(double m) { return 700.0 * (std::pow(10.0, m / 2595.0) - 1.0); }

int fe_create(wf_frontend *fe, const wf_frontend_config *cfg, const float *hush_audio) {
  fe->cfg = *cfg;
  const int n_mels = cfg->n_mels, H = cfg->hush_samples;
  fe->max_frames = cfg->max_total_samples / kHop + cfg->max_streams;
  int rc;
  std::vector<float> hush((size_t)(H > 0 ? H : 1), 0.0f);
  if (H > 0) memcpy(hush.data(), hush_audio, (size_t)H * 4);
  if ((rc = fe_upload(fe, &fe->hush, hush))) return rc;
  std::vector<float> win(kNfft);
  for (int n2 = 0; n2 < 25; ++n2)
    for (int n1 = 0; n1 < 16; ++n1) win[n2 * 16 + n1] = (float)(0.5 - 0.5 * std::cos(2.0 * kPi * ((25 * n1 + 16 * n2) % kNfft) / kNfft));
  if ((rc = fe_upload(fe, &fe->window, win))) return rc;
  // triangular filters, unit peak, equally spaced on the mel scale over [0, 8000] Hz
  std::vector<double> edges(n_mels + 2);
  const double m_hi = hz_to_mel(8000.0);
  for (int k = 0; k < n_mels + 2; ++k) edges[k] = mel_to_hz(m_hi * k / (n_mels + 1));
  std::vector<float> taps;
  std::vector<uint32_t> filters(n_mels);
  for (int k = 0; k < n_mels; ++k) {
    int first = 0, n = 0;
    const size_t tap0 = taps.size();
    for (int f = 0; f < kBins; ++f) {
      const double hz = f * 40.0;
      const double up = (hz - edges[k]) / (edges[k + 1] - edges[k]);
      const double down = (edges[k + 2] - hz) / (edges[k + 2] - edges[k + 1]);
      const double w = std::fmax(0.0, std::fmin(up, down));
      if (w > 0.0) {                                            // the bins under a triangle are consecutive
        if (n == 0) first = f;
        taps.push_back((float)w);
        ++n;
      }
    }
    filters[k] = (uint32_t)first | (uint32_t)n << 8 | (uint32_t)tap0 << 16;
    if (n == 0) filters.push_back((uint32_t)k);
  }
  fe->n_taps = (int)taps.size();
  fe->n_empty = (int)filters.size() - n_mels;
  if (fe->n_taps > kMaxTaps) return ffail(WF_E_INVALID_ARG, "%d filter taps, at most %d", fe->n_taps, kMaxTaps);
  if (taps.empty()) taps.push_back(0.0f);
  if ((rc = fe_upload(fe, &fe->taps, taps))) return rc;
  if ((rc = fe_upload(fe, &fe->filters, filters))) return rc;
  fe->max_blocks = fe->max_frames / kFramesSmall + cfg->max_streams;
  if ((rc = fe_alloc(fe, (void **)&fe->range, (size_t)fe->max_blocks * sizeof(float2)))) return rc;
  const size_t idx_bytes = ((size_t)cfg->max_streams + 1) * sizeof(FeStream) + (size_t)fe->max_blocks * 4;
  if ((rc = fe_alloc(fe, (void **)&fe->idx_dev, idx_bytes))) return rc;
  for (int i = 0; i < kIdxSlots; ++i) {
    FE_HIP_TRY(hipHostMalloc((void **)&fe->idx_host[i], idx_bytes, hipHostMallocDefault));
    FE_HIP_TRY(hipEventCreateWithFlags(&fe->idx_evt[i], hipEventDisableTiming));
  }
  FE_HIP_TRY(hipDeviceSynchronize());
  return WF_OK;
}

}  // namespace

extern "C" {

void wf_frontend_destroy(wf_frontend *fe) {
  if (!fe) return;
  (void)hipDeviceSynchronize();
  for (int i = 0; i < kIdxSlots; ++i) {
    if (fe->idx_host[i]) (void)hipHostFree(fe->idx_host[i]);
    if (fe->idx_evt[i]) (void)hipEventDestroy(fe->idx_evt[i]);
  }
  for (void *p : fe->allocs) (void)hipFree(p);
  delete fe;
}

int wf_frontend_create(const wf_frontend_config *cfg, const float *hush_audio, wf_frontend **out) {
  if (!out) return ffail(WF_E_INVALID_ARG, "out is NULL");
  *out = nullptr;
  if (!cfg) return ffail(WF_E_INVALID_ARG, "cfg is NULL");
  if (cfg->n_mels < 1 || cfg->n_mels > 256) return ffail(WF_E_INVALID_ARG, "n_mels = %d, need 1..256", cfg->n_mels);
  if (cfg->hush_samples < 0) return ffail(WF_E_INVALID_ARG, "hush_samples = %d", cfg->hush_samples);
  if (cfg->hush_samples > 0 && !hush_audio) return ffail(WF_E_INVALID_ARG, "hush_audio is NULL but hush_samples = %d", cfg->hush_samples);
  if (cfg->max_streams < 1) return ffail(WF_E_INVALID_ARG, "max_streams = %d", cfg->max_streams);
  if (cfg->max_total_samples < kBins || cfg->max_total_samples > 2000000000LL)
    return ffail(WF_E_INVALID_ARG, "max_total_samples = %lld out of range", (long long)cfg->max_total_samples);
  wf_frontend *fe = new (std::nothrow) wf_frontend();
  if (!fe) return ffail(WF_E_OOM, "host allocation failed");
  int rc = fe_create(fe, cfg, hush_audio);
  if (rc) {
    char keep[512];
    memcpy(keep, wf::error_buffer(), sizeof(keep));
    wf_frontend_destroy(fe);
    memcpy(wf::error_buffer(), keep, sizeof(keep));
    return rc;
  }
  *out = fe;
  return WF_OK;
}

int wf_logmel_batch(wf_frontend *fe, const float *audio_dev, const int64_t *sample_offset, const int32_t *n_samples, int32_t B,
                    void *mel_out_dev, int32_t mel_dtype, int64_t mel_capacity_frames, int32_t *cu_frames_host, void *hip_stream) {
  if (!fe) return ffail(WF_E_INVALID_ARG, "frontend is NULL");
  if (!audio_dev || !sample_offset || !n_samples || !mel_out_dev) return ffail(WF_E_INVALID_ARG, "NULL pointer");
  if (mel_dtype != WF_DTYPE_F32 && mel_dtype != WF_DTYPE_BF16) return ffail(WF_E_INVALID_ARG, "mel_dtype = %d", mel_dtype);
  if (B < 1) return ffail(WF_E_INVALID_ARG, "B = %d, need B >= 1", B);
  if (B > fe->cfg.max_streams) return ffail(WF_E_CAPACITY, "B = %d exceeds max_streams = %d", B, fe->cfg.max_streams);
  const int H = fe->cfg.hush_samples;
  int64_t total = 0, frames = 0;
  for (int i = 0; i < B; ++i) {
    if (n_samples[i] < 0 || sample_offset[i] < 0) return ffail(WF_E_INVALID_ARG, "stream %d: negative length or offset", i);
    const int64_t Np = (int64_t)n_samples[i] + H;
    if (Np < kBins) return ffail(WF_E_INVALID_ARG, "stream %d: %lld samples incl. hush, need >= %d (reflect padding)", i, (long long)Np, kBins);
    total += Np;
    if (total > fe->cfg.max_total_samples)
      return ffail(WF_E_CAPACITY, "total samples incl. hush exceed max_total_samples = %lld (at stream %d)", (long long)fe->cfg.max_total_samples, i);
    frames += Np / kHop;
  }
  if (frames > mel_capacity_frames)
    return ffail(WF_E_CAPACITY, "batch produces %lld frames but mel_capacity_frames = %lld", (long long)frames, (long long)mel_capacity_frames);
  hipStream_t s = (hipStream_t)hip_stream;

  // A batch that would not give every compute unit a large block takes small ones: more of them, each shorter.
  const bool small = frames < kSmallBatch;
  const int fpb = small ? kFramesSmall : kFramesLarge;
  FeArgs a{};
  a.audio = audio_dev; a.hush = fe->hush; a.window = fe->window; a.taps = fe->taps; a.filters = fe->filters;
  a.range = fe->range; a.out = mel_out_dev;
  a.B = B; a.H = H; a.n_mels = fe->cfg.n_mels; a.n_taps = fe->n_taps; a.n_empty = fe->n_empty;
  const bool out_bf16 = mel_dtype == WF_DTYPE_BF16;
  // ---- stream metadata: in the kernel arguments where they fit (no copy ahead of the kernels), else by an upload
  const bool inl = B <= kInline;
  const int slot = fe->idx_next;
  if (!inl && fe->idx_used[slot]) FE_HIP_TRY(hipEventSynchronize(fe->idx_evt[slot]));
  FeStream *meta = inl ? a.local : (FeStream *)fe->idx_host[slot];
  int32_t *bs = inl ? nullptr : (int32_t *)(fe->idx_host[slot] + ((size_t)fe->cfg.max_streams + 1) * sizeof(FeStream));
  int32_t f0 = 0, blocks = 0;
  for (int i = 0; i < B; ++i) {
    const int32_t T = (int32_t)(((int64_t)n_samples[i] + H) / kHop);
    meta[i] = FeStream{sample_offset[i], n_samples[i], f0, blocks, 0};
    if (cu_frames_host) cu_frames_host[i] = f0;
    f0 += T;
    const int32_t nb = (T + fpb - 1) / fpb;
    if (bs)
      for (int32_t b = 0; b < nb; ++b) bs[blocks + b] = i;
    blocks += nb;
  }
  meta[B] = FeStream{0, 0, f0, blocks, 0};
  if (cu_frames_host) cu_frames_host[B] = f0;
  if (blocks == 0) return WF_OK;
  a.blocks = blocks;
  if (!inl) {
    const size_t head = ((size_t)fe->cfg.max_streams + 1) * sizeof(FeStream);
    FE_HIP_TRY(hipMemcpyAsync(fe->idx_dev, fe->idx_host[slot], head + (size_t)blocks * 4, hipMemcpyHostToDevice, s));
    FE_HIP_TRY(hipEventRecord(fe->idx_evt[slot], s));
    fe->idx_used[slot] = true;
    fe->idx_next = (slot + 1) % kIdxSlots;
    a.streams = (const FeStream *)fe->idx_dev;
    a.block_stream = (const int32_t *)(fe->idx_dev + head);
  }
  if (small) {
    if (out_bf16) launch_logmel<kFramesSmall, 256, __bf16>(a, s);
    else launch_logmel<kFramesSmall, 256, float>(a, s);
  } else {
    if (out_bf16) launch_logmel<kFramesLarge, 128, __bf16>(a, s);
    else launch_logmel<kFramesLarge, 128, float>(a, s);
  }
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return ffail(WF_E_HIP, "front-end launch: %s", hipGetErrorString(err));
  return WF_OK;
}

}  // extern "C"
