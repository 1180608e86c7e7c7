// STFT and inverse STFT around the separation path (arXiv 2212.05271, Section 3: feature extraction and
// iSTFT are among the operations run on the GPU; the paper fixes 513 bins, i.e. a 1024-point transform).
//
// Definition (the paper is silent on window, hop and padding): periodic Hann window of 1024 samples, hop
// 256, the signal zero-padded by 768 samples on both sides, T = ceil(N / 256) + 3 frames; the inverse is
// irfft * window / 1.5 (= sum over the four shifts of the squared window), overlap-added, padding stripped.
//
// A 1024-point real transform is done as a 512-point complex FFT of the even/odd-packed frame plus the
// split step.  The 512-point transform is 8 x 8 x 8: one wavefront per transform, eight values per lane,
// three passes of 8-point butterflies in registers with two exchanges through LDS in between (a radix-2
// transform that lives in LDS is bound by LDS bandwidth: it moves every value through LDS nine times).
// Twiddles come from one table exp(-2 pi i k / 1024), k = 0..512, and the window from another, both evaluated in fp64 and
// rounded once; the tables are computed on the device by the first call of a context, and every workgroup copies what it
// reads per transform into LDS.
//
// Workgroup order: consecutive workgroup ids go to different XCDs (each with its own L2), so the id is
// remapped such that every XCD walks a contiguous range of frames: neighbouring frames share three quarters
// of their samples, and their 64-byte output runs are neighbours in memory.
#include "gss_internal.h"
#include "gss_rules.h"

namespace {

constexpr int kN = 1024;        // real transform length
constexpr int kH = 512;         // complex transform length
constexpr int kBins = 513;
constexpr int kHop = 256;
constexpr int kPad = kN - kHop;
constexpr int kFftWaves = 8;

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

constexpr int kXcds = 8;

// table[k] = exp(-2 pi i k / 1024), k = 0 .. 512; table[513 + n] = the periodic Hann window at the samples 2n and 2n + 1.
constexpr int kTableSize = kH + 1 + kH;
__device__ __forceinline__ float2* window_of(float2* table) { return table + kH + 1; }
__device__ __forceinline__ const float2* window_of(const float2* table) { return table + kH + 1; }
__global__ void twiddle_table_kernel(float2* __restrict__ table) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k > kH) return;
  double sn, cs;
  sincospi(-2.0 * (double)k / (double)kN, &sn, &cs);
  table[k] = make_float2((float)cs, (float)sn);
  if (k < kH)
    window_of(table)[k] = make_float2((float)(0.5 - 0.5 * cospi(4.0 * (double)k / (double)kN)),
                                      (float)(0.5 - 0.5 * cospi((4.0 * (double)k + 2.0) / (double)kN)));
}

// LDS copies of the first n twiddles and of the window times `scale`, by the whole workgroup (the caller synchronises).  The
// window as a table of pairs: from the cosines among the twiddles it took two reads with four-way bank conflicts per pair.
__device__ __forceinline__ void fill_tables(float2* tw, int n, float2* win, float scale, const float2* __restrict__ table) {
  for (int k = threadIdx.x; k < n; k += blockDim.x) tw[k] = table[k];
  for (int k = threadIdx.x; k < kH; k += blockDim.x) {
    const float2 w = window_of(table)[k];
    win[k] = make_float2(w.x * scale, w.y * scale);
  }
}

// Work item of workgroup `id` out of `n` when the grid has kXcds * ceil(n / kXcds) workgroups: XCD x = id % 8
// gets the contiguous items [x * per, (x + 1) * per).  Returns -1 for the padding workgroups.
__device__ __forceinline__ long xcd_contiguous(unsigned id, long n) {
  const long per = (n + kXcds - 1) / kXcds;
  const long w = (long)(id % kXcds) * per + id / kXcds;
  return (id / kXcds < per && w < n) ? w : -1;
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// W_1024^idx for 0 <= idx < 1024 from the half table: W^idx = -W^(idx - 512).
__device__ __forceinline__ float2 twiddle(const float2* tw, int idx) {
  const float2 w = tw[idx <= kH ? idx : idx - kH];
  return idx <= kH ? w : make_float2(-w.x, -w.y);
}

// 8-point DFT in registers, natural order in and out: v[k] <- sum_n v[n] exp(-2 pi i n k / 8).
__device__ __forceinline__ void dft8(float2 (&v)[8]) {
  constexpr float kR = 0.70710678118654752440f;
  float2 a[4], b[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    a[j] = make_float2(v[j].x + v[j + 4].x, v[j].y + v[j + 4].y);
    b[j] = make_float2(v[j].x - v[j + 4].x, v[j].y - v[j + 4].y);
  }
  // b[j] *= W8^j
  b[1] = make_float2((b[1].x + b[1].y) * kR, (b[1].y - b[1].x) * kR);
  b[2] = make_float2(b[2].y, -b[2].x);
  b[3] = make_float2((b[3].y - b[3].x) * kR, -(b[3].x + b[3].y) * kR);
  // two 4-point DFTs: even outputs from a, odd outputs from b
  auto dft4 = [](const float2 (&c)[4], float2& x0, float2& x1, float2& x2, float2& x3) {
    const float2 e0 = make_float2(c[0].x + c[2].x, c[0].y + c[2].y);
    const float2 e1 = make_float2(c[0].x - c[2].x, c[0].y - c[2].y);
    const float2 o0 = make_float2(c[1].x + c[3].x, c[1].y + c[3].y);
    const float2 d = make_float2(c[1].x - c[3].x, c[1].y - c[3].y);
    const float2 o1 = make_float2(d.y, -d.x);                  // -i (c1 - c3)
    x0 = make_float2(e0.x + o0.x, e0.y + o0.y);
    x2 = make_float2(e0.x - o0.x, e0.y - o0.y);
    x1 = make_float2(e1.x + o1.x, e1.y + o1.y);
    x3 = make_float2(e1.x - o1.x, e1.y - o1.y);
  };
  dft4(a, v[0], v[2], v[4], v[6]);
  dft4(b, v[1], v[3], v[5], v[7]);
}

constexpr int kExStride = 72;                 // float2 per row of the exchange buffer (64 + padding)
// float2 per transform in LDS (inverse): at least 8 * kExStride (the exchange), 513 (a spectrum) and, so that eight transforms side
// by side can be read and written eight-at-a-time per bin without bank conflicts, 2 modulo 16.
constexpr int kRow = 578;
static_assert(kRow >= 8 * kExStride && kRow >= kBins && kRow % 16 == 2, "row pitch of the transforms in LDS");

// Per-lane constants of the 512-point transform: the twiddles between its passes.
struct FftLane {
  float2 wa[7];     // W_512^(lane * r),          r = 1..7
  float2 wb[7];     // W_64^((lane % 8) * p),     p = 1..7
};
__device__ __forceinline__ void fft_lane_init(FftLane& c, const float2* tw, int lane) {
#pragma unroll
  for (int r = 1; r < 8; ++r) {
    c.wa[r - 1] = twiddle(tw, 2 * lane * r);
    c.wb[r - 1] = twiddle(tw, 16 * (lane & 7) * r);
  }
}

// Forward 512-point complex FFT by one wavefront.  In: v[r] = x[64 r + lane].  Out: v[p] = the transform at k =
// fft_bin(lane) + 64 p; the exchange buffer is free on return.  With n = 64 n1 + n2, k = k1 + 8 k2:
//   pass 1 (lane = n2):            8-point DFT over n1, times W_512^(n2 k1)
//   exchange: rows k1, columns n2 = 8 m1 + m0;   pass 2 (lane = (k1, m0)): DFT over m1, times W_64^(m0 p1)
//   exchange: [k1][p1][m0], 9-float2 pitch;      pass 3 (lane = (k1, p1)): DFT over m0 -> k = k1 + 8 p1 + 64 p0
__device__ __forceinline__ void fft512(float2 (&v)[8], float2* ex, const FftLane& c, int lane) {
  const int hi = lane >> 3, lo = lane & 7;
  dft8(v);
#pragma unroll
  for (int r = 1; r < 8; ++r) v[r] = cmul(v[r], c.wa[r - 1]);
#pragma unroll
  for (int r = 0; r < 8; ++r) ex[r * kExStride + lane] = v[r];
  wave_sync();
#pragma unroll
  for (int m1 = 0; m1 < 8; ++m1) v[m1] = ex[hi * kExStride + 8 * m1 + lo];
  wave_sync();
  dft8(v);
#pragma unroll
  for (int p = 1; p < 8; ++p) v[p] = cmul(v[p], c.wb[p - 1]);
#pragma unroll
  for (int p = 0; p < 8; ++p) ex[hi * kExStride + 9 * p + lo] = v[p];
  wave_sync();
#pragma unroll
  for (int m0 = 0; m0 < 8; ++m0) v[m0] = ex[hi * kExStride + 9 * lo + m0];
  wave_sync();
  dft8(v);
}
__device__ __forceinline__ int fft_bin(int lane) { return (lane >> 3) + 8 * (lane & 7); }

// Items of workgroup w of `wgs`: an even, contiguous share of n.
__device__ __forceinline__ long share_begin(long w, long wgs, long n) { return (long)((unsigned long)w * (unsigned long)n / (unsigned long)wgs); }

// ----------------------------------------------------------------------------------------------
// STFT.  A workgroup of W wavefronts takes steps of (segment, frame) items; a step is UNITS units of W transforms, one per wavefront: a
// unit is all channels of W / D consecutive frames, or 8 channels of a frame with more than 8 (W = 8).  The samples of the next unit
// are requested before the current transforms.  The spectrum replaces the transform in the wavefront's LDS row (the lane that reads the pair Z[k], Z[512 - k] writes X[k] and X[512 - k]), and the workgroup
// writes a bin's values of the step as one run of memory (128 bytes for two units of 8 channels).
//
// Bound: memory and latency.  W = 8: two workgroups per compute unit are resident, held there by 128 registers and, for two
// units, by LDS; each has one unit of samples in flight.  W = 16 (long calls): one workgroup per compute unit with 256-byte runs per
// bin.  At 128 registers 14 to 24 (two units) or 10 (one) are spilled to scratch memory.  Ten minutes of 8 channels: 504 us -> 434
// with the spectrum written past the caches (STREAM) -> 370 us = 4.2 TB/s with W = 16 as well (a large copy: 4.7).  On the way: an
// even share of consecutive frames per workgroup instead of turns 583 us, one workgroup per frame, 64-byte runs 722 us; turns of
// 4 or 8 steps, whose frames share samples in the compute unit's own cache, 497 to 533 us: neighbouring workgroups then write
// further apart.  Three workgroups per compute unit at 80 registers: 55 to 70 spilled, twice as slow.
//
// One unit per step for short calls (gss_stft): 8 channels 7.7, 10.7, 17.2 us at 130, 510, 1020 frames (two units 11.0, 12.5,
// 17.0; one workgroup per frame 8.1, 11.2, 20.6).
// ----------------------------------------------------------------------------------------------
constexpr int kStftWgsPerCu = 2;                           // resident workgroups; no more are launched
// Row pitch: at least 8 * kExStride (the exchange) and 513 (a spectrum).
constexpr int kStftRow = 577;
static_assert(kStftRow >= 8 * kExStride && kStftRow >= kBins, "row pitch of the transforms in LDS");
struct __attribute__((packed, aligned(4))) PairUnaligned { float a, b; };
// A store that does not stay in the caches (STREAM).
template <bool STREAM>
__device__ __forceinline__ void put(float2* p, float2 v) {
  if constexpr (STREAM) __builtin_nontemporal_store(__builtin_bit_cast(double, v), reinterpret_cast<double*>(p));
  else *p = v;
}
template <int W, int UNITS, bool STREAM>
__global__ __launch_bounds__(64 * W, 4) void stft_kernel(const float* __restrict__ x, float2* __restrict__ Y,
                                                                const float2* __restrict__ table, int D, long N, int T,
                                                                long n_items) {
  // (two units: the split's half of the table only, so that two workgroups fit into a compute unit; the lanes' constants come
  // from memory, one more latency at the start)
  constexpr int kTw = UNITS == 1 ? kH + 1 : kH / 2;
  __shared__ float2 tw[kTw];
  __shared__ float2 win[kH];
  __shared__ float2 rows[UNITS * W][kStftRow];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Every XCD has an even, contiguous share of the items, which its workgroups take step by step in turn: at any time they
  // write neighbouring frames.
  const int xcd = (int)(blockIdx.x % kXcds);
  const long j = blockIdx.x / kXcds, per_xcd = gridDim.x / kXcds;
  const bool by_frame = D <= 8;                            // the units of a step: frames, or groups of eight channels
  const int per_unit = D <= 8 ? W / D : 1;                 // frames per unit
  const int per_step = by_frame ? UNITS * per_unit : 1;    // frames per step
  constexpr int kChans = 8 * UNITS;                        // more than 8 channels: channels per step
  const long item1 = share_begin(xcd + 1, kXcds, n_items);
  long i = share_begin(xcd, kXcds, n_items) + j * per_step, block_end = i + per_step;
  if (i >= item1) return;

  const int my_frame = D <= 8 ? wave / D : 0, my_chan = D <= 8 ? wave % D : wave;
  // this wavefront's samples of unit u of the step at item i, channels from d0 on
  float2 raw[8];
  auto request = [&](long i, int d0, int u) {
    const int s = (int)((unsigned)i / (unsigned)T);        // (fewer than 2^31 items)
    const int fr = by_frame ? u * per_unit + my_frame : 0, d = d0 + my_chan + (by_frame ? 0 : 8 * u);
    const int t = (int)i - s * T + fr;
    const long start = (long)t * kHop - kPad;              // first sample of the frame (may be negative)
    const bool on = my_frame < per_unit && t < T && i + fr < item1 && d < D;
    const float* __restrict__ xs = x + ((long)s * D + (on ? d : 0)) * N;
    if (on && start >= 0 && start + kN <= N) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const PairUnaligned v = *reinterpret_cast<const PairUnaligned*>(xs + start + 2 * (lane + 64 * m));   // (4-byte aligned)
        raw[m] = make_float2(v.a, v.b);
      }
    } else {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const long p0 = start + 2 * (lane + 64 * m), p1 = p0 + 1;
        raw[m].x = on && p0 >= 0 && p0 < N ? xs[p0] : 0.f;
        raw[m].y = on && p1 >= 0 && p1 < N ? xs[p1] : 0.f;
      }
    }
  };
  int d0 = 0;
  request(i, 0, 0);
  fill_tables(tw, kTw, win, 1.f, table);
  FftLane fc;
  if constexpr (UNITS > 1) fft_lane_init(fc, table, lane);
  __syncthreads();
  if constexpr (UNITS == 1) fft_lane_init(fc, tw, lane);
  while (i < item1) {
    const int s = (int)((unsigned)i / (unsigned)T), t = (int)i - s * T;
    const long end = block_end < item1 ? block_end : item1;
    int nf = (int)(end - i);                               // frames of this step that are in the same segment
    nf = T - t < nf ? T - t : nf;
    const int nd = by_frame ? D : (D - d0 < kChans ? D - d0 : kChans);
    const bool more = !by_frame && d0 + kChans < D;        // the frame has channels left
    long in = more ? i : i + nf;
    if (in >= block_end) {                                 // the workgroup's next block of frames
      in = block_end + (per_xcd - 1) * per_step;
      block_end = in + per_step;
    }
    const int dn = more ? d0 + kChans : 0;
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      // windowed frame, even/odd packed: z[n] = w[2n] x[2n] + i w[2n+1] x[2n+1]
      float2 v[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const float2 w = win[lane + 64 * m];
        v[m] = make_float2(w.x * raw[m].x, w.y * raw[m].y);
      }
      if (u + 1 < UNITS) request(i, d0, u + 1);
      else if (in < item1) request(in, dn, 0);
      const int fr = by_frame ? u * per_unit + my_frame : 0, dd = my_chan + (by_frame ? 0 : 8 * u);
      if (my_frame < per_unit && fr < nf && dd < nd) {
        float2* __restrict__ Z = rows[u * W + wave];
        fft512(v, Z, fc, lane);
        const int kb = fft_bin(lane);
#pragma unroll
        for (int p = 0; p < 8; ++p) Z[kb + 64 * p] = v[p];
        wave_sync();
        // split: with e = (Z[k] + conj Z[512-k]) / 2, o = (Z[k] - conj Z[512-k]) / 2, Z[512] = Z[0]:
        // X[k] = e - i w^k o, X[512-k] = conj(e + i w^k o); X[256] = conj Z[256]
#pragma unroll
        for (int m = 0; m < 4; ++m) {
          const int k = lane + 64 * m;
          const float2 zk = Z[k];
          const float2 zc = Z[(kH - k) & (kH - 1)];
          const float2 e = make_float2(0.5f * (zk.x + zc.x), 0.5f * (zk.y - zc.y));
          const float2 o = make_float2(0.5f * (zk.x - zc.x), 0.5f * (zk.y + zc.y));
          const float2 wo = cmul(tw[k], o);
          Z[k] = make_float2(e.x + wo.y, e.y - wo.x);
          Z[kH - k] = make_float2(e.x - wo.y, -(e.y + wo.x));
        }
        if (lane == 0) Z[kH / 2].y = -Z[kH / 2].y;
      }
    }
    __syncthreads();
    // bin k: the step's nf frames x nd channels, one run of memory (several frames: all their channels)
    const int nr = nf * nd, q = by_frame ? per_unit * D : W;     // values per bin, of the first unit
    float2* __restrict__ out = Y + ((long)s * kBins * T + t) * D + d0;
    const long pitch = (long)T * D;
    constexpr int kFull = W * UNITS, kShift = kFull == 8 ? 3 : kFull == 16 ? 4 : 5;        // (a full step: the first unit has W values)
    if (nr == kFull) {
      for (int e = threadIdx.x; e < kBins * kFull; e += 64 * W)
        put<STREAM>(out + (e >> kShift) * pitch + (e & (kFull - 1)), rows[e & (kFull - 1)][e >> kShift]);
    } else {
      for (int e = threadIdx.x; e < kBins * nr; e += 64 * W) {
        const int k = (int)((unsigned)e / (unsigned)nr), r = e - k * nr;
        put<STREAM>(out + k * pitch + r, rows[r < q ? r : W + r - q][k]);
      }
    }
    __syncthreads();
    i = in;
    d0 = dn;
  }
}

// ----------------------------------------------------------------------------------------------
// Inverse STFT, overlap-add included.  A workgroup of W wavefronts forms `W steps - 3` consecutive blocks of 256 samples of one segment
// from W steps frames (the three in front of its first block once more); a step is W frames, one per wavefront, read as
// runs of 8 W bytes of X[bin][frame] and requested a step ahead.  The windowed frames stay in LDS; block th is the sum of
// its four frames, oldest first, and the three blocks that the next step completes are carried over as partial sums.
//
// Bound: latency, with the LDS busy for half of the time.  Which W and how many steps: plan_istft.  Long calls: one workgroup of
// 16 wavefronts per compute unit (registers), with one step requested ahead: 128 segments of 18 s 216 us = 3.4 TB/s, X read once
// and x written once (two workgroups of 8 wavefronts, 64-byte runs 270 us; the same steps per workgroup as those 248: the number
// of steps is chosen so that the rounds of workgroups are full; window from the cosine table in a pass of its own through LDS
// 291; through frames in memory, 1.9 GB instead of 0.74 GB: 618 us).  10 segments of 25 s 46 -> 32 us, 30 of 9 s 50 -> 33.  The
// spectrum, the transform and the windowed frame share one LDS row per wavefront; the last pass's values are windowed in registers.
// ----------------------------------------------------------------------------------------------
template <int W>
__global__ __launch_bounds__(64 * W, 4) void istft_kernel(const float2* __restrict__ X, float* __restrict__ x,
                                                              const float2* __restrict__ table, long N, int T, int steps,
                                                              long wgs) {
  __shared__ float2 tw[kH + 1];
  __shared__ float2 win[kH];                               // window / 1.5, irfft's 1 / N
  __shared__ float2 rows[W][kRow];
  __shared__ float carry[3][kHop];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long wg = xcd_contiguous(blockIdx.x, wgs);
  if (wg < 0) return;
  const int nb = W * steps - 3;                            // blocks per workgroup
  const int per_seg = (T - 3 + nb - 1) / nb;               // blocks 3 .. T - 1 hold samples
  const int s = (int)((unsigned long)wg / (unsigned)per_seg);
  const int b0 = 3 + (int)(wg - (long)s * per_seg) * nb;   // first block; its frames are b0 - 3 .. b0
  const int b1 = b0 + nb < T ? b0 + nb : T;
  constexpr int kLoads = (kBins * W + 64 * W - 1) / (64 * W);
  const float2* __restrict__ Xs = X + (long)s * kBins * T;
  float2 raw[kLoads];
  auto request = [&](int f0) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = threadIdx.x + u * 64 * W;
      const int k = e / W, t = f0 + (e & (W - 1));
      raw[u] = make_float2(0.f, 0.f);
      if (e < kBins * W && t < T) raw[u] = Xs[(long)k * T + t];
    }
  };
  request(b0 - 3);
  fill_tables(tw, kH + 1, win, 1.0f / (1.5f * (float)kN), table);
  for (int c = threadIdx.x; c < 3 * kHop; c += 64 * W) carry[c / kHop][c % kHop] = 0.f;
  __syncthreads();
  FftLane fc;
  fft_lane_init(fc, tw, lane);
  float2* __restrict__ z = rows[wave];
  const int part = threadIdx.x >> 8, c = threadIdx.x & (kHop - 1);
  for (int f0 = b0 - 3; f0 < b1; f0 += W) {
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int e = threadIdx.x + u * 64 * W;
      if (e < kBins * W) rows[e & (W - 1)][e / W] = raw[u];
    }
    __syncthreads();
    if (f0 + W < b1) request(f0 + W);
    // pack the half spectrum of a real signal into a 512-point complex one, conjugated so that a forward
    // transform inverts it:  Zc[k] = conj( (X[k] + conj X[512-k]) + i conj(w^k) (X[k] - conj X[512-k]) )
    // (a frame beyond the last one is zero and stays zero)
    float2 v[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int k = lane + 64 * m;
      float2 xk = z[k];
      float2 xc = z[kH - k];
      if (k == 0) { xk.y = 0.f; xc.y = 0.f; }    // DC and Nyquist of a real signal are real (as irfft assumes)
      const float2 e = make_float2(xk.x + xc.x, xk.y - xc.y);
      const float2 o = make_float2(xk.x - xc.x, xk.y + xc.y);
      const float2 wc = make_float2(tw[k].x, -tw[k].y);
      const float2 wo = cmul(wc, o);
      v[m] = make_float2(e.x - wo.y, -(e.y + wo.x));          // conj(e + i wo)
    }
    wave_sync();
    fft512(v, z, fc, lane);
    // x[2n] = Re, x[2n+1] = -Im (undo the conjugate), windowed on the way to the row
    const int nb0 = fft_bin(lane);
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const float2 w = win[nb0 + 64 * p];
      z[nb0 + 64 * p] = make_float2(v[p].x * w.x, -v[p].y * w.y);
    }
    __syncthreads();
    // block f0 + j: frames f0 + j - 3 .. f0 + j, frame f0 + q being row q
    auto sample = [&](int row, int seg) { return reinterpret_cast<const float*>(rows[row])[seg * kHop + c]; };
    float sum[4];
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int j = (W / 4) * jj + part;
      float acc = j < 3 ? carry[j < 3 ? j : 0][c] : 0.f;
#pragma unroll
      for (int q = 3; q >= 0; --q)
        if (j >= q) acc += sample(j - q, q);
      sum[jj] = acc;
    }
#pragma unroll
    for (int jj = 0; jj < (W == 8 ? 2 : 1); ++jj) {           // block f0 + W + j so far
      const int j = (W / 4) * jj + part;
      if (j < 3) {
        float acc = 0.f;
#pragma unroll
        for (int q = 3; q >= 1; --q)
          if (q > j) acc += sample(W + j - q, q);
        carry[j][c] = acc;
      }
    }
#pragma unroll
    for (int jj = 0; jj < 4; ++jj) {
      const int th = f0 + (W / 4) * jj + part;
      const long n = (long)th * kHop - kPad + c;
      if (th >= b0 && th < b1 && n < N) x[(long)s * N + n] = sum[jj];
    }
    __syncthreads();
  }
}

// A copy of a spectrum that shares memory with the output (gss_istft).
__global__ void copy_spectrum_kernel(const float2* __restrict__ X, float2* __restrict__ copy, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) copy[i] = X[i];
}

// The context's twiddle table, created on first use; the fill is ordered before the caller's kernels on `st`.
int get_twiddles(gss_ctx* ctx, hipStream_t st, const float2** out) {
  if (!ctx->twiddles) {
    void* p = nullptr;
    if (hipMalloc(&p, kTableSize * sizeof(float2)) != hipSuccess) return GSS_ENOMEM;
    hipLaunchKernelGGL(twiddle_table_kernel, dim3((kH + 256) / 256), dim3(256), 0, st, (float2*)p);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess) {
      (void)hipFree(p);
      return GSS_EHIP;
    }
    ctx->twiddles = p;
  }
  *out = (const float2*)ctx->twiddles;
  return GSS_OK;
}

}  // namespace

extern "C" int gss_stft(gss_ctx* ctx, const float* x, int S, int D, int64_t N, int n_fft, int hop,
                        float* Y, int T, void* stream) {
  if (!ctx || !x || !Y || S <= 0 || D <= 0 || N <= 0 || T <= 0) return GSS_EINVAL;
  if (n_fft != kN || hop != kHop) return GSS_EUNSUPPORTED;
  if ((N + hop - 1) / hop + 3 != T) return GSS_EINVAL;
  if ((long)S * T > 0x7ffffff0L) return GSS_EUNSUPPORTED;
  if (hipSetDevice(ctx->device) != hipSuccess) return GSS_EHIP;
  const float2* table = nullptr;
  const int rc = get_twiddles(ctx, (hipStream_t)stream, &table);
  if (rc != GSS_OK) return rc;
  const long n_items = (long)S * T, most = (long)ctx->num_cu * kStftWgsPerCu;
  const int per_unit = D <= 8 ? 8 / D : 1;
  // Long calls: 16 wavefronts per workgroup, runs of 256 bytes per bin (8 channels), one workgroup per compute unit.  8 / 16 wavefronts,
  // us: 8 channels, 512 MB 164 / 170, 640 MB 189 / 194, 768 MB 237 / 233, 1.23 GB 428 / 370, 3.8 GB 1673 / 1390; 6 channels 288 MB 138 /
  // 136, 577 MB 315 / 251; 4 channels 616 MB 291 / 246; 5 channels 962 MB 608 / 426.  Around 300 MB, at 270, 300, 320 and 360 MB, 16 over
  // 8: 1 channel 0.99, 0.95, 0.95, 0.89, 2 channels 1.04, 0.95, 0.97, 0.94, 3 channels 1.04, 1.03, 0.99, 0.94, 4 channels 1.12, 1.00, 1.00,
  // 0.98, 5 channels 0.97, 0.96, 0.95, 0.86, 6 channels 1.02, 0.98, 0.97, 0.92, 7 channels 1.05, 1.00, 0.97, 0.94.  (Single lengths of
  // 4 channels suit 8 wavefronts far better than their neighbours do: 3 x 6496 frames, 320 MB, 118 / 132.)
  const double out_bytes = (double)S * kBins * T * D * sizeof(float2);
  const bool wide = D <= 8 && out_bytes > (D == 8 ? 700e6 : 300e6);
  const long steps1 = (n_items + per_unit - 1) / per_unit;
  // Short calls take steps of one unit: the chip is not full otherwise, and each workgroup would do two units in a row.  The line
  // lies at four rounds of the resident workgroups (8 channels, one / two units: 510 frames, one round, 10.7 / 12.5 us; 2040, four
  // rounds, 29.9 / 31.1; 3000 37.9 / 38.1; 6000 79.8 / 68.7).  24 channels are three units per frame, of which pairs leave one
  // alone (510 frames 24.2 / 27.1, 6000 frames 275 / 288); other counts beyond 8 gain nothing from single units.
  const int units = (D <= 8 ? steps1 <= 4 * most : D % 16 == 8) ? 1 : 2;
  const long per_step = wide ? 2 * (16 / D) : D <= 8 ? units * per_unit : 1, steps = (n_items + per_step - 1) / per_step;
  const long res = wide ? most / 2 : most;
  const long grid = ((steps < res ? steps : res) + kXcds - 1) / kXcds * kXcds;
  // A spectrum that no cache holds until it is read anyway is written past them, so that the samples, which four neighbouring frames
  // share, stay there: where the runs are whole 64-byte pieces.  With / without, us: 1.23 GB (8 channels) 434 / 504, 231 MB (24) 87 /
  // 112, 197 MB (16) 110 / 130; but 128 MB (8) 48 / 46, and runs of other lengths: 6 channels, 577 MB 535 / 315.
  const bool past = D % 8 == 0 && out_bytes > 190e6;
  const auto kern = wide ? (past ? stft_kernel<16, 2, true> : stft_kernel<16, 2, false>)
                    : units == 1 ? (past ? stft_kernel<8, 1, true> : stft_kernel<8, 1, false>) : (past ? stft_kernel<8, 2, true> : stft_kernel<8, 2, false>);
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * (wide ? 16 : kFftWaves)), 0, (hipStream_t)stream,
                     x, (float2*)Y, table, D, (long)N, T, n_items);
  return hipGetLastError() == hipSuccess ? GSS_OK : GSS_EHIP;
}

extern "C" int gss_istft(gss_ctx* ctx, const float* X, int S, int T, int n_fft, int hop,
                         float* x, int64_t N, void* stream) {
  if (!ctx || !X || !x || S <= 0 || T <= 0 || N <= 0) return GSS_EINVAL;
  if (n_fft != kN || hop != kHop) return GSS_EUNSUPPORTED;
  if ((N + hop - 1) / hop + 3 != T) return GSS_EINVAL;
  if (S > 65535) return GSS_EUNSUPPORTED;                  // (a limit of the call, not of the kernel)
  if (hipSetDevice(ctx->device) != hipSuccess) return GSS_EHIP;
  if ((long)S * ((T + 7) / 8) > 0x7fffffffL) return GSS_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  const float2* table = nullptr;
  int rc = get_twiddles(ctx, st, &table);
  if (rc != GSS_OK) return rc;
  // Output over the input: workgroups write samples while others still read frames, so these are read from a copy.
  const long n_spec = (long)S * kBins * T;
  const uintptr_t in0 = (uintptr_t)X, in1 = in0 + n_spec * sizeof(float2), out0 = (uintptr_t)x, out1 = out0 + (size_t)S * N * sizeof(float);
  if (in0 < out1 && out0 < in1) {
    rc = gss_ensure_scratch(ctx, n_spec * sizeof(float2));
    if (rc != GSS_OK) return rc;
    hipLaunchKernelGGL(copy_spectrum_kernel, dim3(ctx->num_cu * 8), dim3(256), 0, st, (const float2*)X, (float2*)ctx->scratch, n_spec);
    X = (const float*)ctx->scratch;
  }
  const IstftPlan p = plan_istft(S, T, ctx->num_cu);
  const long wgs = S * p.per_seg;
  const long grid = (wgs + kXcds - 1) / kXcds * kXcds;
  if (grid > 0x7fffffffL) return GSS_EUNSUPPORTED;
  hipLaunchKernelGGL((p.waves == 8 ? istft_kernel<8> : istft_kernel<16>), dim3((unsigned)grid), dim3(64 * p.waves), 0, st, (const float2*)X, x,
                     table, (long)N, T, p.steps, wgs);
  return hipGetLastError() == hipSuccess ? GSS_OK : GSS_EHIP;
}
