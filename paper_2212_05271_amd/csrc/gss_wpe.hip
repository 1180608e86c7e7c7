// WPE dereverberation (arXiv 2212.05271, Section 2.1: the late reverberation X^tail of the signal model is
// estimated with the weighted-prediction-error algorithm of the works cited there and subtracted) for gfx950.
//
// Per (segment, frequency), with ytilde_t the stack of the L delayed observations y_{t-Delta} .. y_{t-Delta-L+1}
// (N = D L components, component tau*D + d = y_{t-Delta-tau, d}) and x = y at the start, each iteration is
//
//   power  : lambda_t = mean_d |x_{t,d}|^2, floored at 1e-10 of its maximum over the segment's frames
//   cov    : R = sum_t ytilde_t ytilde_t^H / lambda_t  (N x N),  P = sum_t ytilde_t y_t^H / lambda_t  (N x D),
//            fp64 partial sums per chunk of frames
//   solve  : R += 1e-10 tr(R)/N I,  G = R^-1 P
//   apply  : x_t = y_t - G^H ytilde_t  (and lambda for the next iteration, or the complex64 output)
//
// R and P are accumulated on the fp64 matrix cores.  Everything up to the output is fp64: R is built from strongly
// correlated delayed copies of one signal and the solve amplifies rounding errors of the sums by its condition number.
#include "gss_internal.h"

#include "gss_device.h"

namespace {

constexpr int kWpeThreads = 256;

// Staging loop of a workgroup: elements e = first, first + stride, ... below n; load(e) fetches one from memory,
// store(e, v) puts it where it belongs (LDS).  BATCH loads are issued before the first of them is stored: written
// as a plain loop, each element waits out a full memory latency before the next load goes out.
template <int BATCH, class V, class Load, class Store>
__device__ __forceinline__ void staged_copy(int first, int n, int stride, Load load, Store store) {
  for (int e0 = first; e0 < n; e0 += BATCH * stride) {
    V v[BATCH];
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int e = e0 + u * stride;
      v[u] = V{};
      if (e < n) v[u] = load(e);
    }
#pragma unroll
    for (int u = 0; u < BATCH; ++u) {
      const int e = e0 + u * stride;
      if (e < n) store(e, v[u]);
    }
  }
}

constexpr int kWpeTile = 64;                  // frames per LDS window of the covariance kernel
constexpr double kWpeEpsPowerRel = 1e-10;
constexpr double kWpeLoadRel = 1e-10;

__device__ inline int clamp_T(const int32_t* T_len, int s, int Tmax) {
  int T = T_len ? T_len[s] : Tmax;
  return T < 0 ? 0 : (T > Tmax ? Tmax : T);
}

// Maximum of lam[0..T) over a workgroup (every thread gets it).  `red` holds one double per wavefront.
__device__ inline double block_max(const double* __restrict__ lam, int T, double* red) {
  double m = 0.0;
  for (int t = threadIdx.x; t < T; t += blockDim.x) m = fmax(m, lam[t]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
  const int wave = threadIdx.x / kWave;
  if ((threadIdx.x & (kWave - 1)) == 0) red[wave] = m;
  __syncthreads();
  double r = 0.0;
  for (int w = 0; w < (int)(blockDim.x / kWave); ++w) r = fmax(r, red[w]);
  __syncthreads();
  return r;
}

// Frame kernels (power, apply) run one workgroup per block of 256 frames of a (segment, frequency) row.
// Workgroups are dealt to the 8 accelerator dies round-robin by their index; xcd_block() turns the index into
// the logical block so that consecutive logical blocks (the blocks of one row, which share the row's
// prediction coefficients and the frames at their common edge) run on the same die and meet in its L2.
// The grid has 8 * ceil(n / 8) workgroups; the surplus ones get an index >= n and leave.
__device__ __forceinline__ long xcd_block(unsigned b, long per_xcd) { return (long)(b & 7u) * per_xcd + (long)(b >> 3); }

// lambda of the observation itself (first iteration).  The block's frames are read as one contiguous run
// (coalesced), |y|^2 per component goes to LDS, then thread = frame sums its D values in channel order.
// fb = frames per block (256 for D <= kPowerMaxD, 64 for larger arrays: fb * (D | 1) doubles of LDS).
constexpr int kPowerMaxD = 8;
__global__ __launch_bounds__(kWpeThreads) void wpe_power_kernel(const float2* __restrict__ Y, const int32_t* __restrict__ T_len,
                                                                double* __restrict__ lam, int F, int Tmax, int D,
                                                                int blocks_per_sf, long n_blocks, long per_xcd, int fb) {
  __shared__ double sP[kWpeThreads * (kPowerMaxD + 1)];
  const long blk = xcd_block(blockIdx.x, per_xcd);
  if (blk >= n_blocks) return;
  const long sf = blk / blocks_per_sf;
  const int t0 = (int)(blk % blocks_per_sf) * fb;
  const int T = clamp_T(T_len, (int)(sf / F), Tmax);
  const int pitch = D | 1;                                // odd: the frames' rows start in different banks
  const float2* __restrict__ Yblk = Y + (sf * Tmax + t0) * D;
  const int n_valid = (T - t0 < fb ? (T - t0 > 0 ? T - t0 : 0) : fb) * D;
  staged_copy<4, float2>(
      threadIdx.x, fb * D, kWpeThreads,
      [&](int e) { return e < n_valid ? Yblk[e] : make_float2(0.f, 0.f); },
      [&](int e, float2 v) {
        const int r = e / D, d = e - r * D;
        const double re = v.x, im = v.y;
        sP[r * pitch + d] = re * re + im * im;
      });
  __syncthreads();
  const int t = t0 + threadIdx.x;
  if ((int)threadIdx.x >= fb || t >= Tmax) return;
  double p = 0.0;
  for (int d = 0; d < D; ++d) p += sP[threadIdx.x * pitch + d];
  lam[sf * Tmax + t] = p / (double)D;
}

// Tiles of the augmented matrix [R | P] (N rows of N + D entries): 16 x 16 complex tiles, nt = ceil(N / 16) tile rows;
// row p holds the tiles of R from the diagonal on (columns p .. nt - 1; R is Hermitian) and then the ntd = ceil(D / 16)
// tiles of P (columns nt .. nt + ntd - 1).  A tile is stored as 256 double2 in the order in which the lanes of a
// wavefront hold it: entry (i, j) at 16 i + j.
typedef double double4v __attribute__((ext_vector_type(4)));
constexpr int kTileEntries = 256;
__host__ __device__ constexpr int wpe_tile_base(int p, int nt, int ntd) { return p * (nt + ntd) - p * (p - 1) / 2; }
__host__ __device__ constexpr int wpe_num_tiles(int nt, int ntd) { return wpe_tile_base(nt, nt, ntd); }

// D += A B of 16 x 4 and 4 x 16 doubles.  Lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and D[l / 16 + 4 v][l % 16]
// for v = 0..3: entry v of a tile's lane is entry 64 v + l of the tile's storage.
__device__ __forceinline__ double4v mfma_f64(double a, double b, double4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// LDS addresses as plain numbers: a read at a register plus a constant number of elements.
typedef double double2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned lds_address(const void* p) {
  unsigned a = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
  asm("" : "+v"(a));
  return a;
}
template <class V>
__device__ __forceinline__ V lds_at(unsigned address, int elem) {
  return ((const __attribute__((address_space(3))) V*)(uintptr_t)address)[elem];
}

// Covariance accumulation on the fp64 matrix cores.  A workgroup takes a chunk of 64-frame windows of one (segment,
// frequency).  Per window the frames t0-Delta-L+1 .. t0+63 are staged in LDS, converted to fp64 once, P >= D values
// apart: component n = tau D + d of ytilde_t is value d of row t - Delta - tau, so a lane's operand is at a position of
// its own plus a multiple of the frame.  A wavefront owns TPW tiles and adds, four frames at a time, the tile products
// sum_t (w_t a_i(t)) conj(b_j(t)).  The complex product takes three real ones, S1 = sum w Re a Re b,
// S2 = sum w Im a Im b and S3 = sum w (Re a + Im a)(Re b - Im b): the real part is S1 + S2, the imaginary part
// S3 - S1 + S2.  Lanes of rows or columns >= N (or >= D) repeat the last one; nothing uses their results.
// Few tiles (small D * taps): `split` wavefronts share their tiles, each takes a part of the window's frames; their sums
// meet in LDS at the end.  Many tiles (large arrays): G workgroups per chunk (blockIdx.x = chunk slot * G + g).
// part[(chunk slot * tiles + tile) * 256 ..]: the tile's entries.
//
// Bound: the fp64 matrix rate.  Vector instructions do not run beside a fp64 matrix instruction of the same SIMD (busy
// times of the two add up), so the loop is written for few of them: Re - Im is kept in LDS beside the value, the
// frame pitch is a compile-time constant (operand addresses are one register per tile plus constant offsets for four
// steps), and the weighted left operand is formed once per tile row.  Measured, 10 taps: 513 x 1560 x 8 440 us (vector
// FMAs on 4 x 4 blocks: 639 us), 513 x 1500 x 24 3.25 ms (5.42 ms); the matrix cores are busy 82 % of the time.
template <int P, int TPW>
__global__ __launch_bounds__(kWpeThreads, 2) void wpe_cov_kernel(const float2* __restrict__ Y, const int32_t* __restrict__ T_len,
                                                                 const double* __restrict__ lam, double2* __restrict__ part,
                                                                 int F, int Tmax, int D, int taps, int delay, ChunkMap cmap,
                                                                 int G, int split) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  const int past = delay + taps - 1;
  const int win_frames = kWpeTile + past;
  double2* __restrict__ sWin = reinterpret_cast<double2*>(lds_raw);                    // [win_frames][P]
  double* __restrict__ sDif = reinterpret_cast<double*>(sWin + (size_t)win_frames * P);   // [win_frames][P]: re - im
  double* __restrict__ sWt = sDif + (size_t)win_frames * P;                               // [kWpeTile]
  double* __restrict__ sRed = sWt + kWpeTile;

  const unsigned slot = blockIdx.x / (unsigned)G;
  const int g = (int)(blockIdx.x % (unsigned)G);
  long sf;
  int chunk, tpc;
  chunk_decode(cmap, slot, sf, chunk, tpc);
  const int T = clamp_T(T_len, (int)(sf / F), Tmax);
  const int N = D * taps;
  const int nt = (N + 15) / 16, ntd = (D + 15) / 16;
  const int n_tiles = wpe_num_tiles(nt, ntd);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int part_of = wave % split;                      // which of the wavefronts on the same tiles
  const int first = (g * (kWpeThreads / kWave / split) + wave / split) * TPW;   // the wavefront's first tile
  const int steps = kWpeTile / 4 / split;                // groups of four frames per window (4, 8 or 16)

  // Positions of the tiles' operands in the window: lane (k, i) = (l / 16, l % 16) holds component i of the tile at
  // frame k of the group.  The TPW consecutive tiles of a wavefront lie in at most two tile rows (wpe_tiling_fits): the
  // first n0 of them in row p0, the others in the next.
  const int k4 = lane >> 4, li = lane & 15;
  int apos0, apos1, n0 = TPW;
  int bpos[TPW];
  {
    const int f0 = past + 4 * steps * part_of + k4;      // window row of the lane's first frame
    auto delayed = [&](int tile) {
      int n = 16 * tile + li;
      n = n < N ? n : N - 1;
      const int tau = n / D;
      return (f0 - delay - tau) * P + (n - tau * D);
    };
    auto current = [&](int tile) {
      const int d = 16 * tile + li;
      return f0 * P + (d < D ? d : D - 1);
    };
    int p = 0;
    while (p + 1 < nt && wpe_tile_base(p + 1, nt, ntd) <= first) ++p;
    int c = p + first - wpe_tile_base(p, nt, ntd);
    if (c >= nt + ntd) c = p;                            // (surplus tiles repeat the last row: in bounds, not stored)
    apos0 = delayed(p);
    apos1 = apos0;
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      if (c >= nt + ntd) {                               // the next row of tiles
        p = p + 1 < nt ? p + 1 : p;
        c = p;
        n0 = n0 == TPW ? q : n0;
        apos1 = delayed(p);
      }
      bpos[q] = c < nt ? delayed(c) : current(c - nt);
      ++c;
    }
  }
  n0 = __builtin_amdgcn_readfirstlane(n0);

  const double* __restrict__ lrow = lam + sf * Tmax;
  const double floor_l = kWpeEpsPowerRel * block_max(lrow, T, sRed);
  const float2* __restrict__ Yrow = Y + sf * (long)Tmax * D;

  double4v s1[TPW], s2[TPW], s3[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    s1[q] = double4v{0.0, 0.0, 0.0, 0.0};
    s2[q] = double4v{0.0, 0.0, 0.0, 0.0};
    s3[q] = double4v{0.0, 0.0, 0.0, 0.0};
  }

  const int tile_end = (T + kWpeTile - 1) / kWpeTile;
  const int tile_lo = chunk * tpc;
  const int tile_hi = tile_lo + tpc < tile_end ? tile_lo + tpc : tile_end;
  // where the thread's first value of a window goes, and the step to its next one (kWpeThreads values further on)
  const int r0 = (int)threadIdx.x / D, d0 = (int)threadIdx.x - r0 * D;
  const int step_d = kWpeThreads % D, step_pos = kWpeThreads / D * P + step_d;
  // The power of the thread's frame of a window, requested one window ahead, and with it one value of every 128-byte line
  // of the window's new frames, so that the staging loads find them in cache: the wavefronts of a compute unit tend to
  // reach the staging together, and nothing hides a memory latency there.
  auto power_of = [&](int t) { return threadIdx.x < kWpeTile && t < T ? lrow[t] : 0.0; };
  double l_next = tile_lo < tile_hi ? power_of(tile_lo * kWpeTile + (int)threadIdx.x) : 0.0;
  for (int tile = tile_lo; tile < tile_hi; ++tile) {
    const int t0 = tile * kWpeTile;
    // The window's frames and the next window's new ones, as far as they exist, are one run of n_run values.  Its start
    // takes 64 bits (a row may be longer than 2^32 values), positions inside it 32 (those before it wrap around).
    const int t_run = t0 > past ? t0 - past : 0;
    const char* __restrict__ Yrun = reinterpret_cast<const char*>(Yrow + (long)t_run * D);
    const unsigned n_run = (unsigned)((t0 - t_run + (T - t0 < 2 * kWpeTile ? T - t0 : 2 * kWpeTile)) * D);
    __syncthreads();                                    // the previous tile's window is no longer read
    {
      const unsigned g0 = (unsigned)((t0 - past - t_run) * D);
      int d = d0, pos = r0 * P + d0;
      staged_copy<8, float2>(
          threadIdx.x, win_frames * D, kWpeThreads,
          [&](int m) {
            const unsigned e = g0 + (unsigned)m;
            return e < n_run ? *reinterpret_cast<const float2*>(Yrun + e * 8u) : make_float2(0.f, 0.f);
          },
          [&](int, float2 v) {
            const double re = v.x, im = v.y;              // converted once here, not at every use
            sWin[pos] = make_double2(re, im);
            sDif[pos] = re - im;
            d += step_d;
            pos += step_pos;
            if (d >= D) {
              d -= D;
              pos += P - D;
            }
          });
    }
    if (threadIdx.x < kWpeTile) {
      double w = 0.0;
      if (t0 + (int)threadIdx.x < T) {
        const double l = fmax(l_next, floor_l);
        w = l > 0.0 ? 1.0 / l : 0.0;                   // all-zero bin: no weight, R = 0, bin left unchanged
      }
      sWt[threadIdx.x] = w;
    }
    l_next = power_of(t0 + kWpeTile + (int)threadIdx.x);
    float touched = 0.f;
    {
      const unsigned e = (unsigned)((t0 + kWpeTile - t_run) * D) + threadIdx.x * 16u;
      if ((int)threadIdx.x < kWpeTile * D / 16 && e < n_run) touched = *reinterpret_cast<const float*>(Yrun + e * 8u);
    }
    __syncthreads();
    // LDS addresses the compiler cannot take apart again (it would add the base at every use)
    unsigned a0 = lds_address(sWin + apos0), a1 = lds_address(sWin + apos1), aw = lds_address(sWt + 4 * steps * part_of + k4);
    unsigned ab[TPW], ad[TPW];
#pragma unroll
    for (int q = 0; q < TPW; ++q) {
      ab[q] = lds_address(sWin + bpos[q]);
      ad[q] = lds_address(sDif + bpos[q]);
    }
    // The next operands are requested between the matrix instructions of the current ones: two wavefronts that share a SIMD run
    // in step, so reads issued in a block of their own would leave the matrix core idle in both.  (Behind the last frames: the
    // same again.)
    if constexpr (TPW >= 4) {
      // Sixteen frames (four steps) at a time, tile by tile: twelve products in a row on the same three accumulators.  A product
      // on one of many accumulators that take turns starts six cycles later (72 instead of 66 cycles per product in a
      // micro-benchmark of 15 accumulators): covariance kernel 450 -> 432 us at 513 x 1560 x 8, 3.25 -> 3.10 ms at
      // 513 x 1500 x 24.  Up to three tiles the operands of four steps cost the third wavefront of a SIMD, and the form
      // below is 2 % faster.
      double w[4], ar[4], ai[4], as[4];
      double2v x[4], b[2][4];
      double bd[2][4];
      auto fetch_x = [&](auto UI, unsigned address) { x[UI.value] = lds_at<double2v>(address, 4 * P * UI.value); };
      auto fetch_w = [&](auto UI) { w[UI.value] = lds_at<double>(aw, 4 * UI.value); };
      auto fetch_right = [&](auto SLOT, auto QI, auto UI) {
        constexpr int q = decltype(QI)::value, slot = decltype(SLOT)::value, u = decltype(UI)::value;
        b[slot][u] = lds_at<double2v>(ab[q], 4 * P * u);
        bd[slot][u] = lds_at<double>(ad[q], 4 * P * u);
      };
      auto form_left = [&]() {
  #pragma unroll
        for (int u = 0; u < 4; ++u) {
          ar[u] = w[u] * x[u].x;
          ai[u] = w[u] * x[u].y;
          as[u] = ar[u] + ai[u];
        }
      };
      static_for<0, 4>([&](auto UI) {
        fetch_w(UI);
        fetch_x(UI, a0);
        fetch_right(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, UI);
      });
      auto sixteen = [&](int s, auto PARITY) {
        const unsigned on = s + 4 < steps ? 1u : 0u;
        form_left();
        static_for<0, TPW>([&](auto QI) {
          constexpr int q = QI.value, slot = (q + decltype(PARITY)::value * TPW) & 1;
          constexpr std::integral_constant<int, slot ^ 1> other{};
          constexpr std::integral_constant<int, q + 1 < TPW ? q + 1 : 0> next{};
          int row1 = n0;
          asm volatile("" : "+s"(row1));                    // (tested anew: kept as booleans the tests cost vector instructions)
          if (q > 0 && q == row1) form_left();              // (wave-uniform) the next tile row's operand
          ab[q] += on * 16 * P * sizeof(double2);
          ad[q] += on * 16 * P * sizeof(double);
          if constexpr (q + 1 == TPW) {
            aw += on * 16 * sizeof(double);
            a0 += on * 16 * P * sizeof(double2);
          }
          static_for<0, 4>([&](auto UI) {
            constexpr int u = UI.value;
            s1[q] = mfma_f64(ar[u], b[slot][u].x, s1[q]);
            s2[q] = mfma_f64(ai[u], b[slot][u].y, s2[q]);
            s3[q] = mfma_f64(as[u], bd[slot][u], s3[q]);
            if constexpr (q == 0) fetch_x(UI, a1);
            if constexpr (q + 1 == TPW) {
              fetch_w(UI);
              fetch_x(UI, a0);
            }
            fetch_right(other, next, UI);
            __builtin_amdgcn_sched_barrier(0);
          });
          if constexpr (q == 0) a1 += on * 16 * P * sizeof(double2);
        });
      };
      for (int s = 0; s < steps; s += 8) {
        sixteen(s, std::integral_constant<int, 0>{});
        if (s + 4 < steps) sixteen(s + 4, std::integral_constant<int, 1>{});
      }
    } else {
      // Four frames at a time, the tiles in turn, each tile's next operands as soon as its own are used.
      double w[2];
      double2v x0[2], x1[2], b[TPW];
      double bd[TPW];
      auto fetch_row = [&](auto UI) {
        constexpr int u = decltype(UI)::value;
        w[u & 1] = lds_at<double>(aw, 4 * u);
        x0[u & 1] = lds_at<double2v>(a0, 4 * P * u);
        x1[u & 1] = lds_at<double2v>(a1, 4 * P * u);
      };
      auto fetch_col = [&](auto QI, auto UI) {
        constexpr int q = decltype(QI)::value, u = decltype(UI)::value;
        b[q] = lds_at<double2v>(ab[q], 4 * P * u);
        bd[q] = lds_at<double>(ad[q], 4 * P * u);
      };
      fetch_row(std::integral_constant<int, 0>{});
      static_for<0, TPW>([&](auto QI) { fetch_col(QI, std::integral_constant<int, 0>{}); });
      for (int s = 0; s < steps; s += 4) {
        const unsigned on = s + 4 < steps ? 1u : 0u;
        static_for<0, 4>([&](auto UI) {
          constexpr int u = UI.value;
          constexpr std::integral_constant<int, (u + 1) & 3> next{};
          double ar = w[u & 1] * x0[u & 1].x, ai = w[u & 1] * x0[u & 1].y, as = ar + ai;
          double w1 = w[u & 1];
          const double2v y1 = x1[u & 1];
          static_for<0, TPW>([&](auto QI) {
            constexpr int q = QI.value;
            int row1 = n0;
            asm volatile("" : "+s"(row1));                // (tested anew: kept as booleans the tests cost vector instructions)
            if (q > 0 && q == row1) {                     // (wave-uniform) the next tile row's operand
              asm volatile("" : "+v"(w1));                // (keeps this a branch: six selects at every tile otherwise)
              ar = w1 * y1.x;
              ai = w1 * y1.y;
              as = ar + ai;
            }
            s1[q] = mfma_f64(ar, b[q].x, s1[q]);
            s2[q] = mfma_f64(ai, b[q].y, s2[q]);
            s3[q] = mfma_f64(as, bd[q], s3[q]);
            if constexpr (u == 3) {
              ab[q] += on * 16 * P * sizeof(double2);
              ad[q] += on * 16 * P * sizeof(double);
            }
            fetch_col(QI, next);
            if constexpr (q == 0) {
              if constexpr (u == 3) {
                aw += on * 16 * sizeof(double);
                a0 += on * 16 * P * sizeof(double2);
                a1 += on * 16 * P * sizeof(double2);
              }
              fetch_row(next);
            }
            __builtin_amdgcn_sched_barrier(0);
          });
        });
      }
    }
    asm volatile("" ::"v"(touched));                    // (the load above is not dropped)
  }
  double2* __restrict__ out = part + (size_t)slot * n_tiles * kTileEntries + lane;
  // A tile of every wavefront that is not the first on its tiles, in the window's place (kWpeCovSumBytes): one set of tiles
  // per chunk is written, whatever `split` is.
  double2* __restrict__ sSum = reinterpret_cast<double2*>(lds_raw) + lane;
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    double2 x[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = make_double2(s1[q][v] + s2[q][v], (s3[q][v] - s1[q][v]) + s2[q][v]);
    if (split > 1) {
      __syncthreads();                                  // the window, or the tile before, is no longer read
      if (part_of > 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) sSum[(wave - 1 - wave / split) * kTileEntries + v * kWave] = x[v];
      }
      __syncthreads();
      if (part_of == 0)
        for (int u = 0; u < split - 1; ++u) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const double2 y = sSum[(wave / split * (split - 1) + u) * kTileEntries + v * kWave];
            x[v].x += y.x;
            x[v].y += y.y;
          }
        }
    }
    if (part_of == 0 && first + q < n_tiles) {
#pragma unroll
      for (int v = 0; v < 4; ++v) out[(size_t)(first + q) * kTileEntries + v * kWave] = x[v];
    }
  }
}

// LDS in which the wavefronts that share their tiles add them up: one tile of at most 3 of the 4.
constexpr int kWpeCovSumBytes = 3 * kTileEntries * (int)sizeof(double2);

// Workgroups per compute unit that the chunks are planned for: two wavefronts per SIMD keep its matrix core busy, and
// finer chunks would only add partial sums (more workgroups may be resident).
constexpr int kWpeCovPerCu = 2;

// Tiles per wavefront (2..5), wavefronts that share the same tiles, workgroups per chunk.
struct WpeTiling { int tpw, split, groups; };
// Chosen by the time of one 64-frame window: TPW tiles of 48 matrix instructions of 64 cycles each in every wavefront,
// divided among the wavefronts that share them, plus about 1500 cycles of staging, for each of the groups.
constexpr WpeTiling wpe_tiling(int n_tiles) {
  WpeTiling best{5, 1, 1};
  long best_cost = -1;
  for (int tpw = 5; tpw >= 2; --tpw) {
    const int waves = (n_tiles + tpw - 1) / tpw;
    const int split = waves == 1 ? 4 : waves == 2 ? 2 : 1;
    const int groups = waves <= 2 ? 1 : (waves + 3) / 4;
    const long cost = (long)groups * (tpw * 3072 / split + 1500);
    if (best_cost < 0 || cost < best_cost) {
      best_cost = cost;
      best = WpeTiling{tpw, split, groups};
    }
  }
  return best;
}
// What the covariance kernel takes for granted of every legal system (nt tile rows, ntd column tiles of P; D > 16 has
// nt >= 2): no wavefront's tiles touch three tile rows, and with two column tiles there are three tiles per wavefront or
// more.  The rows get shorter by one down to 1 + ntd tiles, so five tiles from the last one of a row of 4 on (ntd = 1) would
// touch three; a wavefront starts at a multiple of 5, and none of the sizes puts that tile there.
constexpr bool wpe_tiling_fits() {
  for (int ntd = 1; ntd <= (GSS_WPE_LARGE_MAX_D + 15) / 16; ++ntd)
    for (int nt = ntd; nt <= (GSS_WPE_LARGE_MAX_N + 15) / 16; ++nt) {
      const int n_tiles = wpe_num_tiles(nt, ntd), tpw = wpe_tiling(n_tiles).tpw;
      if (tpw < 1 + ntd) return false;
      for (int first = 0, p = 0; first < n_tiles; first += tpw) {
        while (p + 1 < nt && wpe_tile_base(p + 1, nt, ntd) <= first) ++p;
        const int last = first + tpw < n_tiles ? first + tpw - 1 : n_tiles - 1;
        if (p + 2 < nt && wpe_tile_base(p + 2, nt, ntd) <= last) return false;
      }
    }
  return true;
}
static_assert(wpe_tiling_fits(), "a wavefront of the covariance kernel has one left operand for each of two tile rows");

typedef void (*wpe_cov_fn)(const float2*, const int32_t*, const double*, double2*, int, int, int, int, int, ChunkMap, int, int);
template <int P>
inline wpe_cov_fn wpe_cov_tpw(int tpw) {
  if constexpr (P <= 16)
    if (tpw == 2) return wpe_cov_kernel<P, 2>;
  switch (tpw) {
    case 3: return wpe_cov_kernel<P, 3>;
    case 4: return wpe_cov_kernel<P, 4>;
    default: return wpe_cov_kernel<P, 5>;
  }
}
// The kernel for D channels and its frame pitch.
inline wpe_cov_fn wpe_cov_of(int D, int tpw, int& pitch) {
  pitch = D <= 2 ? 2 : D <= 4 ? 4 : (D + 7) / 8 * 8;
  switch (pitch) {
    case 2: return wpe_cov_tpw<2>(tpw);
    case 4: return wpe_cov_tpw<4>(tpw);
    case 8: return wpe_cov_tpw<8>(tpw);
    case 16: return wpe_cov_tpw<16>(tpw);
    case 24: return wpe_cov_tpw<24>(tpw);
    default: return wpe_cov_tpw<32>(tpw);
  }
}
inline int wpe_cov_lds(int pitch, int taps, int delay, int split) {
  const int window =
      (kWpeTile + delay + taps - 1) * pitch * 3 * (int)sizeof(double) + (kWpeTile + kWpeThreads / kWave) * (int)sizeof(double);
  return split > 1 && window < kWpeCovSumBytes ? kWpeCovSumBytes : window;
}
constexpr int kWpeLdsLimit = 160 * 1024;      // LDS of a compute unit
// Largest window accepted (64 KB for the values and the weights).
inline bool wpe_window_fits(int D, int taps, int delay) {
  return ((kWpeTile + delay + taps) * D + 8) * (int)sizeof(double2) + (kWpeTile + kWpeThreads / kWave) * (int)sizeof(double) <=
         64 * 1024;
}

// ----------------------------------------------------------------------------------------------
// Solve R G = P (R loaded on its diagonal), one workgroup of four wavefronts per (segment, frequency).
//
// Blocked Cholesky factorisation R = U^H U on the 16 x 16 tiles, left-looking by tile rows, the tiles of P carried along
// as further columns: for tile row p
//   S(p, i) = A(p, i) - sum_{j < p} U(j, p)^H U(j, i)   for every column i >= p,
//   V = U(p, p)^-1 from S(p, p) = U(p, p)^H U(p, p)     (one wavefront),
//   U(p, i) = V^H S(p, i)                               for i > p,
// which leaves Z = U^-H P in the columns of P; then the back substitution G(p) = V_p Z(p), Z(i) -= U(i, p) G(p) for
// i < p.  A tile in a wavefront's registers, as the matrix instructions leave it (entry (l / 16 + 4 v, l % 16) in lane l),
// is at once the left operand of X^H Y and the right operand of X Y, so the factorisation needs no transposition; the
// back substitution reads the tiles transposed.
// Without pivoting (R is Hermitian positive definite; a pivot <= 1e-300 is floored and flagged).  Rows and columns >= N
// of the last tile row are the identity's.
// part: the covariance kernel's tiles; chunks are added up as they are read, and the first chunk's tiles are overwritten (a
// workgroup's tiles stay in L2).  Out: the coefficients as the apply kernels read them: rt > 0 tiles of 8 channels:
// wpe_apply_coef; rt = 0: Gc[sf][a][d] = conj(G[a][d]).
//
// Bound: for small systems the chain of the 16 sweeps per tile row (LDS round trip and reciprocal, about 400 cycles each),
// for large ones the tile products.  Three workgroups per compute unit (two: 40 % more time), which leaves 168 registers: 16
// vector registers (60 bytes per lane) and 42 scalar ones are spilled.  Measured, 513 bins: 63 us for
// 80 unknowns and 8 right-hand sides, 0.79 ms for 240 and 24 (assembled matrix and Gauss-Jordan in the registers of a
// workgroup: 228 us; 8-column Cholesky in global memory: 4.0 ms).
// ----------------------------------------------------------------------------------------------
constexpr int kSolveThreads = 256;

constexpr int kApplyFewMaxD = 4;              // channels up to which the prediction is applied by the vector kernel
__host__ __device__ inline int wpe_apply_groups(int N) { return (N + 3) / 4; }        // groups of four components
// Entry of the coefficient array for component n, channel d and part (0: the row that yields Re x_d, 1: Im x_d).
__host__ __device__ inline int wpe_apply_coef(int n, int d, int part, int rt) {
  return ((n >> 2) * rt + (d >> 3)) * kWave + (n & 3) * 16 + (d & 3) + 8 * ((d >> 2) & 1) + 4 * part;
}

constexpr int kSolveMaxSlots = 4;             // partial sums per problem that the solve kernel adds up itself

// Problems with many partial sums (the ones left over after the last full round of workgroups are cut into small chunks):
// their tiles are added up here, one workgroup per tile, into the first chunk's.  (One workgroup of the solve kernel
// would read all of them alone: 24 chunks of the last of 513 bins took 1.4 ms at 24 channels, everything else 0.65 ms.)
__global__ __launch_bounds__(kTileEntries) void wpe_sum_chunks_kernel(double2* __restrict__ part, ChunkMap cmap, long sf0,
                                                                      int n_tiles) {
  const long sf = sf0 + blockIdx.x / (unsigned)n_tiles;
  int count;
  const long slot0 = chunk_base(cmap, sf, count);
  const size_t stride = (size_t)n_tiles * kTileEntries;
  double2* __restrict__ t = part + (size_t)slot0 * stride + (size_t)(blockIdx.x % (unsigned)n_tiles) * kTileEntries + threadIdx.x;
  double2 sum = t[0];
  for (int q0 = 1; q0 < count; q0 += 4) {
    double2 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = q0 + u < count ? t[(q0 + u) * stride] : make_double2(0.0, 0.0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      sum.x += v[u].x;
      sum.y += v[u].y;
    }
  }
  t[0] = sum;
}

struct CTile {                                            // the lane's entries of a complex tile
  double4v re, im;
};
__device__ __forceinline__ CTile tile_load(const double2* __restrict__ t, int lane) {
  CTile c;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double2 x = t[lane + kWave * v];
    c.re[v] = x.x;
    c.im[v] = x.y;
  }
  return c;
}
__device__ __forceinline__ CTile tile_load_transposed(const double2* __restrict__ t, int lane) {
  CTile c;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double2 x = t[16 * (lane & 15) + (lane >> 4) + 4 * v];
    c.re[v] = x.x;
    c.im[v] = x.y;
  }
  return c;
}
__device__ __forceinline__ void tile_store(double2* __restrict__ t, const CTile& c, int lane) {
#pragma unroll
  for (int v = 0; v < 4; ++v) t[lane + kWave * v] = make_double2(c.re[v], c.im[v]);
}
// s +- conj(x) y over the tiles' common rows (x as loaded: X^H Y)
template <bool SUB>
__device__ __forceinline__ void tile_xhy(CTile& s, const CTile& x, const CTile& y) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double xr = SUB ? -x.re[k] : x.re[k], xi = SUB ? -x.im[k] : x.im[k];
    s.re = mfma_f64(xr, y.re[k], s.re);
    s.im = mfma_f64(xr, y.im[k], s.im);
    s.re = mfma_f64(xi, y.im[k], s.re);
    s.im = mfma_f64(-xi, y.re[k], s.im);
  }
}
// s +- x y with x loaded transposed (X Y)
template <bool SUB>
__device__ __forceinline__ void tile_xy(CTile& s, const CTile& x, const CTile& y) {
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double xr = SUB ? -x.re[k] : x.re[k], xi = SUB ? -x.im[k] : x.im[k];
    s.re = mfma_f64(xr, y.re[k], s.re);
    s.im = mfma_f64(xr, y.im[k], s.im);
    s.re = mfma_f64(-xi, y.im[k], s.re);
    s.im = mfma_f64(xi, y.re[k], s.im);
  }
}
__device__ __forceinline__ CTile tile_zero() {
  const double4v z = {0.0, 0.0, 0.0, 0.0};
  return CTile{z, z};
}

__global__ __launch_bounds__(kSolveThreads, 3) void wpe_solve_kernel(double2* __restrict__ part, double2* __restrict__ Gc,
                                                                     uint32_t* __restrict__ status, int D, int taps,
                                                                     ChunkMap cmap, int rt) {
  __shared__ double2 sG[2][(GSS_WPE_LARGE_MAX_D + 15) / 16][kTileEntries];
  __shared__ double2 sRow[16];
  __shared__ double sPiv[16];
  __shared__ double sRed[kSolveThreads / kWave];
  const long sf = blockIdx.x;
  const int N = D * taps;
  const int nt = (N + 15) / 16, ntd = (D + 15) / 16, nc = nt + ntd;
  const int n_tiles = wpe_num_tiles(nt, ntd);
  int count;
  const long slot0 = chunk_base(cmap, sf, count);
  if (count > kSolveMaxSlots) count = 1;                   // (wpe_sum_chunks_kernel has added them up)
  double2* __restrict__ A = part + (size_t)slot0 * n_tiles * kTileEntries;       // the tiles of the first chunk
  const size_t slot_stride = (size_t)n_tiles * kTileEntries;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int k4 = lane >> 4, li = lane & 15;
  const int n_coef = rt ? wpe_apply_groups(N) * rt * kWave : N * D;
  double2* __restrict__ out = Gc + sf * (long)n_coef;
  // tile (p, i) of [A | P], later [U | Z]
  auto tile_at = [&](int p, int i) { return A + (size_t)(wpe_tile_base(p, nt, ntd) + i - p) * kTileEntries; };

  // trace of R
  double tr = 0.0;
  for (int a = threadIdx.x; a < N; a += kSolveThreads) {
    const double2* __restrict__ t = tile_at(a >> 4, a >> 4) + 17 * (a & 15);
    for (int q = 0; q < count; ++q) tr += t[q * slot_stride].x;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) tr += __shfl_xor(tr, o);
  if (lane == 0) sRed[wave] = tr;
  __syncthreads();
  tr = 0.0;
#pragma unroll
  for (int w = 0; w < kSolveThreads / kWave; ++w) tr += sRed[w];
  if (!(tr > 0.0)) {                                       // no frame has a past (or silence): G = 0
    for (int e = threadIdx.x; e < n_coef; e += kSolveThreads) out[e] = make_double2(0.0, 0.0);
    return;
  }
  const double load = kWpeLoadRel * tr / (double)N;
  const double tiny = 1e-300;

  // A(p, i): the chunks' sum, loaded and completed to the identity
  auto load_a = [&](int p, int i) {
    CTile c = tile_load(tile_at(p, i), lane);
    for (int q = 1; q < count; ++q) {
      const CTile x = tile_load(tile_at(p, i) + q * slot_stride, lane);
      c.re += x.re;
      c.im += x.im;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * p + k4 + 4 * v, b = 16 * i + li;
      const bool in = a < N && (i >= nt || b < N);
      if (i == p && a == b) {
        c.re[v] = in ? c.re[v] + load : 1.0;
        c.im[v] = 0.0;
      } else if (!in) {
        c.re[v] = 0.0;
        c.im[v] = 0.0;
      }
    }
    return c;
  };
  // S[c] -= sum over j < n of U(j, p)^H U(j, i0 + c), c = 0 and 1 (PAIR: they share the left operands)
  auto update = [&](int p, int i0, int n, auto PAIR, CTile (&S)[2]) {
    constexpr bool pair = decltype(PAIR)::value;
    if (n <= 0) return;
    CTile x = tile_load(tile_at(0, p), lane), y0 = tile_load(tile_at(0, i0), lane), y1 = tile_zero();
    if constexpr (pair) y1 = tile_load(tile_at(0, i0 + 1), lane);
    for (int j = 0; j < n; ++j) {
      CTile xn = x, yn0 = y0, yn1 = y1;
      if (j + 1 < n) {                                    // the next operands are requested ahead
        xn = tile_load(tile_at(j + 1, p), lane);
        yn0 = tile_load(tile_at(j + 1, i0), lane);
        if constexpr (pair) yn1 = tile_load(tile_at(j + 1, i0 + 1), lane);
      }
      tile_xhy<true>(S[0], x, y0);
      if constexpr (pair) tile_xhy<true>(S[1], x, y1);
      x = xn;
      y0 = yn0;
      if constexpr (pair) y1 = yn1;
    }
  };
  constexpr std::integral_constant<bool, false> one{};
  constexpr std::integral_constant<bool, true> two{};

  CTile diag = tile_zero();                               // (wavefront 0) S(p, p)
  if (wave == 0) diag = load_a(0, 0);
  for (int p = 0; p < nt; ++p) {
    // Wavefront 0 factorises S(p, p); the others form S(p, i) for the columns behind the diagonal, and the next diagonal
    // tile up to the terms that exist already.  As far as the factorisation (about five tile products long) leaves
    // time, wavefront 0 takes columns too.
    const int m = nc - p - 1;
    int m0 = p > 0 ? (p * (m - 3) - 20) / (4 * p) : 0;
    m0 = m0 < 0 ? 0 : m0;
    int lo = nc - m0, hi = nc;
    if (wave > 0) {
      lo = p + 1 + (m - m0) * (wave - 1) / 3;
      hi = p + 1 + (m - m0) * wave / 3;
    }
    if (wave == 0) {
      CTile S = diag;
      // S = U^H U by elimination in place: after sweep r, row r of S is row r of the unscaled U from the diagonal on, and
      // the entries below the diagonal of columns <= r hold the inverse of the unit lower factor.  Row r goes through LDS;
      // column r is its conjugate.
      static_for<0, 16>([&](auto RI) {
        constexpr int r = RI.value, vr = r >> 2;
        if (k4 == (r & 3)) sRow[li] = make_double2(S.re[vr], S.im[vr]);
        wave_lds_sync();
        double piv = sRow[r].x;
        const double2 rj = sRow[li];
        double2 ri[4];
#pragma unroll
        for (int v = vr; v < 4; ++v) ri[v] = sRow[k4 + 4 * v];
        wave_lds_sync();
        if (!(piv > tiny)) {
          if (lane == 0) atomicOr(status, GSS_STATUS_NONPD_WPE);
          piv = tiny;
        }
        if (lane == 0) sPiv[r] = piv;
        const double inv = rcp_f64(piv);
        const double cr = rj.x * inv, ci = rj.y * inv;     // row r over the pivot
        const bool col = li == r;
#pragma unroll
        for (int v = vr; v < 4; ++v) {
          // rows below r: S(i, j) -= conj(S(r, i)) S(r, j) / pivot, and -conj(S(r, i)) / pivot in column r
          const double nr = col ? -inv * ri[v].x : fma(-ri[v].x, cr, fma(-ri[v].y, ci, S.re[v]));
          const double ni = col ? inv * ri[v].y : fma(-ri[v].x, ci, fma(ri[v].y, cr, S.im[v]));
          if (v > vr || k4 > (r & 3)) {
            S.re[v] = nr;
            S.im[v] = ni;
          }
        }
      });
      wave_lds_sync();
      // V = U^-1: the inverse of the unit lower factor, rows scaled by pivot^-1/2, conjugated and transposed
      double2* __restrict__ dst = tile_at(p, p);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = k4 + 4 * v;
        const double isq = 1.0 / sqrt(sPiv[i]);
        const double wr = li < i ? S.re[v] : li == i ? 1.0 : 0.0, wi = li < i ? S.im[v] : 0.0;
        dst[16 * li + i] = make_double2(wr * isq, -wi * isq);
      }
    }
    if (wave == 3 && p + 1 < nt) {
      CTile S[2] = {load_a(p + 1, p + 1), tile_zero()};
      update(p + 1, p + 1, p, one, S);
      tile_store(tile_at(p + 1, p + 1), S[0], lane);
    }
    for (int i = lo; i < hi; i += 2) {
      CTile S[2] = {load_a(p, i), tile_zero()};
      if (i + 1 < hi) {
        S[1] = load_a(p, i + 1);
        update(p, i, p, two, S);
        tile_store(tile_at(p, i + 1), S[1], lane);
      } else {
        update(p, i, p, one, S);
      }
      tile_store(tile_at(p, i), S[0], lane);
    }
    __syncthreads();
    {
      const CTile V = tile_load(tile_at(p, p), lane);
      const int i0 = p + 1 + wave;
      CTile S = i0 < nc ? tile_load(tile_at(p, i0), lane) : tile_zero();
      if (wave == 0 && p + 1 < nt) diag = tile_load(tile_at(p + 1, p + 1), lane);
      for (int i = i0; i < nc; i += 4) {
        CTile Sn = S;
        if (i + 4 < nc) Sn = tile_load(tile_at(p, i + 4), lane);
        CTile U = tile_zero();
        tile_xhy<false>(U, V, S);
        tile_store(tile_at(p, i), U, lane);
        if (i == p + 1 && i < nt) tile_xhy<true>(diag, U, U);   // (wavefront 0) the last term of the next diagonal tile
        S = Sn;
      }
    }
    __syncthreads();
  }

  // Back substitution.  Wavefront i mod 4 owns tile row i of Z: it subtracts U(i, p) G(p) for every p > i, and forms G(i) as
  // soon as the last of them is in; G goes to the others through LDS (two buffers, one barrier per tile row).
  auto finish = [&](int p, int c, const CTile& V, const CTile& Z) {
    CTile G = tile_zero();
    tile_xy<false>(G, V, Z);
    tile_store(sG[p & 1][c], G, lane);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * p + k4 + 4 * v, d = 16 * c + li;
      if (rt == 0) {
        if (a < N && d < D) out[a * D + d] = make_double2(G.re[v], -G.im[v]);
      } else if (a < 4 * wpe_apply_groups(N) && d < 8 * rt) {
        // Re x -= Re G Re ytilde + Im G Im ytilde, Im x -= Re G Im ytilde - Im G Re ytilde; zero for what is padding
        const bool in = a < N && d < D;
        const double gr = in ? G.re[v] : 0.0, gi = in ? G.im[v] : 0.0;
        out[wpe_apply_coef(a, d, 0, rt)] = make_double2(-gr, -gi);
        out[wpe_apply_coef(a, d, 1, rt)] = make_double2(gi, -gr);
      }
    }
  };
  if (wave == ((nt - 1) & 3)) {
    const CTile V = tile_load_transposed(tile_at(nt - 1, nt - 1), lane);
    for (int c = 0; c < ntd; ++c) finish(nt - 1, c, V, tile_load(tile_at(nt - 1, nt + c), lane));
  }
  __syncthreads();
  for (int p = nt - 1; p > 0; --p) {
    const int i0 = p - 1 - ((p - 1 - wave) & 3);          // the wavefront's last row above p (negative: none)
    for (int c = 0; c < ntd && i0 >= 0; ++c) {
      const CTile G = tile_load(sG[p & 1][c], lane);
      CTile V = tile_zero();
      if (i0 == p - 1) V = tile_load_transposed(tile_at(i0, i0), lane);
      CTile X = tile_load_transposed(tile_at(i0, p), lane), Z = tile_load(tile_at(i0, nt + c), lane);
      for (int i = i0; i >= 0; i -= 4) {
        CTile Xn = X, Zn = Z;
        if (i >= 4) {                                     // the next operands are requested ahead
          Xn = tile_load_transposed(tile_at(i - 4, p), lane);
          Zn = tile_load(tile_at(i - 4, nt + c), lane);
        }
        tile_xy<true>(Z, X, G);
        if (i == p - 1) finish(i, c, V, Z);
        else tile_store(tile_at(i, nt + c), Z, lane);
        X = Xn;
        Z = Zn;
      }
    }
    __syncthreads();
  }
}

inline void wpe_launch_solve(double2* part, double2* Gc, uint32_t* status, long n_sf, int D, int taps, const ChunkMap& cmap,
                             int rt, hipStream_t st) {
  const int n_tiles = wpe_num_tiles((D * taps + 15) / 16, (D + 15) / 16);
  const bool all = cmap.c_main > kSolveMaxSlots;
  const long sf0 = all ? 0 : cmap.n_main;
  if ((all || cmap.c_tail > kSolveMaxSlots) && sf0 < n_sf)
    hipLaunchKernelGGL(wpe_sum_chunks_kernel, dim3((unsigned)((n_sf - sf0) * n_tiles)), dim3(kTileEntries), 0, st, part, cmap, sf0,
                       n_tiles);
  hipLaunchKernelGGL(wpe_solve_kernel, dim3((unsigned)n_sf), dim3(kSolveThreads), 0, st, part, Gc, status, D, taps, cmap, rt);
}

// Apply for up to kApplyFewMaxD channels: lane = frame.  (A tile of the matrix cores has 16 rows, Re and Im of 8 channels:
// mostly padding here.)  The frames t0-Delta-L+1 .. t0+255 of the bin are staged in LDS (row pitch odd in
// 8-byte units for even D, so that the lanes' rows start in different banks); every lane then subtracts
// the prediction, walking the N components of ytilde_t while the N x D coefficients, which are the same for
// all lanes, come through the scalar path.  FINAL: writes the complex64 output (zero at t >= T); otherwise
// writes lambda_t of the new estimate for the next iteration.
template <int D, bool FINAL>
__global__ __launch_bounds__(kWpeThreads) void wpe_apply_few_kernel(const float2* __restrict__ Y, const int32_t* __restrict__ T_len,
                                                                const double2* __restrict__ Gc, double* __restrict__ lam,
                                                                float2* __restrict__ X, int F, int Tmax, int taps, int delay,
                                                                int blocks_per_sf, int pitch, long n_blocks, long per_xcd) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  float2* __restrict__ sWin = reinterpret_cast<float2*>(lds_raw);
  const long blk = xcd_block(blockIdx.x, per_xcd);
  if (blk >= n_blocks) return;
  const long sf = blk / blocks_per_sf;
  const int t0 = (int)(blk % blocks_per_sf) * kWpeThreads;
  const int T = clamp_T(T_len, (int)(sf / F), Tmax);
  const int t = t0 + threadIdx.x;
  const int N = D * taps;
  if (t0 >= T) {                                         // nothing valid in this block
    if (t < Tmax) {
      if constexpr (FINAL) {
#pragma unroll
        for (int d = 0; d < D; ++d) X[(sf * Tmax + t) * D + d] = make_float2(0.f, 0.f);
      } else {
        lam[sf * Tmax + t] = 0.0;
      }
    }
    return;
  }
  const int past = delay + taps - 1;                     // frames before t0 that the block needs
  const int rows = kWpeThreads + past;
  const float2* __restrict__ Yrow = Y + sf * (long)Tmax * D;
  staged_copy<6, float2>(
      threadIdx.x, rows * D, kWpeThreads,
      [&](int e) {
        const int r = e / D, d = e - r * D;
        const int tt = t0 - past + r;
        return (tt >= 0 && tt < T) ? Yrow[(long)tt * D + d] : make_float2(0.f, 0.f);
      },
      [&](int e, float2 v) {
        const int r = e / D, d = e - r * D;
        sWin[r * pitch + d] = v;
      });
  __syncthreads();
  double xr[D], xi[D];
  const float2* __restrict__ mine = sWin + (threadIdx.x + past) * pitch;
#pragma unroll
  for (int d = 0; d < D; ++d) { xr[d] = (double)mine[d].x; xi[d] = (double)mine[d].y; }
  typedef const __attribute__((address_space(4))) double* cptr_t;
  const cptr_t g4 = (cptr_t)(uintptr_t)(Gc + sf * (long)N * D);
  if constexpr (D % 2 == 0) {
    // The D coefficients of one component of ytilde are wave-uniform and come through the scalar path; two
    // such rows are resident in SGPRs and the loads of the next row are issued during the arithmetic of the
    // current one (the empty asm statements fix that order: the next row's offset becomes known after the
    // first product of the current row, and every sum passes a fence at the end of the row).  LDS and scalar
    // loads share one counter, so the frame values of the next tap are fetched from LDS along with the first
    // coefficient row of the current tap, one tap ahead.  The pipeline fetches one row past the last one
    // it uses; the coefficient array is followed by padding so that this load stays in bounds.
    double cA[2 * D], cB[2 * D];
    auto fetch = [&](double (&c)[2 * D], int off) {
      const cptr_t cg = g4 + off;
#pragma unroll
      for (int x = 0; x < 2 * D; ++x) c[x] = cg[x];
    };
    float2 vcur[D], vnxt[D];
    {
      const float2* __restrict__ src = mine - delay * pitch;
#pragma unroll
      for (int dp = 0; dp < D; ++dp) vcur[dp] = src[dp];
      int off0 = 0;
      asm volatile("" : "+s"(off0));                    // opaque offset: keeps the loads inside this kernel's loop
      fetch(cA, off0);
    }
    for (int tau = 0; tau < taps; ++tau) {
      const int tn = tau + 1 < taps ? tau + 1 : tau;     // the last tap re-reads its own row (stays in bounds)
      const float2* __restrict__ srcn = mine - (delay + tn) * pitch;
#pragma unroll
      for (int dp = 0; dp < D; ++dp) {
        const double vr = (double)vcur[dp].x, vi = (double)vcur[dp].y;
        double (&cur)[2 * D] = (dp & 1) ? cB : cA;
        double (&nxt)[2 * D] = (dp & 1) ? cA : cB;
        xr[0] = fma(-cur[0], vr, fma(cur[1], vi, xr[0]));  // first use of this row: the wait for its loads lands here
        int noff = (tau * D + dp + 1) * 2 * D;
        asm volatile("" : "+s"(noff), "+v"(xr[0]));
        fetch(nxt, noff);
        if (dp == 0) {
#pragma unroll
          for (int q = 0; q < D; ++q) vnxt[q] = srcn[q];
        }
        xi[0] = fma(-cur[0], vi, fma(-cur[1], vr, xi[0]));
#pragma unroll
        for (int d = 1; d < D; ++d) {                    // x_d -= c[d] * v
          xr[d] = fma(-cur[2 * d], vr, fma(cur[2 * d + 1], vi, xr[d]));
          xi[d] = fma(-cur[2 * d], vi, fma(-cur[2 * d + 1], vr, xi[d]));
        }
#pragma unroll
        for (int d = 0; d < D; ++d) asm volatile("" : "+v"(xr[d]), "+v"(xi[d]));
      }
#pragma unroll
      for (int q = 0; q < D; ++q) vcur[q] = vnxt[q];
    }
  } else {
    for (int tau = 0; tau < taps; ++tau) {
      const float2* __restrict__ src = mine - (delay + tau) * pitch;
#pragma unroll
      for (int dp = 0; dp < D; ++dp) {
        const float2 v = src[dp];
        const double vr = (double)v.x, vi = (double)v.y;
        const cptr_t c = g4 + ((long)(tau * D + dp) * D) * 2;
#pragma unroll
        for (int d = 0; d < D; ++d) {                    // x_d -= c[d] * v
          const double cr = c[2 * d], ci = c[2 * d + 1];
          xr[d] = fma(-cr, vr, fma(ci, vi, xr[d]));
          xi[d] = fma(-cr, vi, fma(-ci, vr, xi[d]));
        }
      }
    }
  }
  if (t >= Tmax) return;
  if constexpr (FINAL) {
    float2* __restrict__ o = X + (sf * Tmax + t) * D;
#pragma unroll
    for (int d = 0; d < D; ++d) o[d] = t < T ? make_float2((float)xr[d], (float)xi[d]) : make_float2(0.f, 0.f);
  } else {
    double p = 0.0;
#pragma unroll
    for (int d = 0; d < D; ++d) p += xr[d] * xr[d] + xi[d] * xi[d];
    lam[sf * Tmax + t] = t < T ? p / (double)D : 0.0;
  }
}

// iters == 0: the output is the input (zero at t >= T).
__global__ __launch_bounds__(kWpeThreads) void wpe_copy_kernel(const float2* __restrict__ Y, const int32_t* __restrict__ T_len,
                                                               float2* __restrict__ X, int F, int Tmax, int D, long n) {
  const long i = (long)blockIdx.x * kWpeThreads + threadIdx.x;
  if (i >= n) return;
  const long frame = i / D;
  const int t = (int)(frame % Tmax);
  const int s = (int)(frame / Tmax / F);
  X[i] = t < clamp_T(T_len, s, Tmax) ? Y[i] : make_float2(0.f, 0.f);
}

// Apply on the fp64 matrix cores: x_t = y_t - G^H ytilde_t as a product of real matrices, 16 rows (Re and Im of 8 channels)
// by 4 components of ytilde by 16 frames at a time, once for their real and once for their imaginary parts, added up on
// top of y_t.  RT tiles of 8 channels (8 RT >= D > 8 (RT - 1)); a wavefront owns CT groups of 16 frames.  The frames
// t0-Delta-L+1 .. t0+64 CT-1 are staged in LDS as they came, 8 RT + 1 values apart (odd: the lanes' frames start in
// different banks).  Row i = k + 4 v of a tile is part v & 1 (Re, Im) of channel k + 4 (v >> 1), so that a lane ends up
// with whole complex values.  The coefficients come from memory in the order of the operands (wpe_apply_coef), two groups
// of components ahead.  FINAL: writes the complex64 output (zero at t >= T); otherwise lambda_t of the new estimate.
//
// Bound: the fp64 matrix rate (no padding where D is a multiple of 8).  Measured, 10 taps: 94 us at 513 x 1560 x 8 (one frame
// per lane with the coefficients through the scalar path: 102 us), 0.63 ms at 513 x 1500 x 24 (1.40 ms).
constexpr int kApplyAhead = 4;                // groups of components whose coefficients are in flight (even)

// A value of the window: as it came, or, where only one tile of channels would use each conversion, converted once (each value
// is read `taps` times).
template <int RT>
struct ApplyWindow {
  using type = float2;
  static __device__ __forceinline__ type make(float2 v) { return v; }
};
template <>
struct ApplyWindow<1> {
  using type = double2;
  static __device__ __forceinline__ type make(float2 v) { return make_double2((double)v.x, (double)v.y); }
};

template <int RT, int CT, bool FINAL>
__global__ __launch_bounds__(kWpeThreads, 2) void wpe_apply_kernel(const float2* __restrict__ Y, const int32_t* __restrict__ T_len,
                                                                   const double2* __restrict__ Gc, double* __restrict__ lam,
                                                                   float2* __restrict__ X, int F, int Tmax, int D, int taps,
                                                                   int delay, int blocks_per_sf, long n_blocks, long per_xcd) {
  constexpr int P = 8 * RT + 1, fb = kWpeThreads / kWave * 16 * CT;
  using Win = ApplyWindow<RT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
  typename Win::type* __restrict__ sWin = reinterpret_cast<typename Win::type*>(lds_raw);
  const long blk = xcd_block(blockIdx.x, per_xcd);
  if (blk >= n_blocks) return;
  const unsigned sfu = (unsigned)blk / (unsigned)blocks_per_sf;         // (fewer than 2^31 blocks)
  const int t0 = (int)((unsigned)blk - sfu * (unsigned)blocks_per_sf) * fb;
  const long sf = (long)sfu;
  const int T = clamp_T(T_len, (int)(sfu / (unsigned)F), Tmax);
  const int N = D * taps;
  if (t0 >= T) {                                         // nothing valid in this block
    const int n = Tmax - t0 < fb ? Tmax - t0 : fb;
    if constexpr (FINAL) {
      for (int e = threadIdx.x; e < n * D; e += kWpeThreads) X[(sf * Tmax + t0) * D + e] = make_float2(0.f, 0.f);
    } else {
      for (int e = threadIdx.x; e < n; e += kWpeThreads) lam[sf * Tmax + t0 + e] = 0.0;
    }
    return;
  }
  const int past = delay + taps - 1;
  const int rows = fb + past;
  const float2* __restrict__ Yrow = Y + sf * (long)Tmax * D;
  {
    // the window's frames that exist are one run of n_run values: its start takes 64 bits, positions inside it 32
    const int t_run = t0 > past ? t0 - past : 0;
    const float2* __restrict__ Yrun = Yrow + (long)t_run * D;
    const unsigned n_run = (unsigned)((t0 - t_run + (T - t0 < fb ? T - t0 : fb)) * D), g0 = (unsigned)((t0 - past - t_run) * D);
    const int step_r = kWpeThreads / D, step_d = kWpeThreads - step_r * D, step_pos = step_r * P + step_d;
    const int r0 = (int)((unsigned)threadIdx.x / (unsigned)D);
    int d = (int)threadIdx.x - r0 * D, pos = r0 * P + d;
    staged_copy<8, float2>(
        threadIdx.x, rows * D, kWpeThreads,
        [&](int m) {
          const unsigned e = g0 + (unsigned)m;
          return e < n_run ? Yrun[e] : make_float2(0.f, 0.f);
        },
        [&](int, float2 v) {
          sWin[pos] = Win::make(v);
          d += step_d;
          pos += step_pos;
          if (d >= D) {
            d -= D;
            pos += P - D;
          }
        });
  }
  __syncthreads();
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int k4 = lane >> 4, li = lane & 15;
  const int f0 = wave * 16 * CT + li;                    // the lane's frame within the block, first group
  double4v acc[RT][CT];
#pragma unroll
  for (int r = 0; r < RT; ++r)
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int d = 8 * r + 4 * h + k4;
        const typename Win::type y = sWin[(f0 + 16 * c + past) * P + (d < D ? d : 0)];
        acc[r][c][2 * h] = d < D ? (double)y.x : 0.0;
        acc[r][c][2 * h + 1] = d < D ? (double)y.y : 0.0;
      }
  // component n = 4 s + k4 of ytilde_t: value d of the frame Delta + tau before t (components >= N, which have zero
  // coefficients, repeat the last one)
  const int groups = wpe_apply_groups(N);
  const int n_steps = t0 + wave * 16 * CT < T ? groups : 0;   // (none where no frame of the wavefront is valid)
  const double2* __restrict__ g = Gc + (size_t)sf * groups * RT * kWave + lane;
  int n = k4, d = k4;                                     // (D > 4)
  int pos = (f0 + past - delay) * P + d;
  auto step = [&]() {
    n += 4;
    const bool wrap = d + 4 >= D;
    const int to = wrap ? 4 - D - P : 4, dd = wrap ? 4 - D : 4;
    pos += n < N ? to : 0;
    d += dd;
  };
  auto coef = [&](double2 (&a)[RT], int s) {
#pragma unroll
    for (int r = 0; r < RT; ++r) a[r] = g[(s * RT + r) * kWave];
  };
  auto frames = [&](typename Win::type (&v)[CT]) {
#pragma unroll
    for (int c = 0; c < CT; ++c) v[c] = sWin[pos + 16 * P * c];
    step();
  };
  // (The buffers of the requested operands are picked at compile time: moving them along would wait for the loads.)
  double2 a[kApplyAhead][RT];
  typename Win::type v[2][CT];
  static_for<0, kApplyAhead>([&](auto UI) { coef(a[UI.value], UI.value < groups ? UI.value : 0); });
  frames(v[0]);
  for (int s0 = 0; s0 < n_steps; s0 += kApplyAhead) {
    static_for<0, kApplyAhead>([&](auto UI) {
      constexpr int u = UI.value;
      if (s0 + u < n_steps) {
        double br[CT], bi[CT];
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          br[c] = (double)v[u & 1][c].x;
          bi[c] = (double)v[u & 1][c].y;
        }
        frames(v[(u + 1) & 1]);                           // (behind the last group: read, not used)
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[r][c] = mfma_f64(a[u][r].x, br[c], acc[r][c]);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
          for (int c = 0; c < CT; ++c) acc[r][c] = mfma_f64(a[u][r].y, bi[c], acc[r][c]);
        if (s0 + u + kApplyAhead < n_steps) coef(a[u], s0 + u + kApplyAhead);
      }
    });
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    const int t = t0 + f0 + 16 * c;
    if constexpr (FINAL) {
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const int dd = 8 * r + 4 * h + k4;
          if (t < Tmax && dd < D)
            X[(sf * Tmax + t) * D + dd] =
                t < T ? make_float2((float)acc[r][c][2 * h], (float)acc[r][c][2 * h + 1]) : make_float2(0.f, 0.f);
        }
    } else {
      double p = 0.0;
#pragma unroll
      for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int h = 0; h < 2; ++h)
          if (8 * r + 4 * h + k4 < D) p += acc[r][c][2 * h] * acc[r][c][2 * h] + acc[r][c][2 * h + 1] * acc[r][c][2 * h + 1];
      p += __shfl_xor(p, 16);
      p += __shfl_xor(p, 32);
      if (k4 == 0 && t < Tmax) lam[sf * Tmax + t] = t < T ? p / (double)D : 0.0;
    }
  }
}

// ----------------------------------------------------------------------------------------------
// Host side
// ----------------------------------------------------------------------------------------------
struct WpeApply {
  int fb, lds, rt;                                       // frames per workgroup, LDS bytes, tiles of 8 channels (0: few channels)
  const void* fn[2];                                     // the kernel without and with the output
};
// Up to 4 channels the vector kernel (of the 16 rows of a matrix tile at most half would be used: gss_wpe on 513 x 1000 x 4,
// 10 taps, 3 iterations 616 us against 627; from 5 channels on the matrix kernel is the faster one).  More than 24 channels:
// half as many frames per workgroup (registers, LDS).
inline WpeApply wpe_apply_of(int D, int taps, int delay) {
  WpeApply a;
  a.fb = D > 24 ? 128 : 256;
  a.rt = D <= kApplyFewMaxD ? 0 : (D + 7) / 8;
  const int pitch = a.rt ? 8 * a.rt + 1 : D | 1;
  a.lds = (a.fb + delay + taps - 1) * pitch * (int)(a.rt == 1 ? sizeof(double2) : sizeof(float2));
#define GSS_APPLY(...) { a.fn[0] = (const void*)__VA_ARGS__, false>; a.fn[1] = (const void*)__VA_ARGS__, true>; }
  switch (a.rt ? a.rt + kApplyFewMaxD : D) {
    case 1: GSS_APPLY(wpe_apply_few_kernel<1) break;
    case 2: GSS_APPLY(wpe_apply_few_kernel<2) break;
    case 3: GSS_APPLY(wpe_apply_few_kernel<3) break;
    case 4: GSS_APPLY(wpe_apply_few_kernel<4) break;
    case 5: GSS_APPLY(wpe_apply_kernel<1, 4) break;
    case 6: GSS_APPLY(wpe_apply_kernel<2, 4) break;
    case 7: GSS_APPLY(wpe_apply_kernel<3, 4) break;
    default: GSS_APPLY(wpe_apply_kernel<4, 2) break;
  }
#undef GSS_APPLY
  return a;
}

int run_wpe(gss_ctx* ctx, const float2* Y, const int32_t* T_len, int S, int F, int Tmax, int D, int taps, int delay, int iters,
            float2* X, hipStream_t st) {
  const long n_sf = (long)S * F;
  const int N = D * taps;
  const int tiles = (Tmax + kWpeTile - 1) / kWpeTile;
  const int n_tiles = wpe_num_tiles((N + 15) / 16, (D + 15) / 16);
  const WpeTiling til = wpe_tiling(n_tiles);
  int pitch;
  const wpe_cov_fn cov = wpe_cov_of(D, til.tpw, pitch);
  const int cov_lds = wpe_cov_lds(pitch, taps, delay, til.split);
  const WpeApply ap = wpe_apply_of(D, taps, delay);
  const int fb_power = D > kPowerMaxD ? 64 : 256;
  // (windows of at most 64 KB, in the apply kernel at the smallest odd frame pitch)
  if ((ap.fb + delay + taps - 1) * (D | 1) * (int)sizeof(float2) > 64 * 1024 || !wpe_window_fits(D, taps, delay)) return GSS_EUNSUPPORTED;
  // (the attribute belongs to the process: every call sets the same value, so that one thread's call cannot lower the limit
  // between another's setting it and its launch)
  for (const void* fn : {ap.fn[0], ap.fn[1], (const void*)cov})
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kWpeLdsLimit) != hipSuccess) return GSS_EHIP;
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, cov, kWpeThreads, (size_t)cov_lds) != hipSuccess || per_cu < 1)
    per_cu = 1;
  // several workgroups per chunk: the chunks are planned for that part of the resident workgroups
  long slots = (long)ctx->num_cu * (per_cu < kWpeCovPerCu ? per_cu : kWpeCovPerCu) / til.groups;
  if (slots < 1) slots = 1;
  const ChunkMap cmap = plan_chunk_map(slots, n_sf, tiles, 1, 0, true);
  const long wgs = chunk_map_wgs(cmap, n_sf);
  const long bps_apply = (Tmax + ap.fb - 1) / ap.fb, bps_power = (Tmax + fb_power - 1) / fb_power;
  if (wgs * til.groups > 0x7fffffffL || n_sf * bps_power + 8 > 0x7fffffffL || n_sf * n_tiles > 0x7fffffffL)
    return GSS_EUNSUPPORTED;

  // coefficients: as the apply kernel reads them; the vector kernel's are followed by room for its read-ahead
  const size_t coef_bytes = ap.rt ? (size_t)n_sf * wpe_apply_groups(N) * ap.rt * kWave * sizeof(double2)
                                  : (size_t)n_sf * N * D * sizeof(double2) + 256;
  size_t o = 0;
  const size_t off_lam = o;  o = gss_align_up(o + (size_t)n_sf * Tmax * sizeof(double), 256);
  const size_t off_g = o;    o = gss_align_up(o + coef_bytes, 256);
  const size_t off_part = o; o = gss_align_up(o + (size_t)wgs * n_tiles * kTileEntries * sizeof(double2), 256);
  const int rc = gss_ensure_scratch(ctx, o);
  if (rc != GSS_OK) return rc;
  char* base = (char*)ctx->scratch;
  double* lam = (double*)(base + off_lam);
  double2* Gc = (double2*)(base + off_g);
  double2* part = (double2*)(base + off_part);

  const dim3 block(kWpeThreads);
  const long nb_power = n_sf * bps_power, px_power = (nb_power + 7) / 8;
  long nb_apply = n_sf * bps_apply, px_apply = (nb_apply + 7) / 8;
  hipLaunchKernelGGL(wpe_power_kernel, dim3((unsigned)(8 * px_power)), block, 0, st, Y, T_len, lam, F, Tmax, D,
                     (int)bps_power, nb_power, px_power, fb_power);
  for (int it = 0; it < iters; ++it) {
    gss_profile_begin(ctx, 2, st);
    hipLaunchKernelGGL(cov, dim3((unsigned)(wgs * til.groups)), block, cov_lds, st, Y, T_len, lam, part, F, Tmax, D, taps, delay,
                       cmap, til.groups, til.split);
    gss_profile_end(ctx, 2, st);
    wpe_launch_solve(part, Gc, ctx->status, n_sf, D, taps, cmap, ap.rt, st);
    int bps = (int)bps_apply;
    int apitch = D | 1;
    void* few[] = {&Y, &T_len, &Gc, &lam, &X, &F, &Tmax, &taps, &delay, &bps, &apitch, &nb_apply, &px_apply};
    void* mat[] = {&Y, &T_len, &Gc, &lam, &X, &F, &Tmax, &D, &taps, &delay, &bps, &nb_apply, &px_apply};
    if (hipLaunchKernel(ap.fn[it + 1 < iters ? 0 : 1], dim3((unsigned)(8 * px_apply)), block, ap.rt ? mat : few, (size_t)ap.lds, st) !=
        hipSuccess)
      return GSS_EHIP;
  }
  if (hipGetLastError() != hipSuccess) return GSS_EHIP;
  return GSS_OK;
}

}  // namespace

extern "C" int gss_wpe(gss_ctx* ctx, const float* Y, const int32_t* T_len, int S, int F, int Tmax, int D,
                       int taps, int delay, int iters, float* X, void* stream) {
  if (!ctx || !Y || !X || Y == X) return GSS_EINVAL;
  if (S <= 0 || F <= 0 || Tmax <= 0 || D <= 0 || taps <= 0 || delay <= 0 || iters < 0) return GSS_EINVAL;
  if (D > GSS_WPE_LARGE_MAX_D || (long)D * taps > GSS_WPE_LARGE_MAX_N || delay > 64) return GSS_EUNSUPPORTED;
  if (hipSetDevice(ctx->device) != hipSuccess) return GSS_EHIP;
  hipStream_t st = (hipStream_t)stream;
  const float2* Yc = (const float2*)Y;
  float2* Xc = (float2*)X;
  if (iters == 0) {
    const long n = (long)S * F * Tmax * D;
    const long blocks = (n + kWpeThreads - 1) / kWpeThreads;
    if (blocks > 0x7fffffffL) return GSS_EUNSUPPORTED;
    hipLaunchKernelGGL(wpe_copy_kernel, dim3((unsigned)blocks), dim3(kWpeThreads), 0, st, Yc, T_len, Xc, F, Tmax, D, n);
    return hipGetLastError() == hipSuccess ? GSS_OK : GSS_EHIP;
  }
  return run_wpe(ctx, Yc, T_len, S, F, Tmax, D, taps, delay, iters, Xc, st);
}
