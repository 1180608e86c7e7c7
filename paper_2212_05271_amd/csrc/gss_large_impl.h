// EM and MVDR kernels for large arrays, 9 <= D <= 32 channels (e.g. multi-array set-ups with 24
// microphones).  Same algorithm, same fp64 arithmetic and the same pass / factor structure as the D <= 8
// kernels (arXiv 2212.05271, Section 2.2 and 2.3); what changes is the mapping: D is a run-time value, and both
// contractions of a pass run on the fp64 matrix cores in real arithmetic.
//
//   * A frame is the vector u of its 2 D reals (re, im of every channel, as in memory), padded to 16 NB entries,
//     NB = ceil(D / 8).
//   * E-step: the class matrix enters as W = the inverse of its Cholesky factor (B = L L^H, W = L^-1), and
//     q = y^H B^-1 y = |W y|^2: a product of the real form of W (2 D x 2 D, block lower triangular, 16 x 16 tiles) with 16
//     frames, then a sum of squares.  No cancellation beyond that of W y, whose entries are the square roots of those of
//     B^-1: better conditioned than the quadratic form itself.
//   * M-step sums: sum_t w_t u_t u_t^T by 16 x 16 tiles on and above the diagonal; the Hermitian sums are
//     Re = (re re) + (im im), Im = (im re) - (re im) of them, formed once at the end.
//   * A last block of up to 4 channels (H = 1: up to 2, H = 2: 3 or 4; H = 0: more) is 4 H rows of W and columns of the sums
//     instead of 16, by the 4 x 4 x 4 products.
//   * A class that is inactive in a group of 16 frames is skipped for the group in both steps.
#pragma once

#include "gss_internal.h"

#include "gss_device.h"

namespace {

constexpr int kLargeWaves = 4;

__host__ __device__ inline int item_index(int i, int j, int D) { return i * D - i * (i - 1) / 2 + (j - i); }   // i <= j
__host__ __device__ inline int num_items(int D) { return D * (D + 1) / 2; }

__device__ __forceinline__ double ipow_rt(double x, int n) {   // x^n, n >= 1
  double r = 1.0, b = x;
  while (n) {
    if (n & 1) r *= b;
    b *= b;
    n >>= 1;
  }
  return r;
}


// ----------------------------------------------------------------------------------------------
// Geometry of the matrix-core kernels
// ----------------------------------------------------------------------------------------------
typedef double double4v __attribute__((ext_vector_type(4)));
typedef double double2v __attribute__((ext_vector_type(2)));
// D += A B of 16 x 4 and 4 x 16 doubles.  Lane l holds A[l % 16][l / 16] and B[l / 16][l % 16], and D[l / 16 + 4 v][l % 16]
// for v = 0..3.
__device__ __forceinline__ double4v mfma_f64(double a, double b, double4v c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// Four products of 4 x 4 and 4 x 4 doubles, a fifth of the time of the above.  Lane 16 k + 4 b + i holds A[i][k] and B[k][i] of
// product b, and D[k][i].  So a lane's A above is A of the rows 4 b .. 4 b + 3, and its B above is B of the columns 4 b .. 4 b + 3.
__device__ __forceinline__ double mfma4_f64(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}
// Sum over the four rows of 16 lanes, in every lane.
__device__ __forceinline__ double sum_rows_f64(double v) {
  auto add = [](auto lo, auto hi) { return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]); };
  v = add(__builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false),
          __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false));
  return add(__builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false),
             __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false));
}

// Largest of the four lane rows' values, in every lane.
__device__ __forceinline__ int max_rows_i32(int v) {
  const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const int m = (int)a[0] > (int)a[1] ? (int)a[0] : (int)a[1];
  const auto b = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  return (int)b[0] > (int)b[1] ? (int)b[0] : (int)b[1];
}

// Real entries per frame row in LDS: 16 NB and 4 more.  The operands of a tile product are rows 4 g + s of 16 frames (lane
// row g, step s): four rows apart is 128 modulo the 256 bytes that LDS delivers per cycle, so such a read has no conflicts.
__host__ __device__ constexpr int large_pitch(int NB) { return 16 * NB + 4; }
// Tiles of W (block lower triangular, by rows) and the doubles of a class: lane l = 16 g + m of a tile (i, j) holds
// W[16 i + m][16 j + 4 g + s], s = 0..3, the left operand of step s: as two pairs, [tile][s / 2][lane][s % 2].
__host__ __device__ constexpr int large_tiles(int NB) { return NB * (NB + 1) / 2; }
__host__ __device__ constexpr int large_coef(int NB) { return 256 * large_tiles(NB); }

// The last block of channels: H = 0: 16 reals, 1 or 2: 4 H (see above); the blocks that are taken in full.  With the block in full
// calls whose classes are all active most of the time lost to the vector units: 513 x 1500 frames, 3 iterations, all classes
// active in 9 of 10 frames, items on the vector units / block in full / now: 9 channels and 8 classes 0.85 / 1.16 / 0.85 ms, 12 and 5
// 0.74 / 0.80 / 0.68, 17 and 5 1.02 / 1.33 / 1.13, 17 and 8 1.36 / 1.98 / 1.78, 25 and 8 4.54 / 3.60 / 2.90; speaker turns: 9 and 5
// 0.55 / 0.45 / 0.43, 17 and 5 0.90 / 0.78 / 0.71, 25 and 5 1.79 / 1.27 / 1.09.  19 and 20 channels with 7 or 8 classes keep the
// block in full: the 8 accumulators and 2 for the rest of every class do not fit in registers (8 classes 1.04 against 1.24).
inline int large_rest(int D, int K) {
  const int c = (D - 1) % 8 + 1;
  return c <= 2 ? 1 : c <= 4 && !(D > 16 && D <= 24 && K > 6) ? 2 : 0;
}
__host__ __device__ constexpr int full_blocks(int NB, int H) { return H > 0 ? NB - 1 : NB; }

// Tiles of the weighted sums: which of the NB (NB + 1) / 2 tiles on and above the diagonal a wavefront of the workgroup adds
// up, over which of the four groups of 16 frames of a tile of frames.  A wavefront has one left operand (row of tiles `left`)
// and `count` right ones; left > right is the transposed tile.  Every wavefront gets the same number of products (1, 3, 6 and
// 10 tiles in four: one, three, six and ten groups x tiles), with few accumulators: 8 count K registers.  The first `full` right
// operands of every wavefront take all groups.  `phase`: when the wavefront's sums of the tile join the others' at the end
// (0: they are the first).
template <int NB>
struct LargeShare;
template <>
struct LargeShare<1> {
  static constexpr int count = 1;
  static constexpr int left[4] = {0, 0, 0, 0};
  static constexpr int right[4][1] = {{0}, {0}, {0}, {0}};
  static constexpr int groups[4][1] = {{1}, {2}, {4}, {8}};
  static constexpr int full = 0, phases = 4;
  static constexpr int phase[4][1] = {{0}, {1}, {2}, {3}};
};
template <>
struct LargeShare<2> {
  static constexpr int count = 2;
  static constexpr int left[4] = {0, 0, 1, 1};
  static constexpr int right[4][2] = {{0, 1}, {0, 1}, {1, 0}, {1, 0}};
  static constexpr int groups[4][2] = {{3, 1}, {12, 4}, {3, 2}, {12, 8}};
  static constexpr int full = 0, phases = 4;
  static constexpr int phase[4][2] = {{0, 0}, {1, 1}, {0, 2}, {1, 3}};
};
template <>
struct LargeShare<3> {
  static constexpr int count = 2;
  static constexpr int left[4] = {0, 0, 1, 2};
  static constexpr int right[4][2] = {{0, 1}, {2, 1}, {1, 2}, {2, 1}};
  static constexpr int groups[4][2] = {{15, 3}, {15, 12}, {15, 3}, {15, 12}};
  static constexpr int full = 1, phases = 2;
  static constexpr int phase[4][2] = {{0, 0}, {0, 1}, {0, 0}, {0, 1}};
};
template <>
struct LargeShare<4> {
  static constexpr int count = 3;
  static constexpr int left[4] = {0, 3, 1, 2};
  static constexpr int right[4][3] = {{0, 1, 2}, {3, 0, 1}, {1, 2, 3}, {2, 3, 0}};
  static constexpr int groups[4][3] = {{15, 15, 3}, {15, 15, 12}, {15, 15, 3}, {15, 15, 12}};
  static constexpr int full = 2, phases = 2;
  static constexpr int phase[4][3] = {{0, 0, 0}, {0, 0, 1}, {0, 0, 0}, {0, 0, 1}};
};
// The 4 H columns of a last block of few channels: which 16 rows of them a wavefront adds up, over which groups of frames; the
// rows of its other tiles where there is a choice.
template <int NB>
struct RestShare;
template <>
struct RestShare<2> {
  static constexpr int row[4] = {0, 1, 0, 1}, groups[4] = {3, 3, 12, 12}, phase[4] = {0, 0, 1, 1};
};
template <>
struct RestShare<3> {
  static constexpr int row[4] = {0, 2, 1, 2}, groups[4] = {15, 3, 15, 12}, phase[4] = {0, 0, 0, 1};
};
template <>
struct RestShare<4> {
  static constexpr int row[4] = {0, 3, 1, 2}, groups[4] = {15, 15, 15, 15}, phase[4] = {0, 0, 0, 0};
};
// A wavefront's share in registers (wave-uniform).
template <int NB, int H>
struct LargeRole {
  using S = LargeShare<full_blocks(NB, H)>;
  int left, right[S::count], groups[S::count], phase[S::count], rest_row = 0, rest_groups = 0, rest_phase = -1;
  __device__ __forceinline__ explicit LargeRole(int wave) {
    left = 0;
#pragma unroll
    for (int w = 0; w < kLargeWaves; ++w)
      if (wave == w) {
        left = S::left[w];
#pragma unroll
        for (int r = 0; r < S::count; ++r) {
          right[r] = S::right[w][r];
          groups[r] = S::groups[w][r];
          phase[r] = S::phase[w][r];
        }
        if constexpr (H > 0) {
          rest_row = RestShare<NB>::row[w];
          rest_groups = RestShare<NB>::groups[w];
          rest_phase = RestShare<NB>::phase[w];
        }
      }
  }
};
// A wavefront's sums of KW classes: its 16 x 16 tiles, and 16 x 4 H of the last block of channels (lane l: row 4 (l / 4 % 4) + l / 16,
// column 4 h + l % 4).
template <int NB, int H, int KW>
struct LargeAcc {
  static constexpr int C = LargeShare<full_blocks(NB, H)>::count;
  double4v full[KW][C];
  double rest[KW][H > 0 ? H : 1];
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int k = 0; k < KW; ++k) {
#pragma unroll
      for (int r = 0; r < C; ++r) full[k][r] = double4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int h = 0; h < (H > 0 ? H : 1); ++h) rest[k][h] = 0.0;
    }
  }
};

// A wavefront's 16 frames of a tile: lane (g, n) = (lane / 16, lane % 16) has frame n's channels 8 b + 2 g and the one behind it
// for every b < NB, which is the right operand of the E-step's products (entries 16 b + 4 g .. + 3 of u).  Channels from D on
// and frames from T on are zero.
template <int NB>
struct LargeFrames {
  float2 v[NB][2];
  unsigned abits, mask;                                     // (mask: the masks of a tile further on, the same in every lane)
  __device__ __forceinline__ void request(const float2* __restrict__ Yrow, const uint8_t* __restrict__ abrow, int t, int T,
                                          int D, int g) {
    abits = abrow[t < T ? t : 0];
    request(Yrow, t, T, D, g);
  }
  __device__ __forceinline__ void request(const float2* __restrict__ Yrow, int t, int T, int D, int g) {
    struct __attribute__((packed, aligned(8))) pair { float x0, y0, x1, y1; };
    const bool valid = t < T;
    const float2* __restrict__ src = Yrow + (long)(valid ? t : 0) * D + 2 * g;     // (frame 0 exists where a tile is live)
#pragma unroll
    for (int b = 0; b + 1 < NB; ++b) {
      const pair q = *reinterpret_cast<const pair*>(src + 8 * b);
      v[b][0] = make_float2(q.x0, q.y0);
      v[b][1] = make_float2(q.x1, q.y1);
    }
    // the last block of channels may end inside: channel 0 or 1 of the block before in the place of one that is not there (no
    // branch: a load under one is waited for where the branch ends)
    constexpr int c = 8 * (NB - 1);
    v[NB - 1][0] = src[c + 2 * g < D ? c : c - 8];
    v[NB - 1][1] = src[c + 2 * g + 1 < D ? c + 1 : c - 7];
  }
  __device__ __forceinline__ void convert(double (&u)[NB][4], int t, int T, int D, int g) const {
    const bool valid = t < T;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        u[b][2 * e] = (double)v[b][e].x;
        u[b][2 * e + 1] = (double)v[b][e].y;
      }
    // (both conditions are the same in every lane: hardly ever true, or never)
    if (__builtin_amdgcn_readfirstlane(t - (t & 15)) + 16 > T || (D & 7) != 0) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) u[b][e] = valid && 8 * b + 2 * g + (e >> 1) < D ? u[b][e] : 0.0;
    }
  }
};

// Adds w_k u u^T over the tile's 64 frames to the wavefront's tiles, for the classes of each group of 16 frames (byte g of
// `masks`).  sW: [KW][64] weights.  Step s of a group takes frames 4 g + s (lane row g): a lane's four weights are contiguous,
// and the four products of a tile follow each other on the same accumulators (a product on other accumulators starts about
// ten of its 64 cycles later).
template <int NB, int H, int KW>
__device__ __forceinline__ void accumulate_large(const double* __restrict__ sY, const double* __restrict__ sW,
                                                 const LargeRole<NB, H>& role, unsigned masks, int lane,
                                                 LargeAcc<NB, H, KW>& acc) {
  using S = LargeShare<full_blocks(NB, H)>;
  constexpr int P = large_pitch(NB), C = S::count;
  const double* __restrict__ p = sY + 4 * (lane >> 4) * P + (lane & 15);
  const double* __restrict__ pr = sY + 4 * (lane >> 4) * P + 16 * (NB - 1) + (lane & 3);
  const double* __restrict__ pw = sW + 4 * (lane >> 4);
  // Requested ahead of their use: the operands of the next group of frames and the weights of the next class, whatever the
  // masks say (an unused read costs less than a wait; 4 x 4 tiles, and 3 x 3 with a rest: the registers allow the weights only).
  constexpr bool kAheadOps = NB < 4 && (NB < 3 || H == 0);
  double l[2][4], b[2][C][4];
  double x[H > 0 ? 4 : 1], y[H > 0 ? H : 1][4];           // the last block's: rows, columns
  auto operands = [&](int slot, int g) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      l[slot][s] = p[(16 * g + s) * P + 16 * role.left];
#pragma unroll
      for (int r = 0; r < C; ++r) b[slot][r][s] = p[(16 * g + s) * P + 16 * role.right[r]];
    }
  };
  if constexpr (kAheadOps) operands(0, 0);
  static_for<0, 4>([&](auto GI) {
    constexpr int g = GI.value, cur = kAheadOps ? g & 1 : 0;
    if constexpr (!kAheadOps) operands(0, g);
    double2 w[2][2];
    w[0][0] = *reinterpret_cast<const double2*>(pw + 16 * g);
    w[0][1] = *reinterpret_cast<const double2*>(pw + 16 * g + 2);
    if constexpr (H > 0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        x[s] = p[(16 * g + s) * P + 16 * role.rest_row];
#pragma unroll
        for (int h = 0; h < H; ++h) y[h][s] = pr[(16 * g + s) * P + 4 * h];
      }
    }
    if constexpr (kAheadOps && g < 3) operands(cur ^ 1, g + 1);
    unsigned mask = (masks >> (8 * g)) & 0xffu;
    static_for<0, KW>([&](auto KI) {
      constexpr int k = KI.value;
      if constexpr (k + 1 < KW) {
        w[(k + 1) & 1][0] = *reinterpret_cast<const double2*>(pw + (k + 1) * kWave + 16 * g);
        w[(k + 1) & 1][1] = *reinterpret_cast<const double2*>(pw + (k + 1) * kWave + 16 * g + 2);
      }
      if (class_on(mask, k)) {
        const double2 w0 = w[k & 1][0], w1 = w[k & 1][1];
        const double a[4] = {w0.x * l[cur][0], w0.y * l[cur][1], w1.x * l[cur][2], w1.y * l[cur][3]};
#pragma unroll
        for (int r = 0; r < C; ++r) {
          if (r < S::full || class_on((unsigned)role.groups[r], g)) {
#pragma unroll
            for (int s = 0; s < 4; ++s) acc.full[k][r] = mfma_f64(a[s], b[cur][r][s], acc.full[k][r]);
          }
        }
        if constexpr (H > 0) {
          if (class_on((unsigned)role.rest_groups, g)) {
            const double v[4] = {w0.x * x[0], w0.y * x[1], w1.x * x[2], w1.y * x[3]};
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
              for (int s = 0; s < 4; ++s) acc.rest[k][h] = mfma4_f64(v[s], y[h][s], acc.rest[k][h]);
          }
        }
      }
    });
  });
}

// The workgroup's sums as packed partial sums out[k][m][2] (m: item (i, j), i <= j): the wavefronts put their tiles into LDS, in
// a fixed order where several have the same one, as many classes at a time as there is room for; then Re and Im of the items
// are formed from them.  red: large_red_doubles.
constexpr int kRedTile = 16 * 17;                           // a tile, rows 17 apart
__host__ __device__ constexpr int large_red_classes(int K, int NB) {
  const int room = 2 * (kWave * large_pitch(NB) + K * kWave) / (kRedTile * large_tiles(NB));
  return room < K ? room : K;
}
__host__ __device__ constexpr int upper_tile(int i, int j, int NB) { return i * NB - i * (i - 1) / 2 + (j - i); }   // i <= j
template <int NB, int H, int KW, int BATCH>
__device__ __forceinline__ void reduce_large(const LargeAcc<NB, H, KW>& acc, const LargeRole<NB, H>& role,
                                             double* __restrict__ red, double* __restrict__ out, int D, int lane) {
  using S = LargeShare<full_blocks(NB, H)>;
  constexpr int C = S::count, kClass = kRedTile * large_tiles(NB);
  static_assert(S::phases >= 2, "the last block's sums join in the first two");
  const int row = lane >> 4, col = lane & 15, M = num_items(D);
#pragma unroll
  for (int k0 = 0; k0 < KW; k0 += BATCH) {
    __syncthreads();
#pragma unroll
    for (int ph = 0; ph < S::phases; ++ph) {
      if constexpr (H > 0) {
        if (role.rest_phase == ph) {
          double* __restrict__ dst = red + kRedTile * upper_tile(role.rest_row, NB - 1, NB) + 17 * (4 * ((lane >> 2) & 3) + row) + (lane & 3);
#pragma unroll
          for (int c = 0; c < BATCH; ++c)
            if (k0 + c < KW) {
#pragma unroll
              for (int h = 0; h < H; ++h) {
                const double x = acc.rest[k0 + c < KW ? k0 + c : 0][h];
                dst[c * kClass + 4 * h] = ph == 0 ? x : dst[c * kClass + 4 * h] + x;
              }
            }
        }
      }
#pragma unroll
      for (int r = 0; r < C; ++r) {
        if (role.phase[r] == ph) {
          const bool turned = role.left > role.right[r];
          const int tile = turned ? upper_tile(role.right[r], role.left, NB) : upper_tile(role.left, role.right[r], NB);
          double* __restrict__ dst = red + kRedTile * tile + (turned ? 17 * col + row : 17 * row + col);
          const int step = turned ? 4 : 4 * 17;
#pragma unroll
          for (int c = 0; c < BATCH; ++c)
            if (k0 + c < KW) {
#pragma unroll
              for (int v = 0; v < 4; ++v) {
                const double x = acc.full[k0 + c < KW ? k0 + c : 0][r][v];
                dst[c * kClass + v * step] = ph == 0 ? x : dst[c * kClass + v * step] + x;
              }
            }
        }
      }
      __syncthreads();
    }
    for (int x = threadIdx.x; x < D * D; x += kWave * kLargeWaves) {
      const int i = x / D, j = x - i * D;
      if (i <= j) {
        const double* __restrict__ e = red + kRedTile * upper_tile(i >> 3, j >> 3, NB) + 17 * 2 * (i & 7) + 2 * (j & 7);
        double* __restrict__ o = out + ((long)k0 * M + item_index(i, j, D)) * 2;
#pragma unroll
        for (int c = 0; c < BATCH; ++c)
          if (k0 + c < KW)
            *reinterpret_cast<double2*>(o + (long)c * M * 2) =
                make_double2(e[c * kClass] + e[c * kClass + 18], e[c * kClass + 17] - e[c * kClass + 1]);
      }
    }
  }
}

// ----------------------------------------------------------------------------------------------
// EM pass, 9 <= D <= 32.  Grid: block0 + blockIdx.x = chunk + C * (f + F * s).  The workgroup's four wavefronts share every tile of 64
// frames: wavefront w has frames 16 w .. 16 w + 15 in the E-step, straight from memory (requested before the sums of the tile
// before), puts them into LDS as fp64 and, with their weights in place, takes its share of the tiles of the sums
// (LargeShare).  Two buffers for frames and weights, so one barrier per tile.  The final pass has no sums: no tile in LDS, no
// barrier, and every wavefront walks the tiles on its own.
//   coef : W of every class (large_coef doubles each), or null for B = I (first pass)
//   masks: per tile four bytes, the classes that are active in each group of 16 frames
// Dynamic LDS: large_lds_doubles, reused for the final reduction.
//
// Bound: the fp64 matrix rate (2 * 96 products of 64 cycles per class and tile at 24 channels: 144 us of a pass over 513 x 1500
// frames, 5 classes, 2.3 of them active), and vector instructions, which do not run beside a matrix instruction of the same
// SIMD: the wavefront that is between its products gets one in for every product of the other, so it runs at a raised
// priority there, lane rows share the posterior's classes, and the lane rows' parts are added up by their reader.  That
// pass takes 240 us (340 us with the products of frames formed on the vector units, item by item, in both steps); the final
// pass 122 us (181).  Ways there: frames through LDS with two barriers per tile 274 us, every lane all classes; loads under a
// branch (waited for at its end) 258; masks through the scalar path, W two tiles ahead, no priorities 249.
// ----------------------------------------------------------------------------------------------
// Wavefronts per SIMD: one where the accumulators of two would not fit (25 to 32 channels, 7 or 8 classes: 128 to 192 registers and
// as many again for operands; 25 channels, 8 classes 2.09 ms with one, 2.46 with two and 120 spilled registers).
constexpr int pass_waves_per_simd(int K, int NB) { return NB == 4 && K > 6 ? 1 : 2; }
__host__ __device__ constexpr int large_lds_doubles(int K, int NB, bool final_pass) {
  const int fixed = 2 * K + kWave * K;                      // constants and counts
  return fixed + (final_pass ? 4 * (K + 1) * kWave : 2 * (kWave * large_pitch(NB) + K * kWave));
}

template <int K, int NB, int H, bool FINAL>
__global__ __launch_bounds__(kWave * kLargeWaves, pass_waves_per_simd(K, NB)) void em_pass_large(
    gss_yview yv, const uint8_t* __restrict__ abyte, const uint32_t* __restrict__ masks,
    const int32_t* __restrict__ T_len,
    const double* __restrict__ coef, const double* __restrict__ cmant, const int32_t* __restrict__ cexp,
    double* __restrict__ part, double* __restrict__ npart, float* __restrict__ gamma, uint32_t* __restrict__ status,
    int F, int Tmax, int D, ChunkMap cmap, unsigned block0) {
  extern __shared__ __attribute__((aligned(16))) double lds_large[];
  constexpr int P = large_pitch(NB), NF = full_blocks(NB, H);
  constexpr int kBuf = FINAL ? 0 : kWave * P + K * kWave;   // one buffer: weights, then the tile
  constexpr int kRows = (K + 3) / 4;                        // classes of a lane row in the posterior
  constexpr unsigned kmask = (1u << K) - 1u;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = lane >> 4, n = lane & 15;
  long sf;
  int chunk, tiles_per_chunk;
  const unsigned block = block0 + blockIdx.x;
  chunk_decode(cmap, block, sf, chunk, tiles_per_chunk);
  const int s = (int)((unsigned)sf / (unsigned)F);
  const int f = (int)((unsigned)sf % (unsigned)F);
  int T;
  const float2* __restrict__ Yrow = y_row(yv, T_len, s, f, D, Tmax, T);
  const int t_end = FINAL ? Tmax : T;

  double2* __restrict__ sC = reinterpret_cast<double2*>(lds_large);    // [K] mantissa and exponent of pi_k / det B_k
  double* __restrict__ sN = lds_large + 2 * K;              // [4][K][16] class counts of the wavefronts' frames
  double* __restrict__ sBuf = sN + kWave * K;
  const double* __restrict__ cf = coef ? coef + sf * (long)(K * large_coef(NB)) + 2 * lane : nullptr;
  const uint8_t* __restrict__ abrow = abyte + (long)s * Tmax;
  const int tiles_total = (Tmax + kWave - 1) / kWave;
  typedef const __attribute__((address_space(4))) uint32_t* mask_ptr_t;
  const mask_ptr_t mrow = (mask_ptr_t)(uintptr_t)(masks + (long)s * tiles_total);
  const uint32_t* __restrict__ mvec = masks + (long)s * tiles_total + (lane >> 6);   // the same, through the vector path
  float* __restrict__ grow = FINAL ? gamma + ((long)s * K * F + f) * Tmax : nullptr;
  const long gk = (long)F * Tmax;

  const LargeRole<NB, H> role(wave);
  LargeAcc<NB, H, FINAL ? 1 : K> acc;
  acc.clear();
  for (int x = threadIdx.x; x < kWave * K; x += kWave * kLargeWaves) sN[x] = 0.0;
  if (threadIdx.x < K)
    sC[threadIdx.x] = cf ? make_double2(cmant[sf * K + threadIdx.x], (double)cexp[sf * K + threadIdx.x])
                         : make_double2(0.5, 1.0);

  const int tile_lo = chunk * tiles_per_chunk;
  int tile_hi = tile_lo + tiles_per_chunk;
  const int tile_end = (t_end + kWave - 1) / kWave;
  tile_hi = tile_hi < tile_end ? tile_hi : tile_end;
  if constexpr (FINAL) {
    // zeros of the classes that are not active in a group of 16 frames
    for (int tile = tile_lo; tile < tile_hi; ++tile) {
      const unsigned any = mrow[tile], live = (any >> (8 * wave)) & kmask;
      const int t = tile * kWave + 16 * wave + n;
      for (int k = g; k < K; k += 4)
        if (((live >> k) & 1u) == 0u && t < Tmax) grow[k * gk + t] = 0.f;
      if (live == 0u && any != 0u) {
        // frames without energy are flagged in every tile that has an active class; the walk below passes this group by
        const float2* __restrict__ y = Yrow + (long)(t < T ? t : 0) * D;
        double n2 = 0.0;
        for (int d = g; d < D; d += 4) n2 += (double)y[d].x * (double)y[d].x + (double)y[d].y * (double)y[d].y;
        n2 = sum_rows_f64(n2);
        if (g == 0 && t < T && !(n2 >= GSS_EPS_NORM_SQ)) atomicOr(status, GSS_STATUS_ZERO_FRAME);
      }
    }
  }
  __syncthreads();

  // The masks of the tiles (final pass: those of this wavefront's frames), 0 behind the last; the one after the next live tile is
  // requested with the frames of the next.  live_tile: from `tile` with mask m on, the first that has an active class.
  auto mask_of = [&](int tile) {
    const unsigned m = mrow[tile < tile_hi ? tile : tile_lo];
    return tile >= tile_hi ? 0u : FINAL ? m & (0xffu << (8 * wave)) : m;
  };
  auto live_tile = [&](int tile, unsigned& m) {
    while (m == 0u && tile < tile_hi) m = mask_of(++tile);
    return tile;
  };
  unsigned mq = tile_lo < tile_hi ? mask_of(tile_lo) : 0u;
  int tile = live_tile(tile_lo, mq);
  if (tile < tile_hi) {
    LargeFrames<NB> frames;
    frames.request(Yrow, abrow, tile * kWave + 16 * wave + n, T, D, g);
    // W comes from memory piece by piece (its tiles in their order, of those of a last block of few channels 4 rows at a time,
    // which every group of 4 lanes has), kRing pieces ahead of their use, across the classes (behind the last class: the same
    // again) and from one tile of frames to the next: a register set is refilled when its products have been issued
    constexpr int NM = large_tiles(NF), NT = NM + (H > 0 ? NB * H : 0);
    // (as far as registers allow: 24 channels, 3 iterations, 6 segments, 2 classes, 900 frames 1589 us with 3 ahead, 1544 with 6, 6
    // classes, 100 frames 932 and 905, one segment of 5 classes the same; 28 channels, 6 classes: 7 ahead spill in the loop,
    // 1.52 ms, 2 ahead 1.27)
    constexpr bool kAhead6 = NT == 6 && H == 0 && K <= 6 && !FINAL, kAhead2 = NB == 4 && H > 0 && K >= 4 && K <= 6;
    constexpr int kRing = kAhead2 ? 2 : kAhead6 ? 6 : NT % 5 == 0 ? 5 : NT % 7 == 0 ? 7 : 3;
    static_assert(NT % kRing == 0, "a class starts with the first register set");
    const int rest_lane = 2 * ((lane & 3) - n);             // from the lane's place in a tile to the first 4 rows'
    double2v w[kRing][2];
    auto fetch = [&](double2v (&dst)[2], const double* __restrict__ c, auto TI) {
      constexpr int t = decltype(TI)::value, rest = t < NM ? 0 : t - NM, rh = H > 0 ? H : 1;
      constexpr int at = t < NM ? 256 * t : 256 * (NM + rest / rh) + 8 * (rest % rh);
      const double* __restrict__ src = t < NM ? c + at : c + rest_lane + at;
      dst[0] = *reinterpret_cast<const double2v*>(src);
      dst[1] = *reinterpret_cast<const double2v*>(src + 128);
    };
    auto fetch_first = [&](unsigned m) {                    // the first tiles of the first class of this wavefront's frames
      const unsigned own = (m >> (8 * wave)) & kmask;
      const double* __restrict__ c = cf + (long)(own != 0u ? __builtin_ctz(own) : 0) * large_coef(NB);
      static_for<0, kRing>([&](auto TI) { fetch(w[TI.value], c, TI); });
    };
    if (cf) fetch_first(mq);
    int buf = 0;
    unsigned mnext = mask_of(tile + 1);
    for (;;) {
      double* __restrict__ sW = sBuf + buf * kBuf;          // [K][64] weights
      double* sT = sW + K * kWave;                          // [64][P]
      // [K + 1][16 frames][4 lane rows]: the lane rows' parts of the q and (last) of |y|^2; where the wavefront's frames go after
      static_assert((K + 1) * kWave <= 16 * P, "a wavefront's rows must hold the parts");
      double* sQ = FINAL ? sBuf + wave * (K + 1) * kWave : sT + 16 * wave * P;
      const int t = tile * kWave + 16 * wave + n;
      const unsigned live = (mq >> (8 * wave)) & kmask;     // classes of this wavefront's 16 frames
      const int next = live_tile(tile + 1, mnext);
      double u[NB][4];
      const unsigned abits = t < T ? frames.abits : 0u;
      frames.convert(u, t, T, D, g);
      if constexpr (!FINAL) {
        // the next tile's frames and the masks of the one after (behind the last tile: the same again, so that the loads need
        // no branch)
        frames.request(Yrow, abrow, (next < tile_hi ? next : tile) * kWave + 16 * wave + n, T, D, g);
        frames.mask = mvec[next + 1 < tile_hi ? next + 1 : tile];
      }
      double n2 = 0.0;
      if (live != 0u) {
        // ---- E-step: q_k = |W_k y|^2 of the lane's frame (the same in the four lane rows) ----
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int e = 0; e < 4; ++e) n2 = fma(u[b][e], u[b][e], n2);
        sQ[K * kWave + 4 * n + g] = n2;
        if (cf) {
          __builtin_amdgcn_s_setprio(0);
          unsigned left = live;
          int k = __builtin_ctz(left);
          const double* __restrict__ ck = cf + (long)k * large_coef(NB);
          while (left != 0u) {
            left &= left - 1u;
            const int kn = left != 0u ? __builtin_ctz(left) : k;
            const double* __restrict__ cn = cf + (long)kn * large_coef(NB);
            double qs = 0.0;
            double4v z[2];
            auto refill = [&](auto TI) {
              constexpr int t = decltype(TI)::value, ta = t + kRing;
              __builtin_amdgcn_sched_barrier(0);            // (the scheduler would put all of a class's loads in one place)
              fetch(w[t % kRing], ta < NT ? ck : cn, std::integral_constant<int, (ta < NT ? ta : ta - NT)>{});
            };
            static_for<0, NF>([&](auto II) {
              constexpr int i = II.value;
              z[i & 1] = double4v{0.0, 0.0, 0.0, 0.0};
              static_for<0, i + 1>([&](auto JI) {
                constexpr int j = JI.value, tl = i * (i + 1) / 2 + j;
                const double2v w0 = w[tl % kRing][0], w1 = w[tl % kRing][1];
                z[i & 1] = mfma_f64(w0.x, u[j][0], z[i & 1]);
                z[i & 1] = mfma_f64(w0.y, u[j][1], z[i & 1]);
                z[i & 1] = mfma_f64(w1.x, u[j][2], z[i & 1]);
                z[i & 1] = mfma_f64(w1.y, u[j][3], z[i & 1]);
                refill(std::integral_constant<int, tl>{});
                if constexpr (i > 0 && j == 0) {            // the row before: its products are done by now
#pragma unroll
                  for (int v = 0; v < 4; ++v) qs = fma(z[(i - 1) & 1][v], z[(i - 1) & 1][v], qs);
                }
              });
            });
            if constexpr (H > 0) {                          // lane row g: rows 4 h + g of the last block
              double zr[H];
#pragma unroll
              for (int h = 0; h < H; ++h) zr[h] = 0.0;
              static_for<0, NB * H>([&](auto RI) {
                constexpr int j = RI.value / H, h = RI.value % H, tl = NM + RI.value;
                const double2v w0 = w[tl % kRing][0], w1 = w[tl % kRing][1];
                zr[h] = mfma4_f64(w0.x, u[j][0], zr[h]);
                zr[h] = mfma4_f64(w0.y, u[j][1], zr[h]);
                zr[h] = mfma4_f64(w1.x, u[j][2], zr[h]);
                zr[h] = mfma4_f64(w1.y, u[j][3], zr[h]);
                refill(std::integral_constant<int, tl>{});
              });
#pragma unroll
              for (int v = 0; v < 4; ++v) qs = fma(z[(NF - 1) & 1][v], z[(NF - 1) & 1][v], qs);
#pragma unroll
              for (int h = 0; h < H; ++h) qs = fma(zr[h], zr[h], qs);
            } else {
#pragma unroll
              for (int v = 0; v < 4; ++v) qs = fma(z[(NF - 1) & 1][v], z[(NF - 1) & 1][v], qs);
            }
            sQ[k * kWave + 4 * n + g] = qs;                 // (added up by the reader: no chain of lane permutes per class)
            k = kn;
            ck = cn;
          }
          __builtin_amdgcn_s_setprio(2);
        }
        wave_lds_sync();
      }
      if constexpr (FINAL) {
        if (next < tile_hi) {
          frames.request(Yrow, abrow, next * kWave + 16 * wave + n, T, D, g);
          frames.mask = mvec[next + 1 < tile_hi ? next + 1 : next];
          if (cf) fetch_first(mnext);
        }
      }
      if (live != 0u) {
        // ---- posterior over the active classes: pi_k / det B_k * q_k^-D, mantissa / exponent form.  Lane row g takes the
        // live classes number g and g + 4; the largest exponent and the sum go over the lane rows. ----
        auto parts = [&](int k) {
          const double2 x0 = *reinterpret_cast<const double2*>(sQ + k * kWave + 4 * n);
          const double2 x1 = *reinterpret_cast<const double2*>(sQ + k * kWave + 4 * n + 2);
          return (x0.x + x0.y) + (x1.x + x1.y);
        };
        n2 = parts(K);
        const double n2c = fmax(n2, GSS_EPS_NORM_SQ);
        const double qfloor = GSS_EPS_Q * n2c;
        double rq[kRows], v[kRows];
        int kc[kRows], ex[kRows], emax = -(1 << 28);
        unsigned left = live;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          const unsigned l1 = left & (left - 1u), l2 = l1 & (l1 - 1u), l3 = l2 & (l2 - 1u);
          const unsigned mine = g == 0 ? left : g == 1 ? l1 : g == 2 ? l2 : l3;
          kc[r] = mine != 0u ? __builtin_ctz(mine) : -1;
          v[r] = 0.0;
          rq[r] = 0.0;
          ex[r] = -(1 << 28);
          if (r == 0 || left != 0u) {
            const int k = kc[r] < 0 ? 0 : kc[r];
            const double2 c = sC[k];
            const double q = cf ? parts(mine != 0u ? k : __builtin_ctz(live)) : n2;
            rq[r] = rcp_f64(fmax(q, qfloor));
            const double x = rq[r] * n2c;
            const double mu = __builtin_amdgcn_frexp_mant(x);
            const int eu = __builtin_amdgcn_frexp_exp(x);
            const double pw = ipow_rt(mu, D);              // >= 2^-32
            v[r] = c.x * __builtin_amdgcn_frexp_mant(pw);
            const bool a = mine != 0u && ((abits >> k) & 1u);
            ex[r] = a ? (int)c.y + eu * D + __builtin_amdgcn_frexp_exp(pw) : -(1 << 28);
            emax = ex[r] > emax ? ex[r] : emax;
          }
          left = l3 & (l3 - 1u);
        }
        emax = max_rows_i32(emax);
        double Z = 0.0;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
          int de = ex[r] - emax;
          de = de < -1100 ? -1100 : de;
          v[r] = ex[r] > -(1 << 28) ? ldexp(v[r], de) : 0.0;
          Z += v[r];
        }
        Z = sum_rows_f64(Z);
        const double rz = Z > 0.0 ? rcp_f64(Z) : 0.0;
        if constexpr (FINAL) {
          if (g == 0 && t < T && !(n2 >= GSS_EPS_NORM_SQ)) atomicOr(status, GSS_STATUS_ZERO_FRAME);
#pragma unroll
          for (int r = 0; r < kRows; ++r)
            if (kc[r] >= 0 && t < Tmax) grow[kc[r] * gk + t] = (float)(v[r] * rz);
          wave_lds_sync();                               // the parts have been read
        } else {
#pragma unroll
          for (int r = 0; r < kRows; ++r)
            if (kc[r] >= 0) {
              const double gm = v[r] * rz;
              sN[(wave * K + kc[r]) * 16 + n] += gm;
              sW[kc[r] * kWave + 16 * wave + n] = gm * rq[r];
            }
        }
      }
      if constexpr (!FINAL) {
        wave_lds_sync();                                 // the parts have been read
        double* dst = sT + (16 * wave + n) * P + 4 * g;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          *reinterpret_cast<double2*>(dst + 16 * b) = make_double2(u[b][0], u[b][1]);
          *reinterpret_cast<double2*>(dst + 16 * b + 2) = make_double2(u[b][2], u[b][3]);
        }
        __syncthreads();                                 // every frame and its weights are in place
        if (cf) fetch_first(next < tile_hi ? mnext : mq);
        __builtin_amdgcn_s_setprio(0);
        accumulate_large<NB, H, K>(sT, sW, role, mq, lane, acc);
        __builtin_amdgcn_s_setprio(2);
        buf ^= 1;
      }
      if (next >= tile_hi) break;
      tile = next;
      mq = mnext;
      mnext = tile + 1 < tile_hi ? __builtin_amdgcn_readfirstlane(frames.mask) : 0u;
      if constexpr (FINAL) mnext &= 0xffu << (8 * wave);
    }
  }
  if constexpr (!FINAL) {
    reduce_large<NB, H, K, large_red_classes(K, NB)>(acc, role, sBuf, part + (long)block * (2 * K) * num_items(D), D, lane);
    // class counts: the 64 frame columns in their order (written before the barriers of the reduction)
    if (threadIdx.x < K) {
      double sum = 0.0;
      for (int x = 0; x < kWave; ++x) sum += sN[((x >> 4) * K + threadIdx.x) * 16 + (x & 15)];
      npart[(long)block * K + threadIdx.x] = sum;
    }
  }
}

// In-place Gauss-Jordan inversion of the D x D Hermitian positive-definite matrix in (sMr, sMi), thread
// (i, j) = (tid / D, tid % D), all threads of the workgroup call it.  Returns det as mant * 2^exp.
__device__ __forceinline__ void gauss_jordan_large(double (*sMr)[33], double (*sMi)[33], int D, int i, int j, bool on,
                                                   uint32_t* status, uint32_t flag, double& detm, int& dete) {
  detm = 1.0;
  dete = 0;
  for (int p = 0; p < D; ++p) {
    double piv = sMr[p][p];
    if (!(piv > 1e-300)) {
      piv = 1e-300;
      if (threadIdx.x == 0) atomicOr(status, flag);
    }
    detm *= piv;
    dete += __builtin_amdgcn_frexp_exp(detm);
    detm = __builtin_amdgcn_frexp_mant(detm);
    const double rp = 1.0 / piv;
    double nr = 0.0, ni = 0.0;
    if (on) {
      const double air = sMr[i][p], aii = sMi[i][p];
      const double apr = sMr[p][j], api = sMi[p][j];
      if (i == p && j == p) {
        nr = rp;
      } else if (i == p) {
        nr = apr * rp; ni = api * rp;
      } else if (j == p) {
        nr = -air * rp; ni = -aii * rp;
      } else {
        nr = sMr[i][j] - (air * apr - aii * api) * rp;
        ni = sMi[i][j] - (air * api + aii * apr) * rp;
      }
    }
    __syncthreads();
    if (on) { sMr[i][j] = nr; sMi[i][j] = ni; }
    __syncthreads();
  }
}

// ----------------------------------------------------------------------------------------------
// Factor kernel, 9 <= D <= 32: one wavefront per (segment, frequency, class), a workgroup = the K classes of a
// (segment, frequency).  The D x D matrix sits in the registers of the wavefront: lane (a, b) = (lane / 8,
// lane % 8) holds the BS x BS block of rows a BS .. and columns b BS .. (BS = ceil(D / 8) = NB; rows and columns
// beyond D are those of the identity and stay so).  Elimination without pivoting (B is Hermitian positive definite after
// the loading; the product of the pivots is det B), in place: sweep p subtracts row p times a_ip / pivot from the rows i > p
// and leaves -a_ip / pivot in column p, so that the strictly lower triangle ends as that of M = the inverse of the unit
// lower factor, and the diagonal holds the pivots d.  W = d^-1/2 M.  The lanes that hold pivot row p
// publish it in the wavefront's LDS, every lane reads back the entries of its own columns and, conjugated for the pivot column,
// of its own rows.  Nothing is shared between wavefronts, so there is no workgroup barrier.
// A problem of the tail comes in many chunks (513 problems: the last one in 24, which one compute unit took 16 us to read while all
// others were done): its classes have a workgroup each, whose wavefronts take every K-th chunk; the first one goes on.
// Bound: latency, a chain of LDS round trip, reciprocal and update per sweep.  513 problems of 24 channels, 5 classes: 43 us (47 us
// with the pivot column published as well and reals in LDS; whole EM calls 0.3 % (16 channels) to 8 % (32 channels) slower), and
// 38 with the tail's chunks shared.
// ----------------------------------------------------------------------------------------------
template <int BS>
__global__ __launch_bounds__(kWave * GSS_MAX_K) void em_factor_large(
    const double* __restrict__ part, const double* __restrict__ npart,
    double* __restrict__ coef, double* __restrict__ cmant, int32_t* __restrict__ cexp, uint32_t* __restrict__ status,
    int D, int K, ChunkMap cmap, int weight_mode, unsigned sf0, unsigned n_whole) {
  constexpr int W = 8 * BS;                                // padded matrix size
  __shared__ __attribute__((aligned(16))) double2 sPiv[GSS_MAX_K][W];   // per wavefront: pivot row
  extern __shared__ __attribute__((aligned(16))) double sItems[];   // per wavefront: the class's packed sums, 2 M doubles
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // (from workgroup n_whole on: a class of a problem each, whose wavefronts share the sums)
  const bool shared = blockIdx.x >= n_whole;
  const unsigned extra = shared ? blockIdx.x - n_whole : 0u;
  const long sf = sf0 + (shared ? n_whole + extra / (unsigned)K : blockIdx.x);
  const int k = shared ? (int)(extra % (unsigned)K) : wave;
  const int a = lane >> 3, b = lane & 7;
  const int M = num_items(D);
  int C;
  const long slot0 = chunk_base(cmap, sf, C);
  double2* __restrict__ row = sPiv[wave];

  // class counts: lane l < K adds the chunks' counts of class l (in chunk order)
  double nl = 0.0;
  if (lane < K) nl = sum_chunks(npart + slot0 * K + lane, K, C);
  const double Nk = __shfl(nl, k, kWave);
  double Ntot = 0.0;
  for (int kk = 0; kk < K; ++kk) Ntot += __shfl(nl, kk, kWave);

  // R_k = sum over the chunks (in chunk order) of the packed partial sums: as one contiguous run per chunk, kFly of them in
  // flight, into the wavefront's LDS, then the lane's block from there; entry (i, j) with i > j is the conjugate of item (j, i)
  double mr[BS][BS], mi[BS][BS];
  {
    constexpr int kRun = (W * (W + 1) / 2 + kWave - 1) / kWave, kFly = BS == 4 ? 2 : 4;
    double2* __restrict__ sP = reinterpret_cast<double2*>(sItems) + wave * M;
    const double2* __restrict__ pc = reinterpret_cast<const double2*>(part) + (slot0 * K + k) * (long)M;
    double2 sum[kRun];
#pragma unroll
    for (int x = 0; x < kRun; ++x) sum[x] = make_double2(0.0, 0.0);
    const int first = shared ? wave : 0, step = shared ? K : 1;   // the chunks first, first + step, ...
    for (int c0 = first; c0 < C; c0 += kFly * step) {
      double2 v[kFly][kRun];
#pragma unroll
      for (int c = 0; c < kFly; ++c)
#pragma unroll
        for (int x = 0; x < kRun; ++x) {
          v[c][x] = make_double2(0.0, 0.0);
          if (c0 + c * step < C && lane + kWave * x < M) v[c][x] = pc[(long)(c0 + c * step) * K * M + lane + kWave * x];
        }
#pragma unroll
      for (int c = 0; c < kFly; ++c)
#pragma unroll
        for (int x = 0; x < kRun; ++x) {
          sum[x].x += v[c][x].x;
          sum[x].y += v[c][x].y;
        }
    }
#pragma unroll
    for (int x = 0; x < kRun; ++x)
      if (lane + kWave * x < M) sP[lane + kWave * x] = sum[x];
    if (shared) {                                          // the wavefronts' sums, in their order
      __syncthreads();
      if (wave != 0) return;
      for (int w = 1; w < K; ++w)
        for (int x = lane; x < M; x += kWave) {
          const double2 v = sP[w * M + x];
          sP[x].x += v.x;
          sP[x].y += v.y;
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int r = 0; r < BS; ++r)
#pragma unroll
      for (int c = 0; c < BS; ++c) {
        const int i = a * BS + r, j = b * BS + c;
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        const double2 v = sP[hi < D ? item_index(lo, hi, D) : 0];
        mr[r][c] = v.x;
        mi[r][c] = v.y;
      }
  }
  double trl = 0.0;
#pragma unroll
  for (int r = 0; r < BS; ++r)
#pragma unroll
    for (int c = 0; c < BS; ++c) {
      const int i = a * BS + r, j = b * BS + c;
      const bool in = i < D && j < D;
      mr[r][c] = in ? mr[r][c] : 0.0;
      mi[r][c] = in ? (i < j ? mi[r][c] : (i > j ? -mi[r][c] : 0.0)) : 0.0;
      if (r == c && a == b) trl += mr[r][c];
    }
  const double tr = wave_sum_f64(trl);
  // B = D R / max(N, eps); dead if its trace <= eps; else rescaled to trace D (= R * D / tr R); loading delta I
  const double trB = (double)D * tr / fmax(Nk, GSS_EPS_N);
  const bool dead = !(trB > GSS_EPS_N);
  const double sc = dead ? 0.0 : (double)D / tr;
#pragma unroll
  for (int r = 0; r < BS; ++r)
#pragma unroll
    for (int c = 0; c < BS; ++c) {
      const int i = a * BS + r, j = b * BS + c;
      const bool in = i < D && j < D;
      double vr = dead ? 0.0 : mr[r][c] * sc, vi = dead ? 0.0 : mi[r][c] * sc;
      if (i == j) {
        vr = dead ? 1.0 : vr;
        vi = 0.0;
        vr = in ? vr + GSS_DELTA : 1.0;                    // beyond D: the identity
      }
      mr[r][c] = vr;
      mi[r][c] = vi;
    }

  double detm = 1.0;
  int dete = 0;
  // (kept as a loop: unrolled, the 8 BS sweeps are straight-line code that every wavefront runs once, and the
  // kernel then waits for instruction fetches most of the time)
#pragma unroll 1
  for (int pg = 0; pg < 8; ++pg) {
    static_for<0, BS>([&](auto PP) {
      constexpr int pp = decltype(PP)::value;
      const int p = pg * BS + pp;
      if (p < D) {                                         // the same in every lane
        if (a == pg) {
#pragma unroll
          for (int c = 0; c < BS; ++c) row[b * BS + c] = make_double2(mr[pp][c], mi[pp][c]);
        }
        wave_lds_sync();
        double piv = row[p].x;
        double pr[BS], pim[BS], cr[BS], cim[BS];
#pragma unroll
        for (int c = 0; c < BS; ++c) {
          const double2 v = row[b * BS + c], h = row[a * BS + c];
          pr[c] = v.x; pim[c] = v.y;
          cr[c] = h.x; cim[c] = -h.y;                      // the pivot column below the pivot: what is left there is Hermitian
        }
        wave_lds_sync();                                   // read before the next sweep writes
        if (!(piv > 1e-300)) {
          piv = 1e-300;
          if (lane == 0) atomicOr(status, GSS_STATUS_NONPD_B);
        }
        detm *= piv;
        dete += __builtin_amdgcn_frexp_exp(detm);
        detm = __builtin_amdgcn_frexp_mant(detm);
        const double rp = rcp_f64(piv);
        // The rows below the pivot take m - (column entry)(row entry) / pivot; with pivot + 1 in place of the row entry of
        // the pivot column this leaves -(column entry) / pivot there.
        const bool pcol = b == pg;
        pr[pp] = pcol ? piv + 1.0 : pr[pp];
        pim[pp] = pcol ? 0.0 : pim[pp];
#pragma unroll
        for (int r = 0; r < BS; ++r) {
          const bool below = a > pg || (a == pg && r > pp);
          cr[r] = below ? cr[r] * rp : 0.0;
          cim[r] = below ? cim[r] * rp : 0.0;
        }
#pragma unroll
        for (int r = 0; r < BS; ++r)
#pragma unroll
          for (int c = 0; c < BS; ++c) {
            const double air = cr[r], aii = cim[r], apr = pr[c], api = pim[c];
            mr[r][c] -= air * apr - aii * api;
            mi[r][c] -= air * api + aii * apr;
          }
      }
    });
  }

  // W in the pass kernel's layout: the entry (i, j) = w of a tile is [[re, -im], [im, re]] of its real form, and these four are
  // neighbours there.  Zero above the diagonal and beyond D.
  if (a == b) {
#pragma unroll
    for (int r = 0; r < BS; ++r) row[a * BS + r].x = 1.0 / sqrt(fmax(mr[r][r], 1e-300));
  }
  wave_lds_sync();
  double* __restrict__ cf = coef + (sf * K + k) * (long)large_coef(BS);
#pragma unroll
  for (int r = 0; r < BS; ++r) {
    const int i = a * BS + r;
    const double ds = row[i].x;
#pragma unroll
    for (int c = 0; c < BS; ++c) {
      const int j = b * BS + c;
      const int bi = i >> 3, bj = j >> 3;
      if (bj <= bi) {
        const bool in = i < D && j <= i;
        const double re = in ? (i == j ? ds : mr[r][c] * ds) : 0.0;
        const double im = in && i != j ? mi[r][c] * ds : 0.0;
        double* __restrict__ dst = cf + 256 * (bi * (bi + 1) / 2 + bj) + 128 * (j & 1) + 2 * (16 * ((j & 7) >> 1) + 2 * (i & 7));
        *reinterpret_cast<double2*>(dst) = make_double2(re, -im);
        *reinterpret_cast<double2*>(dst + 2) = make_double2(im, re);
      }
    }
  }
  if (lane == 0) {
    const double pi = weight_mode == 1 ? Nk / fmax(Ntot, GSS_EPS_N) : 1.0 / (double)K;
    const double cst = fmax(pi, GSS_EPS_PI) / detm;
    cmant[sf * K + k] = __builtin_amdgcn_frexp_mant(cst);
    cexp[sf * K + k] = __builtin_amdgcn_frexp_exp(cst) - dete;
  }
}

// ----------------------------------------------------------------------------------------------
// Masked covariances, 9 <= D <= 32: the sums of the EM pass with two weights per frame, gamma of the target and the sum of the
// others.  Grid: blockIdx.x = chunk + C * (f + F * s).  Output: part[chunk][2][m][2] (0: target, 1: background).
// Bound: the fp64 matrix rate (24 channels: 48 products of 64 cycles per 16 frames, 63 us for 513 x 1500 by the counters); the
// next tile is requested before the sums.  513 x 1500 frames of 24 channels 164 -> 109 us (a lane with a few items, formed on
// the vector units, and a partial tile per wavefront at the end); whole call, 4 to 6 classes: 9 channels 175 -> 99 us, 16
// 208 -> 116, 24 247 -> 192, 32 484 -> 297 (both sides with a candidate's powers on all threads), 250 frames of 24 channels
// 139 -> 74.  4 H columns of the last block instead of 16: 9 channels 102 -> 87 us, 12 119 -> 111, 17 177 -> 166, 25 276 -> 253
// (513 x 1560).
// ----------------------------------------------------------------------------------------------
__host__ __device__ constexpr int cov_lds_doubles(int NB) { return 2 * (kWave * large_pitch(NB) + 2 * kWave); }

template <int NB, int H>
__global__ __launch_bounds__(kWave * kLargeWaves, 2) void mvdr_cov_large(
    gss_yview yv, const float* __restrict__ gamma, const int32_t* __restrict__ T_len,
    const int32_t* __restrict__ target, double* __restrict__ part, uint32_t* __restrict__ status,
    int F, int Tmax, int D, int K, ChunkMap cmap) {
  extern __shared__ __attribute__((aligned(16))) double lds_large[];
  constexpr int P = large_pitch(NB);
  constexpr int kBuf = kWave * P + 2 * kWave;               // one buffer: weights, then the tile
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int g = lane >> 4, n = lane & 15;
  long sf;
  int chunk, tiles_per_chunk;
  chunk_decode(cmap, blockIdx.x, sf, chunk, tiles_per_chunk);
  const int s = (int)((unsigned)sf / (unsigned)F);
  const int f = (int)((unsigned)sf % (unsigned)F);
  int T;
  const float2* __restrict__ Yrow = y_row(yv, T_len, s, f, D, Tmax, T);
  int tgt = target[s];
  if (tgt < 0 || tgt >= K) {
    if (threadIdx.x == 0 && chunk == 0 && f == 0) atomicOr(status, GSS_STATUS_BAD_TARGET);
    tgt = tgt < 0 ? 0 : K - 1;
  }
  const float* __restrict__ grow = gamma + ((long)s * K * F + f) * Tmax;
  const long gk = (long)F * Tmax;

  const LargeRole<NB, H> role(wave);
  LargeAcc<NB, H, 2> acc;
  acc.clear();
  const int tile_lo = chunk * tiles_per_chunk;
  int tile_hi = tile_lo + tiles_per_chunk;
  const int tile_end = (T + kWave - 1) / kWave;
  tile_hi = tile_hi < tile_end ? tile_hi : tile_end;
  LargeFrames<NB> frames;
  float gv[GSS_MAX_K];
  auto request = [&](int tile) {
    const int t = tile * kWave + 16 * wave + n;
    frames.request(Yrow, t, T, D, g);
    const float* __restrict__ p = grow + (t < T ? t : 0);
#pragma unroll
    for (int k = 0; k < GSS_MAX_K; ++k) gv[k] = p[k < K ? k * gk : 0];
  };
  if (tile_lo < tile_hi) request(tile_lo);
  int buf = 0;
  for (int tile = tile_lo; tile < tile_hi; ++tile) {
    double* sW = lds_large + buf * kBuf;                    // [2][64] weights
    double* sT = sW + 2 * kWave;                            // [64][P]
    const int t = tile * kWave + 16 * wave + n;
    double u[NB][4];
    frames.convert(u, t, T, D, g);
    double wt = 0.0, wb = 0.0;
#pragma unroll
    for (int k = 0; k < GSS_MAX_K; ++k)
      if (k < K) {
        if (k == tgt) wt = (double)gv[k];
        else wb += (double)gv[k];
      }
    if (tile + 1 < tile_hi) request(tile + 1);
    double* dst = sT + (16 * wave + n) * P + 4 * g;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      *reinterpret_cast<double2*>(dst + 16 * b) = make_double2(u[b][0], u[b][1]);
      *reinterpret_cast<double2*>(dst + 16 * b + 2) = make_double2(u[b][2], u[b][3]);
    }
    if (g < 2) sW[g * kWave + 16 * wave + n] = t < T ? (g == 0 ? wt : wb) : 0.0;
    __syncthreads();                                        // (one barrier per tile: the buffers take turns)
    accumulate_large<NB, H, 2>(sT, sW, role, 0x03030303u, lane, acc);
    buf ^= 1;
  }
  reduce_large<NB, H, 2, large_red_classes(2, NB)>(acc, role, lds_large, part + (long)blockIdx.x * 4 * num_items(D), D, lane);
}

// One workgroup per (segment, frequency), D*D active threads.  H[sf][r][d], pw[sf][r][2] as for D <= 8.
__global__ __launch_bounds__(1024) void mvdr_solve_large(
    const double* __restrict__ part, double2* __restrict__ H, double* __restrict__ pw,
    uint32_t* __restrict__ status, int D, ChunkMap cmap) {
  __shared__ double sKr[32][33], sKi[32][33], sBr[32][33], sBi[32][33], sMr[32][33], sMi[32][33];
  double (*sGr)[33] = sMr;   // G and then H overwrite the inverse once it has been consumed
  double (*sGi)[33] = sMi;
  const int M = num_items(D);
  const long sf = blockIdx.x;
  int C;
  const long slot0 = chunk_base(cmap, sf, C);
  const int tid = threadIdx.x;
  const int i = tid / D, j = tid % D;
  const bool on = tid < D * D;
  if (on && i <= j) {
    const int m = item_index(i, j, D);
    double kr = 0.0, ki = 0.0, br = 0.0, bi = 0.0;
    for (int c = 0; c < C; ++c) {
      const double* p = part + ((slot0 + c) * 2 * (long)M + m) * 2;  // [k = 0 target, 1 background][m][re, im]
      kr += p[0]; ki += p[1]; br += p[2 * M]; bi += p[2 * M + 1];
    }
    if (i == j) { ki = 0.0; bi = 0.0; }
    sKr[i][j] = kr; sKi[i][j] = ki; sBr[i][j] = br; sBi[i][j] = bi;
    if (i != j) { sKr[j][i] = kr; sKi[j][i] = -ki; sBr[j][i] = br; sBi[j][i] = -bi; }
  }
  __syncthreads();
  double trb = 0.0, trk = 0.0;
  for (int r = 0; r < D; ++r) { trb += sBr[r][r]; trk += sKr[r][r]; }
  if (!(trb > 0.0)) {
    if (trk > 0.0 && tid == 0) atomicOr(status, GSS_STATUS_NONPD_PHI);
    if (on) H[(sf * D + j) * D + i] = make_double2(0.0, 0.0);
    if (tid < D) { pw[(sf * D + tid) * 2 + 0] = 0.0; pw[(sf * D + tid) * 2 + 1] = 0.0; }
    return;
  }
  __syncthreads();
  if (on) {
    if (i == j) sBr[i][i] += GSS_DELTA_BF * trb / (double)D;
  }
  __syncthreads();
  if (on) { sMr[i][j] = sBr[i][j]; sMi[i][j] = sBi[i][j]; }
  __syncthreads();
  double detm;
  int dete;
  gauss_jordan_large(sMr, sMi, D, i, j, on, status, GSS_STATUS_NONPD_PHI, detm, dete);
  double gr = 0.0, gi = 0.0;
  if (on) {
    for (int m = 0; m < D; ++m) {
      const double ar = sMr[i][m], ai = sMi[i][m], br = sKr[m][j], bi = sKi[m][j];
      gr += ar * br - ai * bi;
      gi += ar * bi + ai * br;
    }
  }
  __syncthreads();
  if (on) { sGr[i][j] = gr; sGi[i][j] = gi; }
  __syncthreads();
  double tr = 0.0;
  for (int r = 0; r < D; ++r) tr += sGr[r][r];
  const double inv = 1.0 / (tr + GSS_EPS_TRACE);
  __syncthreads();
  if (on) {
    const double hr = sGr[i][j] * inv, hi = sGi[i][j] * inv;
    H[(sf * D + j) * D + i] = make_double2(hr, hi);
    sGr[i][j] = hr; sGi[i][j] = hi;
  }
  __syncthreads();
  // powers of candidate r: h_r^H Phi h_r; thread (a, r) = (i, j) forms its term Re(conj(h_ar) (Phi h_r)_a), then thread r adds
  // them in the order of a (every candidate on one thread, D^2 dependent steps: one segment of 24 channels 286 us, now 247)
  double tk = 0.0, tb = 0.0;
  if (on) {
    double tkr = 0.0, tki = 0.0, tbr = 0.0, tbi = 0.0;         // (Phi h_r)[a]
    for (int b = 0; b < D; ++b) {
      const double hr = sGr[b][j], hi = sGi[b][j];
      tkr += sKr[i][b] * hr - sKi[i][b] * hi;  tki += sKr[i][b] * hi + sKi[i][b] * hr;
      tbr += sBr[i][b] * hr - sBi[i][b] * hi;  tbi += sBr[i][b] * hi + sBi[i][b] * hr;
    }
    const double hr = sGr[i][j], hi = sGi[i][j];
    tk = hr * tkr + hi * tki;
    tb = hr * tbr + hi * tbi;
  }
  __syncthreads();
  if (on) {
    sKr[i][j] = tk;                                            // (the covariances have been used)
    sKi[i][j] = tb;
  }
  __syncthreads();
  if (tid < D) {
    double pk = 0.0, pb = 0.0;
    for (int a = 0; a < D; ++a) {
      pk += sKr[a][tid];
      pb += sKi[a][tid];
    }
    pw[(sf * D + tid) * 2 + 0] = pk;
    pw[(sf * D + tid) * 2 + 1] = pb;
  }
}

__global__ __launch_bounds__(256) void mvdr_apply_large(
    gss_yview yv, const double2* __restrict__ H, const int32_t* __restrict__ ref,
    const int32_t* __restrict__ T_len, float2* __restrict__ X, int F, int Tmax, int D, int C, int frames_per_chunk,
    int ref_per_f) {
  __shared__ double2 sh[GSS_MAX_D];
  const int chunk = blockIdx.x % C;
  const long sf = blockIdx.x / C;
  const int s = (int)(sf / F);
  int T;
  const float2* __restrict__ Yrow = y_row(yv, T_len, s, (int)(sf % F), D, Tmax, T);
  int r = ref[ref_per_f ? sf : (long)s];
  r = r < 0 ? 0 : (r >= D ? D - 1 : r);
  if (threadIdx.x < D) sh[threadIdx.x] = H[(sf * D + r) * D + threadIdx.x];
  __syncthreads();
  float2* __restrict__ Xrow = X + sf * (long)Tmax;
  const int t_lo = chunk * frames_per_chunk;
  int t_hi = t_lo + frames_per_chunk;
  t_hi = t_hi < Tmax ? t_hi : Tmax;
  for (int t = t_lo + threadIdx.x; t < t_hi; t += blockDim.x) {
    double xr = 0.0, xi = 0.0;
    if (t < T) {
      for (int d = 0; d < D; ++d) {
        const float2 v = Yrow[(long)t * D + d];
        const double2 h = sh[d];
        xr += h.x * (double)v.x + h.y * (double)v.y;
        xi += h.x * (double)v.y - h.y * (double)v.x;
      }
    }
    Xrow[t] = make_float2((float)xr, (float)xi);
  }
}

// Resident workgroup slots of a tile kernel with its dynamic LDS size.
template <typename Kern>
long large_slots(const gss_ctx* ctx, Kern kern, int lds_bytes) {
  int per_cu = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, kWave * kLargeWaves, (size_t)lds_bytes) != hipSuccess ||
      per_cu < 1)
    per_cu = 1;
  return (long)ctx->num_cu * per_cu;
}

// Scratch memory that a call may take before its problems share it in groups: some 20,000 problems of 9 to 16 channels and 8
// classes, forty rounds of workgroups, so that the launches of a group do not show.
constexpr size_t kLargeScratch = (size_t)1 << 30;

template <int K, int NB, int H>
int run_em_large(gss_ctx* ctx, const gss_yview& Y, const uint8_t* act, const int32_t* T_len, int S, int F, int Tmax,
                 int D, int iters, int weight_mode, float* gamma, hipStream_t st) {
  const long n_sf = (long)S * F;
  const int M = num_items(D);
  constexpr int lds_acc = large_lds_doubles(K, NB, false) * (int)sizeof(double);
  constexpr int lds_fin = large_lds_doubles(K, NB, true) * (int)sizeof(double);
  if (hipFuncSetAttribute((const void*)em_pass_large<K, NB, H, false>, hipFuncAttributeMaxDynamicSharedMemorySize,
                          lds_acc) != hipSuccess)
    return GSS_EHIP;
  // the factor kernel adds the chunks of every class in LDS (up to 68 KB: 8 classes of 32 channels); one limit for every call
  const int factor_lds = K * M * 2 * (int)sizeof(double);
  constexpr int factor_max = K * (8 * NB) * (8 * NB + 1) * (int)sizeof(double);
  if (hipFuncSetAttribute((const void*)em_factor_large<NB>, hipFuncAttributeMaxDynamicSharedMemorySize, factor_max) != hipSuccess)
    return GSS_EHIP;
  const int tiles = (Tmax + kWave - 1) / kWave;
  const ChunkMap acc_map = plan_chunk_map(large_slots(ctx, em_pass_large<K, NB, H, false>, lds_acc), n_sf, tiles, 1, 0, true);
  const ChunkMap fin_map = plan_chunk_map(large_slots(ctx, em_pass_large<K, NB, H, true>, lds_fin), n_sf, tiles, 1, 0, true);
  const long wgs_acc = chunk_map_wgs(acc_map, n_sf), wgs_fin = chunk_map_wgs(fin_map, n_sf);
  if (wgs_acc > 0x7fffffffL || wgs_fin > 0x7fffffffL || n_sf * K > 0x7fffffffL) return GSS_EUNSUPPORTED;
  if ((long)S * tiles > 0x7fffffffL) return GSS_EUNSUPPORTED;
  // Problems [p0, p1) in one go: working memory for `n` problems and `wgs` workgroups of the accumulating pass.
  struct Offsets { size_t cm, ce, part, npart, abyte, masks, end; };
  auto layout = [&](long n, long wgs) {
    Offsets q;
    q.cm = gss_align_up((size_t)n * K * large_coef(NB) * sizeof(double), 256);
    q.ce = gss_align_up(q.cm + (size_t)n * K * sizeof(double), 256);
    q.part = gss_align_up(q.ce + (size_t)n * K * sizeof(int32_t), 256);
    q.npart = gss_align_up(q.part + (size_t)wgs * M * K * 2 * sizeof(double), 256);
    q.abyte = gss_align_up(q.npart + (size_t)wgs * K * sizeof(double), 256);
    q.masks = gss_align_up(q.abyte + (size_t)S * Tmax, 256);
    q.end = gss_align_up(q.masks + (size_t)S * tiles * sizeof(uint32_t), 256);
    return q;
  };
  auto first_block = [](const ChunkMap& m, long p) {
    int count;
    return chunk_base(m, p, count);
  };
  long group = n_sf;                                       // problems in one go
  Offsets off = layout(n_sf, wgs_acc);
  // W's tiles are two to five times as large as the packed Hermitian coefficients (16 bytes per item, the items of a row in
  // groups of 8).  A call takes no more scratch than it would with these, or than kLargeScratch or the context's present scratch
  // if that is more: groups of problems share the memory.  The chunks of a problem stay the same, and with them every bit of
  // the result.  Scratch of a given size: what fits is what would fit with the packed coefficients, and what the header
  // promises to fit.
  int packed = 0;
  for (int r = 1; r <= D; ++r) packed += (r + 7) / 8 * 16;
  const size_t need = (size_t)n_sf * K * (packed * sizeof(double) + 12) + (size_t)wgs_acc * K * (M * 16 + 8) +
                      (size_t)S * (Tmax + tiles * sizeof(uint32_t));
  size_t most_scratch = ctx->scratch_cap;
  if (!ctx->scratch_fixed) {
    most_scratch = need > most_scratch ? need : most_scratch;
    most_scratch = kLargeScratch > most_scratch ? kLargeScratch : most_scratch;
  } else if (need > ctx->scratch_cap && n_sf * K * D * D > 3500000L) {
    return GSS_ETOOBIG;
  }
  const Offsets one = layout(1, acc_map.c_main > acc_map.c_tail ? acc_map.c_main : acc_map.c_tail);
  if (off.end > most_scratch && one.end > most_scratch) {  // (the activity alone fills it)
    group = 1;
    off = one;
    most_scratch = one.end;
  }
  for (long groups = 2; off.end > most_scratch && group > 1; ++groups) {
    group = (n_sf + groups - 1) / groups;
    long most = 0;
    for (long p0 = 0; p0 < n_sf; p0 += group) {
      const long p1 = p0 + group < n_sf ? p0 + group : n_sf;
      const long wgs = first_block(acc_map, p1) - first_block(acc_map, p0);
      most = wgs > most ? wgs : most;
    }
    off = layout(group, most);
  }
  int rc = gss_ensure_scratch(ctx, off.end);
  if (rc != GSS_OK) return rc;
  char* base = (char*)ctx->scratch;
  uint8_t* abyte = (uint8_t*)(base + off.abyte);
  uint32_t* masks = (uint32_t*)(base + off.masks);
  const dim3 block(kWave * kLargeWaves);
  hipLaunchKernelGGL(em_pack_activity<true>, dim3((unsigned)(S * tiles)), dim3(kWave), 0, st, Y, act, T_len, abyte, masks, K,
                     Tmax, tiles);
  for (long p0 = 0; p0 < n_sf; p0 += group) {
    const long p1 = p0 + group < n_sf ? p0 + group : n_sf;
    const unsigned np = (unsigned)(p1 - p0);
    // problems of the tail, in many chunks, have a workgroup per class in the factor kernel
    const long whole = acc_map.c_tail > 4 && acc_map.n_main < p1 ? (acc_map.n_main > p0 ? acc_map.n_main - p0 : 0) : np;
    const unsigned n_whole = (unsigned)whole;
    const long a0 = first_block(acc_map, p0), f0 = first_block(fin_map, p0);
    const unsigned na = (unsigned)(first_block(acc_map, p1) - a0), nf = (unsigned)(first_block(fin_map, p1) - f0);
    // (the kernels index by problem and workgroup of the whole call)
    double* coef = (double*)base - p0 * K * large_coef(NB);
    double* cm = (double*)(base + off.cm) - p0 * K;
    int32_t* ce = (int32_t*)(base + off.ce) - p0 * K;
    double* part = (double*)(base + off.part) - a0 * M * K * 2;
    double* npart = (double*)(base + off.npart) - a0 * K;
    for (int it = 0; it < iters; ++it) {
      gss_profile_begin(ctx, 0, st);
      hipLaunchKernelGGL((em_pass_large<K, NB, H, false>), dim3(na), block, lds_acc, st, Y, abyte, masks, T_len,
                         it == 0 ? (const double*)nullptr : coef, cm, ce, part, npart, (float*)nullptr, ctx->status, F, Tmax, D,
                         acc_map, (unsigned)a0);
      gss_profile_end(ctx, 0, st);
      gss_profile_begin(ctx, 1, st);
      hipLaunchKernelGGL(em_factor_large<NB>, dim3(n_whole + (np - n_whole) * K), dim3(kWave * K), factor_lds, st, part, npart, coef, cm, ce,
                         ctx->status, D, K, acc_map, weight_mode, (unsigned)p0, n_whole);
      gss_profile_end(ctx, 1, st);
    }
    hipLaunchKernelGGL((em_pass_large<K, NB, H, true>), dim3(nf), block, lds_fin, st, Y, abyte, masks, T_len,
                       iters == 0 ? (const double*)nullptr : coef, cm, ce, (double*)nullptr, (double*)nullptr, gamma, ctx->status,
                       F, Tmax, D, fin_map, (unsigned)f0);
  }
  if (hipGetLastError() != hipSuccess) return GSS_EHIP;
  return GSS_OK;
}

template <int K>
int dispatch_nb(gss_ctx* ctx, const gss_yview& Y, const uint8_t* act, const int32_t* T_len, int S, int F, int Tmax,
                int D, int iters, int weight_mode, float* gamma, hipStream_t st) {
  const int rest = large_rest(D, K);
  auto blocks = [&](auto NB) {
    constexpr int nb = decltype(NB)::value;
    return rest == 1   ? run_em_large<K, nb, 1>(ctx, Y, act, T_len, S, F, Tmax, D, iters, weight_mode, gamma, st)
           : rest == 2 ? run_em_large<K, nb, 2>(ctx, Y, act, T_len, S, F, Tmax, D, iters, weight_mode, gamma, st)
                       : run_em_large<K, nb, 0>(ctx, Y, act, T_len, S, F, Tmax, D, iters, weight_mode, gamma, st);
  };
  if (D <= 16) return blocks(std::integral_constant<int, 2>{});
  if (D <= 24) return blocks(std::integral_constant<int, 3>{});
  return blocks(std::integral_constant<int, 4>{});
}

template <int NB, int H>
int run_mvdr_large(gss_ctx* ctx, const gss_yview& Y, const float* gamma, const int32_t* T_len, int S, int F, int Tmax,
                   int D, int K, const int32_t* target, int32_t* ref, int ref_per_f, float2* X, hipStream_t st) {
  const long n_sf = (long)S * F;
  const int M = num_items(D);
  constexpr int lds = cov_lds_doubles(NB) * (int)sizeof(double);
  if (hipFuncSetAttribute((const void*)mvdr_cov_large<NB, H>, hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
    return GSS_EHIP;
  const int tiles = (Tmax + kWave - 1) / kWave;
  const ChunkMap cmap = plan_chunk_map(large_slots(ctx, mvdr_cov_large<NB, H>, lds), n_sf, tiles, 1, 0, true);
  const long wgs = chunk_map_wgs(cmap, n_sf);
  if (wgs > 0x7fffffffL) return GSS_EUNSUPPORTED;
  size_t o = 0;
  const size_t off_part = o; o = gss_align_up(o + (size_t)wgs * M * 4 * sizeof(double), 256);
  const size_t off_H = o;    o = gss_align_up(o + (size_t)n_sf * D * D * sizeof(double2), 256);
  const size_t off_pw = o;   o = gss_align_up(o + (size_t)n_sf * D * 2 * sizeof(double), 256);
  int rc = gss_ensure_scratch(ctx, o);
  if (rc != GSS_OK) return rc;
  char* base = (char*)ctx->scratch;
  double* part = (double*)(base + off_part);
  double2* filters = (double2*)(base + off_H);
  double* pw = (double*)(base + off_pw);
  hipLaunchKernelGGL((mvdr_cov_large<NB, H>), dim3((unsigned)wgs), dim3(kWave * kLargeWaves), lds, st, Y, gamma, T_len,
                     target, part, ctx->status, F, Tmax, D, K, cmap);
  const int sthreads = (D * D + 63) / 64 * 64;
  hipLaunchKernelGGL(mvdr_solve_large, dim3((unsigned)n_sf), dim3(sthreads), 0, st, part, filters, pw, ctx->status, D, cmap);
  gss_launch_mvdr_ref(pw, ref, ctx->status, S, F, D, ref_per_f, st);
  const int fpc = 1024;
  const int CA = (Tmax + fpc - 1) / fpc;
  if (n_sf * CA > 0x7fffffffL) return GSS_EUNSUPPORTED;
  hipLaunchKernelGGL(mvdr_apply_large, dim3((unsigned)(n_sf * CA)), dim3(256), 0, st, Y, filters, ref, T_len, X, F, Tmax, D,
                     CA, fpc, ref_per_f);
  if (hipGetLastError() != hipSuccess) return GSS_EHIP;
  return GSS_OK;
}

}  // namespace
