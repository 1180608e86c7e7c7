// Device-side building blocks shared by the EM and the MVDR kernels (internal, not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <type_traits>

#include "gss_internal.h"

namespace {

constexpr int kWave = 64;

// ----------------------------------------------------------------------------------------------
// fp64 helpers (no transcendental functions anywhere in the EM loop)
// ----------------------------------------------------------------------------------------------
__device__ __forceinline__ double rcp_f64(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  r = fma(fma(-x, r, 1.0), r, r);
  return r;
}

// One Newton step only: relative error about 2e-15 (the hardware estimate is good to 5e-8).  For the
// posterior's 1 / q and 1 / Z, where a few ulps change nothing that survives the fp32 output.
__device__ __forceinline__ double rcp_f64_fast(double x) {
  const double r = __builtin_amdgcn_rcp(x);
  return fma(fma(-x, r, 1.0), r, r);
}

// Sum of a double over the 64 lanes of the wavefront, the same value in every lane, in a fixed order.  Within
// a row of 16 lanes four butterfly steps through the lane-permute modifier of the vector move (on the two
// halves of the double): neighbours, pairs, the mirrored half of 8, the mirrored row; then the four row sums
// are read into scalar registers and added.  No LDS traffic (a shuffle goes through the LDS crossbar and costs
// a round trip per step).
__device__ __forceinline__ double wave_sum_f64(double v) {
  auto step = [](double x, auto CTRL) {
    constexpr int ctrl = decltype(CTRL)::value;
    const int lo = __double2loint(x), hi = __double2hiint(x);
    const int plo = __builtin_amdgcn_update_dpp(0, lo, ctrl, 0xf, 0xf, false);
    const int phi = __builtin_amdgcn_update_dpp(0, hi, ctrl, 0xf, 0xf, false);
    return x + __hiloint2double(phi, plo);
  };
  v = step(v, std::integral_constant<int, 0xB1>{});     // quad_perm [1, 0, 3, 2]
  v = step(v, std::integral_constant<int, 0x4E>{});     // quad_perm [2, 3, 0, 1]
  v = step(v, std::integral_constant<int, 0x141>{});    // row_half_mirror
  v = step(v, std::integral_constant<int, 0x140>{});    // row_mirror
  const int lo = __double2loint(v), hi = __double2hiint(v);
  double r[4];
#pragma unroll
  for (int q = 0; q < 4; ++q)
    r[q] = __hiloint2double(__builtin_amdgcn_readlane(hi, 16 * q), __builtin_amdgcn_readlane(lo, 16 * q));
  return (r[0] + r[1]) + (r[2] + r[3]);
}

// The values that lane 8 * (lane / 8) + N holds, in every lane of that group of 8: a row of 16 lanes is served by
// two lane-permute moves, each confined to one half of the row by its bank mask.  Every lane of the wavefront
// must be active.  (s_nop: a vector write of a source needs two wait states before the permute reads it.)
template <int N, int M>
__device__ __forceinline__ void class_row_bcast(const double (&src)[M], double (&dst)[M]) {
#define GSS_CLASS_BCAST(d, s)                                                       \
  "v_mov_b64_dpp %" #d ", %" #s " row_newbcast:%[lo] row_mask:0xf bank_mask:0x3\n\t" \
  "v_mov_b64_dpp %" #d ", %" #s " row_newbcast:%[hi] row_mask:0xf bank_mask:0xc\n\t"
  constexpr int m4 = M / 4 * 4;
#pragma unroll
  for (int m = 0; m < m4; m += 4)
    asm("s_nop 1\n\t" GSS_CLASS_BCAST(0, 4) GSS_CLASS_BCAST(1, 5) GSS_CLASS_BCAST(2, 6) GSS_CLASS_BCAST(3, 7)
        : "=&v"(dst[m]), "=&v"(dst[m + 1]), "=&v"(dst[m + 2]), "=&v"(dst[m + 3])
        : "v"(src[m]), "v"(src[m + 1]), "v"(src[m + 2]), "v"(src[m + 3]), [lo] "n"(N), [hi] "n"(N + 8));
#pragma unroll
  for (int m = m4; m < M; ++m)
    asm("s_nop 1\n\t" GSS_CLASS_BCAST(0, 1) : "=&v"(dst[m]) : "v"(src[m]), [lo] "n"(N), [hi] "n"(N + 8));
#undef GSS_CLASS_BCAST
}

template <int N>
__device__ __forceinline__ double ipow(double x) {
  if constexpr (N == 1) {
    return x;
  } else if constexpr (N % 2 == 0) {
    const double h = ipow<N / 2>(x);
    return h * h;
  } else {
    return x * ipow<N - 1>(x);
  }
}

// Compile-time loop: f(std::integral_constant<int, B>{}), ..., f(std::integral_constant<int, E_ - 1>{}).
template <int B, int E_, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (B < E_) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E_>(f);
  }
}

// Sums of N per-lane doubles over the 64 lanes of the wavefront, all at once and in a fixed order: six
// butterfly steps, and at each step a lane keeps only half of its values (of each pair of values one lane of
// the exchanging pair keeps the first and the other the second), so the work halves from step to step
// instead of every value paying six steps.  Afterwards lane l holds in v[j] the wavefront's total of value
// 64 j + transposed_index(l) (where that is below N; the other entries are meaningless).  The first four steps
// stay inside a row of 16 lanes and use the lane-permute modifier of the vector move (mirrored row, mirrored
// half, pairs, neighbours, in this order: each permutation leaves the bits that earlier steps selected on
// unchanged), the last two cross the rows with a shuffle.  Every lane of the wavefront must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_permute_f64(double x) {
  const int lo = __double2loint(x), hi = __double2hiint(x);
  const int plo = __builtin_amdgcn_update_dpp(0, lo, CTRL, 0xf, 0xf, false);
  const int phi = __builtin_amdgcn_update_dpp(0, hi, CTRL, 0xf, 0xf, false);
  return __hiloint2double(phi, plo);
}
__device__ __forceinline__ int transposed_index(int lane) {
  return (int)(__brev((unsigned)(lane & 15)) >> 28) | (lane & 48);
}
template <int N>
__device__ __forceinline__ void transpose_reduce(double (&v)[N], int lane) {
  auto step = [&](auto CNT, bool second, auto perm) {
    constexpr int n = decltype(CNT)::value;
    static_for<0, n / 2>([&](auto MI) {
      constexpr int m = MI.value;
      const double a = v[2 * m], b = v[2 * m + 1];
      const double keep = second ? b : a, send = second ? a : b;
      v[m] = keep + perm(send);
    });
    if constexpr (n & 1) {            // a value without a partner: both lanes keep its sum
      const double a = v[n - 1];
      v[n / 2] = a + perm(a);
    }
  };
  constexpr int n1 = (N + 1) / 2, n2 = (n1 + 1) / 2, n3 = (n2 + 1) / 2, n4 = (n3 + 1) / 2, n5 = (n4 + 1) / 2;
  step(std::integral_constant<int, N>{}, (lane & 8) != 0, [](double x) { return dpp_permute_f64<0x140>(x); });   // row_mirror
  step(std::integral_constant<int, n1>{}, (lane & 4) != 0, [](double x) { return dpp_permute_f64<0x141>(x); });  // row_half_mirror
  step(std::integral_constant<int, n2>{}, (lane & 2) != 0, [](double x) { return dpp_permute_f64<0x4E>(x); });   // quad_perm [2, 3, 0, 1]
  step(std::integral_constant<int, n3>{}, (lane & 1) != 0, [](double x) { return dpp_permute_f64<0xB1>(x); });   // quad_perm [1, 0, 3, 2]
  step(std::integral_constant<int, n4>{}, (lane & 16) != 0, [](double x) { return __shfl_xor(x, 16, kWave); });
  step(std::integral_constant<int, n5>{}, (lane & 32) != 0, [](double x) { return __shfl_xor(x, 32, kWave); });
}

// Position (row i, column j >= i, part: 0 diagonal, 1 real, 2 imaginary) of packed index idx.
__host__ __device__ constexpr int packed_i(int idx, int D) {
  int i = 0;
  for (int r = 1; r < D; ++r)
    if (idx >= gss_packed_row(r, D)) i = r;
  return i;
}
__host__ __device__ constexpr int packed_j(int idx, int D) {
  const int i = packed_i(idx, D);
  const int off = idx - gss_packed_row(i, D);
  return off == 0 ? i : i + 1 + (off - 1) / 2;
}
__host__ __device__ constexpr int packed_part(int idx, int D) {
  const int off = idx - gss_packed_row(packed_i(idx, D), D);
  return off == 0 ? 0 : 1 + ((off - 1) & 1);
}

// Entry IDX of the Hermitian outer product y y^H in the packed order (see gss_packed_row), fp64.
template <int D, int IDX>
__device__ __forceinline__ double packed_entry(const double (&yr)[D], const double (&yi)[D]) {
  constexpr int i = packed_i(IDX, D), j = packed_j(IDX, D), part = packed_part(IDX, D);
  if constexpr (part == 0) return yr[i] * yr[i] + yi[i] * yi[i];
  else if constexpr (part == 1) return yr[i] * yr[j] + yi[i] * yi[j];   // Re(y_i conj(y_j))
  else return yi[i] * yr[j] - yr[i] * yi[j];                            // Im(y_i conj(y_j))
}

// First frame of (segment s, frequency f) in the view and the number T of valid frames of the segment:
// T_len[s] (all Tmax frames if T_len is NULL) clipped to [0, Tmax] and to what the underlying array holds
// behind the segment's first frame.
__device__ __forceinline__ const float2* y_row(const gss_yview& v, const int32_t* __restrict__ T_len, int s, int f,
                                               int D, int Tmax, int& T) {
  long off = v.frame0 ? (long)v.frame0[s] : 0;
  off = off < 0 ? 0 : (off > v.t_limit ? v.t_limit : off);
  int t = T_len ? T_len[s] : Tmax;
  t = t < 0 ? 0 : (t > Tmax ? Tmax : t);
  const long room = v.t_limit - off;
  T = (long)t > room ? (int)room : t;
  return v.base + (long)s * v.s_stride + (long)f * v.f_stride + off * D;
}
__device__ __forceinline__ int y_frames(const gss_yview& v, const int32_t* __restrict__ T_len, int s, int Tmax) {
  int T;
  (void)y_row(v, T_len, s, 0, 1, Tmax, T);
  return T;
}

// Orders this wavefront's LDS traffic: everything written before is visible to every lane of the
// wavefront after.  (The LDS executes one wavefront's instructions in order; this only has to stop the
// compiler from moving accesses across and make it wait for outstanding ones.)
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A class whose bit is clear in a tile's activity mask has posterior 0 in every frame of the tile and adds nothing
// to any sum: the pass kernels skip its arithmetic for the whole tile under wave-uniform branches.
// Activity in the form the pass kernels read: abyte[s][t] has bit k set when class k may be active in frame t
// (a_{t,k} of Eq. (5); 0 at t >= T_len[s]), tmask[s][tile] is the OR of the bytes of the tile's 64 frames, or (GROUPS) four
// bytes, those of its groups of 16 frames.
// Grid: one wavefront per (segment, tile).
template <bool GROUPS>
__global__ __launch_bounds__(kWave) void em_pack_activity(
    gss_yview yv, const uint8_t* __restrict__ act, const int32_t* __restrict__ T_len, uint8_t* __restrict__ abyte,
    uint32_t* __restrict__ tmask, int K, int Tmax, int tiles) {
  const int s = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int lane = threadIdx.x;
  const int T = y_frames(yv, T_len, s, Tmax);
  const int t = tile * kWave + lane;
  unsigned b = 0;
  if (t < T)
    for (int k = 0; k < K; ++k) b |= (act[((long)s * K + k) * Tmax + t] != 0 ? 1u : 0u) << k;
  if (t < Tmax) abyte[(long)s * Tmax + t] = (uint8_t)b;
  if constexpr (GROUPS) b <<= 8 * (lane >> 4);
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) b |= (unsigned)__shfl_xor((int)b, off, kWave);
  if (lane == 0) tmask[(long)s * tiles + tile] = b;
}

// The double-precision FMA with the row-broadcast selector on its first factor: acc += c[lane n of the row] * p.  Every lane of the
// wavefront must be active (the selector reads other lanes).  The instruction is written as an asm statement, which hides it
// from the compiler's hazard handling: a lane-selecting instruction must not issue within two wait states of a vector
// instruction that writes one of its registers, so a statement starts with two idle states.
//
// q[e mod 3] += c[lane e of the row] * P[e] for e = 0 .. NG - 1 (16, or what is left of D * D entries: 9, 4, 1) in
// one statement: between separate statements the compiler puts an idle state in front of every third FMA, which
// costs a wavefront an issue slot like any other instruction.  With three accumulators in turn each is read two issue slots
// after it was written, and the two idle states in front separate the first FMA from the last write of its registers.
template <int NG>
__device__ __forceinline__ void fma_bcast_chain(double (&q)[3], double c, const double (&P)[NG]) {
  static_assert(NG == 16 || NG == 9 || NG == 4 || NG == 1, "entries of a block of 16");
#define GSS_BCAST_FMA(acc, e) "v_fmac_f64_dpp %[" #acc "], %[c], %[p" #e "] row_newbcast:" #e " row_mask:0xf bank_mask:0xf\n\t"
  if constexpr (NG == 16)
    asm("s_nop 1\n\t"
        GSS_BCAST_FMA(q0, 0) GSS_BCAST_FMA(q1, 1) GSS_BCAST_FMA(q2, 2) GSS_BCAST_FMA(q0, 3)
        GSS_BCAST_FMA(q1, 4) GSS_BCAST_FMA(q2, 5) GSS_BCAST_FMA(q0, 6) GSS_BCAST_FMA(q1, 7)
        GSS_BCAST_FMA(q2, 8) GSS_BCAST_FMA(q0, 9) GSS_BCAST_FMA(q1, 10) GSS_BCAST_FMA(q2, 11)
        GSS_BCAST_FMA(q0, 12) GSS_BCAST_FMA(q1, 13) GSS_BCAST_FMA(q2, 14) GSS_BCAST_FMA(q0, 15)
        : [q0] "+v"(q[0]), [q1] "+v"(q[1]), [q2] "+v"(q[2])
        : [c] "v"(c), [p0] "v"(P[0]), [p1] "v"(P[1]), [p2] "v"(P[2]), [p3] "v"(P[3]), [p4] "v"(P[4]), [p5] "v"(P[5]),
          [p6] "v"(P[6]), [p7] "v"(P[7]), [p8] "v"(P[8]), [p9] "v"(P[9]), [p10] "v"(P[10]), [p11] "v"(P[11]),
          [p12] "v"(P[12]), [p13] "v"(P[13]), [p14] "v"(P[14]), [p15] "v"(P[15]));
  else if constexpr (NG == 9)
    asm("s_nop 1\n\t"
        GSS_BCAST_FMA(q0, 0) GSS_BCAST_FMA(q1, 1) GSS_BCAST_FMA(q2, 2) GSS_BCAST_FMA(q0, 3) GSS_BCAST_FMA(q1, 4)
        GSS_BCAST_FMA(q2, 5) GSS_BCAST_FMA(q0, 6) GSS_BCAST_FMA(q1, 7) GSS_BCAST_FMA(q2, 8)
        : [q0] "+v"(q[0]), [q1] "+v"(q[1]), [q2] "+v"(q[2])
        : [c] "v"(c), [p0] "v"(P[0]), [p1] "v"(P[1]), [p2] "v"(P[2]), [p3] "v"(P[3]), [p4] "v"(P[4]), [p5] "v"(P[5]),
          [p6] "v"(P[6]), [p7] "v"(P[7]), [p8] "v"(P[8]));
  else if constexpr (NG == 4)
    asm("s_nop 1\n\t"
        GSS_BCAST_FMA(q0, 0) GSS_BCAST_FMA(q1, 1) GSS_BCAST_FMA(q2, 2) GSS_BCAST_FMA(q0, 3)
        : [q0] "+v"(q[0]), [q1] "+v"(q[1]), [q2] "+v"(q[2])
        : [c] "v"(c), [p0] "v"(P[0]), [p1] "v"(P[1]), [p2] "v"(P[2]), [p3] "v"(P[3]));
  else
    asm("s_nop 1\n\t" GSS_BCAST_FMA(q0, 0) : [q0] "+v"(q[0]) : [c] "v"(c), [p0] "v"(P[0]));
#undef GSS_BCAST_FMA
}

// acc[b] += sum over n of w[lane n of the row] * x[b][n], n = 0 .. 15, b = 0 .. NB - 1 (1 to 4), with the
// accumulators in turn, so that an FMA does not wait for the one before it (one accumulator: three partial sums).  Statements of
// 16 FMAs or fewer, each with the two idle states in front (a statement may be moved up to the write of w).
template <int NB, int n0>
__device__ __forceinline__ void fma_bcast_rows_4(double (&acc)[NB], double w, const double (&x)[NB][16]) {
#define GSS_ROW_FMA(a, p, n) "v_fmac_f64_dpp %[a" #a "], %[w], %[x" #a #p "] row_newbcast:%[n" #n "] row_mask:0xf bank_mask:0xf\n\t"
#define GSS_ROW_IN(b) [x##b##0] "v"(x[b][n0]), [x##b##1] "v"(x[b][n0 + 1]), [x##b##2] "v"(x[b][n0 + 2]), [x##b##3] "v"(x[b][n0 + 3])
#define GSS_ROW_LANES [n0] "n"(n0), [n1] "n"(n0 + 1), [n2] "n"(n0 + 2), [n3] "n"(n0 + 3)
  if constexpr (NB == 4)
    asm("s_nop 1\n\t"
        GSS_ROW_FMA(0, 0, 0) GSS_ROW_FMA(1, 0, 0) GSS_ROW_FMA(2, 0, 0) GSS_ROW_FMA(3, 0, 0)
        GSS_ROW_FMA(0, 1, 1) GSS_ROW_FMA(1, 1, 1) GSS_ROW_FMA(2, 1, 1) GSS_ROW_FMA(3, 1, 1)
        GSS_ROW_FMA(0, 2, 2) GSS_ROW_FMA(1, 2, 2) GSS_ROW_FMA(2, 2, 2) GSS_ROW_FMA(3, 2, 2)
        GSS_ROW_FMA(0, 3, 3) GSS_ROW_FMA(1, 3, 3) GSS_ROW_FMA(2, 3, 3) GSS_ROW_FMA(3, 3, 3)
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2]), [a3] "+v"(acc[3])
        : [w] "v"(w), GSS_ROW_IN(0), GSS_ROW_IN(1), GSS_ROW_IN(2), GSS_ROW_IN(3), GSS_ROW_LANES);
  else if constexpr (NB == 3)
    asm("s_nop 1\n\t"
        GSS_ROW_FMA(0, 0, 0) GSS_ROW_FMA(1, 0, 0) GSS_ROW_FMA(2, 0, 0) GSS_ROW_FMA(0, 1, 1) GSS_ROW_FMA(1, 1, 1) GSS_ROW_FMA(2, 1, 1)
        GSS_ROW_FMA(0, 2, 2) GSS_ROW_FMA(1, 2, 2) GSS_ROW_FMA(2, 2, 2) GSS_ROW_FMA(0, 3, 3) GSS_ROW_FMA(1, 3, 3) GSS_ROW_FMA(2, 3, 3)
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1]), [a2] "+v"(acc[2])
        : [w] "v"(w), GSS_ROW_IN(0), GSS_ROW_IN(1), GSS_ROW_IN(2), GSS_ROW_LANES);
  else
    asm("s_nop 1\n\t"
        GSS_ROW_FMA(0, 0, 0) GSS_ROW_FMA(1, 0, 0) GSS_ROW_FMA(0, 1, 1) GSS_ROW_FMA(1, 1, 1)
        GSS_ROW_FMA(0, 2, 2) GSS_ROW_FMA(1, 2, 2) GSS_ROW_FMA(0, 3, 3) GSS_ROW_FMA(1, 3, 3)
        : [a0] "+v"(acc[0]), [a1] "+v"(acc[1])
        : [w] "v"(w), GSS_ROW_IN(0), GSS_ROW_IN(1), GSS_ROW_LANES);
#undef GSS_ROW_FMA
#undef GSS_ROW_IN
#undef GSS_ROW_LANES
}
template <int NB>
__device__ __forceinline__ void fma_bcast_rows(double (&acc)[NB], double w, const double (&x)[NB][16]) {
  static_assert(NB >= 1 && NB <= 4, "blocks of 16 entries");
  if constexpr (NB == 1) {
    double t[3] = {acc[0], 0.0, 0.0};
    fma_bcast_chain<16>(t, w, x[0]);
    acc[0] = t[0] + (t[1] + t[2]);
  } else {
    fma_bcast_rows_4<NB, 0>(acc, w, x);
    fma_bcast_rows_4<NB, 4>(acc, w, x);
    fma_bcast_rows_4<NB, 8>(acc, w, x);
    fma_bcast_rows_4<NB, 12>(acc, w, x);
  }
}

// Sums of N per-lane doubles over the four rows of 16 lanes (lane l of every row belongs together), in a fixed order: two
// exchange steps, at each of which a lane keeps one value of every pair, by the instructions that swap halves (rows) of two
// registers.  Afterwards lane l of row q holds in v[j] the total of value row_sum_index(q, j) (where that is below N).
__device__ __forceinline__ int row_sum_index(int q, int j) { return 4 * j + ((q & 1) << 1 | (q >> 1 & 1)); }
template <int N>
__device__ __forceinline__ void row_sums(double (&v)[N]) {
  auto step = [&](auto CNT, auto HALVES) {
    constexpr int n = decltype(CNT)::value;
    static_for<0, (n + 1) / 2>([&](auto MI) {
      constexpr int m = MI.value;
      const double a = v[2 * m], b = 2 * m + 1 < n ? v[2 * m + 1 < n ? 2 * m + 1 : 0] : 0.0;
      unsigned al = __double2loint(a), ah = __double2hiint(a), bl = __double2loint(b), bh = __double2hiint(b);
      if constexpr (decltype(HALVES)::value) {
        const auto lo = __builtin_amdgcn_permlane32_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        v[m] = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
      } else {
        const auto lo = __builtin_amdgcn_permlane16_swap(al, bl, false, false), hi = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
        v[m] = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
      }
    });
  };
  step(std::integral_constant<int, N>{}, std::true_type{});
  step(std::integral_constant<int, (N + 1) / 2>{}, std::false_type{});
}

// Wave-uniform test of bit k of `mask`, re-evaluated from the one scalar register that holds the mask at every
// use (the empty asm statement keeps the compiler from caching the K booleans in scalar register pairs).
__device__ __forceinline__ bool class_on(unsigned mask, int k) {
  asm volatile("" : "+s"(mask));
  return (mask >> k) & 1u;
}

// A workgroup of the EM's pass kernel and of the MVDR covariances is kPassWaves wavefronts; each wavefront owns whole tiles of 64
// frames and a private LDS region.
//
// The covariances of a tile: lane = (frame group tg, lane type i), D lane types and 64 / D frame groups (lanes left over idle along).
// Lane type i owns D of the D * D reals of the packed Hermitian matrix: Re and Im of y_i conj(y_b), b = (i + d) mod D, for the
// circular distances d = 1 .. (D - 1) / 2, the real diagonal entry |y_i|^2, and for even D one half of the pair at distance
// D / 2: Re of y_i conj(y_(i + D/2)) for i < D / 2 and Im of y_(i - D/2) conj(y_i) otherwise.  Both halves are
// y_i.re * a + y_i.im * b of a second operand (a, b) = y_(i + D/2) or -i y_(i - D/2), which the lane reads from the tile (a
// row carries the turned copies of the lower half), so every lane type runs the same instructions.  The pairs at circular
// distances up to D / 2 are all pairs once; where b < i the slot holds the conjugate of the stored (upper-triangle) entry,
// i.e. its imaginary part with the opposite sign.
//
// A row is D complex channels, then the turned copies, in 16-byte units.  D = 8: 12 units and one of padding, a group takes 8
// consecutive frames: LDS delivers 256 bytes per cycle, rows 8 * 208 bytes apart are 128 modulo 256, and a 16-byte read of the
// wavefront's 8 rows takes 4 cycles (frames tg, tg + 8, ...: 9 cycles; calls of one segment 1 to 9 % slower).  D < 8: frames
// tg, tg + 64 / D, ..., no padding: the rows read together are one run of memory (odd D) or start at an odd multiple of 16
// bytes (D = 2 and 6).
constexpr int kPassWaves = 4;
template <int D>
struct TileLayout {
  static_assert(D >= 1 && D <= 8, "channels of the tile kernels");
  static constexpr bool even = D % 2 == 0;
  static constexpr int full = (D - 1) / 2;                  // circular distances whose pairs a lane type owns in full
  static constexpr int reads = 1 + full + (even ? 1 : 0);   // channels that a lane reads per frame
  static constexpr int turned = 2 * D;                      // offset of the turned copies within a row (doubles)
  static constexpr int pad = D == 8 ? 2 : 0;
  static constexpr int row = 2 * D + (even ? D : 0) + pad;  // doubles per frame row
  static constexpr int groups = kWave / D;
  static constexpr int steps = kWave / groups;              // frames that every group has
  static constexpr int rest = kWave - groups * steps;       // groups that have one more
  static constexpr bool blocked = D == 8;                   // a group's frames: consecutive, or `groups` apart
  __host__ __device__ static constexpr int first(int tg) { return blocked ? steps * tg : tg; }
  static constexpr int next = blocked ? 1 : groups;         // rows from one frame of a group to its next
  static_assert(!blocked || rest == 0, "consecutive frames need equal groups");
};

// Writes one frame row of the y tile: channel d at 2 d and the turned copies of the lower half of the channels.
template <int D>
__device__ __forceinline__ void store_tile_row(double* __restrict__ row, const double (&yr)[D], const double (&yi)[D]) {
  using L = TileLayout<D>;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    *reinterpret_cast<double2*>(&row[2 * d]) = make_double2(yr[d], yi[d]);
    if (L::even && d < D / 2) *reinterpret_cast<double2*>(&row[L::turned + 2 * d]) = make_double2(yi[d], -yr[d]);
  }
}

// Offsets within a row of the channels that lane type i reads: itself, i + 1, ..., and for even D the second operand of the
// pair at distance D / 2.
template <int D>
__device__ __forceinline__ int tile_operand(int i, int n) {
  using L = TileLayout<D>;
  if (n <= L::full) return 2 * (i + n < D ? i + n : i + n - D);
  return i < D / 2 ? 2 * (i + D / 2) : L::turned + 2 * (i - D / 2);
}
// The lane type's D entries of a frame from the operands it has read.
template <int D>
__device__ __forceinline__ void tile_entries(const double2 (&y)[TileLayout<D>::reads], double (&e)[D]) {
  using L = TileLayout<D>;
  const double2 x = y[0];
#pragma unroll
  for (int d = 0; d < L::full; ++d) {
    const double2 b = y[1 + d];
    e[2 * d] = x.x * b.x + x.y * b.y;
    e[2 * d + 1] = x.y * b.x - x.x * b.y;
  }
  e[2 * L::full] = x.x * x.x + x.y * x.y;
  if constexpr (L::even) e[D - 1] = x.x * y[L::reads - 1].x + x.y * y[L::reads - 1].y;
}

struct SlotEntry { int i, j, part, sign; };     // part: 0 real diagonal, 1 Re, 2 Im
__host__ __device__ constexpr SlotEntry slot_entry(int i, int n, int D) {
  const int full = (D - 1) / 2;
  if (n < 2 * full) {
    const int part = 1 + (n & 1), b = (i + n / 2 + 1) % D;
    if (i < b) return SlotEntry{i, b, part, 1};
    return SlotEntry{b, i, part, part == 2 ? -1 : 1};
  }
  if (n == 2 * full) return SlotEntry{i, i, 0, 1};
  return i < D / 2 ? SlotEntry{i, i + D / 2, 1, 1} : SlotEntry{i - D / 2, i, 2, 1};
}
// Packed index (gss_packed_row order) and sign of slot n of lane type i, at [n * D + i].
template <int D>
struct SlotTable { short index[kWave]; signed char sign[kWave]; };
template <int D>
constexpr SlotTable<D> make_slot_table() {
  SlotTable<D> t{};
  for (int o = 0; o < kWave; ++o) { t.index[o] = -1; t.sign[o] = 1; }
  for (int o = 0; o < D * D; ++o) {
    const SlotEntry e = slot_entry(o % D, o / D, D);
    t.index[o] = (short)(gss_packed_row(e.i, D) + (e.part == 0 ? 0 : 1 + 2 * (e.j - e.i - 1) + (e.part - 1)));
    t.sign[o] = (signed char)e.sign;
  }
  return t;
}

// The covariances of a tile: lane (tg, i) accumulates acc[n][k] += w_k[r] * (slot n of lane type i)[r] over the frames r of its group.
// sY: [64][TileLayout<D>::row] doubles, sW: [64][WS] doubles (two weights per frame: target and background).
template <int D, int WS>
__device__ __forceinline__ void accumulate_tile(const double* __restrict__ sY, const double* __restrict__ sW,
                                                int tg, int i, double (&acc)[D][2]) {
  using L = TileLayout<D>;
  int o[L::reads];
#pragma unroll
  for (int n = 0; n < L::reads; ++n) o[n] = tile_operand<D>(i, n);
  auto frame = [&](int r) {
    double w[2], e[D];
    double2 y[L::reads];
#pragma unroll
    for (int k = 0; k < 2; ++k) w[k] = sW[r * WS + k];
#pragma unroll
    for (int n = 0; n < L::reads; ++n) y[n] = *reinterpret_cast<const double2*>(&sY[r * L::row + o[n]]);
    tile_entries<D>(y, e);
#pragma unroll
    for (int n = 0; n < D; ++n)
#pragma unroll
      for (int k = 0; k < 2; ++k) acc[n][k] = fma(w[k], e[n], acc[n][k]);
  };
#pragma unroll 2
  for (int j = 0; j < L::steps; ++j) frame(L::first(tg) + j * L::next);
  if constexpr (L::rest > 0) {
    if (tg < L::rest) frame(tg + L::steps * L::next);
  }
}

// Reduction of the per-lane accumulators of a workgroup of kPassWaves wavefronts into packed partial
// sums: out[k * E + packed index] for both matrices k of size D.  Sums are taken in a fixed order (frame
// groups ascending, then wavefronts ascending).
//   wbuf: LDS private to the calling wavefront, reduce_wave_doubles(D) doubles (its tile region);
//   red:  LDS scratch of the workgroup, kPassWaves * 128 doubles, may overlap the wbuf regions.
// The function starts with a barrier (every wavefront is done with its tiles).  First every wavefront
// sums over its frame groups through its own LDS region: entry n of all lanes goes out as one contiguous
// row (lane = D tg + i), and lane o = D n + i reads the values of slot (i, n) back (lanes from D * D on: the last
// slot once more).  Then the wavefronts' sums meet in `red`.
constexpr int kReduceRow = 72;                         // doubles per row of 64 (+ 8: spreads the banks)
__host__ __device__ constexpr int reduce_wave_doubles(int D) { return 2 * D * kReduceRow; }
template <int D>
__device__ __forceinline__ void reduce_and_store_partials(const double (&acc)[D][2], double* wbuf, double* red, double* __restrict__ out,
                                                          int lane, int wave) {
  constexpr int E = D * D;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int n = 0; n < D; ++n) wbuf[(k * D + n) * kReduceRow + lane] = acc[n][k];
  wave_lds_sync();
  const int o = lane < E ? lane : E - 1;
  const int n = o / D, i = o - n * D;
  double S[2] = {0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int tg = 0; tg < TileLayout<D>::groups; ++tg) S[k] += wbuf[(k * D + n) * kReduceRow + tg * D + i];
  __syncthreads();                           // the private regions are free: `red` may overlap them
#pragma unroll
  for (int k = 0; k < 2; ++k) red[(wave * 2 + k) * 64 + lane] = S[k];
  __syncthreads();
  for (int x = threadIdx.x; x < 2 * 64; x += kWave * kPassWaves) {
    const int k = x / 64, slot = x % 64;
    double sum = 0.0;
#pragma unroll
    for (int w = 0; w < kPassWaves; ++w) sum += red[(w * 2 + k) * 64 + slot];
    static constexpr SlotTable<D> kSlots = make_slot_table<D>();
    if (slot < E) out[k * E + kSlots.index[slot]] = kSlots.sign[slot] < 0 ? -sum : sum;
  }
}

// Sum of n values src[0], src[stride], ... in their order, eight loads in flight (in a plain loop every one waits out a memory
// latency before the next goes out; the problems of a launch's tail have the most chunks, and everything waits for them).
__device__ __forceinline__ double sum_chunks(const double* __restrict__ src, long stride, int n) {
  double sum = 0.0;
  for (int c0 = 0; c0 < n; c0 += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = c0 + u < n ? src[(c0 + u) * stride] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) sum += v[u];
  }
  return sum;
}

// Workgroups of `threads` threads of kernel `kern` that one compute unit holds at a time (`dflt` if the
// runtime cannot say).
template <typename Kern>
inline int resident_wgs(Kern kern, int threads, int dflt, size_t lds_bytes = 0) {
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kern, threads, lds_bytes) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    n = dflt;
  }
  return n;
}

// How the (segment, frequency) problems are cut into workgroups.  The first n_main problems get c_main
// chunks of tpc_main tiles each; the remaining ones (the tail that would otherwise run alone on an almost
// empty chip after the last full round of workgroups) are cut finer, into c_tail chunks of tpc_tail tiles.
// Workgroup b writes partial-sum slot b.
struct ChunkMap {
  int n_main, c_main, tpc_main, c_tail, tpc_tail;
};
__host__ __device__ inline void chunk_decode(const ChunkMap& m, unsigned b, long& sf, int& chunk, int& tpc) {
  // 32-bit arithmetic: the grid has fewer than 2^31 workgroups
  const unsigned main_wgs = (unsigned)m.n_main * (unsigned)m.c_main;
  if (b < main_wgs) {
    sf = (long)(b / (unsigned)m.c_main);
    chunk = (int)(b % (unsigned)m.c_main);
    tpc = m.tpc_main;
  } else {
    const unsigned r = b - main_wgs;
    sf = (long)((unsigned)m.n_main + r / (unsigned)m.c_tail);
    chunk = (int)(r % (unsigned)m.c_tail);
    tpc = m.tpc_tail;
  }
}
__host__ __device__ inline long chunk_base(const ChunkMap& m, long sf, int& count) {
  if (sf < m.n_main) {
    count = m.c_main;
    return sf * m.c_main;
  }
  count = m.c_tail;
  return (long)m.n_main * m.c_main + (sf - m.n_main) * m.c_tail;
}

inline long chunk_map_wgs(const ChunkMap& m, long n_sf) {
  return (long)m.n_main * m.c_main + (n_sf - m.n_main) * m.c_tail;
}

// Chunking of n_sf problems of `tiles` tiles each for a kernel with `slots` resident workgroups; chunks are
// multiples of `round_up` tiles.  Splitting a problem over several workgroups costs a partial-sum round
// trip and a second reduction, so it is done only as far as needed to fill the slots (tpc_override > 0
// fixes the tiles per chunk of the main part instead).  Tail: if the workgroups left over after the last
// full round of slots fill less than a quarter of the chip, the problems they belong to are cut finer so
// that the remainder spreads out.
inline ChunkMap plan_chunk_map(long slots, long n_sf, int tiles, int round_up, int tpc_override, bool allow_tail) {
  ChunkMap m;
  auto chunks_for = [&](int tpc) { return (tiles + tpc - 1) / tpc; };
  auto tpc_for = [&](long c) {
    int tpc = (int)((tiles + c - 1) / c);
    tpc = (tpc + round_up - 1) / round_up * round_up;
    return tpc;
  };
  long c_target = (slots + n_sf - 1) / n_sf;
  if (c_target < 1) c_target = 1;
  m.tpc_main = tpc_override > 0 ? tpc_override : tpc_for(c_target);
  m.c_main = chunks_for(m.tpc_main);
  m.n_main = (int)n_sf;
  m.c_tail = m.c_main;
  m.tpc_tail = m.tpc_main;
  const long wgs = n_sf * m.c_main;
  const long rem = wgs % slots;
  if (allow_tail && wgs > slots && rem > 0 && rem * 4 <= slots) {
    const long tail_sf = (rem + m.c_main - 1) / m.c_main;
    const long want = slots / (2 * tail_sf) > 1 ? slots / (2 * tail_sf) : 1;    // chunks per tail problem
    const int tpc_t = tpc_for(want * m.c_main);
    if (tpc_t < m.tpc_main) {
      m.n_main = (int)(n_sf - tail_sf);
      m.tpc_tail = tpc_t;
      m.c_tail = chunks_for(tpc_t);
    }
  }
  return m;
}


}  // namespace
