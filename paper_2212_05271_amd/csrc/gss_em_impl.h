// Guided cACGMM EM (arXiv 2212.05271, Section 2.2, Eq. (2)-(5)) for gfx950.
//
// One EM iteration = M-step (class scatter matrices B_{f,k} and weights pi_{f,k} from the posteriors)
// followed by an E-step (posteriors from Eq. (3)-(5)).  The E-step that ends iteration i and the M-step
// that starts iteration i+1 use the same quadratic forms q = y^H B^-1 y, so they are fused into one
// pass over Y:
//
//   pass i (i = 0 .. iters):   per frame: q_k, posterior gamma_k, weight w_k = gamma_k / q_k;
//                              i < iters: accumulate R_k = sum_t w_k y y^H, N_k = sum_t gamma_k
//                              i = iters: write gamma
//   factor i (i = 1 .. iters): B_k from (R_k, N_k), regularise, invert, log-det -> coefficients for pass i
//
// Pass 0 has B = I and uniform weights, which are the initial posteriors
// gamma^0 = activity / (number of active classes) and q^0 = 1 (PASS_FIRST).
//
// Arithmetic.  The quadratic form is evaluated as the real inner product <B^-1, y y^H> over the D*D real
// degrees of freedom of the Hermitian outer product.  That form cancels heavily when B is
// ill-conditioned, so the outer product, the inner product and the scatter accumulation are done in
// fp64 from the RAW fp32 observations (products of fp32 numbers are exact in fp64); the unit
// normalisation of Eq. (2) is applied to q afterwards (q is homogeneous of degree 2 in y) and cancels
// in the M-step weight.  On this chip fp64 FMA issues at the same rate as unpacked fp32 FMA, so this
// costs registers, not time.  The posterior is fp64 as well, evaluated as pi_k / det B_k * q_k^-D and
// normalised over the classes (no logarithm, no exponential; for D <= 8 every term is a normal double);
// only the gamma that leaves the library is rounded to fp32.
#pragma once

#include "gss_internal.h"

#include "gss_device.h"
#include "gss_rules.h"


namespace {

// ----------------------------------------------------------------------------------------------
// Coefficient initialisation: B = I, log-term 0  (pass 0).
// coef[sf][k][E] packed as gss_packed_row(); cconst[sf][k] = pi_k / det B_k (any common factor cancels in
// the posterior).
// ----------------------------------------------------------------------------------------------
__global__ void em_init_coef(double* __restrict__ coef, double* __restrict__ cconst, int D, int K, long n_sf) {
  const int E = D * D;
  long total = n_sf * (long)K * E;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < total; i += (long)gridDim.x * blockDim.x) {
    int e = (int)(i % E);
    // diagonal entries sit at gss_packed_row(r, D)
    double v = 0.0;
    for (int r = 0; r < D; ++r)
      if (e == gss_packed_row(r, D)) v = 1.0;
    coef[i] = v;
  }
  long nl = n_sf * (long)K;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < nl; i += (long)gridDim.x * blockDim.x) {
    cconst[i] = 1.0;
  }
}

// ----------------------------------------------------------------------------------------------
// Pass kernel for D <= 8.  Workgroup = kPassWaves wavefronts on the same (segment, frequency); every
// wavefront owns a contiguous range of tiles of 64 frames and a private LDS region, and there is no
// workgroup barrier inside the tile loop.
//
// Class coefficients.  The packed coefficients of B_k^-1 (D * D reals per class) are the same for every
// frame.  Lane l of every row of 16 lanes holds entry 16 r + (l mod 16) of register r, and the FMAs of phase 1 read them with the
// row-broadcast lane selector of the double-precision vector FMA (v_fmac_f64 ... row_newbcast:n takes its
// first factor from lane n of the executing lane's row).  No scalar loads in the inner loop.  They are resident for the whole
// kernel where registers have room beside the outer product (resident_coefs); otherwise a class's registers are fetched from an
// LDS copy in front of its FMAs (8 channels, 5 classes: 64 segments 14.5 ms; resident, 10 registers spilled, 14.7; fetched a class
// ahead 14.5).
//
// Classes that are not active anywhere in a tile (activity mask, Eq. (5)) have posterior 0 in all of its
// frames and add nothing to any sum: the tile's arithmetic for them is skipped under wave-uniform branches.
//
// Phase 1 (lane = frame): the Hermitian outer product P in fp64, all D * D reals in registers; q_k = <coef_k, P> takes D * D
//   row-broadcast FMAs per live class; posterior over the active classes; weights w_k = gamma_k / q_k.
// Phase 2 (lane = (row of 16 frames, entry of a block of 16)): the blocks of P are transposed within their rows of 16 lanes through
//   8 KB of LDS, and lane (row, e) adds w_k[n] * P[e][n] over the 16 frames n of its row: the weights are where they were computed,
//   in lane n of the row, and the FMAs take them through the same row selector.  An accumulator per class and block, which stays
//   in its register across the tiles; nothing is formed twice, and no weight goes through LDS.
//   The frames of the next live tile are requested from memory before phase 2 (stream_tiles): a wavefront used to wait 1300 of
//   the 9700 cycles of a tile for them (8 channels, 5 classes, two wavefronts per SIMD).
//
// Bound: the vector ALUs, with the clock held at 2.1 GHz by their power (2.4 GHz under a fill kernel), so what counts is the number
// of vector instructions, not the waits.  With y and the weights in LDS and the products formed again from y by 8 lane types in
// phase 2 a tile of 8 channels took about 830 of them with its share of the end of an iteration (shared by 17 tiles), now 665: 195 and 149
// per live class (counted; 2.8 classes in a batch of speech), and a 17th of 949 (m_step_in_wave).
// Times, us: 64 segments of up to 1875 frames, 8 channels, 5 classes, 15 iterations 15931 -> 14517; 3 segments of up to 701, 6
// channels, 4 classes, 10 iterations 430 -> 350; 24 segments of up to 700, 5 iterations, 8 channels and 2 / 5 / 8 classes 730 -> 725
// / 1079 -> 978 / 1971 -> 1281 (the accumulators no longer spill), 5 channels and 5 classes 653 -> 520.  Fewer tests of the class
// mask (20 instead of 55 per tile, over 32 FMAs each) left the times as they were.
//
// Grid: blockIdx.x = chunk + C * (f + F * s).  A chunk is `tiles_per_chunk` tiles of 64 frames.
// ----------------------------------------------------------------------------------------------

// Tile layout: the D * D packed entries of the outer product in blocks of 16, which phase 2 takes transposed (lane = entry of a
// block), and up to 4 entries left over (6 and 7 channels), which a lane adds up for its own frame as in the direct layout.
template <int D>
struct TileSums {
  static constexpr int E = D * D;
  static constexpr int rest = E % 16 <= 4 ? E % 16 : 0;
  static constexpr int blocks = (E - rest + 15) / 16;
};
// Doubles between the rows (entries) of a block of 16 x 64 in LDS: a lane writes its frame's entries, 512 bytes in a row for the
// wavefront, and reads two frames of its entry at a time; 16 rows 528 bytes apart are 16 bytes apart modulo 256, which is what
// LDS delivers per cycle.
constexpr int kBlockRow = kWave + 2;
constexpr int kBlockDoubles = 16 * kBlockRow;

// Registers (pairs) of 16 coefficients per class, and whether a wavefront keeps them all resident: they have to fit beside the outer
// product, the accumulators, counts, posterior terms and partial sums, with some 40 registers left of 256 for everything else.
__host__ __device__ constexpr int coef_regs(int D) { return (D * D + 15) / 16; }
__host__ __device__ constexpr bool resident_coefs(int D, int K) {
  return D <= 4 || 2 * (D * D + K * coef_regs(D) + 3 * K + 3 + K * coef_regs(D)) <= 215;
}

template <int D, int K, bool DIRECT>
struct PassAcc {
  static constexpr int rows = DIRECT ? K : TileSums<D>::blocks + TileSums<D>::rest, cols = DIRECT ? D * D : K;
  using type = double[rows][cols];
};
template <int A, int B>
__device__ __forceinline__ void zero_acc(double (&acc)[A][B]) {
#pragma unroll
  for (int a = 0; a < A; ++a)
#pragma unroll
    for (int b = 0; b < B; ++b) acc[a][b] = 0.0;
}

// The lane's frame of a tile as stored in memory and its activity bits: loaded by the caller of pass_tile
// ahead of time (the whole-EM kernel keeps the one tile of a tiny problem for all iterations, and requests
// the next tile of a streamed problem before it works on the current one).
template <int D>
struct TileRegs {
  float2 y[D];
  unsigned abits;
};
// A lane whose frame lies beyond T reads frame 0 instead (it exists whenever the tile's mask is not empty); its
// activity bits are cleared by pass_tile, not here: nothing in this function waits for a loaded value, so the
// loads of the next tile stay in flight while the current one is worked on.
template <int D>
__device__ __forceinline__ void load_tile_regs(TileRegs<D>& r, const float2* __restrict__ Yrow,
                                               const uint8_t* __restrict__ abrow, int t0, int lane, int T) {
  const int t = t0 + lane;
  const bool valid = t < T;
#pragma unroll
  for (int d = 0; d < D; ++d) r.y[d] = Yrow[(long)(valid ? t : 0) * D + d];
  r.abits = abrow[valid ? t : 0];
}

// One tile of 64 frames starting at frame t0.  `tmask` (wave-uniform) is the tile's activity mask.
//   creg : the resident coefficient registers [K * coef_regs(D)] (used when RESIDENT)
//   sC   : LDS copy of the coefficients, [K * coef_regs(D)][16] doubles (used otherwise)
//   sY   : the wavefront's LDS for a block of 16 entries of its 64 frames (tile layout)
//   cc   : class constants pi_k / det B_k (wave-uniform)
//   cur  : the lane's frame, loaded by the caller (nothing is read from Yrow / abrow): TILE_KEEP leaves it as it is;
//          TILE_STREAM replaces it by the lane's frame of the tile at next_t0, requested before phase 2, when the
//          posterior's registers are free, and wants a mask that is not empty.
enum TileSource { TILE_LOAD, TILE_KEEP, TILE_STREAM };
// PASS_FIRST: B = I and uniform weights, so q = |y|^2 and the active classes share the posterior: no coefficients and none of phase
// 1's D * D FMAs per class (6 iterations, 8 channels and 5 classes: 12 segments of up to 300 frames 409 -> 392 us, 5 channels 225 ->
// 202; 15 iterations of 64 segments 1 %).
enum PassKind { PASS_FIRST, PASS_NEXT, PASS_FINAL };
template <int D, int K, PassKind KIND, bool RESIDENT, bool DIRECT, TileSource SRC = TILE_LOAD>
__device__ __forceinline__ void pass_tile(
    const float2* __restrict__ Yrow, const uint8_t* __restrict__ abrow, const double (&creg)[RESIDENT ? K * coef_regs(D) : 1],
    const double* __restrict__ sC, const double (&cc)[K], float* __restrict__ gamma_row /* + k*F*Tmax */,
    uint32_t* __restrict__ status, long gamma_kstride, int T, int Tmax, int t0, int lane, unsigned tmask,
    double* __restrict__ sY, typename PassAcc<D, K, DIRECT>::type& acc, double (&nacc)[K],
    TileRegs<D>* cur = nullptr, int next_t0 = 0) {
  constexpr int E = D * D;
  constexpr int R = coef_regs(D);
  constexpr bool FINAL = KIND == PASS_FINAL;
  tmask &= (1u << K) - 1u;
  const int t = t0 + lane;
  if constexpr (SRC != TILE_STREAM) {
    if (tmask == 0u) {                        // no frame of the tile has an active class
      if constexpr (FINAL) {
        if (t < Tmax) {
#pragma unroll
          for (int k = 0; k < K; ++k) gamma_row[k * gamma_kstride + t] = 0.f;
        }
      }
      return;
    }
  }

  // ---- phase 1: load y ----
  // A lane whose frame lies beyond T reads frame 0 instead (it exists whenever a tile is processed at all, or is
  // padding in the final pass); its activity bits are zero, so its posterior and weights are zero.
  const bool valid = t < T;
  double yr[D], yi[D];
  unsigned abits;
  if constexpr (SRC != TILE_LOAD) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      float2 v = cur->y[d];
      if constexpr (SRC == TILE_STREAM) asm volatile("" : "+v"(v.x), "+v"(v.y));   // (held in 32 bits up to here)
      yr[d] = (double)v.x;
      yi[d] = (double)v.y;
    }
    abits = valid ? cur->abits : 0u;
  } else {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const float2 v = Yrow[(long)(valid ? t : 0) * D + d];
      yr[d] = (double)v.x;
      yi[d] = (double)v.y;
    }
    abits = abrow[valid ? t : 0];
    abits = valid ? abits : 0u;
  }

  // ---- the outer product, and q_k = <coef_k, y y^H>: 16 FMAs per block on three partial sums (an FMA does not wait for the one
  // before it).  v_k = pi_k / det B_k * q_k^-D with q_k = max(qraw_k / n2c, eps_q), normalised over k below.  For D <= 8 this
  // needs no scaling: B has trace D and eigenvalues >= 1e-6, so 1e-6 <= q <= 1e6 on unit vectors (floored at 1e-10), q^-D lies
  // in [1e-48, 1e80], 1 / det B in [1, 1e42] and pi in [1e-30, 1]: every v_k is a normal double. ----
  double P[R * 16], n2 = 0.0;
  static_for<0, E>([&](auto EI) {
    constexpr int e = EI.value;
    P[e] = packed_entry<D, e>(yr, yi);
    if constexpr (packed_part(e, D) == 0) n2 += P[e];
  });
#pragma unroll
  for (int e = E; e < R * 16; ++e) P[e] = 0.0;
  const double n2c = fmax(n2, GSS_EPS_NORM_SQ);
  const double qfloor = GSS_EPS_Q * n2c;
  const double rq_first = KIND == PASS_FIRST ? rcp_f64_fast(fmax(n2, qfloor)) : 0.0;
  const double p_first = fma(rq_first, 0.0, 1.0);     // 1, and for an infinite frame not a number, as q^-D is in the passes that follow
  double rq[K], v[K], Z = 0.0;
  static_for<0, K>([&](auto KI) {
    constexpr int k = KI.value;
    rq[k] = 0.0;
    v[k] = 0.0;
    if constexpr (KIND == PASS_FIRST) {
      rq[k] = rq_first;
      v[k] = ((abits >> k) & 1u) ? p_first : 0.0;
      Z += v[k];
    } else if (class_on(tmask, k)) {
      double c[R], q[3] = {0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (RESIDENT) c[r] = creg[k * R + r]; else c[r] = sC[(k * R + r) * 16 + (lane & 15)];
      }
      static_for<0, R>([&](auto RI) {
        constexpr int r = RI.value, ng = E - 16 * r < 16 ? E - 16 * r : 16;
        double Pb[ng];
#pragma unroll
        for (int e = 0; e < ng; ++e) Pb[e] = P[16 * r + e];
        fma_bcast_chain<ng>(q, c[r], Pb);
      });
      rq[k] = rcp_f64_fast(fmax(q[0] + q[1] + q[2], qfloor));   // 1 / (q * n2c): the M-step weight is gamma * rq
      const double p = cc[k] * ipow<D>(rq[k] * n2c);            // (1 / q)^D
      v[k] = ((abits >> k) & 1u) ? p : 0.0;
      Z += v[k];
    }
  });
  const double rz = Z > 0.0 ? rcp_f64_fast(Z) : 0.0;
  if constexpr (FINAL) {
    if (valid && !(n2 >= GSS_EPS_NORM_SQ)) atomicOr(status, GSS_STATUS_ZERO_FRAME);
    if (t < Tmax) {
#pragma unroll
      for (int k = 0; k < K; ++k) gamma_row[k * gamma_kstride + t] = (float)(v[k] * rz);
    }
  } else if constexpr (DIRECT) {
    static_for<0, K>([&](auto KI) {
      constexpr int k = KI.value;
      if (class_on(tmask, k)) {
        const double g = v[k] * rz;
        nacc[k] += g;
        const double w = g * rq[k];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[k][e] = fma(w, P[e], acc[k][e]);
      }
    });
  } else {
    // ---- phase 2: lane = (row of 16 frames, entry e of a block).  The blocks change places through LDS one after the other (the
    // LDS executes a wavefront's instructions in order); the weights of the row's 16 frames lie in the row's own lanes. ----
    constexpr int NB = TileSums<D>::blocks;
    double w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double g = v[k] * rz;
      nacc[k] += g;
      w[k] = g * rq[k];
    }
    if constexpr (SRC == TILE_STREAM) load_tile_regs<D>(*cur, Yrow, abrow, next_t0, lane, T);
    double x[NB][16];
    double* __restrict__ sw = sY + lane;
    const double* __restrict__ sr = sY + (lane & 15) * kBlockRow + (lane & 48);
    static_for<0, NB>([&](auto BI) {
      constexpr int b = BI.value;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (16 * b + e < E) sw[e * kBlockRow] = P[16 * b + e];
      wave_lds_sync();
#pragma unroll
      for (int n = 0; n < 16; n += 2) {
        const double2 p2 = *reinterpret_cast<const double2*>(sr + n);
        x[b][n] = p2.x;
        x[b][n + 1] = p2.y;
      }
      wave_lds_sync();
    });
    static_for<0, K>([&](auto KI) {
      constexpr int k = KI.value;
      if (class_on(tmask, k)) {
        double a[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) a[b] = acc[b][k];
        fma_bcast_rows<NB>(a, w[k], x);
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[b][k] = a[b];
#pragma unroll
        for (int j = 0; j < TileSums<D>::rest; ++j) acc[NB + j][k] = fma(w[k], P[16 * NB + j], acc[NB + j][k]);
      }
    });
  }
}

// The accumulating pass over tiles lo .. hi - 1 in the tile layout: every live tile's frames are requested while the live
// tile before it is in phase 2.
template <int D, int K, PassKind KIND, bool RESIDENT, class MaskPtr>
__device__ __forceinline__ void stream_tiles(
    const float2* __restrict__ Yrow, const uint8_t* __restrict__ abrow, MaskPtr tmrow,
    const double (&creg)[RESIDENT ? K * coef_regs(D) : 1], const double* __restrict__ sC, const double (&cc)[K], int T,
    int Tmax, int lo, int hi, int by, int lane, double* __restrict__ sY,
    typename PassAcc<D, K, false>::type& acc, double (&nacc)[K]) {
  constexpr unsigned kmask = (1u << K) - 1u;
  int tile = lo;
  unsigned m = 0u;
  while (tile < hi && (m = tmrow[tile] & kmask) == 0u) tile += by;
  if (tile >= hi) return;
  TileRegs<D> cur;
  load_tile_regs<D>(cur, Yrow, abrow, tile * kWave, lane, T);
  for (;;) {
    int next = tile + by;
    unsigned mn = 0u;
    while (next < hi && (mn = tmrow[next] & kmask) == 0u) next += by;
    const bool last = next >= hi;
    // (after the last live tile its own frames are requested again, so that the load needs no branch)
    pass_tile<D, K, KIND, RESIDENT, false, TILE_STREAM>(Yrow, abrow, creg, sC, cc, nullptr, nullptr, 0, T, Tmax, tile * kWave, lane, m, sY,
                                           acc, nacc, &cur, (last ? tile : next) * kWave);
    if (last) break;
    tile = next;
    m = mn;
  }
}

// Direct layout: the wavefront's totals of the accumulators acc[k][e] and the class counts nacc[k], written as
// out[k * E + e] and out[K * E + k] (LDS; the caller orders the traffic).
template <int D, int K>
__device__ __forceinline__ void direct_values(const typename PassAcc<D, K, true>::type& acc, const double (&nacc)[K],
                                              double (&v)[K * D * D + K]) {
  constexpr int E = D * D;
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int e = 0; e < E; ++e) v[k * E + e] = acc[k][e];
    v[K * E + k] = nacc[k];
  }
}
template <int D, int K>
__device__ __forceinline__ void store_direct_sums(const typename PassAcc<D, K, true>::type& acc, const double (&nacc)[K],
                                                  double* __restrict__ out, int lane) {
  constexpr int N = K * D * D + K;
  double v[N];
  direct_values<D, K>(acc, nacc, v);
  transpose_reduce<N>(v, lane);
  const int n0 = transposed_index(lane);
#pragma unroll
  for (int j = 0; j < (N + kWave - 1) / kWave; ++j)
    if (n0 + kWave * j < N) out[n0 + kWave * j] = v[j];
}
// The same by way of LDS, 16 values at a time, four lanes adding up 16 frames each of a value: a third of the instructions, where
// 9 KB per wavefront are there (buf: 16 rows of kReduceRow doubles; rows 64 bytes apart modulo 256, so that the four lanes of
// four rows read without bank conflicts).
template <int D, int K>
__device__ __forceinline__ void store_direct_sums_lds(const typename PassAcc<D, K, true>::type& acc, const double (&nacc)[K],
                                                      double* __restrict__ buf, double* __restrict__ out, int lane) {
  constexpr int N = K * D * D + K;
  double v[N];
  direct_values<D, K>(acc, nacc, v);
  const double* __restrict__ src = buf + (lane >> 2) * kReduceRow + 2 * (lane & 3);
#pragma unroll
  for (int n0 = 0; n0 < N; n0 += 16) {
#pragma unroll
    for (int n = n0; n < (n0 + 16 < N ? n0 + 16 : N); ++n) buf[(n - n0) * kReduceRow + lane] = v[n];
    wave_lds_sync();
    double2 p[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = *reinterpret_cast<const double2*>(src + 8 * i);
    wave_lds_sync();
    double h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = (p[i].x + p[i].y) + (p[i + 4].x + p[i + 4].y);
    double sum = (h[0] + h[1]) + (h[2] + h[3]);
    sum += dpp_permute_f64<0xB1>(sum);                   // quad_perm [1, 0, 3, 2]
    sum += dpp_permute_f64<0x4E>(sum);                   // quad_perm [2, 3, 0, 1]
    const int n = n0 + (lane >> 2);
    if ((lane & 3) == 0 && n < N) out[n] = sum;
  }
}

// Tile layout: the same, out[k * E + e] and out[K * E + k].
template <int D, int K>
__device__ __forceinline__ void store_tile_sums(const typename PassAcc<D, K, false>::type& acc, const double (&nacc)[K],
                                                double* __restrict__ out, int lane) {
  constexpr int E = D * D, NB = TileSums<D>::blocks, NR = TileSums<D>::rest, N = K * NB;
  double v[N], u[K * (NR + 1)];
#pragma unroll
  for (int k = 0; k < K; ++k) {
#pragma unroll
    for (int b = 0; b < NB; ++b) v[k * NB + b] = acc[b][k];
#pragma unroll
    for (int j = 0; j < NR; ++j) u[k * NR + j] = acc[NB + j][k];
    u[K * NR + k] = nacc[k];
  }
  row_sums<N>(v);
#pragma unroll
  for (int j = 0; j < (N + 3) / 4; ++j) {
    const int i = row_sum_index(lane >> 4, j), k = i / NB, e = 16 * (i - k * NB) + (lane & 15);
    if (i < N && e < E) out[k * E + e] = v[j];
  }
  transpose_reduce<K * (NR + 1)>(u, lane);
  const int i = transposed_index(lane);                  // (at most 64 values)
  if (i < K * NR) {
    const int k = i / (NR > 0 ? NR : 1);
    out[k * E + 16 * NB + (i - k * NR)] = u[0];
  } else if (i < K * (NR + 1)) {
    out[K * E + (i - K * NR)] = u[0];
  }
}

template <int D, int K, PassKind KIND>
__global__ __launch_bounds__(kWave * kPassWaves, 2) void em_pass_small(
    gss_yview yv, const uint8_t* __restrict__ abyte, const uint32_t* __restrict__ tmask,
    const int32_t* __restrict__ T_len,
    const double* __restrict__ coef, const double* __restrict__ cconst,
    double* __restrict__ part, double* __restrict__ npart, float* __restrict__ gamma, uint32_t* __restrict__ status,
    int F, int Tmax, ChunkMap cmap) {
  constexpr bool FINAL = KIND == PASS_FINAL, FIRST = KIND == PASS_FIRST;
  constexpr int E = D * D;
  constexpr int R = coef_regs(D);
  constexpr bool RESIDENT = resident_coefs(D, K);
  constexpr bool DIRECT = direct_layout(D, K, false);   // no blocks in LDS then
  // per wavefront: a block on its way through LDS; then the wavefront's sums
  constexpr int kSumDoubles = (K * E + K + 1) / 2 * 2;
  constexpr int kTileDoubles = DIRECT || kSumDoubles > kBlockDoubles ? kSumDoubles : kBlockDoubles;
  constexpr int kCoefDoubles = RESIDENT || FIRST ? 0 : K * R * 16;
  constexpr int kTilesDoubles = FINAL ? 2 : kPassWaves * kTileDoubles;
  __shared__ __attribute__((aligned(16))) double lds[kTilesDoubles + kCoefDoubles];

  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  long sf;
  int chunk, tiles_per_chunk;
  chunk_decode(cmap, blockIdx.x, sf, chunk, tiles_per_chunk);
  const int s = (int)((unsigned)sf / (unsigned)F);
  const int f = (int)((unsigned)sf % (unsigned)F);
  int T;
  const float2* __restrict__ Yrow = y_row(yv, T_len, s, f, D, Tmax, T);
  const int t_end = FINAL ? Tmax : T;       // the final pass also writes the zero padding

  const double* __restrict__ cf = coef + sf * (long)(K * E);
  double* __restrict__ sY = lds + (FINAL ? 0 : wave * kTileDoubles);
  double* __restrict__ sC = lds + kTilesDoubles;

  // The class coefficients: register r of class k holds entries 16 r .. 16 r + 15 of its packed coefficients,
  // entry 16 r + (lane mod 16) in every lane (a lane past the end of the class reads the last entry of the
  // array instead: its value is never used).
  double creg[RESIDENT ? K * R : 1];
  if constexpr (FIRST) {
    creg[0] = 0.0;
  } else if constexpr (RESIDENT) {
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int e = 16 * r + (lane & 15);
        creg[k * R + r] = cf[k * E + (e < E ? e : E - 1)];
      }
  } else {
    creg[0] = 0.0;
    for (int x = threadIdx.x; x < K * R * 16; x += kWave * kPassWaves) {
      const int k = x / (R * 16), e = x % (R * 16);
      sC[x] = cf[k * E + (e < E ? e : E - 1)];
    }
    __syncthreads();
  }
  // class constants pi_k / det B_k (wave-uniform, read through the scalar path)
  double cc[K];
  if constexpr (FIRST) {
#pragma unroll
    for (int k = 0; k < K; ++k) cc[k] = 1.0;
  } else {
    typedef const __attribute__((address_space(4))) double* cc_ptr_t;
    const cc_ptr_t ccp = (cc_ptr_t)(uintptr_t)(cconst + sf * K);
#pragma unroll
    for (int k = 0; k < K; ++k) cc[k] = ccp[k];
  }

  typename PassAcc<D, K, DIRECT>::type acc;
  double nacc[K];
  zero_acc(acc);
#pragma unroll
  for (int k = 0; k < K; ++k) nacc[k] = 0.0;
  const uint8_t* __restrict__ abrow = abyte + (long)s * Tmax;
  const int tiles_total = (Tmax + kWave - 1) / kWave;
  // the tile masks are read through the scalar path (they were written by an earlier kernel)
  typedef const __attribute__((address_space(4))) uint32_t* mask_ptr_t;
  const mask_ptr_t tmrow = (mask_ptr_t)(uintptr_t)(tmask + (long)s * tiles_total);
  float* __restrict__ gamma_row = FINAL ? gamma + ((long)s * K * F + f) * Tmax : nullptr;
  const long gamma_kstride = (long)F * Tmax;

  // The chunk's tiles are split into one contiguous range per wavefront (lengths differ by at most one); the
  // assignment depends only on the tile count, so the sums are bitwise reproducible.
  const int tile_lo = chunk * tiles_per_chunk;
  int tile_hi = tile_lo + tiles_per_chunk;
  const int tile_end = (t_end + kWave - 1) / kWave;
  tile_hi = tile_hi < tile_end ? tile_hi : tile_end;
  const int n_tiles = tile_hi > tile_lo ? tile_hi - tile_lo : 0;
  const int my_lo = tile_lo + (n_tiles * wave) / kPassWaves;
  const int my_hi = tile_lo + (n_tiles * (wave + 1)) / kPassWaves;
  if constexpr (DIRECT || FINAL) {
    for (int tile = my_lo; tile < my_hi; ++tile)
      pass_tile<D, K, KIND, RESIDENT, DIRECT>(Yrow, abrow, creg, sC, cc, gamma_row, status, gamma_kstride, T, Tmax, tile * kWave,
                                       lane, tmrow[tile], sY, acc, nacc);
  } else {
    stream_tiles<D, K, KIND, RESIDENT>(Yrow, abrow, tmrow, creg, sC, cc, T, Tmax, my_lo, my_hi, 1, lane, sY, acc, nacc);
  }
  if (FINAL) return;

  // every wavefront's totals meet in LDS and are added in the order of the wavefronts
  constexpr int N = K * E + K;
  if constexpr (DIRECT) store_direct_sums<D, K>(acc, nacc, sY, lane);
  else store_tile_sums<D, K>(acc, nacc, sY, lane);
  __syncthreads();
  for (int x = threadIdx.x; x < N; x += kWave * kPassWaves) {
    double sum = lds[x];
#pragma unroll
    for (int w = 1; w < kPassWaves; ++w) sum += lds[w * kTileDoubles + x];
    if (x < K * E) part[(long)blockIdx.x * (K * E) + x] = sum;
    else npart[(long)blockIdx.x * K + (x - K * E)] = sum;
  }
}

// ----------------------------------------------------------------------------------------------
// End of an iteration in one wavefront (5 channels and more): the accumulators are added up, the K class matrices B_k =
// D R_k / N_k scaled to trace D, loaded with delta I (identity for a class without data) and inverted in place; the packed
// coefficients of B_k^-1 go to sC[K][coef_regs(D) * 16] (LDS) and the class constants pi_k / det B_k to cc (wave-uniform).
// Lane (k, i) = (le / 8, le % 8) holds row i of the matrix of class k in registers.  Every lane of the wavefront must be active.
//
// Between the lanes that add up and the lanes that eliminate, the matrices pass through LDS as full rows (row pitch of 9
// complex numbers: the rows of two classes are read without bank conflicts): an entry of the upper triangle is written to both
// of its places, and a row is read with D loads and no choices.  The coefficients are collected from the inverse in the same
// way.  A wavefront of a batch runs this once per iteration for 17 tiles on average (64 segments of up to 1875 frames), where it
// was 1500 vector instructions against the 610 of a tile; now 949.
// ----------------------------------------------------------------------------------------------
constexpr int kMatRow = 18;                              // doubles per row of a class matrix in LDS
__host__ __device__ constexpr int mat_doubles(int D) { return D * kMatRow; }
// The two places of packed entry e within a class matrix, and the factor of the second: conj for an imaginary part, and the (zero)
// imaginary part for a diagonal entry.  place | second << 8 | factor << 16.
template <int D>
struct MatPlaces { int code[kWave]; };
template <int D>
constexpr MatPlaces<D> make_mat_places() {
  MatPlaces<D> t{};
  for (int e = 0; e < D * D; ++e) {
    const int i = packed_i(e, D), j = packed_j(e, D), part = packed_part(e, D);
    const int at = i * kMatRow + 2 * j + (part == 2 ? 1 : 0);
    const int second = part == 0 ? at + 1 : j * kMatRow + 2 * i + (part == 2 ? 1 : 0);
    t.code[e] = at | second << 8 | (part == 0 ? 0 : part == 1 ? 1 : -1) * (1 << 16);
  }
  return t;
}
// Sums of N per-lane doubles over the wavefront, the same in the 8 lanes of group g for value 8 r + g: out[r].  buf: 8 rows of
// kBlockRow doubles.
template <int N>
__device__ __forceinline__ void lane_sums(const double (&v)[N], double* __restrict__ buf, int le, double (&out)[(N + 7) / 8]) {
#pragma unroll
  for (int r = 0; r < (N + 7) / 8; ++r) {
#pragma unroll
    for (int n = 8 * r; n < (8 * r + 8 < N ? 8 * r + 8 : N); ++n) buf[(n - 8 * r) * kBlockRow + le] = v[n];
    wave_lds_sync();
    double2 p[4];
    const double* __restrict__ src = buf + (le >> 3) * kBlockRow + 8 * (le & 7);
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = *reinterpret_cast<const double2*>(src + 2 * j);
    wave_lds_sync();
    double sum = ((p[0].x + p[0].y) + (p[1].x + p[1].y)) + ((p[2].x + p[2].y) + (p[3].x + p[3].y));
    sum += dpp_permute_f64<0xB1>(sum);                   // quad_perm [1, 0, 3, 2]
    sum += dpp_permute_f64<0x4E>(sum);                   // quad_perm [2, 3, 0, 1]
    sum += dpp_permute_f64<0x141>(sum);                  // row_half_mirror
    out[r] = sum;
  }
}
template <int D, int K>
__device__ __forceinline__ void m_step_in_wave(const typename PassAcc<D, K, false>::type& acc, const double (&nacc)[K],
                                               double* __restrict__ sM, const int* __restrict__ sPlaces, double* __restrict__ sC,
                                               double (&cc)[K], int le, int weight_mode, uint32_t* __restrict__ status) {
  constexpr int E = D * D, R = coef_regs(D), NB = TileSums<D>::blocks, NR = TileSums<D>::rest, N = K * NB;
  const int fk = le >> 3, fi = le & 7;                  // class and row of this lane
  const bool on = fk < K && fi < D;
  auto put = [&](int k, int e, double v) {
    const int code = sPlaces[e];
    sM[k * mat_doubles(D) + (code & 0xff)] = v;
    sM[k * mat_doubles(D) + (code >> 8 & 0xff)] = v * (double)(code >> 16);
  };
  // ---- sums: the class counts and the entries of the last block, then the blocks ----
  double u[K * (NR + 1)], us[(K * (NR + 1) + 7) / 8];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    u[k] = nacc[k];
#pragma unroll
    for (int j = 0; j < NR; ++j) u[K + k * NR + j] = acc[NB + j][k];
  }
  lane_sums<K * (NR + 1)>(u, sM, le, us);
  const double Nk = us[0];
  if constexpr (NR > 0) {
#pragma unroll
    for (int r = 0; r < (K * (NR + 1) + 7) / 8; ++r) {
      const int n = 8 * r + fk - K;
      if (fi == 0 && n >= 0 && n < K * NR) put(n / NR, 16 * NB + n % NR, us[r]);
    }
  }
  double v[N];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int b = 0; b < NB; ++b) v[k * NB + b] = acc[b][k];
  row_sums<N>(v);
#pragma unroll
  for (int j = 0; j < (N + 3) / 4; ++j) {
    const unsigned i0 = row_sum_index(le >> 4, 0);       // value 4 j + i0 = entry e of class k
    const unsigned k = 4 % NB == 0 ? j * (4 / NB) + i0 / NB : (4 * j + i0) / NB;
    const unsigned b = 4 % NB == 0 ? i0 % NB : 4 * j + i0 - k * NB, e = 16 * b + (le & 15);
    if ((4 * j + 3 < N && 16 * NB <= E) || (k < (unsigned)K && e < (unsigned)E)) put(k, e, v[j]);
  }
  wave_lds_sync();

  // ---- row fi of class fk (lanes without one read along) ----
  double* __restrict__ row = sM + (fk < K ? fk : K - 1) * mat_doubles(D) + (fi < D ? fi : D - 1) * kMatRow;
  double ar[D], ai[D];
#pragma unroll
  for (int j = 0; j < D; ++j) {
    const double2 m = *reinterpret_cast<const double2*>(row + 2 * j);
    ar[j] = m.x;
    ai[j] = m.y;
  }
  double tr = fi < D ? row[2 * (fi < D ? fi : 0)] : 0.0;
  tr += dpp_permute_f64<0xB1>(tr);
  tr += dpp_permute_f64<0x4E>(tr);
  tr += dpp_permute_f64<0x141>(tr);
  // B = D R / max(N, eps); dead if its trace <= eps; else rescaled to trace D (= R * D / tr R)
  // (the test without its division, the scale with a reciprocal: both sit in front of the sweeps)
  const bool dead = !((double)D * tr > GSS_EPS_N * fmax(Nk, GSS_EPS_N));
  const double sc = dead ? 0.0 : (double)D * rcp_f64(tr), load = dead ? 1.0 + GSS_DELTA : GSS_DELTA;
  if (__ballot(dead) != 0) {                             // (entries may be infinite)
#pragma unroll
    for (int j = 0; j < D; ++j) {
      ar[j] = dead ? 0.0 : ar[j];
      ai[j] = dead ? 0.0 : ai[j];
    }
  }
#pragma unroll
  for (int j = 0; j < D; ++j) {
    ar[j] = fma(ar[j], sc, j == fi ? load : 0.0);
    ai[j] *= sc;
  }
  // Gauss-Jordan sweeps.  The 8 lanes of a class sit in one half of a row of 16 lanes, so the pivot row
  // reaches them through the lane-permute move (class_row_bcast): nothing goes through LDS, nothing waits.
  // Executed by all lanes (the permute reads lanes, so none may be switched off); lanes without a row carry
  // values that are never stored.  Row minus (a_ip / pivot) x pivot row; the pivot row itself minus (1 - 1 / pivot) x itself
  // (pivots are at most D, so the difference cancels to an eighth of its terms at worst).
  double det = 1.0;
  static_for<0, D>([&](auto PI) {
    constexpr int p = PI.value;
    double pr[D], pi[D];
    class_row_bcast<p>(ar, pr);
    class_row_bcast<p>(ai, pi);
    double piv = pr[p];
    if (!(piv > 1e-300)) {
      piv = 1e-300;
      if (on && fi == 0) atomicOr(status, GSS_STATUS_NONPD_B);
    }
    det *= piv;
    const double rp = rcp_f64(piv);
    const bool is_piv = fi == p;
    const double fr = ar[p] * rp, fim = ai[p] * rp;      // M_ip / pivot
    const double cr = is_piv ? 1.0 - rp : fr, ci = is_piv ? 0.0 : fim;
#pragma unroll
    for (int j = 0; j < D; ++j) {
      if (j != p) {
        ar[j] = fma(ci, pi[j], fma(-cr, pr[j], ar[j]));
        ai[j] = fma(-ci, pr[j], fma(-cr, pi[j], ai[j]));
      }
    }
    ar[p] = is_piv ? rp : -fr;
    ai[p] = -ci;
  });
  // packed coefficients of q = sum_i A_ii P_ii + 2 sum_{i<j} (Re A_ij Re P_ij + Im A_ij Im P_ij), A = the
  // Hermitian part of the computed inverse: the coefficient of the pair i < j is A_ij + conj(A_ji), not 2 A_ij.
  // (Rounding leaves the computed inverse slightly non-Hermitian.  For an ill-conditioned B, e.g. a class with
  // fewer frames than channels, whose inverse has entries of 1e6, the quadratic form of the Hermitian part is
  // still good to 1e-10 for the class's own frames, while that of one triangle mirrored is off by up to 1e-4.)
  if (on) {
#pragma unroll
    for (int j = 0; j < D; ++j) *reinterpret_cast<double2*>(row + 2 * j) = make_double2(ar[j], j == fi ? 0.0 : ai[j]);
  }
  wave_lds_sync();
  if (le < E) {
    const int code = sPlaces[le];
    const double f = (double)(code >> 16);
    const double* __restrict__ m0 = sM + (code & 0xff);
    const double* __restrict__ m1 = sM + (code >> 8 & 0xff);
#pragma unroll
    for (int k = 0; k < K; ++k) sC[k * (R * 16) + le] = fma(f, m1[k * mat_doubles(D)], m0[k * mat_doubles(D)]);
  }
  // (every lane of a class computes the class constant; it is kept in scalar registers across the tile loop)
  auto of_class = [](double x, int k) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), 8 * k), __builtin_amdgcn_readlane(__double2loint(x), 8 * k));
  };
  double Ntot = 0.0;
#pragma unroll
  for (int k = 0; k < K; ++k) Ntot += of_class(Nk, k);
  const double pi_k = weight_mode == 1 ? Nk * rcp_f64(fmax(Ntot, GSS_EPS_N)) : 1.0 / (double)K;
  const double cck = fmax(pi_k, GSS_EPS_PI) * rcp_f64(det);
#pragma unroll
  for (int k = 0; k < K; ++k) cc[k] = of_class(cck, k);
}

// The M-step for few channels from the packed sums sR[K][E] and the class counts sN[K] (LDS), the class constants to sCC[K] (LDS),
// every class in one lane: lane k mod 8 has the packed matrix of class k in registers and eliminates
// it alone, B = L diag(d) L^H, M = L^-1, B^-1 = M^H diag(1 / d) M (Hermitian by construction).  Nothing crosses lanes between
// the reads of the sums and the writes of the coefficients.  Up to 4 channels its chain of dependent instructions is shorter
// than that of the sweeps with a row per lane: one segment of 200 frames, 10 iterations, 2 channels and 3 classes 36.8 -> 32.6
// us, 3 channels and 5 classes 62.0 -> 56.4, 24 segments of up to 700 frames, 4 channels and 5 classes 857 -> 805 us.
constexpr int kLaneFactorMaxD = 4;
template <int D, int K>
__device__ __forceinline__ void factor_class_in_lane(const double* __restrict__ sR, const double* __restrict__ sN,
                                                     double* __restrict__ sC, double* __restrict__ sCC, int le,
                                                     int weight_mode, uint32_t* __restrict__ status) {
  constexpr int E = D * D;
  constexpr int R = coef_regs(D);
  const int k = (le & 7) < K ? (le & 7) : K - 1;
  const bool on = le < K;
  double h[E], n[K];
#pragma unroll
  for (int e = 0; e < E; ++e) h[e] = sR[k * E + e];
#pragma unroll
  for (int c = 0; c < K; ++c) n[c] = sN[c];
  const double Nk = sN[k];
  double tr = 0.0, Ntot = 0.0;
#pragma unroll
  for (int d = 0; d < D; ++d) tr += h[gss_packed_row(d, D)];
#pragma unroll
  for (int c = 0; c < K; ++c) Ntot += n[c];
  const bool dead = !((double)D * tr > GSS_EPS_N * fmax(Nk, GSS_EPS_N));
  if constexpr (D == 2) {
    // B = (2 / tr) R', R' = R + delta tr / 2 I: B^-1 = (tr / 2) adj R' / det R' and det B = det R' (2 / tr)^2, one reciprocal
    // behind the sums instead of four in a row (the M-step 900 -> 600 cycles)
    const double half = dead ? 1.0 : 0.5 * tr;
    const double a = fma(GSS_DELTA, half, dead ? 1.0 : h[0]), d = fma(GSS_DELTA, half, dead ? 1.0 : h[3]);
    const double br = dead ? 0.0 : h[1], bi = dead ? 0.0 : h[2];
    double det = fma(a, d, -fma(br, br, bi * bi));
    if (!(det > 0.0)) {
      det = 1e-300;
      if (on) atomicOr(status, GSS_STATUS_NONPD_B);
    }
    const double s = half * rcp_f64(det);
    const double pi_k = weight_mode == 1 ? Nk * rcp_f64(fmax(Ntot, GSS_EPS_N)) : 1.0 / (double)K;
    if (on) {
      double* __restrict__ sCk = sC + k * (R * 16);
      sCk[0] = d * s;
      sCk[1] = -2.0 * br * s;
      sCk[2] = -2.0 * bi * s;
      sCk[3] = a * s;
      sCC[k] = fmax(pi_k, GSS_EPS_PI) * (half * s);
    }
    return;
  }
  const double sc = dead ? 0.0 : (double)D * rcp_f64(tr);
  // upper triangle: hr/hi[i][j] = entry (i, j), i <= j
  double hr[D][D], hi[D][D];
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const int p = gss_packed_row(i, D);
    hr[i][i] = (dead ? 1.0 : h[p] * sc) + GSS_DELTA;
#pragma unroll
    for (int j = i + 1; j < D; ++j) {
      hr[i][j] = dead ? 0.0 : h[p + 1 + 2 * (j - i - 1)] * sc;
      hi[i][j] = dead ? 0.0 : h[p + 2 + 2 * (j - i - 1)] * sc;
    }
  }
  double det = 1.0, rd[D];
  double lr[D][D], li[D][D];                            // unit lower factor, i > p; then its inverse
#pragma unroll
  for (int p = 0; p < D; ++p) {
    double piv = hr[p][p];
    if (!(piv > 1e-300)) {
      piv = 1e-300;
      if (on) atomicOr(status, GSS_STATUS_NONPD_B);
    }
    det *= piv;
    rd[p] = rcp_f64(piv);
#pragma unroll
    for (int i = p + 1; i < D; ++i) {
      lr[i][p] = hr[p][i] * rd[p];                      // conj(H_pi) / d_p
      li[i][p] = -hi[p][i] * rd[p];
#pragma unroll
      for (int j = i; j < D; ++j) {
        hr[i][j] -= lr[i][p] * hr[p][j] - li[i][p] * hi[p][j];
        if (j > i) hi[i][j] -= lr[i][p] * hi[p][j] + li[i][p] * hr[p][j];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < D; ++c)
#pragma unroll
    for (int i = c + 1; i < D; ++i) {
      double mr = lr[i][c], mi = li[i][c];
#pragma unroll
      for (int m = c + 1; m < i; ++m) {                 // (rows m < i of column c are the inverse's already)
        mr += lr[i][m] * lr[m][c] - li[i][m] * li[m][c];
        mi += lr[i][m] * li[m][c] + li[i][m] * lr[m][c];
      }
      lr[i][c] = -mr;
      li[i][c] = -mi;
    }
  double* __restrict__ sCk = sC + k * (R * 16);
#pragma unroll
  for (int i = 0; i < D; ++i) {
    const int pi0 = gss_packed_row(i, D);
#pragma unroll
    for (int j = i; j < D; ++j) {
      // entry (i, j) of the inverse: sum over p >= j of conj(M_pi) M_pj / d_p, M_jj = 1
      double ar, ai = 0.0;
      if (i == j) {
        ar = rd[i];
#pragma unroll
        for (int p = i + 1; p < D; ++p) ar += (lr[p][i] * lr[p][i] + li[p][i] * li[p][i]) * rd[p];
      } else {
        ar = lr[j][i] * rd[j];
        ai = -li[j][i] * rd[j];
#pragma unroll
        for (int p = j + 1; p < D; ++p) {
          ar += (lr[p][i] * lr[p][j] + li[p][i] * li[p][j]) * rd[p];
          ai += (lr[p][i] * li[p][j] - li[p][i] * lr[p][j]) * rd[p];
        }
      }
      if (on) {
        if (i == j) {
          sCk[pi0] = ar;
        } else {
          sCk[pi0 + 1 + 2 * (j - i - 1)] = 2.0 * ar;
          sCk[pi0 + 2 + 2 * (j - i - 1)] = 2.0 * ai;
        }
      }
    }
  }
  const double pi_k = weight_mode == 1 ? Nk * rcp_f64(fmax(Ntot, GSS_EPS_N)) : 1.0 / (double)K;
  if (on) sCC[k] = fmax(pi_k, GSS_EPS_PI) * rcp_f64(det);
}

// ----------------------------------------------------------------------------------------------
// Factor kernel for D <= 8: one workgroup per (segment, frequency), one wavefront per class.
// Sums the chunk partials in a fixed order (deterministic), forms B = D R / N, regularises (trace D,
// + delta I; identity for a class without data), inverts by in-place Gauss-Jordan sweeps in fp64
// (pivots = Schur complements, positive for a Hermitian positive-definite matrix; their product is
// det B) and writes the packed coefficients of B^-1 and the class constant pi_k / det B_k of the next pass.
// Bound: latency.  With the lane's entry in a register across the sweeps, one expression for all lanes and reciprocals in place of
// divisions one segment of 1560 frames, 20 iterations, takes 732 instead of 741 us, 6 channels, 600 frames, 10 iterations 166 instead of 172.
// ----------------------------------------------------------------------------------------------
template <int D, int K>
__global__ __launch_bounds__(kWave * K) void em_factor_small(
    const double* __restrict__ part, const double* __restrict__ npart,
    double* __restrict__ coef, double* __restrict__ cconst, uint32_t* __restrict__ status,
    ChunkMap cmap, int weight_mode) {
  constexpr int E = D * D;
  __shared__ double sR[K][E];
  __shared__ double sMr[K][D][D], sMi[K][D][D];
  __shared__ double sN[K];

  const long sf = blockIdx.x;
  const int k = threadIdx.x / kWave;
  const int l = threadIdx.x % kWave;
  int C;
  const long slot0 = chunk_base(cmap, sf, C);

  if (l < E) {
    sR[k][l] = sum_chunks(part + (slot0 * K + k) * (long)E + l, (long)K * E, C);
  }
  if (l == 0) {
    sN[k] = sum_chunks(npart + slot0 * K + k, K, C);
  }
  __syncthreads();

  const int i = l / D, j = l % D;
  const bool on = l < E;
  double tr = 0.0;
#pragma unroll
  for (int r = 0; r < D; ++r) tr += sR[k][gss_packed_row(r, D)];
  const double Nk = sN[k];
  // B = D R / max(N, eps); dead if its trace <= eps; else rescale to trace D  (=> R * D / tr R)
  // (the test without its division, the reciprocals in place of divisions: they sit in front of the sweeps)
  const bool dead = !((double)D * tr > GSS_EPS_N * fmax(Nk, GSS_EPS_N));
  double mr = 0.0, mi = 0.0;
  if (on) {
    if (dead) {
      mr = (i == j) ? 1.0 : 0.0;
    } else {
      const double sc = (double)D * rcp_f64(tr);
      if (i == j) {
        mr = sR[k][gss_packed_row(i, D)] * sc;
      } else {
        const int lo = i < j ? i : j, hi = i < j ? j : i;
        const int p = gss_packed_row(lo, D) + 1 + 2 * (hi - lo - 1);
        mr = sR[k][p] * sc;
        mi = sR[k][p + 1] * sc;
        if (i > j) mi = -mi;                 // lower triangle = conjugate
      }
    }
    if (i == j) mr += GSS_DELTA;
    sMr[k][i][j] = mr;
    sMi[k][i][j] = mi;
  }
  wave_lds_sync();          // from here on every wavefront works on its own class matrix only

  double detm = 1.0;   // det B = detm * 2^dete, renormalised after every pivot
  int dete = 0;
  for (int p = 0; p < D; ++p) {
    double piv = sMr[k][p][p];
    if (!(piv > 1e-300)) {
      piv = 1e-300;
      if (l == 0) atomicOr(status, GSS_STATUS_NONPD_B);
    }
    detm *= piv;
    dete += __builtin_amdgcn_frexp_exp(detm);
    detm = __builtin_amdgcn_frexp_mant(detm);
    const double rp = rcp_f64(piv);
    // (one expression for every lane, as in m_step_in_wave; the lane's entry stays in registers)
    const int ic = on ? i : 0;
    const double air = sMr[k][ic][p], aii = sMi[k][ic][p];
    const double apr = sMr[k][p][j], api = sMi[k][p][j];
    const bool prow = i == p, pcol = j == p;
    const double fr = air * rp, fim = aii * rp;
    const double cr = prow ? 1.0 - rp : fr, ci = prow ? 0.0 : fim;
    const double nr = fma(ci, api, fma(-cr, apr, mr)), ni = fma(-ci, apr, fma(-cr, api, mi));
    mr = pcol ? (prow ? rp : -fr) : nr;
    mi = pcol ? -ci : ni;
    wave_lds_sync();
    if (on) { sMr[k][i][j] = mr; sMi[k][i][j] = mi; }
    wave_lds_sync();
  }

  // packed coefficients of q = sum_i A_ii P_ii + 2 sum_{i<j} (Re A_ij Re P_ij + Im A_ij Im P_ij), A = B^-1
  if (on && i <= j) {
    double* __restrict__ cf = coef + (sf * K + k) * (long)E;
    // (the Hermitian part of the computed inverse: A_ij + conj(A_ji), see m_step_in_wave)
    if (i == j) {
      cf[gss_packed_row(i, D)] = sMr[k][i][i];
    } else {
      const int p = gss_packed_row(i, D) + 1 + 2 * (j - i - 1);
      cf[p] = sMr[k][i][j] + sMr[k][j][i];
      cf[p + 1] = sMi[k][i][j] - sMi[k][j][i];
    }
  }
  if (l == 0) {
    double pi;
    if (weight_mode == 1) {
      double tot = 0.0;
      for (int kk = 0; kk < K; ++kk) tot += sN[kk];
      pi = Nk * rcp_f64(fmax(tot, GSS_EPS_N));
    } else {
      pi = 1.0 / (double)K;
    }
    const double c = fmax(pi, GSS_EPS_PI) * rcp_f64(detm);            // pi_k / det B_k = c * 2^-dete
    cconst[sf * K + k] = ldexp(c, -dete);
  }
}

// Order in which the whole-EM kernel takes the segments of a ragged batch: longest first (equal lengths in index
// order), so that the long problems start early and the launch does not end with a few wavefronts still walking
// the longest segments.  order[rank] = segment; one thread per segment counts the segments ahead of its own.
// Beyond kOrderMaxSegments the order is left as it is (the count is quadratic in the number of segments).
constexpr int kOrderMaxSegments = 4096;
__global__ __launch_bounds__(256) void em_order_segments(gss_yview yv, const int32_t* __restrict__ T_len, int Tmax, int S,
                                                         int32_t* __restrict__ order) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  if (S > kOrderMaxSegments) {
    order[s] = s;
    return;
  }
  const int T = y_frames(yv, T_len, s, Tmax);
  int rank = 0;
  for (int o = 0; o < S; ++o) {
    const int To = y_frames(yv, T_len, o, Tmax);
    rank += (To > T || (To == T && o < s)) ? 1 : 0;
  }
  order[rank] = s;
}

// Whether the whole-EM kernel requests the next tile's frames before phase 2 (tile layout): not with 8 channels and 8 classes, where
// the 17 registers are missed (12 segments of up to 300 frames, 5 iterations 517 us, requested ahead 541).
__host__ __device__ constexpr bool request_ahead(int D, int K) { return D * K < 64; }

// One pass of a wavefront of the whole-EM kernel over its tiles below tile_end: the one resident tile `pre` (ONE_TILE), or
// tiles wave, wave + NW, ...  With the direct layout there are registers to spare (36 accumulators at most), and the frames of
// the next tile are requested from memory before the current tile is worked on.
template <int D, int K, int NW, bool ONE_TILE, PassKind KIND, bool RESIDENT, bool DIRECT, class MaskPtr>
__device__ __forceinline__ void whole_pass(
    const float2* __restrict__ Yrow, const uint8_t* __restrict__ abrow, MaskPtr tmrow,
    const double (&creg)[RESIDENT ? K * coef_regs(D) : 1], const double* __restrict__ sC, const double (&cc)[K],
    float* __restrict__ gamma_row, uint32_t* __restrict__ status, long gamma_kstride, int T, int Tmax, int tile_end,
    int wave, int lane, unsigned my_mask, TileRegs<D>& pre, double* __restrict__ sY,
    typename PassAcc<D, K, DIRECT>::type& acc, double (&nacc)[K]) {
  constexpr bool FINAL = KIND == PASS_FINAL;
  if constexpr (ONE_TILE) {
    if (wave < tile_end)
      pass_tile<D, K, KIND, RESIDENT, DIRECT, TILE_KEEP>(Yrow, abrow, creg, sC, cc, gamma_row, status, gamma_kstride, T, Tmax,
                                             wave * kWave, lane, __builtin_amdgcn_readfirstlane(my_mask), sY, acc,
                                             nacc, &pre);
  } else if constexpr (DIRECT) {
    constexpr unsigned kmask = (1u << K) - 1u;
    TileRegs<D> cur{};                                   // (replaced below when the first tile is live)
    int tile = wave;
    unsigned m = 0u;
    if (tile < tile_end) {
      m = tmrow[tile] & kmask;
      if (m != 0u) load_tile_regs<D>(cur, Yrow, abrow, tile * kWave, lane, T);
    }
    while (tile < tile_end) {
      const int next = tile + NW;
      TileRegs<D> nxt = cur;
      unsigned mn = 0u;
      if (next < tile_end) {
        mn = tmrow[next] & kmask;
        if (mn != 0u) load_tile_regs<D>(nxt, Yrow, abrow, next * kWave, lane, T);
      }
      // (the mask is the same in every lane; the compiler has to be told after the loop-carried copy)
      pass_tile<D, K, KIND, RESIDENT, DIRECT, TILE_KEEP>(Yrow, abrow, creg, sC, cc, gamma_row, status, gamma_kstride, T, Tmax,
                                             tile * kWave, lane, __builtin_amdgcn_readfirstlane(m), sY, acc, nacc,
                                             &cur);
      cur = nxt;
      m = mn;
      tile = next;
    }
  } else if constexpr (FINAL || !request_ahead(D, K)) {
    for (int tile = wave; tile < tile_end; tile += NW)
      pass_tile<D, K, KIND, RESIDENT, DIRECT>(Yrow, abrow, creg, sC, cc, gamma_row, status, gamma_kstride, T, Tmax, tile * kWave,
                                       lane, tmrow[tile], sY, acc, nacc);
  } else {
    stream_tiles<D, K, KIND, RESIDENT>(Yrow, abrow, tmrow, creg, sC, cc, T, Tmax, wave, tile_end, NW, lane, sY, acc, nacc);
  }
}

// ----------------------------------------------------------------------------------------------
// Whole-EM kernel: a workgroup of NW wavefronts owns one (segment, frequency) for all iterations.  Per
// iteration every wavefront walks its tiles (pass_tile above), sums its accumulators over the rows of lanes
// through LDS, and factorises the K class matrices itself, so that the coefficients of the next iteration go
// from LDS straight back into its registers: no partial sums in memory, no second kernel, no launch per
// iteration, and the same fixed summation order on every run.
//   NW = 1: for batches with many problems (segments x frequencies >> resident wavefronts); the wavefront
//           walks all tiles of its problem; nothing is shared between wavefronts.
//   NW = 4: for few problems of few channels.  ONE_TILE, at most NW tiles (256 frames): wavefront w owns tile w and keeps
//           its frames in registers for all iterations, so an iteration reads nothing from memory.  More tiles:
//           wavefront w walks tiles w, w + NW, ...  The wavefronts' sums meet in LDS, and the first wavefront adds them up and
//           factorises for all of them (by each for itself on two sets of buffers, one barrier instead of two per iteration:
//           one segment of 200 frames, 10 iterations, 2 channels and 3 classes 26.6 -> 20.7 us (19.8 with the closed form at 2 channels), with
//           store_direct_sums_lds, 1500 frames, 8 iterations 54.0 -> 48.9; 4 channels and 5 classes 119 -> 112).
//
// End of an iteration: up to 4 channels a lane per class (factor_class_in_lane), otherwise a lane per row of a class
// (m_step_in_wave).
//
// Walk and resident tile are kernels of their own: in one kernel they need up to 57 registers more (4 channels and 2 classes 204,
// now 151 and 139), and with them a wavefront per SIMD less (one segment of 1860 frames, 3 iterations, 2 channels and 7 classes 66.0
// -> 52.3 us).
// ----------------------------------------------------------------------------------------------
// Wavefronts per SIMD that the kernel is compiled for.  With a tile per wavefront three, also where that spills up to 42 registers
// (2 and 4 channels, 8 classes): the 513 problems of a segment do not fit the chip at two (60 frames, 3 / 4 channels and 8 classes 1.68 /
// 1.64 times as long).  Up to 2 channels the tile loop lives in two registers for every
// accumulator, coefficient, partial sum and count, and some 40 more; the compiler takes one or two more than a step of the
// register file allows (2 channels: 74 with 2 classes, 169 with 8) unless it is told: 24 segments of up to 700 frames, 2
// classes, 3 iterations 88 -> 80 us, 48 segments of up to 300 frames, 8 classes 244 -> 209.
__host__ __device__ constexpr int whole_waves_per_simd(int D, int K, int NW) {
  if (D > 2) return 2;
  const int regs = 2 * K * (D * D + 4) + 40, waves = 512 / ((regs + 7) / 8 * 8), most = NW > 1 ? 4 : 8;   // (four wavefronts: LDS)
  return waves < most ? waves : most;
}
template <int D, int K, int NW, bool ONE_TILE>
__global__ __launch_bounds__(kWave * NW, ONE_TILE ? 3 : whole_waves_per_simd(D, K, NW)) void em_whole_small(
    gss_yview yv, const uint8_t* __restrict__ act, const uint8_t* __restrict__ abyte, const uint32_t* __restrict__ tmask,
    const int32_t* __restrict__ T_len, const int32_t* __restrict__ seg_order, float* __restrict__ gamma,
    uint32_t* __restrict__ status, int F, int Tmax, int iters, int weight_mode) {
  constexpr int E = D * D;
  constexpr int R = coef_regs(D);
  constexpr bool RESIDENT = resident_coefs(D, K);
  constexpr bool DIRECT = direct_layout(D, K, ONE_TILE);   // no blocks in LDS then
  constexpr int kCoefDoubles = K * R * 16;             // packed coefficients, padded to whole registers
  constexpr int kSumDoubles = K * E + K;               // packed weighted scatter sums, then the class counts
  // The sums, counts and class constants of the M-step live only between the last tile of a pass and the first
  // tile of the next one: they share the memory of the blocks.  So do the coefficients when they are resident in registers
  // during a pass (otherwise the pass reads them from LDS and they keep a place of their own).
  constexpr bool IN_WAVE = D > kLaneFactorMaxD;        // m_step_in_wave: the class matrices instead of sums, counts and constants
  constexpr int kMstepKept = IN_WAVE ? K * mat_doubles(D) : kSumDoubles + K;
  constexpr int kMstepDoubles = kMstepKept + (RESIDENT ? kCoefDoubles : 0);
  // (NW > 1: the sums of every wavefront, and the buffers of the M-step, are in a part of their own; the wavefront's part is a
  // block's or store_direct_sums_lds's)
  constexpr int kBlocks = DIRECT ? (NW > 1 ? 16 * kReduceRow : 0) : kBlockDoubles;
  constexpr int kTileDoubles = NW > 1 ? kBlocks : ((kMstepDoubles > kBlocks ? kMstepDoubles : kBlocks) + 1) / 2 * 2;
  constexpr int kWaveDoubles = kTileDoubles + (RESIDENT ? 0 : kCoefDoubles);
  constexpr int kShareDoubles = NW > 1 ? NW * kSumDoubles + kMstepDoubles : 0;
  static_assert(NW == 1 || RESIDENT, "coefficients from the shared part go to registers");
  __shared__ __attribute__((aligned(16))) double lds[NW * kWaveDoubles + kShareDoubles];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / kWave) : 0;
  double* __restrict__ sY = lds + wave * kWaveDoubles;
  double* __restrict__ sR = NW > 1 ? lds + NW * kWaveDoubles : sY;   // [K][E] packed weighted scatter sums
  double* __restrict__ sN = sR + K * E;                // [K] class counts
  double* __restrict__ sCC = sN + K;                   // [K] class constants pi / det B
  double* __restrict__ sC = RESIDENT ? sR + kMstepKept : sY + kTileDoubles;   // [K][R * 16] coefficients of B^-1 for the next pass
  double* __restrict__ sShare = lds + NW * kWaveDoubles + kMstepDoubles;      // [NW][kSumDoubles] sums of the wavefronts (NW > 1)
  __shared__ int sPlaces[IN_WAVE ? kWave : 1];
  static_assert(!IN_WAVE || NW == 1, "one table of places");
  if constexpr (IN_WAVE) {
    static constexpr MatPlaces<D> kPlaces = make_mat_places<D>();
    sPlaces[lane] = kPlaces.code[lane];
  }

  // workgroup -> (segment, frequency): the segments in the order of seg_order (longest first), if given
  const long sf = blockIdx.x;
  int s = (int)((unsigned)sf / (unsigned)F);
  const int f = (int)((unsigned)sf % (unsigned)F);
  if (seg_order) {
    typedef const __attribute__((address_space(4))) int32_t* order_ptr_t;
    s = ((order_ptr_t)(uintptr_t)seg_order)[s];
  }
  int T;
  const float2* __restrict__ Yrow = y_row(yv, T_len, s, f, D, Tmax, T);
  const uint8_t* __restrict__ abrow = abyte + (long)s * Tmax;
  const int tiles_total = (Tmax + kWave - 1) / kWave;
  typedef const __attribute__((address_space(4))) uint32_t* mask_ptr_t;
  const mask_ptr_t tmrow = (mask_ptr_t)(uintptr_t)(tmask + (long)s * tiles_total);
  float* __restrict__ gamma_row = gamma + ((long)s * K * F + f) * Tmax;
  const long gamma_kstride = (long)F * Tmax;
  const int tiles = (T + kWave - 1) / kWave;

  // ONE_TILE: this wavefront's one tile: its mask, and the lane's frame in registers.
  // (Otherwise wavefront w walks tiles w, w + NW, ...)
  TileRegs<D> pre;
  unsigned my_mask = 0u;
#pragma unroll
  for (int d = 0; d < D; ++d) pre.y[d] = make_float2(0.f, 0.f);
  pre.abits = 0u;
  if constexpr (ONE_TILE) {
    // (its activity straight from the input: packing it would be a launch of its own in front of this one)
    const int t = wave * kWave + lane;
    unsigned bits = 0u;
    if (t < T) {
#pragma unroll
      for (int k = 0; k < K; ++k) bits |= (act[((long)s * K + k) * Tmax + t] != 0 ? 1u : 0u) << k;
    }
#pragma unroll
    for (int k = 0; k < K; ++k) my_mask |= (__ballot((int)((bits >> k) & 1u)) != 0 ? 1u : 0u) << k;
    if (my_mask != 0u) {                                // a frame below T exists
#pragma unroll
      for (int d = 0; d < D; ++d) pre.y[d] = Yrow[(long)(t < T ? t : 0) * D + d];
    }
    pre.abits = bits;
  }

  // (written by the end of the first iteration)
  double creg[RESIDENT ? K * R : 1];
  double cc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) cc[k] = 1.0;
#pragma unroll
  for (int r = 0; r < (RESIDENT ? K * R : 1); ++r) creg[r] = 0.0;

  // Everything the end of an iteration derives from the lane number is derived there anew, from a copy of
  // the lane number that the compiler cannot see through: values computed ahead of the iteration loop would be
  // live across the tile loop, where there is no register for them, and come back from scratch memory one
  // dependent load at a time.
  wave_lds_sync();
  for (int it = 0; it < iters; ++it) {
    typename PassAcc<D, K, DIRECT>::type acc;
    double nacc[K];
    zero_acc(acc);
#pragma unroll
    for (int k = 0; k < K; ++k) nacc[k] = 0.0;
    if (it == 0)
      whole_pass<D, K, NW, ONE_TILE, PASS_FIRST, RESIDENT, DIRECT>(Yrow, abrow, tmrow, creg, sC, cc, nullptr, status, gamma_kstride,
                                                                   T, Tmax, tiles, wave, lane, my_mask, pre, sY, acc, nacc);
    else
      whole_pass<D, K, NW, ONE_TILE, PASS_NEXT, RESIDENT, DIRECT>(Yrow, abrow, tmrow, creg, sC, cc, nullptr, status, gamma_kstride,
                                                                  T, Tmax, tiles, wave, lane, my_mask, pre, sY, acc, nacc);

    int le = lane;                                      // the lane number again, opaque
    asm volatile("" : "+v"(le));
    if constexpr (IN_WAVE) {
      m_step_in_wave<D, K>(acc, nacc, sY, sPlaces, sC, cc, le, weight_mode, status);
      wave_lds_sync();
    } else {
      // ---- sums over the lanes -> packed sR[k][e]; class counts -> sN[k] ----
      // (NW > 1: the wavefronts' sums meet in LDS; the first one adds them up and runs the M-step for all of
      // them: run by each of them it took issue slots that the others of the SIMD miss)
      if constexpr (NW > 1) {
        double* __restrict__ sOut = sShare + wave * kSumDoubles;
        if constexpr (DIRECT) store_direct_sums_lds<D, K>(acc, nacc, sY, sOut, le);
        else store_tile_sums<D, K>(acc, nacc, sOut, le);
        __syncthreads();                                // every wavefront's sums of this iteration are in place
        if (wave == 0) {
          for (int e = le; e < kSumDoubles; e += kWave) {
            double sum = sShare[e];
#pragma unroll
            for (int w = 1; w < NW; ++w) sum += sShare[w * kSumDoubles + e];
            sR[e] = sum;                                // sN follows sR
          }
          wave_lds_sync();
          factor_class_in_lane<D, K>(sR, sN, sC, sCC, le, weight_mode, status);
        }
        __syncthreads();
      } else {
        if constexpr (DIRECT) store_direct_sums<D, K>(acc, nacc, sR, le);
        else store_tile_sums<D, K>(acc, nacc, sR, le);
        wave_lds_sync();
        // ---- M-step: B_k from (R_k, N_k), regularised, inverted; coefficients and class constants ----
        factor_class_in_lane<D, K>(sR, sN, sC, sCC, le, weight_mode, status);
        wave_lds_sync();
      }
#pragma unroll
      for (int k = 0; k < K; ++k) {
        // the class constant is the same in every lane: kept in scalar registers across the tile loop
        const double c = sCC[k];
        cc[k] = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(c)),
                                 __builtin_amdgcn_readfirstlane(__double2loint(c)));
      }
    }
    if constexpr (RESIDENT) {
#pragma unroll
      for (int k = 0; k < K; ++k)
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int e = 16 * r + (le & 15);
          creg[k * R + r] = sC[k * (R * 16) + (e < E ? e : E - 1)];
        }
    }
    wave_lds_sync();
  }

  // final pass: the posteriors = the masks, zero padding included
  {
    typename PassAcc<D, K, DIRECT>::type acc;
    double nacc[K];
    zero_acc(acc);
#pragma unroll
    for (int k = 0; k < K; ++k) nacc[k] = 0.0;
    whole_pass<D, K, NW, ONE_TILE, PASS_FINAL, RESIDENT, DIRECT>(Yrow, abrow, tmrow, creg, sC, cc, gamma_row, status, gamma_kstride, T,
                                                   Tmax, tiles_total, wave, lane, my_mask, pre, sY, acc, nacc);
  }
}

// ----------------------------------------------------------------------------------------------
// Host-side plan and dispatch
// ----------------------------------------------------------------------------------------------
struct EmPlan {
  ChunkMap acc;          // chunking of the accumulating passes
  ChunkMap fin;          // chunking of the final pass
  long wgs_acc, wgs_fin;
  size_t off_coef, off_cc, off_part, off_npart, off_abyte, off_tmask, off_order, total;
};

EmPlan make_plan(const gss_ctx* ctx, long n_sf, int S, int Tmax, int D, int K, int wgs_per_cu, int wgs_per_cu_fin) {
  EmPlan p;
  const int tiles = (Tmax + kWave - 1) / kWave;
  const int round_up = kPassWaves;                     // a chunk is a whole number of rounds of tiles
  const long slots = (long)ctx->num_cu * wgs_per_cu;
  p.acc = plan_chunk_map(slots, n_sf, tiles, round_up, 0, true);
  p.wgs_acc = chunk_map_wgs(p.acc, n_sf);
  p.fin = plan_chunk_map((long)ctx->num_cu * wgs_per_cu_fin, n_sf, tiles, round_up, 0, true);
  p.wgs_fin = chunk_map_wgs(p.fin, n_sf);
  const size_t E = (size_t)D * D;
  size_t o = 0;
  p.off_coef = o;  o = gss_align_up(o + (size_t)n_sf * K * E * sizeof(double) + 64, 256);
  p.off_cc = o;    o = gss_align_up(o + (size_t)n_sf * K * sizeof(double), 256);
  p.off_part = o;  o = gss_align_up(o + (size_t)p.wgs_acc * K * E * sizeof(double), 256);
  p.off_npart = o; o = gss_align_up(o + (size_t)p.wgs_acc * K * sizeof(double), 256);
  p.off_abyte = o; o = gss_align_up(o + (size_t)S * Tmax, 256);
  p.off_tmask = o; o = gss_align_up(o + (size_t)S * tiles * sizeof(uint32_t), 256);
  p.off_order = o; o = gss_align_up(o + (size_t)S * sizeof(int32_t), 256);
  p.total = o;
  return p;
}

template <int D, int K>
int run_small(gss_ctx* ctx, const gss_yview& Y, const uint8_t* act, const int32_t* T_len, int S, int F, int Tmax,
              int iters, int weight_mode, float* gamma, hipStream_t st) {
  const long n_sf = (long)S * F;
  // resident workgroups per compute unit of the two pass kernels: asked once per instantiation
  static const int wgs_per_cu = resident_wgs(em_pass_small<D, K, PASS_NEXT>, kWave * kPassWaves, 2);
  static const int wgs_per_cu_fin = resident_wgs(em_pass_small<D, K, PASS_FINAL>, kWave * kPassWaves, 2);
  // From 5 channels on chunks for two workgroups per compute unit also where registers and LDS have room for more.  The 513 problems of
  // a segment are a chunk each then, and the 513th goes to the free places in pieces; planned for three, all of them are
  // cut in two, and the launch is a round and a third (1560 frames, 5 iterations, 5 channels and 3 classes 156 -> 127 us, 7
  // channels and 2 classes 175 -> 144).
  const int plan_wgs = D <= kWholeQuadMaxD || wgs_per_cu < 2 ? wgs_per_cu : 2;
  const EmPlan p = make_plan(ctx, n_sf, S, Tmax, D, K, plan_wgs, wgs_per_cu_fin);
  int rc = gss_ensure_scratch(ctx, p.total);
  if (rc != GSS_OK) return rc;
  char* base = (char*)ctx->scratch;
  double* coef = (double*)(base + p.off_coef);
  double* cc = (double*)(base + p.off_cc);
  double* part = (double*)(base + p.off_part);
  double* npart = (double*)(base + p.off_npart);
  uint8_t* abyte = (uint8_t*)(base + p.off_abyte);
  uint32_t* tmask = (uint32_t*)(base + p.off_tmask);
  int32_t* order = (int32_t*)(base + p.off_order);
  const int tiles = (Tmax + kWave - 1) / kWave;

  if ((long)S * tiles > 0x7fffffffL) return GSS_EUNSUPPORTED;
  if (p.wgs_acc > 0x7fffffffL || p.wgs_fin > 0x7fffffffL) return GSS_EUNSUPPORTED;
  const dim3 block(kWave * kPassWaves);
  // Many problems: one wavefront runs the whole EM of a problem (no partial sums, no factor launches).  Few problems: each one
  // is cut into chunks over several workgroups, one pass and one factor launch per iteration, unless it has few tiles: two
  // launches per iteration cost more than the whole EM of such a problem in one wavefront.
  const bool choose = ctx->em_whole_min_problems < 0;
  bool whole = choose ? use_whole(D, (double)n_sf / ctx->num_cu, tiles, T_len != nullptr) : n_sf >= (long)ctx->em_whole_min_problems;
  // Up to 4 channels there is the variant with four wavefronts per problem (use_quad), and as tiles are cheap (a launch costs as
  // much as a few dozen of them) few problems go to the whole-EM kernel as well unless a pass is so long that
  // the launches per iteration no longer matter.
  bool tiny = false;
  if constexpr (D <= kWholeQuadMaxD) {
    if (choose) {
      static const int ones_per_cu = resident_wgs(em_whole_small<D, K, kWholeQuad, true>, kWave * kWholeQuad, 2);
      static const int walks_per_cu = resident_wgs(em_whole_small<D, K, kWholeQuad, false>, kWave * kWholeQuad, 2);
      const int quads_per_cu = tiles <= kWholeQuad ? ones_per_cu : walks_per_cu;
      tiny = use_quad(D, K, (double)n_sf / ctx->num_cu, tiles, iters, T_len ? S : 1);
      const int row = tiny ? (tiles + kWholeQuad - 1) / kWholeQuad + 1 : tiles;
      if (row <= whole_max_tiles(tiny, quads_per_cu)) whole = true;
    }
  }
  whole = iters > 0 && whole && n_sf <= 0x7fffffffL;
  // (tiny problems with a resident tile per wavefront read the activity themselves: 4 to 5 us of launch and kernel less.  Not
  // where the masks are written over the activity: a workgroup may start when another one is done.)
  const uintptr_t act0 = (uintptr_t)act, act1 = act0 + (size_t)S * K * Tmax, out0 = (uintptr_t)gamma,
                  out1 = out0 + (size_t)n_sf * K * Tmax * sizeof(float);
  if (!whole || (tiles <= kWholeQuad && act0 < out1 && out0 < act1)) tiny = false;
  if (!(tiny && tiles <= kWholeQuad))
    hipLaunchKernelGGL(em_pack_activity<false>, dim3((unsigned)(S * tiles)), dim3(kWave), 0, st, Y, act, T_len, abyte, tmask, K,
                       Tmax, tiles);
  if (whole) {
    // a ragged batch is taken longest segment first
    const int32_t* seg_order = nullptr;
    if (S > 1 && T_len) {
      hipLaunchKernelGGL(em_order_segments, dim3((unsigned)((S + 255) / 256)), dim3(256), 0, st, Y, T_len, Tmax, S, order);
      seg_order = order;
    }
    gss_profile_begin(ctx, 0, st);
    if constexpr (D <= kWholeQuadMaxD) {
      if (tiny)
        hipLaunchKernelGGL((tiles <= kWholeQuad ? em_whole_small<D, K, kWholeQuad, true> : em_whole_small<D, K, kWholeQuad, false>),
                           dim3((unsigned)n_sf), dim3(kWave * kWholeQuad), 0, st, Y, act, abyte, tmask, T_len, seg_order, gamma,
                           ctx->status, F, Tmax, iters, weight_mode);
    }
    if (!tiny)
      hipLaunchKernelGGL((em_whole_small<D, K, 1, false>), dim3((unsigned)n_sf), dim3(kWave), 0, st, Y, act, abyte, tmask, T_len,
                         seg_order, gamma, ctx->status, F, Tmax, iters, weight_mode);
    gss_profile_end(ctx, 0, st);
    if (hipGetLastError() != hipSuccess) return GSS_EHIP;
    return GSS_OK;
  }
  if (iters == 0) hipLaunchKernelGGL(em_init_coef, dim3(1024), dim3(256), 0, st, coef, cc, D, K, n_sf);
  for (int it = 0; it < iters; ++it) {
    gss_profile_begin(ctx, 0, st);
    hipLaunchKernelGGL((it == 0 ? em_pass_small<D, K, PASS_FIRST> : em_pass_small<D, K, PASS_NEXT>), dim3((unsigned)p.wgs_acc), block, 0, st, Y, abyte, tmask, T_len, coef,
                       cc, part, npart, (float*)nullptr, ctx->status, F, Tmax, p.acc);
    gss_profile_end(ctx, 0, st);
    gss_profile_begin(ctx, 1, st);
    hipLaunchKernelGGL((em_factor_small<D, K>), dim3((unsigned)n_sf), dim3(kWave * K), 0, st, part, npart, coef, cc,
                       ctx->status, p.acc, weight_mode);
    gss_profile_end(ctx, 1, st);
  }
  hipLaunchKernelGGL((em_pass_small<D, K, PASS_FINAL>), dim3((unsigned)p.wgs_fin), block, 0, st, Y, abyte, tmask, T_len, coef, cc,
                     (double*)nullptr, (double*)nullptr, gamma, ctx->status, F, Tmax, p.fin);
  if (hipGetLastError() != hipSuccess) return GSS_EHIP;
  return GSS_OK;
}

}  // namespace
