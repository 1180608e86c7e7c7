// Which kernel a call takes where the library has several for it: functions of its sizes alone, without a device, so that a host
// compiler builds and checks them by themselves.
#pragma once

namespace {

// ----------------------------------------------------------------------------------------------
// EM up to 8 channels
// ----------------------------------------------------------------------------------------------
// Few channels: the lane that owns a frame in phase 1 has all D * D entries of its outer product in registers
// anyway (one block of at most 16), and in the direct layout adds w_k * P[e] to K * D * D accumulators of its own: no
// phase 2.  The accumulators are acc[k][e] then (packed order), and the sums over the lanes are taken at the end of the pass
// (transpose_reduce).  `one`: the kernel whose wavefronts have one tile each.
// The line lies where the layouts were measured against each other: the direct one costs no LDS round trip, but its accumulators
// keep wavefronts from the SIMDs and take longer to add up.  Direct / tile layout, us, 32 segments of up to 700 frames, 5
// iterations: 3 channels and 3 / 4 / 5 / 8 classes 266 / 276, 312 / 313, 404 / 364, 582 / 496, 4 channels and 2 / 3 / 5 classes
// 304 / 302, 411 / 350, 571 / 445.  One segment of 200 frames, a tile per wavefront, 10 iterations: 3 channels and 2 / 5 classes
// 32.7 / 28.5, 54.6 / 39.3, 4 channels and 2 / 5 classes 43.4 / 45.6, 68.7 / 61.2.  (4 segments of 3 channels and 5 to 7 classes,
// two wavefronts per SIMD, are 4 to 7 % faster with the direct one.)
constexpr bool direct_layout(int D, int K, bool one) {
  return D <= 2 || (!one && ((D == 3 && K <= 4) || (D == 4 && K <= 2)));
}

// Where the whole-EM kernel with a wavefront per problem is used: tiles per problem, by the problems per compute unit (`load`; 2 for
// the 513 bins of a segment) and whether the segments have lengths of their own, so that the wavefronts end at different times.
// The line lies where the routes were measured against each other, 8 iterations, time in one launch over time in chunks:
//   segments of   330 frames   400         701         1200        1875 frames (8 channels and 5 classes, uniform / ragged)
//   1             0.92         0.97        1.22        1.44        1.70
//   2             0.82 / 0.71  0.90 / 0.72 1.06 / 0.87 1.18 / 1.05 1.33 / 1.23
//   3             0.66 / 0.64  0.69 / 0.70 0.84 / 0.83 0.97 / 0.98 1.06 / 1.15
//   4             0.73 / 0.63  0.79 / 0.61 0.95 / 0.68 1.03 / 0.79 1.12 / 0.86
//   5             0.65 / 0.62  0.70 / 0.64 0.80 / 0.77 0.89 / 0.88 0.92 / 0.96
//   8             0.67 / 0.60  0.70 / 0.62 0.80 / 0.68 0.84 / 0.75 0.95 / 0.78
// and within 0.1 of that at 5 to 8 channels and 3 to 8 classes.  With fewer problems than compute units the chunks of a problem have a
// compute unit each: below load 0.7 5 tiles 0.91 to 1.14 (5 and 6 / 7 and 8 channels), 6 tiles 0.98 to 1.37, 8 and 9 1.33 to 2.0.  For
// the loads between those of whole segments of 513 bins the line is on the safe side: 1.1 to 1.8 and 2.1 to 3.9 8 and 9 tiles 0.76
// to 0.88, 10 to 12 0.82 to 1.01.  Problems of more than 32 tiles of one length end in a partly filled round and wait for 12
// segments (3 iterations, 8 segments of 4000 frames 1.05 to 1.2, 12 segments 0.98 to 1.14).
// Up to 4 channels: 0.5 to 0.95 times from 8 per compute unit on (4 channels, 5 classes, 2500 frames of one length 1.15: longer ones
// wait for 8 segments; 4 segments of up to 700 frames, 4 channels and 8 classes 190 us in chunks, 120 in one launch).
inline bool use_whole(int D, double load, int tiles, bool ragged) {
  if (D <= 4) return load >= (tiles <= 32 ? 8 : 16) || tiles <= 5;
  if (tiles > 32) return load >= 24;
  const int most = load >= 10 ? 32 : load >= 8 ? (ragged ? 32 : 16) : load >= 6 ? (ragged ? 19 : 16) : load >= 4 ? (ragged ? 10 : 9) : load < 1 ? 5 : D >= 7 ? 6 : 7;
  return tiles <= most;
}
// Up to 4 channels: tiles in a row up to which a pass costs less than its launches; where two workgroups of four wavefronts fit a
// compute unit, the 513 problems of a segment take two rounds (4000 frames of 4 channels and 5 classes 1.2 times as long as in chunks).
constexpr int whole_max_tiles(bool quad, int wgs_per_cu) { return quad && wgs_per_cu <= 2 ? 12 : 25; }
// Four wavefronts per problem instead of one, up to 4 channels: fewer tiles in a row, but barriers, and one of the four adds up and
// factorises while the others wait, which costs the more the more problems share a compute unit (`load`): 0.95 `load` - 1.9 tiles,
// and 1.15 `load` at 2 channels, where one wavefront per problem leaves room for many.  `lengths` segments of their own lengths (1:
// all alike) save fewer tiles than the longest one says.  A tile per wavefront: a launch goes as well (the activity is read in
// place), which counts the more the fewer and shorter the iterations; at 2 channels and 7 or 8 classes that kernel keeps 28 and 42
// registers in scratch memory, which costs it 1.5 tiles (one tile of one segment 1.27).  Of the walks with the direct layout at 3
// and 4 channels two workgroups fit a compute unit: 1.2 `load` tiles (three segments of 6 or 7 tiles 1.25).
// Four / one, time of the call, 5 iterations and more, mean over 1 to 4 channels and 2 to 8 classes:
//   tiles         1     2     3     4     5-6   7-9   10-14 15-22 23-30
//   1 segment     0.92  0.80  0.75  0.65  0.75  0.68  0.62  0.56  0.53    (513 bins: load 2)
//   2             1.30  1.01  0.91  0.80  0.92  0.81  0.79  0.69  0.67
//   3             1.55  1.24  1.12  1.02  1.05  1.00  0.95  0.89  0.83
//   4             1.55  1.22  1.03  0.94  1.10  0.97  0.91  0.86  0.85
//   6             1.73  1.37  1.16  1.12  1.19  1.02  0.96  0.90  0.92
//   9 to 24       1.98  1.56  1.44  1.27  1.38  1.26  1.14  1.06  0.99
// and with 1 to 3 iterations one tile of 1, 2, 3, 6 segments 0.82, 0.90, 1.06, 1.48.  Over 4122 calls (1 to 8 classes, 1 to 24 segments
// of 30 to 1900 frames, 33 to 513 bins, 1 to 15 iterations) the choice takes 0.4 % longer than the better of both on average,
// and more than a tenth longer in 55 of them (by `load` squared and the tiles alone 1.8 % and 300); over 1721 calls of 2 to 4 channels,
// 125 frames and 5 iterations or more, two thirds of them with lengths of their own, 0.07 % and 3.
constexpr int kWholeQuad = 4;                 // wavefronts per problem of the variant for few problems
constexpr int kWholeQuadMaxD = 4;             // ... which is built for up to this many channels
inline bool use_quad(int D, int K, double load, int tiles, int iters, int lengths) {
  const int row = (tiles + kWholeQuad - 1) / kWholeQuad;
  double saved = (lengths > 1 ? 0.65 + 0.45 / lengths : 1.0) * (tiles - row);
  if (row == 1) saved += 150.0 / ((double)iters * (D + 1) * (K + 2)) - (D == 2 && K >= 7 ? 1.5 : 0.0);
  else if (D >= 3 && direct_layout(D, K, false)) return saved >= 1.2 * load;
  return saved >= (D == 2 ? 1.15 : 0.95) * load - 1.9;
}

// ----------------------------------------------------------------------------------------------
// Inverse STFT: a workgroup of `waves` wavefronts forms waves * steps - 3 blocks from waves * steps frames, in `per_seg` workgroups
// per segment.  16 wavefronts fill a compute unit and read runs of 128 bytes; 8 leave room for a second workgroup, and alone on their
// compute unit they take two thirds of the time per step.  The times of a round (every compute unit busy once) of c steps, in
// tenths of a microsecond, are fitted to 5245 calls (1 to 400 segments of 1000 samples to a minute, by kernel time):
//   steps                          1     2     3     4     8     16
//   16 wavefronts                  8.7   13.8  18.9  23.9  44    84 us   36 + 51 c
//   8, one per compute unit        6.2   9.4   12.7  16.1  29    55      32 + 34 c (c up to 8)
//   8, two per compute unit        9.8   15.0  20.5  27    50    92      44 + 57 c
// One segment of 2 to 50 s 8.9 -> 6.6 us against 16 wavefronts always, 168 segments of 0.2 s 14.1 -> 9.9; calls that keep 16
// wavefronts keep their steps: the fewest in a row over the rounds of workgroups, with one more per workgroup for its start
// and the three frames that are done twice.
// ----------------------------------------------------------------------------------------------
struct IstftPlan {
  int waves, steps;
  long per_seg;
};
constexpr int kIstftMaxSteps16 = 32, kIstftMaxSteps8 = 8;
inline IstftPlan plan_istft(long S, long T, int num_cu) {
  auto parts = [&](int waves, int c) { return (T - 3 + waves * c - 4) / (waves * c - 3); };
  auto rounds = [&](long n) { return (S * n + num_cu - 1) / num_cu; };
  IstftPlan p{16, 1, parts(16, 1)};
  for (int c = 2; c <= kIstftMaxSteps16; ++c) {
    const long n = parts(16, c);
    if (rounds(n) * (c + 1) < rounds(p.per_seg) * (p.steps + 1)) p = {16, c, n};
  }
  long best = rounds(p.per_seg) * (36 + 51 * p.steps);
  for (int c = 1; c <= kIstftMaxSteps8; ++c) {
    const long n = parts(8, c), r = rounds(n), cost = r / 2 * (44 + 57 * c) + r % 2 * (32 + 34 * c);
    if (cost < best) {
      best = cost;
      p = {8, c, n};
    }
  }
  return p;
}

}  // namespace
