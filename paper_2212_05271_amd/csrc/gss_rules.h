// Which kernel a call takes where the library has several for it: functions of its sizes alone, without a device, so that a host
// compiler builds and checks them by themselves.
#pragma once

namespace {

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
