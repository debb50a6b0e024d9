// The stream-K cut of the decoder projections (linear.hip): which run of
// chunks each block takes and, for the epilogues, which run holds a chunk.
#pragma once

#include <stdint.h>

namespace ooo {

// The stream-K cut: C chunks (tile-major) in B runs, q = C / B, r = C % B; r
// runs hold one chunk more: the first ones, or (spread) evenly dealt, run b
// from chunk floor(C b / B) = q b + floor(r b / B) on.  Where B runs cover the
// tiles periodically, the even cut lets blocks B / period apart, on one XCD,
// stream the same columns of X at the same time.  That matters once X is
// larger than the XCD's 4 MiB L2: with 40 tiles of 432 chunks (K 27648, O
// 5120) longer runs first against spread take 124.2 / 99.6 us at 256 rows (14
// MB of X), 74.9 / 64.7 at 128 and 64.4 / 63.4 at 100, 52.7 / 51.9 at 64
// (3.5 MB), but 46.7 / 50.8 at 17 and 45.0 / 47.7 at one.
struct Runs {
  int q, r, B, seg;
  // longer runs of lo(b): floor((mul b + 1/2) step), mul = r and step = 1 / B
  // spread (r b < B^2, and the quotient's fraction is a multiple of 1 / B,
  // which half a step and a relative error of 2^-22 do not cross), mul =
  // step = 1 otherwise, r at most
  int mul;
  float step;
  // runs per chunk before chunk `head` and from there on (spread: all before)
  int head;
  float rate0, rate1;
  __host__ __device__ __forceinline__ int lo(int b) const {
    const int longer = (int)(((float)(mul * b) + 0.5f) * step);
    return q * b + (longer < r ? longer : r);
  }
  // the run that holds chunk x: an estimate that is at most one off, corrected
  __host__ __device__ __forceinline__ int of(int x) const {
    int b = x < head ? (int)((float)x * rate0) : r + (int)((float)(x - head) * rate1);
    b = b < B - 1 ? b : B - 1;
    return b - (lo(b) > x) + (lo(b + 1) <= x);
  }
};

// The cut of C chunks (1 <= C < 2^31) in B runs.
inline Runs cut_runs(long long C, int B, int KC, bool spread) {
  Runs u{};
  u.B = B;
  u.q = (int)(C / B);
  u.r = (int)(C % B);
  u.seg = (int)((C / B + (u.r > 0)) / KC) + 2;  // tiles a run can touch
  u.mul = spread ? u.r : 1;
  u.step = spread ? 1.f / (float)B : 1.f;
  u.head = spread ? INT32_MAX : u.r * (u.q + 1);
  u.rate0 = spread ? (float)((double)B / (double)C) : 1.f / (float)(u.q + 1);
  u.rate1 = 1.f / (float)u.q;
  return u;
}

}  // namespace ooo
