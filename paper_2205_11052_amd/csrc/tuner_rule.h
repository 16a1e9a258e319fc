// Which stage kernels the launch-shape tuner times.
#pragma once

#include <cstdint>

namespace dgw {

// The FP32 kernels round differently (relative 1e-6 after some hundred stages).
// On a whole MI355X (256 compute units) FP32 therefore doesn't time one against
// the other: the kernel follows from the order and the elements of all shots,
// and only its launch shape is timed.  Kernel 0 runs where it is named here,
// kernel 1 elsewhere, kernel 2 nowhere.
//
// The ranges record what the timing itself chose, at every order over 48 to 82944
// elements (three tunings of each of 80 sizes; all but three agreed), when
// kernel 1 still read every operator tile from L2: order 6, 24576 elements, 201
// against 221 us; order 3, 24576 elements, 31 against 35; order 1, 82944
// elements, 28 against 38.  The middle ranges are where the last wave of kernel
// 1's work-groups on 256 compute units was nearly empty.  Kernel 1 has become
// faster since (order 6: 169 us); the ranges are kept so that a run gives the
// bits it gave, not because they are the fastest choice.  On any other number of
// compute units they stand for nothing and every kernel is timed.
struct TunerRange {
  int N;
  bool aniso;
  int64_t from, to;
};
constexpr int64_t kNoEnd = INT64_MAX;
constexpr TunerRange kNodePerThread[] = {
    {1, false, 5100, kNoEnd}, {3, false, 3700, kNoEnd}, {4, false, 0, 1000},
    {4, false, 1650, 3700},   {5, false, 5100, 9100},   {6, false, 0, 29000},
    {1, true, 3700, kNoEnd},  {2, true, 1650, kNoEnd},  {3, true, 0, kNoEnd},
    {4, true, 1650, 2500},    {5, true, 0, 530},        {5, true, 1000, 1650},
    {6, true, 0, 20000}};

inline bool tuner_times(int kernel, int N, int precision, bool aniso, int64_t elems, int ncu) {
  if (precision == 64 || ncu != 256) return true;
  int named = 1;
  for (const TunerRange &r : kNodePerThread)
    if (r.N == N && r.aniso == aniso && elems >= r.from && elems < r.to) named = 0;
  return kernel == named;
}

}  // namespace dgw
