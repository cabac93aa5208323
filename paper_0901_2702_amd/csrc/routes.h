// Which kernel takes a call, by the sizes of the instrument and of the call:
// the group inverter and its synthesis (group.hip: a wave per few pixels, a
// synthesis point per lane) or a pixel per lane (kernels.hip).  The results
// are the same bits.  Host code that needs no HIP, so that the rules can be
// held against the measured times on the CPU.
#pragma once

#include <stdint.h>

namespace vfisv {

// Synthesis points of an instrument and the chunks of 64 that they take in
// the group kernels, which spend a whole chunk's time on a part of one.
struct Extent {
  bool band;
  int points;
  int chunks;
};

// What a fit is for: a launch whose schedule the caller chose, a plain fit,
// the learned path's short fit and its re-fit.
enum FitUse { FIT_SCHEDULED, FIT_PLAIN, FIT_SHORT, FIT_REFIT };

constexpr int64_t GROUP_ANY = INT64_MAX;

// The most pixels of a fit that the group inverter is faster for, 0 if it is
// for none.  lm_kernel's time is flat up to 65,536 pixels, its lanes, and goes
// with the points; the group inverter's goes with pixels and whole chunks.
// Measured, time in lm_kernel / here (default options):
//  dense, plain: 7 points 4,096 1.87, 16,384 0.97, 131,072 0.49; 29 points
//   32,768 1.07, 57,344 0.80; 45 points 81,920 1.01, 131,072 0.88; 59 points
//   (HMI) 131,072 1.08, 196,608 0.97; 64 points 196,608 1.03.
//  dense, short fits from the network's start (more trials are accepted, whose
//   Jacobian lm_kernel computes ahead): 7 points 4,096 1.06, 16,384 0.73; 29
//   points 16,384 1.41, 32,768 0.85; 59 points 45,056 1.14, 65,536 0.90.
//   Re-fits cross later (lm_kernel then runs lane pairs up to 36,044 pixels):
//   29 points 32,768 1.21, 59 points 57,344 1.34.
//  banded, plain: 3 samples 16,384 1.28, 32,768 0.80, 1,000,000 0.36; 8
//   samples 49,152 1.20, 131,072 0.83; 13 (a full chunk) 196,608 1.09,
//   524,288 0.92; 14 (a second chunk) 57,344 1.11, 131,072 0.83; 20 131,072
//   1.03, 393,216 0.86; 29 (two full) 1,000,000 1.03; 30 262,144 1.01, 524,288
//   0.86; 61 1,000,000 1.16; 112 524,288 1.16.
//  banded, short: 5 samples 16,384 1.41, 32,768 0.81; 14 32,768 1.16, 65,536
//   0.75; 20 57,344 1.08, 131,072 0.97; 112 131,072 1.29, 262,144 1.07.
//   Re-fits: 8 samples 57,344 1.00; 14 98,304 1.04, 163,840 0.88; 20 262,144
//   1.05; 112 262,144 1.44; after a network that has learned nothing (more
//   trials each) 14 32,768 1.25, 65,536 0.77; 20 57,344 1.11, 65,536 0.95.
// A banded limit is n0 rho / (1 - rho), rho being the ratio of the two costs
// per pixel in large launches and n0 the pixels that the flat part is worth.
// (131,072 in the learned path is no crossover for wide spectra: both sides
// of it are faster here, 163,840 of 112 samples 1.17 short, 1.66 re-fits.)
// A fit of few trials is a pixel's set-up more than its passes: HMI pixels
// with max_iter 0 1,024 0.76 and 16,384 0.58, max_iter 2 1,024 1.69 and 16,384
// 0.92, near the minimum max_iter 3 16,384 1.09 and 32,768 0.93, max_iter 5
// 32,768 1.16 and 57,344 0.84; 112 samples max_iter 0 262,144 1.84, max_iter 1
// 16,384 1.60, 32,768 1.05, 57,344 0.72, max_iter 3 32,768 1.31, 49,152 0.91.
// Partly filled chunks cross far earlier, as lm_kernel's latency goes with the
// points: 19 points max_iter 0 512 0.84, max_iter 2 2,048 0.52, max_iter 3 2,048
// 0.73; 14 samples max_iter 3 32,768 0.81; full ones do not: near the minimum 13
// samples max_iter 3 16,384 1.21, 32,768 0.97, 29 samples 49,152 0.93.
inline int64_t fit_group_max(const Extent& e, FitUse use, int max_iter) {
  if (use == FIT_SCHEDULED || e.chunks < 1) return 0;
  const bool plain = use == FIT_PLAIN;
  int64_t most;
  if (e.band) {
    const double n0[3][3] = {{26e3, 35e3, 58e3}, {18e3, 20e3, 20e3}, {26e3, 30e3, 45e3}};
    const double rho = (0.6 * e.points + 10.0) / (32.0 * e.chunks + 22.0);
    most = plain ? GROUP_ANY : 131072;
    if (rho < 0.97) {
      const double n = n0[use - FIT_PLAIN][e.chunks < 3 ? e.chunks - 1 : 2] * rho / (1.0 - rho);
      if (n < (double)most) most = (int64_t)n;
    }
  } else if (plain) {
    most = e.points <= 29 ? 1200 * (int64_t)e.points : 34804 + 3482 * (int64_t)(e.points - 29);
  } else {
    most = e.points > 3 ? 1006 * (int64_t)e.points - 2010 : 1024;
  }
  const double fill = e.points / (64.0 * e.chunks), fill2 = fill * fill;
  int64_t few = GROUP_ANY;
  if (max_iter < 3) {
    const int64_t n = (int64_t)(max_iter < 2 ? 512 : 2048) << (e.chunks < 7 ? e.chunks - 1 : 6);
    few = (int64_t)((n < 32768 ? n : 32768) * fill2);
  } else if (max_iter < 10) {
    few = (int64_t)((e.chunks > 1 ? 40960 : 24576) * fill2 * fill2);
  }
  if (max_iter == 0 && e.chunks > 5) few = GROUP_ANY;
  return most < few ? most : few;
}

// Whether the synthesis of n models (Weideman's series) goes to waves of a few
// models.  As above: a model per lane takes the points' time whatever n is, up
// to 65,536 models and more, waves of a few models whole chunks' time per
// model.  Measured, model per lane / here:
//  dense, values: 7 points 1,024 1.37, 4,096 0.88, 1,000,000 0.36; 29 points
//   30,011 1.04, 65,536 0.83; 59 points 90,000 1.14, 131,072 0.95; 64 points
//   200,000 1.02.
//  dense, with Jacobian: 7 points 8,192 0.96, 16,384 0.79; 29 points 30,011
//   1.03, 45,000 0.91; 45 points 65,536 1.07, 131,072 0.89; 52 points and more
//   at any size (52 262,144 1.05, 59 1.12).
//  banded, values: 1 sample 16,384 1.44, 30,011 0.65, 1,000,000 0.30; 8 samples
//   45,000 0.99; 10 45,000 1.08, 1,000,000 0.90; 13 (a full chunk) and more at
//   any size except a mostly empty second chunk: 14 30,011 1.09, 45,000 0.92;
//   16 30,011 1.20, 65,536 0.68; 20 1,000,000 1.49, 30 1.55, 112 2.10.
//  banded, with Jacobian: 1 sample 8,192 1.09, 30,011 0.50, 1,000,000 0.23; 8
//   samples 16,384 1.40, 45,000 0.67, 1,000,000 0.92; 14 16,384 1.24, 30,011
//   0.86; instruments whose chunks are nearly full at any size but for a dip
//   where the lanes are just filled: 20 30,011 1.10, 45,000 0.77, 65,536 0.82,
//   114,688 1.10, 1,000,000 1.23; 30 45,000 0.73, 114,688 1.10, 1,000,000 1.25;
//   46 45,000 0.96, 112 1.24.
inline bool synth_by_group(const Extent& e, int64_t n, bool jac) {
  if (e.chunks < 1) return false;
  if (!e.band) {
    if (e.points <= 29) return n <= (jac ? 1000 : 41 * e.points) * (int64_t)e.points;
    if (jac) return e.points >= 50 || n <= 29000 + 3000 * (int64_t)(e.points - 29);
    return n <= 34798 + 2663 * (int64_t)(e.points - 29);
  }
  const double fill = e.points / (64.0 * e.chunks);
  if (n <= (jac ? 600 : 900) * (int64_t)e.points / e.chunks) return true;
  if (!jac) return fill >= (e.chunks == 1 ? 0.95 : 0.64);
  if (fill < (e.chunks == 1 ? 0.78 : 0.64)) return false;
  return fill >= 0.95 || e.chunks > 3 || n >= (e.chunks == 1 ? 196608 : 98304);
}

}  // namespace vfisv
