// The one-bit decode in checked batches of steps (k_sign_gram.hip).
#pragma once

#include "mp_internal.h"

namespace mp {

constexpr int kSignActive = 1024;  // active atoms at once, at most
constexpr int kSignSteps = 128;    // steps of a round, at most
constexpr int kSignBeats = 1024;   // atoms a round's check names, at most
constexpr int kSignRows = 4;       // rows of r per lane of a replay

// What the launches of a round leave each other.
struct SignCarry {
  int nact, nnew;                // active atoms; those of them new in this round (the last)
  int steps, count, stalled;     // steps to take; taken; ended on c* = 0
  int first, nbeat;              // first step an atom beat; atoms that beat one
  int take;                      // steps that stand
  int fill;                      // no atom is active: fill from the correlations
  long long t0;                  // steps before the round
  int atom[kSignActive];         // by position
  int log_pos[kSignSteps], log_atom[kSignSteps];
  double log_c[kSignSteps];
  int beat_step[kSignBeats], beat_atom[kSignBeats];
};

int64_t sign_gram_stride(int64_t m);  // of the Gram entries of one active atom
hipError_t launch_sgram_init(const SignGram& b, int64_t m, hipStream_t s);
// first: no atom is active yet, so there are no steps to take or check.
hipError_t launch_sgram_round(const uint32_t* bits, int64_t ws, int64_t n, int64_t m, int64_t ld,
                              double* c64, double* r64, float* r32, const CorrGeom& geom,
                              const SignGram& b, bool first, long long max_iters, float* x,
                              DevState* st, mp_trace tr, hipStream_t s);

}  // namespace mp
