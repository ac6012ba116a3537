// Correlations carried from step to step by Gram columns: shared declarations.
//
// After step k took c psi_i off the residual, every correlation changes by
// c <psi_m, psi_i> (eq. 9 applied to eq. 11), so a step whose atom's Gram
// column g_i = Psi^T psi_i is known needs no pass over the dictionary.  The
// decode alternates two kernels on one stream:
//
//   pass   (the whole chip) one read of the dictionary gives the correlations
//          c~ = Psi^T r and up to kGramReq Gram columns, as one matrix
//          product with kGramReq + 1 right-hand sides on the FP32 matrix
//          cores; it stays bound by the dictionary's bytes;
//   steps  (one workgroup per signal) takes MP steps on the carried
//          correlations until it selects an atom whose Gram column it does
//          not hold (or the carried error has grown too large, or the run
//          stops); it then asks for that column and those of the best other
//          atoms, which are the likely next choices.
//
// The carried correlations only shortlist.  `GramBounds` bounds their
// difference from the exact products, so every atom whose FP32 inner product
// could be the largest is on the list; the list is scored with the FP32
// inner product of the stepping form (dot_column_f32), and the winner, its
// coefficient, the residual, the norm and the stop test are the stepping
// form's bit for bit.
//
// Against one pass per step (whole decodes, to eps = 1e-5): N = 8192,
// M = 32768, K = 512: 19.5 ms from 384 ms (2,367 steps of about 6 us, 22
// passes of 199 us); N = 2048, M = 8192, K = 128: 2.2 ms from 9.0 ms (562 steps
// of 3.2 us, 8 passes).  A signal without structure (noise,
// every step a new atom) is no slower either: the wanted columns cover the
// next several choices (N = 2048, M = 8192, with 16 right-hand sides: 8.4 us a
// step against 15.0; N = 1000, M = 3001: 437 us a decode against 807).  FP64,
// N = 8192, M = 32768, K = 512: 26.8 ms from 750 ms.
#pragma once

#include "mp_internal.h"

namespace mp {

constexpr int kGramReq = 31;        // Gram columns per pass (with r: 32 right-hand sides)
constexpr int kGramTile = 32;       // atoms of one wave's tile of a pass
constexpr int kGramRaggedWaves = 4; // waves per workgroup of the ragged pass
constexpr int kGramMaxAtoms = 32768;  // of a dictionary that decodes on carried correlations
constexpr int kGramMaxCand = 64;    // atoms scored exactly in one step, at most
constexpr unsigned kGramNone = 0xFFFFu;  // map entry of an atom without a Gram column

// What the steps kernel leaves for the pass, and the other way round.
struct GramCtl {
  int nreq;            // Gram columns wanted: atoms req[0 .. nreq)
  int slot0;           // the first of the nreq slots they go to
  int used;            // slots in use
  int req[kGramReq];
};

// Rounding bounds, all relative to ||r|| (columns of norm at most nrm).
struct GramBounds {
  float pass;          // |c~ - <r, psi>| after a pass
  float col;           // |g~ - <psi_i, psi_m>|
  float step;          // added per step, times ||r||: r's own rounding
  float carry;         // added per step, times the largest |c~|: c~'s own rounding
  float dot;           // |dot_column_f32 - <r, psi>|
};

// One signal's decode; T = float or double, the type of the dictionary, r and
// x~ (the carried correlations and Gram columns are float for both: they
// only shortlist).
template <typename T>
struct GramProb {
  const T* psi;        // ld x m columns
  int64_t ld, n, m;
  int64_t mp;          // stride of the Gram columns, >= the steps kernel's threads x share
  float* c;            // mp carried correlations (written by the pass)
  float* g;            // slots x mp Gram columns
  uint16_t* map;       // m: slot of each atom's Gram column, or kGramNone
  int slots;
  float* rhs;          // 32 x ld: a pass's right-hand sides in operand order
  T* r;                // ld elements
  T* x;
  DevState* st;        // pad[0]: the decode gave up (another form goes on from its steps)
  GramCtl* ctl;
};

// Where a pass's right-hand side i keeps row `row`: float4 64 s + 32 q + i
// holds rows 8 s + 4 q .. + 3.
__host__ __device__ inline int64_t gram_rhs_at(int64_t row, int i) {
  return (row / 4 * (kGramReq + 1) + i) * 4 + row % 4;
}

// Threads and correlations per thread of the steps kernel for m atoms and
// columns of ld elements of `esize` bytes; threads 0 where it does not apply.
// c~ and a Gram column have gram_stride entries.
struct GramShape {
  int threads, per_thread;
};
GramShape gram_shape(int64_t ld, int64_t m, int esize);
inline int64_t gram_stride(const GramShape& sh) {
  const int64_t all = static_cast<int64_t>(sh.threads) * sh.per_thread;
  return all < kGramMaxAtoms ? all : kGramMaxAtoms;
}
GramBounds gram_bounds(int64_t n, double max_norm, bool f64);

template <typename T>
struct GramTrace {
  typedef mp_trace type;
};
template <>
struct GramTrace<double> {
  typedef mp_trace_f64 type;
};

// One pass (first: with r only, and the slot map cleared), then the steps it
// allows.  Both return at once when the state says the run is over.
template <typename T>
hipError_t launch_gram_pass(const GramProb<T>& p, int num_cus, bool first, hipStream_t s);
template <typename T>
hipError_t launch_gram_steps(const GramProb<T>& p, const GramShape& sh, const GramBounds& b,
                             long long max_iters, bool first, typename GramTrace<T>::type tr,
                             hipStream_t s);

// ---- Orthogonal Matching Pursuit (k_omp_gram.hip) ---------------------------
struct OmpCarry {
  int hold;              // the next step waits for a block's pass
  int fit;               // the last selection is to be fitted by the launches after it
  int cur;               // block position of the last selected atom; -1: P holds it already,
                         // or it was not in the block
  long long t0;          // directions before the block
  float err;             // bound on |c~ - <r, psi_m>|
  int slot[kGramReq];    // block positions of the atoms selected from it, in order
  float perr[kGramReq];  // bounds on their columns of P
  GramCtl ctl;           // the block's candidates
};
// The block's two passes, where *hold is set: right-hand sides packed, then
// over the first st->t (at most pq.m) columns of pq; and over p.
hipError_t launch_gram_block(const GramProb<float>& p, const GramProb<float>& pq, const int* hold,
                             int num_cus, hipStream_t s);
hipError_t launch_gram_block_pass(const GramProb<float>& p, const int* hold, int num_cus,
                                  hipStream_t s);
hipError_t launch_omp_carry_init(const OmpBufs& b, hipStream_t s);
hipError_t launch_omp_block(const float* psi, int64_t ld, int64_t n, int64_t m, float* r,
                            const OmpBufs& b, DevState* st, long long t_bound, int num_cus,
                            hipStream_t s);
hipError_t launch_omp_pick(const float* psi, int64_t ld, int64_t m, const float* r,
                           const OmpBufs& b, const GramBounds& bd, bool after_pass,
                           bool want_coef, DevState* st, hipStream_t s);
int64_t omp_tops(int64_t m);   // keys k_omp_carry publishes

// ---- signals that share one dictionary (k_gram_batched.hip) ----------------
struct GramBatch {
  const float* psi;    // ld x m
  int64_t ld, n, m;
  int64_t mp;          // stride of g and c
  const float* g;      // every atom's Gram column: m x mp
  float* c;            // per signal: mp carried correlations
  float* r;            // per signal: ld floats
  float* x;            // per signal: ldx floats (the caller's)
  int64_t ldx;
  DevState* states;    // per signal; pad[0]: gave up
};
GramBounds gram_bounds_full(int64_t n, double max_norm);
hipError_t launch_gram_full(const float* psi, int64_t ld, int64_t m, float* g, int64_t mp,
                            int num_cus, hipStream_t s);
hipError_t launch_gram_binit(const float* Y, int64_t ldy, int64_t n, int64_t ld, float* X,
                             int64_t ldx, int64_t m, float* R, DevState* states,
                             const long long* tcap, long long tcap_all, double eps, int nb,
                             hipStream_t s);
// Round `round`: the correlations of the signals still running, then their
// steps.  again: two words; word round mod 2 is set if some signal goes on
// (both launches return at once where the previous round's word is clear).
// single: one signal's decode, whose ||r||^2 is summed in mp_solve's order.
hipError_t launch_gram_bround(const GramBatch& b, const GramShape& sh, const GramBounds& bd,
                              int nb, int num_cus, long long round, int* again, bool single,
                              mp_trace tr, hipStream_t s);

// ---- many independent problems (k_gram.hip) ---------------------------------
struct GramGroup {     // one workgroup of the pass: tiles of problem id
  int id, group;
};
struct GramRagged {
  const GramProb<float>* probs;  // device, count (x is filled in from X)
  const RInst* inst;             // device: offsets of y and x~
  const GramBounds* bounds;      // device, count
  const int* order;              // device: problems, most work first
  const GramGroup* groups;       // device: the pass's work list
  int* again;                    // device, two words (see GramBatch)
  int count, ngroups, split;
  int64_t max_ld, lds;           // lds: of the steps kernel
  bool small;                    // every problem has at most 4096 atoms and rows
  bool one;                      // the product is one lane chain (the FP32 form's)
};
GramBounds gram_bounds_one(int64_t n, double max_norm);
// Stride of a problem's Gram columns in a set whose largest are max_ld, max_m
// (m <= 32768), and tiles per workgroup of the pass for `tiles` in all.
int64_t gram_ragged_stride(int64_t max_ld, int64_t max_m, int64_t m);
int gram_ragged_groups(int64_t tiles, int num_cus);
hipError_t launch_gram_rinit(const GramRagged& g, const float* Y, float* X, const long long* caps,
                             long long cap_all, double eps, hipStream_t s);
hipError_t launch_gram_rcopy(const GramProb<float>* probs, const RInst* inst, int count, float* R,
                             hipStream_t s);
hipError_t launch_gram_rround(const GramRagged& g, float* X, long long round, mp_trace tr,
                              hipStream_t s);

}  // namespace mp
