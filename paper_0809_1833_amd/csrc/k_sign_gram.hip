// The one-bit decode (k_sign.hip) in batches of steps taken on part of the
// atoms and checked against all of them.
//
// A step changes every correlation by c* times an exact integer (the Gram
// entry), in FP64, atom by atom: the steps of a few hundred active atoms can
// run ahead in one workgroup without the others, and whether another atom
// would have been selected can be asked of all atoms at once afterwards.  A
// round is four launches:
//
//   steps   one workgroup: up to kSignSteps steps over the active atoms, each
//           a wave-wide maximum, one barrier and a row of the active atoms'
//           Gram entries; the steps' atoms and coefficients are logged;
//   check   all atoms replay the log against their own Gram entries and name
//           the first step at which they beat its atom; all rows of r replay
//           it and leave each step's partial ||r||^2;
//   decide  one workgroup: the steps up to the first stop or the first such
//           beat stand; the state, the trace; the atoms that beat a step
//           become active;
//   commit  all atoms (with x~) and all rows of r take the steps that stand; Gram
//           entries (16-bit integers, exact) of the atoms that became active
//           against every atom.
//
// Every value that stands is computed from the same operands in the same
// order as one launch per step does (k_mp_step_sign), so the results are the
// same bit for bit; which atoms are active decides only how many steps a
// round brings.  Bound by the steps' chain of latencies and the launches of
// a round: a step 0.96 us (about a third are taken again in a later round),
// check 18, decide 10, commit 15 us for 128 of them.  N = 8192, M = 32768,
// K = 512 (2,376 steps): 5.5 ms a decode from 23.4 in one persistent launch
// that exchanged every step between all CUs.
#include <type_traits>

#include "k_common.h"
#include "k_key2.h"
#include "k_sign_gram.h"
#include "mp_internal.h"

namespace mp {

constexpr int kStepThreads = 256;
constexpr int kStepWaves = kStepThreads / kWave;
constexpr int kPerThread = kSignActive / kStepThreads;  // active atoms per thread
constexpr int kCheckThreads = 128;
constexpr int kDecideThreads = 1024;
constexpr int kDecideWaves = kDecideThreads / kWave;
constexpr int kCommitAtoms = kWave;     // atoms per workgroup of the commit, one per lane
constexpr int kCommitThreads = 256;
constexpr int kCommitWaves = kCommitThreads / kWave;
constexpr int kNewGroup = 16;           // new atoms a wave counts at once
constexpr int kNewChunks = 32;          // 16-byte chunks of a column staged at a time
constexpr int kFirstActive = 256;       // active atoms to begin with, about
constexpr int kNewMost = 128;           // atoms that become active in a round, at most
constexpr int kBins = 1024;
constexpr int kReplay = 32;             // Gram entries in flight per lane of a replay
constexpr int kTurn = kReplay + 1;      // stride of a lane's sums in LDS
constexpr unsigned short kNoPos = 0xFFFFu;
static_assert(kSignSteps % kReplay == 0, "a log is whole groups");
static_assert(kPerThread == 4, "a thread's Gram entries are one 8-byte load");

typedef short v4s __attribute__((ext_vector_type(4)));

__device__ inline double wave_max_f64(double v) {
  v = __builtin_fmax(v, dpp_f64<kDppQuadSwap1>(v));
  v = __builtin_fmax(v, dpp_f64<kDppQuadSwap2>(v));
  v = __builtin_fmax(v, dpp_f64<kDppRowRor4>(v));
  v = __builtin_fmax(v, dpp_f64<kDppRowRor8>(v));
  return __builtin_fmax(__builtin_fmax(lane_f64(v, 0), lane_f64(v, 16)),
                        __builtin_fmax(lane_f64(v, 32), lane_f64(v, 48)));
}

// wave_sum's value, bit for bit, in lane 63 alone: no scalar registers, so that
// several sums overlap.  (wave_sum takes lane 0 of each row of 16, where the
// quads Q meet as (Q0 + Q3) + (Q2 + Q1); a rotation by 12 gives the last lane
// of the row the same pairs.)
__device__ inline double wave_sum_lane63(double v) {
  constexpr int kRowRor12 = 0x12C, kRowBcast15 = 0x142, kRowBcast31 = 0x143;
  v += dpp_f64<kDppQuadSwap1>(v);
  v += dpp_f64<kDppQuadSwap2>(v);
  v += dpp_f64<kRowRor12>(v);
  v += dpp_f64<kDppRowRor8>(v);
  v += dpp_f64<kRowBcast15>(v);
  v += dpp_f64<kRowBcast31>(v);
  return v;
}

__global__ __launch_bounds__(256) void k_sgram_init(SignCarry* g, unsigned short* pos, int64_t m) {
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < m;
       i += static_cast<int64_t>(gridDim.x) * 256)
    pos[i] = kNoPos;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    g->nact = g->nnew = g->count = g->stalled = g->take = g->nbeat = 0;
    g->first = kSignSteps;
    g->fill = 1;
    g->steps = 32;
  }
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kStepThreads) void k_sgram_steps(
    const double* __restrict__ c64, const short* __restrict__ h, double inv_n,
    long long max_iters, const DevState* __restrict__ st, SignCarry* __restrict__ g) {
  if (st->done) return;
  const double thr = st->thr;
  struct Rec {
    double mag, c;
    int pos;
  };
  __shared__ Rec rec[2][kStepWaves];
  __shared__ int s_atom[kSignActive];
  __shared__ int s_log[kSignSteps];
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int nact = g->nact;
  int steps = nact > 0 ? g->steps : 0;
  const long long left = max_iters - st->t;
  if (left < steps) steps = static_cast<int>(left);
  // (a position past the active atoms: -1 in every maximum)
  double c[kPerThread];
  bool live[kPerThread];
#pragma unroll
  for (int e = 0; e < kPerThread; ++e) {
    const int p = kPerThread * tid + e;
    live[e] = p < nact;
    const int atom = live[e] ? g->atom[p] : 0;
    s_atom[p] = atom;
    c[e] = live[e] ? c64[atom] : 0.0;
  }
  __syncthreads();
  int s = 0;
  bool stalled = false;
  // ||r||^2 falls by c*^2 a step: where that reaches the threshold further
  // steps would be for nothing (whether the run stops there is decided from r)
  double rr = st->rr;
  for (; s < steps && rr > thr; ++s) {
    // the wave's largest |c|; of equal ones the smallest atom
    double mag[kPerThread], best = -1.0;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e) {
      mag[e] = live[e] ? __builtin_fabs(c[e]) : -1.0;
      best = __builtin_fmax(best, mag[e]);
    }
    const double top = wave_max_f64(best);
    int pos = -1;
    double val = 0.0;
    if (top >= 0.0) {
#pragma unroll
      for (int e = 0; e < kPerThread; ++e)
        for (unsigned long long l = __ballot(mag[e] == top); l != 0; l &= l - 1) {
          const int p = kPerThread * (kWave * wave + __builtin_ctzll(l)) + e;
          const bool less = pos < 0 || s_atom[p] < s_atom[pos];
          pos = __builtin_amdgcn_readfirstlane(less ? p : pos);
        }
      double mine = c[0];
#pragma unroll
      for (int e = 1; e < kPerThread; ++e) mine = pos % kPerThread == e ? c[e] : mine;
      val = lane_f64(mine, pos / kPerThread % kWave);
    }
    if (lane == 0) rec[s & 1][wave] = Rec{top, val, pos};
    __syncthreads();
    // (selects and a second look at ties: with a tie's branch inside the loop
    // the compiler kept the other record's c beside the new position)
    Rec w = rec[s & 1][0];
    int ties = 0;
#pragma unroll
    for (int k = 1; k < kStepWaves; ++k) {
      const Rec o = rec[s & 1][k];
      const bool more = o.mag > w.mag;
      ties = more ? 0 : ties + (o.mag == w.mag ? 1 : 0);
      w.mag = more ? o.mag : w.mag;
      w.c = more ? o.c : w.c;
      w.pos = more ? o.pos : w.pos;
    }
    if (ties != 0) {  // of equal ones the smallest atom, by its place in LDS
      int at = -1;
      for (int k = 0; k < kStepWaves; ++k)
        if (rec[s & 1][k].mag == w.mag && rec[s & 1][k].pos >= 0) {
          const int here = s_atom[rec[s & 1][k].pos];
          const int best = at < 0 ? 0x7FFFFFFF : s_atom[rec[s & 1][at].pos];
          at = here < best ? k : at;
        }
      at = __builtin_amdgcn_readfirstlane(at);
      w.c = rec[s & 1][at].c;
      w.pos = rec[s & 1][at].pos;
    }
    const int row = __builtin_amdgcn_readfirstlane(w.pos);
    const v4s e4 =
        reinterpret_cast<const v4s*>(h + static_cast<int64_t>(row) * kSignActive)[tid];
    if (tid == 0) {
      s_log[s] = w.pos;
      g->log_c[s] = w.c;
    }
    if (w.c == 0.0) {  // (the check asks whether every other atom's is)
      stalled = true;
      break;
    }
    const double a = w.c * inv_n;
    rr -= w.c * w.c;
#pragma unroll
    for (int e = 0; e < kPerThread; ++e)
      c[e] = __builtin_fma(-a, static_cast<double>(static_cast<int>(e4[e])), c[e]);
  }
  __syncthreads();
  if (tid < s + (stalled ? 1 : 0)) {
    g->log_pos[tid] = s_log[tid];
    g->log_atom[tid] = s_atom[s_log[tid]];
  }
  if (tid == 0) {
    g->count = s;
    g->stalled = stalled ? 1 : 0;
  }
}

// ---------------------------------------------------------------------------
// The log in LDS, filled up to whole replay groups with steps that change and
// beat nothing, so that a replay has no branches and its reads run ahead
// (with a test at each step 128 steps took 28 us, most of it LDS latency).
struct SignLog {
  double c[kSignSteps], a[kSignSteps];  // c*, c* / N
  int pos[kSignSteps], atom[kSignSteps];
};
__device__ inline void stage_log(SignLog& l, const SignCarry* __restrict__ g, int count,
                                 double inv_n) {
  const int all = (count + kReplay - 1) / kReplay * kReplay;
  for (int i = static_cast<int>(threadIdx.x); i < all; i += static_cast<int>(blockDim.x)) {
    const bool on = i < count;
    const double c = on ? g->log_c[i] : 0.0;
    l.c[i] = on ? c : __builtin_inf();
    l.a[i] = c * inv_n;
    l.pos[i] = on ? g->log_pos[i] : 0;
    l.atom[i] = on ? g->log_atom[i] : -1;
  }
  __syncthreads();
}

// One atom through the first `count` logged steps.  CHECK: returns the first
// step at which it beats the step's atom (count: none; a step on c* = 0, which
// ends the run whatever its atom, is beaten by c != 0 alone).  Otherwise adds
// to x~ the coefficients of the steps that selected it.
template <bool CHECK>
__device__ inline int replay_atom(const short* __restrict__ gcol, int64_t mstride, int a,
                                  const SignLog& l, int count, double& c, float& x) {
  int beat = count;
  for (int s0 = 0; s0 < count; s0 += kReplay) {
    short e[kReplay];
#pragma unroll
    for (int u = 0; u < kReplay; ++u) {
      const int p = __builtin_amdgcn_readfirstlane(l.pos[s0 + u]);
      e[u] = gcol[static_cast<int64_t>(p) * mstride + a];
    }
#pragma unroll
    for (int u = 0; u < kReplay; ++u) {
      const int s = s0 + u;
      if constexpr (CHECK) {
        const double mine = __builtin_fabs(c), best = __builtin_fabs(l.c[s]);
        const bool won = (mine > best) | ((mine == best) & (best > 0.0) & (a < l.atom[s]));
        beat = won && s < beat ? s : beat;
      } else {
        const float more = x + static_cast<float>(l.c[s]);
        x = a == l.atom[s] ? more : x;
      }
      c = __builtin_fma(-l.a[s], static_cast<double>(static_cast<int>(e[u])), c);
    }
  }
  return beat;
}

// One wave: the rows of workgroup v of the stepping form through the first
// `count` logged steps (r_n -/+ c* / sqrt(N), rows with a set bit get +), R
// per lane.  CHECK: the steps' partial ||r||^2, summed as k_mp_step_sign does;
// otherwise r is stored, and (TRACE) its trace entries from step t0 on.
template <bool CHECK, bool TRACE, int R>
__device__ inline void replay_rows(const uint32_t* __restrict__ bits, int64_t ws, int n,
                                   int64_t row0, int64_t row1, int v, int lane, int count,
                                   double inv_sqrt_n, const SignLog& l,
                                   double* __restrict__ r64, float* __restrict__ r32,
                                   double* __restrict__ parts, int grid, long long t0,
                                   const mp_trace& tr, double* turn) {
  constexpr int U = kReplay / R;  // steps whose words are in flight
  double r[R];
  bool in[R];   // rows of this workgroup
  bool up[R];   // and of Psi
  int word[R], bit[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int64_t i = row0 + lane + kWave * q;
    in[q] = i < row1;
    up[q] = in[q] && i < n;
    r[q] = in[q] ? r64[i] : 0.0;
    word[q] = up[q] ? static_cast<int>(i >> 5) : 0;
    bit[q] = static_cast<int>(i & 31);
  }
  for (int s0 = 0; s0 < count; s0 += U) {
    uint32_t w[U][R];
    double sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int atom = __builtin_amdgcn_readfirstlane(l.atom[s0 + u]);
      const uint32_t* col = bits + static_cast<int64_t>(atom < 0 ? 0 : atom) * ws;
#pragma unroll
      for (int q = 0; q < R; ++q) w[u][q] = col[word[q]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int st = s0 + u;
      const bool on = st < count;
      const double step = l.c[st] * inv_sqrt_n;
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < R; ++q) {
        const double x = r[q] + (((w[u][q] >> bit[q]) & 1u) ? step : -step);
        r[q] = up[q] && on ? x : r[q];
        if constexpr (TRACE)
          if (up[q] && on && t0 + st < tr.cap)
            tr.r[(t0 + st) * tr.ldr + row0 + lane + kWave * q] = static_cast<float>(r[q]);
        const double more = __builtin_fma(r[q], r[q], s);  // (k_mp_step_sign's contraction)
        s = in[q] ? more : s;
      }
      sum[u] = s;
    }
    if constexpr (CHECK) {
      // wave_sum's value of each step, the steps side by side: lane u adds
      // rows 0 and 1 of 16 lanes of step u, lane u + 32 rows 2 and 3, each
      // row's quads Q as (Q0 + Q3) + (Q2 + Q1)
#pragma unroll
      for (int u = 0; u < U; ++u) turn[lane * kTurn + u] = sum[u];
      __builtin_amdgcn_wave_barrier();
      const int u = lane % 32, half = lane / 32;
      double rows[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const double* p = turn + (32 * half + 16 * k) * kTurn + (u < U ? u : 0);
        double quad[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          quad[e] = (p[4 * e * kTurn] + p[(4 * e + 1) * kTurn]) +
                    (p[(4 * e + 2) * kTurn] + p[(4 * e + 3) * kTurn]);
        rows[k] = (quad[0] + quad[3]) + (quad[2] + quad[1]);
      }
      const double pair = rows[0] + rows[1];
      const double all = pair + __shfl_xor(pair, 32, kWave);
      __builtin_amdgcn_wave_barrier();
      if (lane < U && s0 + lane < count)
        parts[static_cast<int64_t>(s0 + lane) * grid + v] = all;
    }
  }
  if constexpr (!CHECK) {
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (up[q] && count > 0) {
        const int64_t i = row0 + lane + kWave * q;
        r64[i] = r[q];
        r32[i] = static_cast<float>(r[q]);
      }
  }
}

template <bool CHECK>
__device__ inline void replay_rows_of(const uint32_t* __restrict__ bits, int64_t ws, int n,
                                      int64_t ld, int rows_per_wg, int v, int lane, int count,
                                      double inv_sqrt_n, const SignLog& l,
                                      double* __restrict__ r64, float* __restrict__ r32,
                                      double* __restrict__ parts, int grid, long long t0,
                                      const mp_trace& tr, double* turn) {
  const int64_t row0 = static_cast<int64_t>(v) * rows_per_wg;
  const int64_t row1 = row0 + rows_per_wg < ld ? row0 + rows_per_wg : ld;
  auto run = [&](auto trace) {
    constexpr bool TRACE = decltype(trace)::value;
    if (rows_per_wg <= kWave)
      replay_rows<CHECK, TRACE, 1>(bits, ws, n, row0, row1, v, lane, count, inv_sqrt_n, l, r64,
                                   r32, parts, grid, t0, tr, turn);
    else
      replay_rows<CHECK, TRACE, kSignRows>(bits, ws, n, row0, row1, v, lane, count, inv_sqrt_n, l,
                                           r64, r32, parts, grid, t0, tr, turn);
  };
  if (!CHECK && tr.r) run(std::true_type{});
  else run(std::false_type{});
}

__global__ __launch_bounds__(kCheckThreads) void k_sgram_check(
    const uint32_t* __restrict__ bits, int64_t ws, int n, int64_t m, int64_t ld,
    const double* __restrict__ c64, double* __restrict__ r64, const short* __restrict__ gcol,
    int64_t mstride, double inv_n, double inv_sqrt_n, int grid, int rows_per_wg, int ablocks,
    double* __restrict__ parts, const DevState* __restrict__ st, SignCarry* g) {
  const int count = g->count, total = count + g->stalled;
  if (st->done || total == 0) return;
  __shared__ SignLog l;
  __shared__ double turn[kCheckThreads / kWave][kWave * kTurn];
  stage_log(l, g, total, inv_n);
  const int lane = static_cast<int>(threadIdx.x) % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  if (static_cast<int>(blockIdx.x) >= ablocks) {
    const int v = (static_cast<int>(blockIdx.x) - ablocks) * (kCheckThreads / kWave) + wave;
    if (v < grid)
      replay_rows_of<true>(bits, ws, n, ld, rows_per_wg, v, lane, count, inv_sqrt_n, l, r64, nullptr,
                        parts, grid, 0, mp_trace{}, turn[wave]);
    return;
  }
  const int64_t a = static_cast<int64_t>(blockIdx.x) * kCheckThreads + threadIdx.x;
  int beat = total;
  if (a < m) {
    double c = c64[a];
    float x = 0.0f;
    beat = replay_atom<true>(gcol, mstride, static_cast<int>(a), l, total, c, x);
  }
  const unsigned long long who = __ballot(beat < total);
  if (who == 0) return;
  int base = 0;
  if (lane == 0)
    base = __hip_atomic_fetch_add(&g->nbeat, static_cast<int>(__popcll(who)), __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
  base = __builtin_amdgcn_readfirstlane(base);
  if (beat < total) {
    (void)__hip_atomic_fetch_min(&g->first, beat, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int at = base + static_cast<int>(__popcll(who & ((1ull << lane) - 1)));
    if (at < kSignBeats) {
      g->beat_step[at] = beat;
      g->beat_atom[at] = static_cast<int>(a);
    }
  }
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kDecideThreads) void k_sgram_decide(
    const double* __restrict__ c64, int64_t m, const double* __restrict__ parts, int grid,
    long long max_iters, unsigned short* __restrict__ pos, DevState* __restrict__ st,
    SignCarry* __restrict__ g, mp_trace tr) {
  const double thr = st->thr;
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid % kWave, wave = tid / kWave;
  if (st->done) {
    if (tid == 0) g->take = g->nnew = 0;
    return;
  }
  __shared__ double red[kSignSteps][16];
  __shared__ double s_rr[kSignSteps], s_c[kSignSteps];
  __shared__ int s_atom[kSignSteps];
  __shared__ int s_stop, s_pos, s_cut;
  __shared__ int hist[kBins];
  __shared__ Key2 s_keys[kDecideWaves];
  const int count = g->count, first = g->first, fill = g->fill;
  const int nbeat = g->nbeat < kSignBeats ? g->nbeat : kSignBeats;
  const long long t0 = st->t;
  int nact = g->nact;
  if (tid == 0) s_stop = kSignSteps;
  if (tid < count) {
    s_c[tid] = g->log_c[tid];
    s_atom[tid] = g->log_atom[tid];
  }
  for (int i = tid; i < kBins; i += kDecideThreads) hist[i] = 0;
  // ||r||^2 after each step: the block sum of k_mp_step_sign over the partials
  // (64 partials of a step at a time, as that sum's waves; then 16 lanes a step)
  const int per = (grid + kWave - 1) / kWave;
  constexpr int U = kSignSteps / kDecideWaves;
  for (int k = 0; k < per; ++k) {
    const int i = k * kWave + lane;
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int s = wave + u * kDecideWaves;
      v[u] = i < grid && s < count ? parts[static_cast<int64_t>(s) * grid + i] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = wave_sum_lane63(v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (lane == kWave - 1) red[wave + u * kDecideWaves][k] = v[u];
  }
  __syncthreads();
  for (int e = tid; e < count * 16; e += kDecideThreads) {  // (whole rows of 16 lanes)
    double v = e % 16 < per ? red[e / 16][e % 16] : 0.0;
    v += dpp_f64<kDppQuadSwap1>(v);
    v += dpp_f64<kDppQuadSwap2>(v);
    v += dpp_f64<kDppRowRor4>(v);
    v += dpp_f64<kDppRowRor8>(v);
    if (e % 16 == 0) s_rr[e / 16] = v;
  }
  __syncthreads();
  if (tid < count && !(s_rr[tid] > thr)) atomicMin(&s_stop, tid);
  __syncthreads();
  const int stop = s_stop;
  int take = count;
  if (stop + 1 < take) take = stop + 1;
  if (first < take) take = first;
  const long long t = t0 + take;
  int reason = -1;
  if (take == stop + 1) reason = MP_STOP_CONVERGED;
  else if (t >= max_iters) reason = MP_STOP_MAX_ITERS;
  else if (g->stalled && take == count && first > count) reason = MP_STOP_STALLED;
  if (tid < take && t0 + tid < tr.cap) {
    if (tr.idx) tr.idx[t0 + tid] = s_atom[tid];
    if (tr.coef) tr.coef[t0 + tid] = static_cast<float>(s_c[tid]);
    if (tr.rr) tr.rr[t0 + tid] = s_rr[tid];
  }
  const bool over = reason != -1;
  bool refill = false;
  int nnew = 0;
  if (!over && fill) {
    // the atoms of largest |c|: whole bins of its leading bits, down to about
    // kFirstActive atoms (every atom where all can be active), and as many as
    // there is room for of a first bin that is larger.  The largest itself is
    // always one, so that the next round's first step stands.
    const int want = m <= kSignActive ? static_cast<int>(m) : kFirstActive;
    const int room = m <= kSignActive ? kSignActive : 2 * kFirstActive;
    auto mag = [&](int64_t a) {
      return __builtin_bit_cast(unsigned, static_cast<float>(__builtin_fabs(c64[a]))) >> 19;
    };
    Key2 best{0, 0};
    for (int64_t a = tid; a < m; a += kDecideThreads)
      best = key2_max(best, make_key2(c64[a], static_cast<int>(a)));
    best = block_max_key2<kDecideThreads>(best, s_keys);
    const int largest = key2_index(best);
    const unsigned top = mag(largest);
    auto bin = [&](int64_t a) {
      const unsigned b = top - mag(a);
      return static_cast<int>(b < kBins ? b : kBins - 1);
    };
    for (int64_t a = tid; a < m; a += kDecideThreads) atomicAdd(&hist[bin(a)], 1);
    __syncthreads();
    if (tid == 0) {
      int b = 0, sum = 0;
      if (want == m) b = kBins;
      while (b < kBins && sum < want) sum += hist[b++];
      s_cut = b;
      s_pos = 1;
      g->atom[0] = largest;
      pos[largest] = 0;
    }
    __syncthreads();
    for (int64_t a = tid; a < m; a += kDecideThreads)
      if (bin(a) < s_cut && a != largest) {
        const int p = atomicAdd(&s_pos, 1);
        if (p < room) {
          g->atom[p] = static_cast<int>(a);
          pos[a] = static_cast<unsigned short>(p);
        }
      }
    __syncthreads();
    nnew = s_pos < room ? s_pos : room;
  } else if (!over && nbeat > 0) {
    // the atoms that beat the earliest steps
    if (nact + kNewMost > kSignActive) {
      refill = true;
      for (int p = tid; p < nact; p += kDecideThreads) pos[g->atom[p]] = kNoPos;
    } else {
      for (int i = tid; i < nbeat; i += kDecideThreads) atomicAdd(&hist[g->beat_step[i]], 1);
      __syncthreads();
      if (tid == 0) s_cut = s_pos = 0;
      __syncthreads();
      // (more than fit beat the first step: some of them)
      if (tid <= count) {
        int sum = 0;
        for (int b = 0; b <= tid; ++b) sum += hist[b];
        if (sum <= kNewMost || sum == hist[tid]) atomicMax(&s_cut, tid + 1);
      }
      __syncthreads();
      for (int i = tid; i < nbeat; i += kDecideThreads)
        if (g->beat_step[i] < s_cut) {
          const int p = atomicAdd(&s_pos, 1);
          if (p < kNewMost) {
            g->atom[nact + p] = g->beat_atom[i];
            pos[g->beat_atom[i]] = static_cast<unsigned short>(nact + p);
          }
        }
      __syncthreads();
      nnew = s_pos < kNewMost ? s_pos : kNewMost;
    }
  }
  if (tid == 0) {
    if (take > 0) st->rr = s_rr[take - 1];
    st->t = t;
    if (over) {
      st->reason = reason;
      st->done = 1;
    }
    g->take = take;
    g->t0 = t0;
    g->nnew = nnew;
    g->nact = refill ? 0 : nact + nnew;
    g->fill = refill ? 1 : 0;
    // steps taken for nothing cost their time: twice what stood
    int steps = g->steps;
    if (first <= count) steps = 2 * take < 16 ? 16 : 2 * take;
    else if (count > 0) steps = 2 * steps;
    g->steps = steps < kSignSteps ? steps : kSignSteps;
    g->first = kSignSteps;
    g->nbeat = 0;
  }
}

// ---------------------------------------------------------------------------
// The Gram entries n - 2 popcount(b_i XOR b_m) of the new atoms i: lane = atom
// m, its bits turned over in LDS (16-byte chunk ch of atom a at a ^ ch of the
// chunk's row, which keeps both sides off each other's banks), the new atoms'
// bits in scalar registers.  Bound by the bit counts.
__global__ __launch_bounds__(kCommitThreads) void k_sgram_commit(
    const uint32_t* __restrict__ bits, int64_t ws, int n, int64_t m, int64_t ld,
    double* __restrict__ c64, double* __restrict__ r64, float* __restrict__ r32,
    short* __restrict__ gcol, int64_t mstride, short* __restrict__ h,
    const unsigned short* __restrict__ pos, double inv_n, double inv_sqrt_n, int grid,
    int rows_per_wg, int rblocks, float* __restrict__ x, const SignCarry* __restrict__ g,
    mp_trace tr) {
  __shared__ v4u own[kNewChunks * kCommitAtoms];
  __shared__ SignLog l;
  const int take = g->take, nnew = g->nnew;
  if (take > 0) stage_log(l, g, take, inv_n);
  const int lane = static_cast<int>(threadIdx.x) % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  if (static_cast<int>(blockIdx.x) < rblocks) {
    const int v = static_cast<int>(blockIdx.x) * kCommitWaves + wave;
    if (v < grid && take > 0 && blockIdx.y == 0)
      replay_rows_of<false>(bits, ws, n, ld, rows_per_wg, v, lane, take, inv_sqrt_n, l, r64, r32,
                         nullptr, grid, g->t0, tr, nullptr);
    return;
  }
  const int64_t a0 = static_cast<int64_t>(static_cast<int>(blockIdx.x) - rblocks) * kCommitAtoms;
  const int64_t a = a0 + lane;
  if (take > 0 && wave == 0 && a < m && blockIdx.y == 0) {
    double c = c64[a];
    float v = x[a];
    (void)replay_atom<false>(gcol, mstride, static_cast<int>(a), l, take, c, v);
    c64[a] = c;
    x[a] = v;
  }
  if (nnew == 0) return;
  const int nch = static_cast<int>(ws / 4);
  const int base = g->nact - nnew;
  const int mine = a < m ? pos[a] : kNoPos;
  constexpr int kAtOnce = kNewGroup * kCommitWaves;
  for (int g0 = kAtOnce * static_cast<int>(blockIdx.y); g0 < nnew;
       g0 += kAtOnce * static_cast<int>(gridDim.y)) {
    const int i0 = g0 + kNewGroup * wave;
    const v4u* col[kNewGroup];
    int acc[kNewGroup];
#pragma unroll
    for (int k = 0; k < kNewGroup; ++k) {
      const int p = base + (i0 + k < nnew ? i0 + k : nnew - 1);
      const int atom = __builtin_amdgcn_readfirstlane(g->atom[p]);
      col[k] = reinterpret_cast<const v4u*>(bits + static_cast<int64_t>(atom) * ws);
      acc[k] = 0;
    }
    for (int c0 = 0; c0 < nch; c0 += kNewChunks) {
      const int len = nch - c0 < kNewChunks ? nch - c0 : kNewChunks;
      __syncthreads();
      for (int i = static_cast<int>(threadIdx.x); i < kNewChunks * kCommitAtoms;
           i += kCommitThreads) {
        const int at = i / kNewChunks, ch = i % kNewChunks;
        const int64_t from = a0 + at < m ? a0 + at : m - 1;
        if (ch < len)
          own[ch * kCommitAtoms + (at ^ ch)] =
              reinterpret_cast<const v4u*>(bits + from * ws)[c0 + ch];
      }
      __syncthreads();
      if (i0 >= nnew) continue;
      for (int ch = 0; ch < len; ++ch) {
        const v4u o = own[ch * kCommitAtoms + (lane ^ ch)];
#pragma unroll
        for (int k = 0; k < kNewGroup; ++k) {
          const v4u b = col[k][c0 + ch];
          acc[k] += __builtin_popcount(o.x ^ b.x);
          acc[k] += __builtin_popcount(o.y ^ b.y);
          acc[k] += __builtin_popcount(o.z ^ b.z);
          acc[k] += __builtin_popcount(o.w ^ b.w);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kNewGroup; ++k) {
      if (i0 + k >= nnew || a >= m) continue;
      const int p = base + i0 + k;
      const short e = static_cast<short>(n - 2 * acc[k]);
      gcol[static_cast<int64_t>(p) * mstride + a] = e;
      if (mine != kNoPos) {
        h[static_cast<int64_t>(p) * kSignActive + mine] = e;
        h[static_cast<int64_t>(mine) * kSignActive + p] = e;
      }
    }
  }
}

// ---------------------------------------------------------------------------
int64_t sign_gram_stride(int64_t m) { return (m + kWave - 1) / kWave * kWave; }

hipError_t launch_sgram_init(const SignGram& b, int64_t m, hipStream_t s) {
  int64_t blocks = (m + 255) / 256;
  if (blocks > 64) blocks = 64;
  k_sgram_init<<<dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s>>>(b.carry, b.pos, m);
  return hipGetLastError();
}

hipError_t launch_sgram_round(const uint32_t* bits, int64_t ws, int64_t n, int64_t m, int64_t ld,
                              double* c64, double* r64, float* r32, const CorrGeom& geom,
                              const SignGram& b, bool first, long long max_iters, float* x,
                              DevState* st, mp_trace tr, hipStream_t s) {
  const double inv_n = 1.0 / static_cast<double>(n);
  const double inv_sqrt_n = 1.0 / sqrt(static_cast<double>(n));
  const int nn = static_cast<int>(n), grid = geom.grid;
  const int rows_per_wg = static_cast<int>((ld + grid - 1) / grid);
  if (rows_per_wg > kWave * kSignRows || grid > kDecideThreads) return hipErrorInvalidValue;
  const int64_t mstride = sign_gram_stride(m);
  hipError_t e;
  if (!first) {
    k_sgram_steps<<<dim3(1), dim3(kStepThreads), 0, s>>>(c64, b.h, inv_n, max_iters, st, b.carry);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int ca = static_cast<int>((m + kCheckThreads - 1) / kCheckThreads);
  const int cr = (grid + kCheckThreads / kWave - 1) / (kCheckThreads / kWave);
  if (!first) {
    k_sgram_check<<<dim3(ca + cr), dim3(kCheckThreads), 0, s>>>(
        bits, ws, nn, m, ld, c64, r64, b.g, mstride, inv_n, inv_sqrt_n, grid, rows_per_wg, ca,
        b.parts, st, b.carry);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  k_sgram_decide<<<dim3(1), dim3(kDecideThreads), 0, s>>>(c64, m, b.parts, grid, max_iters, b.pos,
                                                          st, b.carry, tr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int oa = static_cast<int>((m + kCommitAtoms - 1) / kCommitAtoms);
  const int orows = (grid + kCommitWaves - 1) / kCommitWaves;
  // (only the first active atoms are more than one group of workgroups takes)
  const unsigned slices = first ? kSignActive / (kNewGroup * kCommitWaves) / 2 : 1;
  k_sgram_commit<<<dim3(oa + orows, slices), dim3(kCommitThreads), 0, s>>>(
      bits, ws, nn, m, ld, c64, r64, r32, b.g, mstride, b.h, b.pos, inv_n, inv_sqrt_n, grid,
      rows_per_wg, orows, x, b.carry, tr);
  return hipGetLastError();
}

}  // namespace mp
