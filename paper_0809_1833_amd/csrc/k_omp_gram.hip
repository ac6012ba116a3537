// OMP's selection on carried correlations (k_gram.h): the pass over the
// dictionary runs once for fifteen to twenty atoms instead of once per atom.
//
// A block starts with a pass that gives c~ = Psi^T r and, for up to kGramReq
// candidate atoms, Psi^T w_i with w_i = psi_i - Q Q^T psi_i (the candidates
// made orthogonal to the directions so far).  An atom selected from the block
// then changes every correlation by z <psi_m, q_t> (r -= z q_t), and
//
//   Psi^T q_t = (Psi^T w_i - sum_s h_s Psi^T q_s) / rho,  s in the block,
//
// a sum over at most kGramReq - 1 stored columns of M (k_omp_carry); the
// block ends with the first atom outside it, which is fitted as well: the next
// block's pass starts from the r it leaves, so that every pass, the first
// included, brings a step (decodes of 1 and 4 atoms at N = 4096, M = 8192: 0.15
// and 0.34 ms; 1.05 and 1.14 while such an atom waited for a pass of its own and
// 8 rounds were enqueued before the first look at the state; 0.30 and 0.33 with a
// pass per step).  The factorisation itself (k_omp.hip) is computed as without
// the block, so the carried correlations only shortlist: k_omp_pick bounds their
// difference from the exact products and scores every atom within it by
// dot_column_f32, and the selected atoms, Q, R, z and r are the stepping form's
// bit for bit.  The part of q_t that the
// sum above misses (the rounding of both ways to orthogonalise) is measured,
// not estimated: k_omp_orth leaves its norm.
//
// Bound by a step's seven dependent launches (40 us with the factorisation's)
// and the blocks' passes.  N = 8192, M = 32768, K = 512: 27.7 ms a decode from
// 95.1 ms with a selection pass of 160 us each step.
#include "k_common.h"
#include "k_gram.h"
#include "k_gram_steps.h"
#include "mp_internal.h"

namespace mp {

constexpr int kCarryThreads = 128;   // atoms per workgroup of k_omp_carry
constexpr int kPickThreads = 1024;
constexpr int kPickWaves = kPickThreads / kWave;
constexpr int kPickTop = 4;          // atoms each wave proposes for the next block
constexpr int kOrthRowsB = 64;       // rows per workgroup of k_omp_borth
constexpr int kOrthWavesB = 8;
constexpr int kOrthChunk = 256;      // rows of H staged at a time

__global__ void k_omp_carry_init(OmpCarry* oc) {
  oc->hold = 1;
  oc->fit = 0;
  oc->cur = -1;
  oc->t0 = 0;
  oc->err = 0.0f;
  oc->ctl.nreq = 0;
  oc->ctl.slot0 = 0;
}

// ---------------------------------------------------------------------------
// W = V - Q H for the block's candidates V (rhs: their operand order for the
// pass that follows).  H = Q^T V comes from the pass kernel over Q.  One row
// per lane, the sum over j split over the waves and added in a fixed order.
__global__ __launch_bounds__(kOrthWavesB* kWave) void k_omp_borth(
    const float* __restrict__ psi, int64_t ld, const float* __restrict__ q,
    const float* __restrict__ h, int64_t ldh, const DevState* __restrict__ st,
    const OmpCarry* __restrict__ oc, float* __restrict__ w, float* __restrict__ rhs) {
  if (st->done || !oc->hold) return;
  __shared__ float ps[kOrthWavesB][kGramReq][kOrthRowsB];
  float(*hs)[kOrthChunk] = reinterpret_cast<float(*)[kOrthChunk]>(&ps[0][0][0]);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t t = st->t;
  const int nreq = oc->ctl.nreq;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * kOrthRowsB + lane;
  float acc[kGramReq];
#pragma unroll
  for (int i = 0; i < kGramReq; ++i) acc[i] = 0.0f;
  for (int64_t j0 = 0; j0 < t; j0 += kOrthChunk) {
    const int len = static_cast<int>(t - j0 < kOrthChunk ? t - j0 : kOrthChunk);
    __syncthreads();
    for (int e = threadIdx.x; e < kGramReq * kOrthChunk; e += kOrthWavesB * kWave) {
      const int i = e / kOrthChunk, j = e % kOrthChunk;
      hs[i][j] = i < nreq && j < len ? h[i * ldh + j0 + j] : 0.0f;
    }
    __syncthreads();
#pragma unroll 4
    for (int j = wave; j < len; j += kOrthWavesB) {
      const float v = q[(j0 + j) * ld + row];
#pragma unroll
      for (int i = 0; i < kGramReq; ++i) acc[i] = __builtin_fmaf(hs[i][j], v, acc[i]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kGramReq; ++i) ps[wave][i][lane] = acc[i];
  __syncthreads();
  for (int i = wave; i < nreq; i += kOrthWavesB) {  // one row per lane
    float s = 0.0f;
#pragma unroll
    for (int k = 0; k < kOrthWavesB; ++k) s += ps[k][i][lane];
    const float v = psi[static_cast<int64_t>(oc->ctl.req[i]) * ld + row] - s;
    w[i * ld + row] = v;
    rhs[gram_rhs_at(row, i + 1)] = v;
  }
}

// ---------------------------------------------------------------------------
// c~ after the last step, and each workgroup's two largest keys.  after_pass:
// the launch follows a block's pass, whose c~ is taken as it is if it ran.
// One atom per thread: bound by the latency of its (at most kGramReq + 1)
// loads, 4 MB in all.
__global__ __launch_bounds__(kCarryThreads) void k_omp_carry(
    float* __restrict__ c, float* __restrict__ p, int64_t mp, int64_t m,
    const float* __restrict__ rmat, int64_t tq, const double* __restrict__ z,
    const DevState* __restrict__ st, const OmpCarry* __restrict__ oc, int after_pass,
    uint64_t* __restrict__ tops) {
  const int hold = oc->hold, cur = oc->cur;
  if (st->done || (hold && !after_pass)) return;
  __shared__ uint64_t red[2][kCarryThreads / kWave];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t a = static_cast<int64_t>(blockIdx.x) * kCarryThreads + threadIdx.x;
  uint64_t key = 0;
  if (a < m) {
    float v = c[a];
    if (!hold && cur >= 0) {
      const int64_t tl = st->t - 1;           // the last step's column of R
      const int k = static_cast<int>(tl - oc->t0);
      const float* col = rmat + tl * tq;
      const float inv = 1.0f / col[tl];
      float sum = p[cur * mp + a];
      float g[kGramReq - 1], h[kGramReq - 1];
#pragma unroll
      for (int s = 0; s < kGramReq - 1; ++s) {
        const int at = s < k ? oc->slot[s] : cur;  // (loads past k: not used)
        g[s] = p[at * mp + a];
        h[s] = s < k ? col[oc->t0 + s] : 0.0f;
      }
#pragma unroll
      for (int s = 0; s < kGramReq - 1; ++s) sum = __builtin_fmaf(-h[s], g[s], sum);
      sum *= inv;
      p[cur * mp + a] = sum;
      v = __builtin_fmaf(-static_cast<float>(z[tl]), sum, v);
      c[a] = v;
    }
    key = make_key(v, static_cast<int>(a));
  }
  uint64_t top = wave_max(key);
  uint64_t next = wave_max(key == top ? 0 : key);
  if (lane == 0) {
    red[0][wave] = top;
    red[1][wave] = next;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kCarryThreads / kWave; ++w) {
      const uint64_t t1 = red[0][w], n1 = red[1][w];
      next = umax64(umax64(top < t1 ? top : t1, next), n1);
      top = umax64(top, t1);
    }
    tops[2 * blockIdx.x] = top;
    tops[2 * blockIdx.x + 1] = next;
  }
}

// ---------------------------------------------------------------------------
// One workgroup: the error bound after the last step, the atoms within it,
// the winner, which is the step's selection; where it is not in the block (or
// the correlations have to be renewed first), also the next block's candidates:
// each wave's best atoms not yet fitted, by the correlations before this step.
__global__ __launch_bounds__(kPickThreads) void k_omp_pick(
    const float* __restrict__ psi, int64_t ld, int64_t m, const float* __restrict__ r,
    const float* __restrict__ c, const uint64_t* __restrict__ tops, int ntops, GramBounds bd,
    const float* __restrict__ rmat, int64_t tq, const double* __restrict__ z,
    const double* __restrict__ dpart, int nparts, int after_pass, int want_coef,
    unsigned char* __restrict__ in_s, int* __restrict__ sel, DevState* __restrict__ st,
    OmpState* __restrict__ os, OmpCarry* __restrict__ oc) {
  const int hold = oc->hold;
  if (st->done) return;
  if (hold && !after_pass) {  // no selection
    if (threadIdx.x == 0) oc->fit = 0;
    return;
  }
  __shared__ uint64_t red[kPickWaves];
  __shared__ Key2 keys[kGramMaxCand];
  __shared__ int cand[kGramMaxCand];
  __shared__ uint64_t want[kPickWaves * kPickTop];
  __shared__ int s_n;
  __shared__ float s_err;
  const int tid = static_cast<int>(threadIdx.x);
  const int lane = tid % kWave, wave = tid / kWave;
  const long long t = st->t;
  const float rn = static_cast<float>(__builtin_sqrt(st->rr));
  uint64_t best = 0;
  for (int i = tid; i < ntops; i += kPickThreads) best = umax64(best, tops[2 * i]);
  if (wave == 0 && !hold) {
    // the bound (u = 2^-24): the column of P just made, then c~
    double d2 = 0.0;
    for (int i = lane; i < nparts; i += kWave) d2 += dpart[i];
    d2 = wave_sum(d2);
    if (lane == 0) {
      float err = oc->err;
      if (oc->cur >= 0) {
        const float u = 1.0f / 16777216.0f;
        const int64_t tl = t - 1;
        const int k = static_cast<int>(tl - oc->t0);
        const float* col = rmat + tl * tq;
        float e = bd.col, hsum = 1.0f;
        for (int s = 0; s < k; ++s) {
          const float h = __builtin_fabsf(col[oc->t0 + s]);
          e += h * oc->perr[s];
          hsum += h;
        }
        const float dn = static_cast<float>(__builtin_sqrt(d2));
        e += 1.01f * dn + 2.1f * static_cast<float>(k + 3) * u * hsum;
        e = e / col[tl] * 1.01f + 4.0f * u;
        oc->perr[k] = e;
        oc->slot[k] = oc->cur;
        oc->cur = -1;
        err += __builtin_fabsf(static_cast<float>(z[tl])) * (e + 2.0f * u) + bd.step * rn;
      }
      s_err = err;
    }
  }
  if (tid == 0) s_n = 0;
  best = block_max<kPickThreads>(best, red);
  const float cmax = __builtin_bit_cast(float, static_cast<uint32_t>(best >> 32));
  const float err = hold ? bd.pass * rn : s_err + bd.carry * cmax;
  const float band = 2.002f * (err + bd.dot * rn);
  bool bail = false, renew = false;
  int win = -1, nc = 0;
  float coef = 0.0f;
  if (!(band <= 0.125f * cmax) || !(rn > 1e-24f) || !(rn < 1e30f)) {
    bail = hold != 0;
    renew = true;
  } else {
    const float tau = cmax - band;
    for (int i = tid; i < ntops; i += kPickThreads) {
      const uint64_t k0 = tops[2 * i], k1 = tops[2 * i + 1];
      if (__builtin_bit_cast(float, static_cast<uint32_t>(k0 >> 32)) < tau) continue;
      if (__builtin_bit_cast(float, static_cast<uint32_t>(k1 >> 32)) < tau) {
        const int pos = atomicAdd(&s_n, 1);
        if (pos < kGramMaxCand) cand[pos] = key_index(k0);
      } else {  // several of this group's atoms
        for (int e = 0; e < kCarryThreads; ++e) {
          const int64_t a = static_cast<int64_t>(i) * kCarryThreads + e;
          if (a < m && __builtin_fabsf(c[a]) >= tau) {
            const int pos = atomicAdd(&s_n, 1);
            if (pos < kGramMaxCand) cand[pos] = static_cast<int>(a);
          }
        }
      }
    }
    __syncthreads();
    nc = s_n;
    if (nc > kGramMaxCand) {
      bail = hold != 0;
      renew = true;
    } else if (nc > 1 || want_coef) {
      const v4f* rv = reinterpret_cast<const v4f*>(r);
      for (int k = wave; k < nc; k += kPickWaves) {
        const int a = cand[k];
        const float v = dot_column_narrow<float, false, 4>(
            reinterpret_cast<const v4f*>(psi + static_cast<int64_t>(a) * ld), rv,
            static_cast<int>(ld / 4), lane);
        if (lane == 0) keys[k] = make_key2(static_cast<double>(v), a);
      }
      __syncthreads();
      const Key2 w = wave_max_key2(lane < nc ? keys[lane] : Key2{0, 0});
      win = key2_index(w);
      coef = static_cast<float>(key2_value(w));
    } else {
      win = cand[0];
    }
  }
  int cur = -1;
  if (!renew) {
    const int nreq = oc->ctl.nreq;
    for (int k = 0; k < nreq; ++k)
      if (oc->ctl.req[k] == win) cur = k;
  }
  const bool fitted = !renew && in_s[win] != 0;
  __syncthreads();  // (before the state below changes)
  if (tid == 0) {
    if (bail) {
      st->done = 1;
      st->pad[0] = 1;
    } else if (fitted) {  // an atom already fitted
      st->done = 1;
      st->reason = MP_STOP_STALLED;
    } else {
      if (!renew) {
        os->sel = win;
        os->c = coef;
        sel[t] = win;
        in_s[win] = 1;
      }
      oc->fit = renew ? 0 : 1;
      oc->cur = cur;
      oc->err = err;
      if (hold) oc->t0 = t;
      oc->hold = cur >= 0 ? 0 : 1;
    }
  }
  if (bail || fitted || cur >= 0) return;
  // the next block
  float mine[kPickTop];
  int at[kPickTop];
#pragma unroll
  for (int k = 0; k < kPickTop; ++k) {
    mine[k] = -1.0f;
    at[k] = 0;
  }
  for (int64_t a = tid; a < m; a += kPickThreads) {
    if (in_s[a] || a == win) continue;
    float v = __builtin_fabsf(c[a]);
    int i = static_cast<int>(a);
#pragma unroll
    for (int k = 0; k < kPickTop; ++k)
      if (v > mine[k]) {
        const float tv = mine[k];
        const int ti = at[k];
        mine[k] = v;
        at[k] = i;
        v = tv;
        i = ti;
      }
  }
  for (int k = 0; k < kPickTop; ++k) {
    const uint64_t key = mine[0] >= 0.0f ? make_key(mine[0], at[0]) : 0;
    const uint64_t w = wave_max(key);
    if (lane == 0) want[wave * kPickTop + k] = w;
    if (w != 0 && w == key) {
#pragma unroll
      for (int j = 0; j + 1 < kPickTop; ++j) {
        mine[j] = mine[j + 1];
        at[j] = at[j + 1];
      }
      mine[kPickTop - 1] = -1.0f;
    }
  }
  __syncthreads();
  if (wave == 0) {
    // the best of the proposals, by rank
    const uint64_t k0 = lane < kPickWaves * kPickTop ? want[lane] : 0;
    int rank = 0;
    for (int j = 0; j < kPickWaves * kPickTop; ++j) rank += want[j] > k0;
    if (k0 != 0 && rank < kGramReq) oc->ctl.req[rank] = key_index(k0);
    const int found = static_cast<int>(__popcll(__ballot(k0 != 0)));
    if (lane == 0) oc->ctl.nreq = found < kGramReq ? found : kGramReq;
  }
}

// ---------------------------------------------------------------------------
hipError_t launch_omp_carry_init(const OmpBufs& b, hipStream_t s) {
  k_omp_carry_init<<<dim3(1), dim3(1), 0, s>>>(b.oc);
  return hipGetLastError();
}

// A block, where the device asks for one: the candidates made orthogonal to
// the t <= t_bound directions, then the pass.
hipError_t launch_omp_block(const float* psi, int64_t ld, int64_t n, int64_t m, float* r,
                            const OmpBufs& b, DevState* st, long long t_bound, int num_cus,
                            hipStream_t s) {
  GramProb<float> p{psi, ld, n, m, b.mp, b.c, b.p, nullptr, kGramReq, b.rhs, r, nullptr, st,
                    &b.oc->ctl};
  GramProb<float> pq = p;  // over Q: right-hand side 0 (r) goes to b.hr
  pq.psi = b.q;
  pq.m = t_bound;
  pq.mp = b.ldh;
  pq.c = b.hr;
  pq.g = b.hq;
  hipError_t e = launch_gram_block(p, pq, &b.oc->hold, num_cus, s);
  if (e != hipSuccess) return e;
  k_omp_borth<<<dim3(static_cast<unsigned>(ld / kOrthRowsB)), dim3(kOrthWavesB * kWave), 0, s>>>(
      psi, ld, b.q, b.hq, b.ldh, st, b.oc, b.w15, b.rhs);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  return launch_gram_block_pass(p, &b.oc->hold, num_cus, s);
}

hipError_t launch_omp_pick(const float* psi, int64_t ld, int64_t m, const float* r,
                           const OmpBufs& b, const GramBounds& bd, bool after_pass,
                           bool want_coef, DevState* st, hipStream_t s) {
  const unsigned grid = static_cast<unsigned>((m + kCarryThreads - 1) / kCarryThreads);
  k_omp_carry<<<dim3(grid), dim3(kCarryThreads), 0, s>>>(b.c, b.p, b.mp, m, b.rmat, b.tq, b.z, st,
                                                        b.oc, after_pass ? 1 : 0, b.tops);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_omp_pick<<<dim3(1), dim3(kPickThreads), 0, s>>>(
      psi, ld, m, r, b.c, b.tops, static_cast<int>(grid), bd, b.rmat, b.tq, b.z, b.dpart,
      static_cast<int>(ld / 64), after_pass ? 1 : 0, want_coef ? 1 : 0, b.in_s, b.sel, st, b.os,
      b.oc);
  return hipGetLastError();
}

int64_t omp_tops(int64_t m) { return 2 * ((m + kCarryThreads - 1) / kCarryThreads); }

}  // namespace mp
