// Batched decode on carried correlations (k_gram.h): signals that share one
// dictionary, each decoded by one workgroup.
//
// The signals' atoms together soon cover the dictionary, so all Gram columns
// are computed at once (G = Psi^T Psi, kept by the context) and a signal needs
// nothing from the others between its steps: no rounds, no launch per
// iteration, only the correlations Psi^T R to start from and again each time
// the carried ones have lost too many digits (about once per three decades of
// ||r||).  Both products are one kernel on the FP32 matrix cores.
//
// Bound by the steps of the longest signal (3.6 us each at N = 2048,
// M = 8192).  Against rounds of BF16 products with a selection launch each:
// N = 2048, M = 8192, 256 signals: 6.6 ms from 42 ms (2 ms more the first
// time, for the Gram columns); N = 500, M = 1000, 500 signals: 2.7 ms from
// 7.8 ms.  One signal of a small dictionary, N = 256, M = 1024, 50 steps: 142
// us from 264 in the launch that exchanges every step between workgroups.
#include <algorithm>

#include "k_common.h"
#include "k_gram.h"
#include "k_gram_steps.h"

namespace mp {

// ---------------------------------------------------------------------------
// Init of every signal: r = y (zero padded), x~ = 0, ||y||^2 in FP64, the
// loop's pre-test.  One workgroup per signal.
__global__ __launch_bounds__(256) void k_gram_binit(const float* __restrict__ Y, int64_t ldy,
                                                    int64_t n, int64_t ld, float* __restrict__ X,
                                                    int64_t ldx, int64_t m,
                                                    float* __restrict__ R,
                                                    DevState* __restrict__ states,
                                                    const long long* __restrict__ tcap,
                                                    long long tcap_all, double eps) {
  __shared__ double red[4];
  const int64_t b = blockIdx.x;
  const float* y = Y + b * ldy;
  float* r = R + b * ld;
  float* x = X + b * ldx;
  for (int64_t j = threadIdx.x; j < m; j += 256) x[j] = 0.0f;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < ld; i += 256) {
    const float v = i < n ? y[i] : 0.0f;
    r[i] = v;
    s += static_cast<double>(v) * v;
  }
  const double yy = block_sum<256>(s, red);
  if (threadIdx.x == 0) {
    DevState d{};
    d.yy = yy;
    d.rr = yy;
    d.thr = eps * eps * yy;
    d.max_iters = tcap ? tcap[b] : tcap_all;
    d.reason = MP_STOP_CONVERGED;
    if (!__builtin_isfinite(yy)) {
      d.done = 1;
      d.reason = kStopNonFinite;
    } else if (yy == 0.0) {
      d.done = 1;
      d.reason = MP_STOP_ZERO_INPUT;
    } else if (!(yy > d.thr)) {
      d.done = 1;
    } else if (d.max_iters <= 0) {
      d.done = 1;
      d.reason = MP_STOP_MAX_ITERS;
    }
    states[b] = d;
  }
}

// ---------------------------------------------------------------------------
// out[j][a] = <psi_a, v_j> for all atoms a and columns v_j (v: the signals'
// residuals, or the dictionary itself): a 32 TW x 32 TW tile per workgroup of
// four waves, each 16 TW x 16 TW on v_mfma_f32_16x16x4_f32.
//
// Bound by the matrix cores (a TW = 4 tile does 64 MFMAs of 32 clocks per wave
// for 16 KB of operands), so the operands simply go through double-buffered
// LDS in 32-row chunks: 8 lanes read 128 bytes of a column; chunk f of column
// i sits at position f ^ (i mod 8), which keeps both sides off each other's
// banks.  FP32 chains are cut every kGemmChain rows and the cuts summed in
// FP32.  SYM (v = psi): only tiles on and above the diagonal are computed, and
// stored both ways round.  A residual tile whose signals have all stopped is
// skipped; `again` (not null): skip everything unless the previous launch of
// the steps left it set.
constexpr int kGemmRows = 32;
constexpr int kGemmChain = 64;

template <int TW, bool SYM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_gram_gemm(
    const float* __restrict__ psi, int64_t ld, int m, const float* __restrict__ v, int nv,
    float* __restrict__ out, int64_t ldo, const DevState* __restrict__ states,
    const int* __restrict__ again, int* __restrict__ clear) {
  constexpr int BT = 32 * TW;          // tile side
  constexpr int LR = BT / 32;          // loads per thread and operand: 32 columns each
  const int bi = static_cast<int>(blockIdx.x), bj = static_cast<int>(blockIdx.y);
  if (clear && bi == 0 && bj == 0 && threadIdx.x == 0) *clear = 0;
  if (again && *again == 0) return;
  if (SYM && bj < bi) return;
  const int a0 = bi * BT, j0 = bj * BT;
  const int t = static_cast<int>(threadIdx.x);
  const int lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  if (!SYM) {
    int live = 0;
    for (int j = j0 + t; j < j0 + BT && j < nv; j += 256) live |= states[j].done == 0;
    if (!__syncthreads_or(live)) return;
  }
  __shared__ v4f sa[2][BT * 8], sb[2][BT * 8];
  const int i = lane % 16, q = lane / 16;
  const int wa = wave / 2 * (16 * TW), wb = wave % 2 * (16 * TW);
  // staging: column t / 8 + 32 u of the tile, 16 bytes t % 8 of its chunk
  const v4f* ga[LR];
  const v4f* gb[LR];
  int put[LR];
#pragma unroll
  for (int u = 0; u < LR; ++u) {
    const int cl = t / 8 + 32 * u;
    const int a = a0 + cl < m ? a0 + cl : m - 1;
    const int j = j0 + cl < nv ? j0 + cl : nv - 1;
    ga[u] = reinterpret_cast<const v4f*>(psi + static_cast<int64_t>(a) * ld) + t % 8;
    gb[u] = reinterpret_cast<const v4f*>(v + static_cast<int64_t>(j) * ld) + t % 8;
    put[u] = cl * 8 + ((t % 8) ^ (cl % 8));
  }
  v4f ra[LR], rb[LR];
  auto load = [&](int c) {
#pragma unroll
    for (int u = 0; u < LR; ++u) {
      ra[u] = ga[u][c * (kGemmRows / 4)];
      rb[u] = gb[u][c * (kGemmRows / 4)];
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int u = 0; u < LR; ++u) {
      sa[buf][put[u]] = ra[u];
      sb[buf][put[u]] = rb[u];
    }
  };
  v4f acc[TW][TW], tot[TW][TW];
#pragma unroll
  for (int x = 0; x < TW; ++x)
#pragma unroll
    for (int y = 0; y < TW; ++y) acc[x][y] = tot[x][y] = v4f{0.f, 0.f, 0.f, 0.f};
  const int chunks = static_cast<int>(ld / kGemmRows);  // even: ld is a multiple of 64
  load(0);
  store(0);
  __syncthreads();
  for (int c = 0; c < chunks; ++c) {
    const int buf = c & 1;
    if (c + 1 < chunks) load(c + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kGemmRows / 16; ++s) {
      v4f fa[TW], fb[TW];
#pragma unroll
      for (int x = 0; x < TW; ++x) {
        const int ca = wa + 16 * x + i, cb = wb + 16 * x + i;
        fa[x] = sa[buf][ca * 8 + ((4 * s + q) ^ (ca % 8))];
        fb[x] = sb[buf][cb * 8 + ((4 * s + q) ^ (cb % 8))];
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int x = 0; x < TW; ++x)
#pragma unroll
          for (int y = 0; y < TW; ++y)
            acc[x][y] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(fa[x][e], fb[y][e], acc[x][y], 0, 0, 0);
    }
    if (buf == 1) {  // every kGemmChain = 2 kGemmRows rows
#pragma unroll
      for (int x = 0; x < TW; ++x)
#pragma unroll
        for (int y = 0; y < TW; ++y) {
          tot[x][y] += acc[x][y];
          acc[x][y] = v4f{0.f, 0.f, 0.f, 0.f};
        }
    }
    if (c + 1 < chunks) store(buf ^ 1);
    __syncthreads();
  }
  // lane l: column j = l % 16 of a block, atoms 4 (l / 16) .. + 3
#pragma unroll
  for (int x = 0; x < TW; ++x)
#pragma unroll
    for (int y = 0; y < TW; ++y) {
      const int a = a0 + wa + 16 * x + 4 * q, j = j0 + wb + 16 * y + i;
      const v4f o = tot[x][y];
      if (j < nv) {
        float* p = out + static_cast<int64_t>(j) * ldo + a;
        if (a + 3 < m) {
          *reinterpret_cast<v4f*>(p) = o;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (a + e < m) p[e] = o[e];
        }
        if (SYM) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (a + e < m) out[static_cast<int64_t>(a + e) * ldo + j] = o[e];
        }
      }
    }
}

// The bounds (u = 2^-24): chains of kGemmChain terms, ld / kGemmChain cuts
// added in FP32; the rest as in gram_bounds.
GramBounds gram_bounds_full(int64_t n, double max_norm) {
  const double u = 1.0 / 16777216.0, nn = static_cast<double>(n + 64);
  GramBounds b = gram_bounds(n, max_norm, false);
  const double prod = (std::min<double>(nn, kGemmChain) + nn / kGemmChain + 7) * u * 1.01;
  b.pass = static_cast<float>(prod * max_norm);
  b.col = static_cast<float>(prod * max_norm * max_norm);
  return b;
}

hipError_t launch_gram_binit(const float* Y, int64_t ldy, int64_t n, int64_t ld, float* X,
                             int64_t ldx, int64_t m, float* R, DevState* states,
                             const long long* tcap, long long tcap_all, double eps, int nb,
                             hipStream_t s) {
  k_gram_binit<<<dim3(nb), dim3(256), 0, s>>>(Y, ldy, n, ld, X, ldx, m, R, states, tcap, tcap_all,
                                              eps);
  return hipGetLastError();
}

hipError_t launch_gram_full(const float* psi, int64_t ld, int64_t m, float* g, int64_t mp,
                            int num_cus, hipStream_t s) {
  const int mm = static_cast<int>(m);
  const unsigned big = static_cast<unsigned>((m + 127) / 128);
  if (big * (big + 1) / 2 >= 2u * num_cus)
    k_gram_gemm<4, true><<<dim3(big, big), dim3(256), 0, s>>>(psi, ld, mm, psi, mm, g, mp, nullptr,
                                                              nullptr, nullptr);
  else {
    const unsigned small = static_cast<unsigned>((m + 63) / 64);
    k_gram_gemm<2, true><<<dim3(small, small), dim3(256), 0, s>>>(psi, ld, mm, psi, mm, g, mp,
                                                                  nullptr, nullptr, nullptr);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// VN: threads of the workgroup whose order ||r||^2 is summed in: the batched
// form's 512, or one signal's 1024.
template <int NT, int CPT, int VN>
__global__ __launch_bounds__(NT + 2 * kWave) void k_gram_bsteps(GramBatch b, GramBounds bd,
                                                                mp_trace tr, int* again) {
  extern __shared__ v4f lds[];
  __shared__ StepShared<float, NT, CPT> sh;
  const int64_t j = blockIdx.x;
  DevState* st = b.states + j;
  if (st->done) return;
  const GramProb<float> p{b.psi, b.ld, b.n, b.m, b.mp, b.c + j * b.mp,
                          const_cast<float*>(b.g), nullptr, 0, nullptr, b.r + j * b.ld,
                          b.x + j * b.ldx, st, nullptr};
  mp_trace t = tr;
  if (t.idx) t.idx += j * tr.cap;
  if (t.coef) t.coef += j * tr.cap;
  if (t.rr) t.rr += j * tr.cap;
  if (t.r) t.r += j * tr.cap * tr.ldr;
  const long long cap = st->max_iters;
  if (threadIdx.x < NT) gram_steps<float, NT, CPT, true, true, VN, false>(p, bd, cap, 0, t, lds, sh);
  else gram_steps<float, NT, CPT, false, true, VN, false>(p, bd, cap, 0, t, lds, sh);
  if (threadIdx.x == 0 && !st->done)
    (void)__hip_atomic_fetch_or(again, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int NT, int CPT, int VN>
static hipError_t launch_bsteps_t(const GramBatch& b, const GramBounds& bd, int nb, mp_trace tr,
                                  int* again, hipStream_t s) {
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_gram_bsteps<NT, CPT, VN>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, 2 * 16384 * 4);
  if (attr != hipSuccess) return attr;
  k_gram_bsteps<NT, CPT, VN><<<dim3(nb), dim3(NT + 2 * kWave), static_cast<size_t>(b.ld) * 8, s>>>(
      b, bd, tr, again);
  return hipGetLastError();
}

hipError_t launch_gram_bround(const GramBatch& b, const GramShape& sh, const GramBounds& bd,
                              int nb, int num_cus, long long round, int* again, bool single,
                              mp_trace tr, hipStream_t s) {
  if (b.ld > 16384) return hipErrorInvalidValue;
  // again[par]: some signal of this round's steps goes on
  const int par = static_cast<int>(round & 1);
  const int mm = static_cast<int>(b.m);
  const unsigned ba = static_cast<unsigned>((b.m + 127) / 128), bb = (nb + 127) / 128;
  const int* prev = round > 0 ? again + (par ^ 1) : nullptr;
  if (ba * bb >= 2u * num_cus)
    k_gram_gemm<4, false><<<dim3(ba, bb), dim3(256), 0, s>>>(b.psi, b.ld, mm, b.r, nb, b.c, b.mp,
                                                             b.states, prev, again + par);
  else
    k_gram_gemm<2, false><<<dim3(static_cast<unsigned>((b.m + 63) / 64), (nb + 63) / 64),
                            dim3(256), 0, s>>>(b.psi, b.ld, mm, b.r, nb, b.c, b.mp, b.states,
                                               prev, again + par);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (sh.threads == 256 && sh.per_thread == 4)
    return single ? launch_bsteps_t<256, 4, 1024>(b, bd, nb, tr, again + par, s)
                  : launch_bsteps_t<256, 4, 512>(b, bd, nb, tr, again + par, s);
  if (sh.threads == 256 && sh.per_thread == 16)
    return single ? launch_bsteps_t<256, 16, 1024>(b, bd, nb, tr, again + par, s)
                  : launch_bsteps_t<256, 16, 512>(b, bd, nb, tr, again + par, s);
  if (sh.threads == 512 && sh.per_thread == 16)
    return single ? launch_bsteps_t<512, 16, 1024>(b, bd, nb, tr, again + par, s)
                  : launch_bsteps_t<512, 16, 512>(b, bd, nb, tr, again + par, s);
  if (sh.threads == 512 && sh.per_thread == 32 && !single)
    return launch_bsteps_t<512, 32, 512>(b, bd, nb, tr, again + par, s);
  return hipErrorInvalidValue;
}

}  // namespace mp
