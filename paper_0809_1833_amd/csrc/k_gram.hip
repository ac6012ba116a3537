// The decode on carried correlations (k_gram.h): the pass and the steps.
#include <algorithm>

#include "k_common.h"
#include "k_gram.h"
#include "k_gram_steps.h"

namespace mp {

// ---------------------------------------------------------------------------
// The pass: [c~ | g_req] = Psi^T [r | psi_req], 32 atoms x 32 right-hand sides
// per wave on v_mfma_f32_32x32x2_f32.
//
// Bound by the dictionary's bytes (the products take two thirds of the time
// its bytes do), so its reads are whole 256-byte pieces of a column (16 lanes
// each).  The matrix operand wants lane l to hold atom l % 32 at rows
// 4 (l / 32) of an 8-row step, where no two neighbouring lanes share a column:
// read straight from memory that is one cache access per lane.  Each wave
// therefore turns its 32 atoms x 64 rows over in 8 KB of LDS of its own (no
// barriers; float4 f of atom a at position f ^ a of its row, so that neither
// side meets bank conflicts), with the next pieces (16 KB) in flight in
// registers.  The right-hand sides are laid out in operand order by
// k_gram_pack and come from L2.
//
// Each 32-atom tile's rows are split over `split` waves of the workgroup, so
// that a short dictionary still gives every CU waves; their sums meet in LDS
// in a fixed order.  Every 32 rows (FP64: 16; gram_chain) are an FP32 chain of
// their own, summed in FP64, which keeps the rounding bound of the products at
// that of one chain.
//
// N = 8192, M = 32768: 199 us in a decode (5.4 TB/s of the dictionary's bytes,
// 5.6 of the 1.04 times as many that the counters show; a large copy reaches
// 6.64) and 22 passes; in FP64 310 us (6.9 and 7.1 TB/s).  Passes alone take
// 192; with 16 right-hand sides (16 atoms a wave) 196, and a decode 40 of them.
constexpr int kPassThreads = 512;
constexpr int kPassWaves = kPassThreads / kWave;
constexpr int kPassRows = 64;           // rows of a piece: 8 steps of 8
constexpr int kPassSteps = kPassRows / 8;
// Rows summed in one FP32 chain.
constexpr int gram_chain(bool f64) { return f64 ? 16 : 32; }
constexpr int kRhs = kGramReq + 1;
static_assert(kRhs == 32 && kGramTile == 32, "one 32 x 32 tile per wave");
typedef float v16f __attribute__((ext_vector_type(16)));

// 16 bytes of a column as floats.
__device__ inline void put_floats(float* p, const v4f& v) { *reinterpret_cast<v4f*>(p) = v; }
__device__ inline void put_floats(float* p, const Vec16<double>::type& v) {
  typedef float v2f __attribute__((ext_vector_type(2)));
  *reinterpret_cast<v2f*>(p) = v2f{static_cast<float>(v.x), static_cast<float>(v.y)};
}

// The right-hand sides in operand order (gram_rhs_at): r, the wanted columns,
// then zeros.  The first pass also clears the slot map.
template <typename T>
__device__ inline void gram_pack(const GramProb<T>& p, int first) {
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t all = static_cast<int64_t>(gridDim.x) * 256;
  const int nreq = first ? 0 : p.ctl->nreq;
  for (int64_t e = t; e < p.ld * (kRhs / 4); e += all) {
    const int i = static_cast<int>(e % kRhs);
    const int64_t row4 = e / kRhs;  // float4 of the column
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
    if (i <= nreq) {
      const T* src = i == 0 ? p.r : p.psi + static_cast<int64_t>(p.ctl->req[i - 1]) * p.ld;
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = static_cast<float>(src[4 * row4 + k]);
    }
    reinterpret_cast<v4f*>(p.rhs)[e] = v;
  }
  if (first)
    for (int64_t e = t; e < p.m; e += all) p.map[e] = static_cast<uint16_t>(kGramNone);
}

template <typename T>
__global__ __launch_bounds__(256) void k_gram_pack(GramProb<T> p, int first) {
  if (!p.st->done) gram_pack(p, first);
}

// One workgroup's share of the pass: tiles group * (WAVES / split) ..., with D
// pieces in flight per wave (every thread of the workgroup calls; there are
// barriers).  SHARE (for split == 1, one piece in flight): the waves go through
// the same rows of the right-hand sides, so each loads its part of a piece of
// them and reads the piece from LDS.  A wave starts at its tile's own piece
// and goes round, so that tiles do not all ask for the same rows at once.
template <typename T, int D, int WAVES, bool SHARE = false>
__device__ inline void gram_pass(const GramProb<T>& p, int64_t group, int split, int first) {
  constexpr int NL = kPassRows * kGramTile * sizeof(T) / 16 / kWave;  // 16-byte loads of a piece
  constexpr int LPA = kPassRows * sizeof(T) / 16;                     // of them per atom
  // steps of an FP32 chain: with 16 rows two more flushes of 16 sums cost registers
  // that two pieces in flight do not leave (232 us a pass from 192, 10 registers
  // spilled)
  constexpr int C = gram_chain(sizeof(T) == 8) / 8;
  typedef typename Vec16<T>::type vec;
  __shared__ v4f turn[WAVES][kGramTile * 16];  // then the split sums
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int tiles = WAVES / split;  // per workgroup
  const int part = wave % split;
  const int64_t m0 = (group * tiles + wave / split) * kGramTile;
  const int i = lane % kGramTile, q = lane / kGramTile;
  const int nreq = first ? 0 : p.ctl->nreq;
  const bool live = m0 < p.m;
  double tot[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) tot[e] = 0.0;
  if (SHARE || live) {
    // load j of a piece: 16 bytes (j 64 + lane) % LPA of atom (j 64 + lane) / LPA
    const vec* a0 = reinterpret_cast<const vec*>(p.psi + (live ? m0 : 0) * p.ld);
    unsigned at[NL];  // in 16 bytes
    int put[NL];      // in floats
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int atom = (j * kWave + lane) / LPA, li = (j * kWave + lane) % LPA;
      const int64_t in = m0 + atom < p.m ? atom : live ? p.m - 1 - m0 : 0;
      at[j] = static_cast<unsigned>(in * (p.ld * static_cast<int>(sizeof(T)) / 16) + li);
      const int f = li * (16 / static_cast<int>(sizeof(T)));  // first row of the 16 bytes
      put[j] = 4 * (atom * 16 + ((f / 4) ^ (atom % 16))) + f % 4;
    }
    const v4f* b = reinterpret_cast<const v4f*>(p.rhs);
    v4f* my = turn[wave];
    const int pieces = static_cast<int>(p.ld / kPassRows);
    const int k0 = pieces * part / split, k1 = pieces * (part + 1) / split;
    const int len = k1 > k0 ? k1 - k0 : 1;
    const int rot = static_cast<int>((m0 / kGramTile / (SHARE ? tiles : 1)) % len);
    auto turned = [&](int k) {
      const int t = (k < k1 ? k : k1 - 1) + rot;
      return static_cast<int64_t>(t < k1 ? t : t - len);
    };
    v16f acc[2];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.0f;
    vec va[D][NL];
    constexpr int NB = SHARE ? kPassSteps / WAVES : kPassSteps;  // this wave's of a piece
    static_assert(!SHARE || (D == 1 && NB * WAVES == kPassSteps), "an even part for each wave");
    v4f vb[D][NB];
    const int b0 = SHARE ? wave * NB : 0;
    // (past the end: read again, not used)
    auto load_a = [&](vec(&x)[NL], int k) {
      const vec* ak = a0 + LPA * turned(k);
#pragma unroll
      for (int j = 0; j < NL; ++j) x[j] = __builtin_nontemporal_load(ak + at[j]);
    };
    auto load_b = [&](v4f(&y)[NB], int k) {
      const v4f* bk = b + kPassSteps * kWave * turned(k);
#pragma unroll
      for (int j = 0; j < NB; ++j) y[j] = bk[(b0 + j) * kWave + lane];
    };
    auto flush = [&](v16f& x) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        tot[e] += static_cast<double>(x[e]);
        x[e] = 0.0f;
      }
    };
    auto use = [&](vec(&x)[NL], v4f(&y)[NB], int next, v4f* bl) {
#pragma unroll
      for (int j = 0; j < NL; ++j) put_floats(reinterpret_cast<float*>(my) + put[j], x[j]);
      if (SHARE) {
#pragma unroll
        for (int j = 0; j < NB; ++j) bl[(b0 + j) * kWave + lane] = y[j];
        load_b(y, next);
      }
      __builtin_amdgcn_wave_barrier();
      load_a(x, next);
      __builtin_amdgcn_sched_barrier(0);
      if (SHARE) __syncthreads();
#pragma unroll
      for (int s = 0; s < kPassSteps; ++s) {
        const v4f xa = my[i * 16 + ((2 * s + q) ^ (i % 16))];
        const v4f xb = SHARE ? bl[s * kWave + lane] : y[SHARE ? 0 : s];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[s / C & 1] =
              __builtin_amdgcn_mfma_f32_32x32x2f32(xa[e], xb[e], acc[s / C & 1], 0, 0, 0);
        if (s % C == C - 1 && s > C) flush(acc[(s / C & 1) ^ 1]);  // the chain before
      }
      flush(acc[1]);
      __builtin_amdgcn_sched_barrier(0);
      if (!SHARE) load_b(y, next);
      __builtin_amdgcn_wave_barrier();
    };
    if (k0 < k1) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        load_a(va[d], k0 + d);
        load_b(vb[d], k0 + d);
      }
    }
    if constexpr (!SHARE) {
      for (int k = k0; k < k1; k += D)
#pragma unroll
        for (int d = 0; d < D; ++d)
          if (k + d < k1) use(va[d], vb[d], k + d + D, nullptr);
    } else {
      // One barrier a piece, with two buffers in turn: a wave that fills one has
      // passed the barrier after which no wave reads it.
      __shared__ v4f bsh[2][kPassSteps * kWave];
      for (int k = 0; k < k1; ++k) use(va[0], vb[0], k + 1, bsh[k & 1]);
    }
  }
  __syncthreads();
  double(*red)[16][kWave] = reinterpret_cast<double(*)[16][kWave]>(&turn[0][0]);
#pragma unroll
  for (int e = 0; e < 16; ++e) red[wave][e][lane] = tot[e];
  __syncthreads();
  if (part != 0 || m0 >= p.m) return;
  for (int w = 1; w < split; ++w)
#pragma unroll
    for (int e = 0; e < 16; ++e) tot[e] += red[wave + w][e][lane];
  // this lane: right-hand side i of atoms m0 + 8 g + 4 q .. + 3 (zero past the last)
  if (i > nreq) return;
  float* out = i == 0 ? p.c : p.g + static_cast<int64_t>(p.ctl->slot0 + i - 1) * p.mp;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int64_t base = m0 + 8 * g + 4 * q;
    v4f o;
#pragma unroll
    for (int e = 0; e < 4; ++e) o[e] = base + e < p.m ? static_cast<float>(tot[4 * g + e]) : 0.0f;
    *reinterpret_cast<v4f*>(out + base) = o;
  }
}

// Waves each tile's rows are split over: the fewest that give every CU a
// workgroup (8 waves with 256 registers fill it).
static int pass_split(int64_t tiles, int num_cus) {
  int split = 1;
  while (split < kPassWaves && tiles * split / kPassWaves < num_cus) split *= 2;
  return split;
}

template <typename T>
__global__ __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gram_pass(
    GramProb<T> p, int split, int first) {
  if (!p.st->done) gram_pass<T, sizeof(T) == 4 ? 2 : 1, kPassWaves>(p, static_cast<int64_t>(blockIdx.x), split, first);
}

template <typename T>
hipError_t launch_gram_pass(const GramProb<T>& p, int num_cus, bool first, hipStream_t s) {
  const int64_t packs = p.ld * (kRhs / 4) / 256;  // ld is a multiple of 64
  k_gram_pack<T><<<dim3(static_cast<unsigned>(packs)), dim3(256), 0, s>>>(p, first ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tiles = (p.m + kGramTile - 1) / kGramTile;
  const int split = pass_split(tiles, num_cus);
  const int per = kPassWaves / split;
  k_gram_pass<T><<<dim3(static_cast<unsigned>((tiles + per - 1) / per)), dim3(kPassThreads), 0, s>>>(
      p, split, first ? 1 : 0);
  return hipGetLastError();
}

template hipError_t launch_gram_pass<float>(const GramProb<float>&, int, bool, hipStream_t);
template hipError_t launch_gram_pass<double>(const GramProb<double>&, int, bool, hipStream_t);

// The passes of an OMP block (k_omp_gram.hip).
__global__ __launch_bounds__(256) void k_gram_block_pack(GramProb<float> p,
                                                         const int* __restrict__ hold) {
  if (!p.st->done && *hold) gram_pack(p, 0);
}

// count: columns of p in use (null: all of them).
__global__ __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(2, 2))) void
k_gram_block_pass(GramProb<float> p, int split, const int* __restrict__ hold,
                  const long long* __restrict__ count) {
  if (p.st->done || !*hold) return;
  if (count) p.m = *count;
  if (p.m > 0) gram_pass<float, 2, kPassWaves>(p, static_cast<int64_t>(blockIdx.x), split, 0);
}

static hipError_t block_pass(const GramProb<float>& p, const int* hold, const long long* count,
                             int num_cus, hipStream_t s) {
  const int64_t tiles = (p.m + kGramTile - 1) / kGramTile;
  const int split = pass_split(tiles, num_cus);
  const int per = kPassWaves / split;
  k_gram_block_pass<<<dim3(static_cast<unsigned>((tiles + per - 1) / per)), dim3(kPassThreads), 0,
                      s>>>(p, split, hold, count);
  return hipGetLastError();
}

hipError_t launch_gram_block(const GramProb<float>& p, const GramProb<float>& pq, const int* hold,
                             int num_cus, hipStream_t s) {
  k_gram_block_pack<<<dim3(static_cast<unsigned>(p.ld * (kRhs / 4) / 256)), dim3(256), 0, s>>>(p, hold);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || pq.m <= 0) return e;
  return block_pass(pq, hold, &p.st->t, num_cus, s);
}

hipError_t launch_gram_block_pass(const GramProb<float>& p, const int* hold, int num_cus,
                                  hipStream_t s) {
  return block_pass(p, hold, nullptr, num_cus, s);
}

// The bounds (u = 2^-24): a product of the pass is a chain of at most
// gram_chain terms, rounded once more to FP32 (and, from an FP64 dictionary, both
// operands rounded to FP32 first); dot_column_f32 is two lane chains of at most
// 4 ceil(ld / 512) terms, then 7 additions (in FP64 its rounding is far below the
// rest).  Each is at most (terms + additions) u sum |a b| <= (...) u ||a||
// ||b||; a step adds r's rounding (u ||r'|| against a unit column; far less in
// FP64), c~'s own (u |c~|) and that of the coefficient (u |c|, in col).
static double dot_roundings(int64_t n, int chains) {
  const int64_t ld = (n + 63) / 64 * 64, per = 256 * chains;  // rows in 4 terms of every lane
  return 4.0 * static_cast<double>((ld + per - 1) / per) + 8.0;
}

GramBounds gram_bounds(int64_t n, double max_norm, bool f64) {
  const double u = 1.0 / 16777216.0, nn = static_cast<double>(n + 64);
  const double slack = 1.01;
  const double prod =
      (std::min<double>(nn, gram_chain(f64)) + 7) * u * slack;
  GramBounds b;
  b.pass = static_cast<float>(prod * max_norm);
  b.col = static_cast<float>(prod * max_norm * max_norm);
  b.step = static_cast<float>((f64 ? 1e-3 : 1.01) * u * max_norm * slack);
  b.carry = static_cast<float>(1.01 * u * slack);
  b.dot = static_cast<float>((f64 ? 0.1 : dot_roundings(n, 2)) * u * max_norm * slack);
  return b;
}

// ---------------------------------------------------------------------------
// The steps of one signal (k_gram_steps.h).
template <typename T, int NT, int CPT>
__global__ __launch_bounds__(NT + 2 * kWave) void k_gram_steps(
    GramProb<T> p, GramBounds bd, long long max_iters, int first,
    typename GramTrace<T>::type tr) {
  extern __shared__ v4f lds[];
  typename Vec16<T>::type* r_lds = reinterpret_cast<typename Vec16<T>::type*>(lds);
  __shared__ StepShared<T, NT, CPT> sh;
  if (p.st->done) return;
  if (threadIdx.x < NT) gram_steps<T, NT, CPT, true, false, 1024, false>(p, bd, max_iters, first, tr, r_lds, sh);
  else gram_steps<T, NT, CPT, false, false, 1024, false>(p, bd, max_iters, first, tr, r_lds, sh);
}

constexpr int64_t kStepLds = 150 * 1024;  // r, a column and (FP32) the slot map, at most

static int64_t step_lds(int64_t ld, int64_t m, int esize) {
  return 2 * ld * esize + (esize == 4 ? 2 * m : 0);
}

// The smallest workgroup that holds the correlations: fewer waves make the
// reductions and barriers of a step shorter.  Above 16384 atoms 14 waves share
// them: a wave's correlations and Gram entries then fit the 128 registers of
// four waves per SIMD (8 waves with 64 each spilled 34 registers a lane).  Columns above 4096 rows take
// 512 threads, so that no thread updates more than a few chunks of r.
GramShape gram_shape(int64_t ld, int64_t m, int esize) {
  const GramShape shapes[] = {{256, 4}, {256, 16}, {512, 16}, {512, 32}, {896, 40}};
  if (m > kGramMaxAtoms || step_lds(ld, m, esize) > kStepLds) return GramShape{0, 0};
  for (const GramShape& s : shapes)
    if (m <= static_cast<int64_t>(s.threads) * s.per_thread &&
        (ld * esize <= 16384 || s.threads >= 512))
      return s;
  return GramShape{0, 0};
}

template <typename T, int NT, int CPT>
static hipError_t launch_steps_t(const GramProb<T>& p, const GramBounds& b, long long max_iters,
                                 bool first, typename GramTrace<T>::type tr, hipStream_t s) {
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_gram_steps<T, NT, CPT>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kStepLds);
  if (attr != hipSuccess) return attr;
  k_gram_steps<T, NT, CPT><<<dim3(1), dim3(NT + 2 * kWave),
                             static_cast<size_t>(step_lds(p.ld, p.m, sizeof(T))), s>>>(
      p, b, max_iters, first ? 1 : 0, tr);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gram_steps(const GramProb<T>& p, const GramShape& sh, const GramBounds& b,
                             long long max_iters, bool first, typename GramTrace<T>::type tr,
                             hipStream_t s) {
  if (step_lds(p.ld, p.m, sizeof(T)) > kStepLds) return hipErrorInvalidValue;
  if (sh.threads == 256 && sh.per_thread == 4)
    return launch_steps_t<T, 256, 4>(p, b, max_iters, first, tr, s);
  if (sh.threads == 256 && sh.per_thread == 16)
    return launch_steps_t<T, 256, 16>(p, b, max_iters, first, tr, s);
  if (sh.threads == 512 && sh.per_thread == 16)
    return launch_steps_t<T, 512, 16>(p, b, max_iters, first, tr, s);
  if (sh.threads == 512 && sh.per_thread == 32)
    return launch_steps_t<T, 512, 32>(p, b, max_iters, first, tr, s);
  if (sh.threads == 896 && sh.per_thread == 40)
    return launch_steps_t<T, 896, 40>(p, b, max_iters, first, tr, s);
  return hipErrorInvalidValue;
}
template hipError_t launch_gram_steps<float>(const GramProb<float>&, const GramShape&,
                                             const GramBounds&, long long, bool, mp_trace,
                                             hipStream_t);
template hipError_t launch_gram_steps<double>(const GramProb<double>&, const GramShape&,
                                              const GramBounds&, long long, bool, mp_trace_f64,
                                              hipStream_t);

// ---------------------------------------------------------------------------
// Many independent problems, each with its own dictionary: the kernels above
// over arrays of problems.  A round packs every running problem's right-hand
// sides, passes over their dictionaries (one launch, a list of tile groups)
// and takes their steps (one workgroup each, most work first); the problems
// share nothing.  Bound by the passes' bytes while many problems run (4.4 ms
// at 3.7 TB/s), then by the steps of the longest (2.9 ms).  512 problems of N
// in {128 ... 1024}, M = 4 N: 7.4 ms from 125 ms with a pass per step in one
// persistent launch.
__global__ __launch_bounds__(256) void k_gram_rinit(const GramProb<float>* __restrict__ probs,
                                                    const RInst* __restrict__ inst,
                                                    const float* __restrict__ Y,
                                                    float* __restrict__ X,
                                                    const long long* __restrict__ caps,
                                                    long long cap_all, double eps) {
  __shared__ double red[4];
  const int id = static_cast<int>(blockIdx.x);
  const GramProb<float> p = probs[id];
  const float* y = Y + inst[id].y_off;
  float* x = X + inst[id].x_off;
  for (int64_t j = threadIdx.x; j < p.m; j += 256) x[j] = 0.0f;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < p.ld; i += 256) {
    const float v = i < p.n ? y[i] : 0.0f;
    p.r[i] = v;
    s += static_cast<double>(v) * v;
  }
  const double yy = block_sum<256>(s, red);
  if (threadIdx.x == 0) {
    DevState d{};
    d.yy = yy;
    d.rr = yy;
    d.thr = eps * eps * yy;
    d.max_iters = caps ? caps[id] : cap_all;
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
    *p.st = d;
  }
}

// again: word `par` is set by this round's steps if some problem goes on; the
// whole round returns at once where the previous round's word is clear.
__global__ __launch_bounds__(256) void k_gram_rpack(const GramProb<float>* __restrict__ probs,
                                                    int* again, int par, int first) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) again[par] = 0;
  if (!first && again[par ^ 1] == 0) return;
  const GramProb<float> p = probs[blockIdx.y];
  if (!p.st->done) gram_pack(p, first);
}

// Three waves per SIMD with a piece each in flight.  Where no tile is split
// (many problems), its waves share the right-hand sides through LDS: their
// misses to the L2 halve what a CU can have under way for the dictionaries
// (512 problems of N in {128 ... 1024}: a solve 8.0 ms, shared 7.75, with
// chains of 32 rows instead of 16 7.65, with the tiles' own starting pieces
// 7.4).  In the pass over one long dictionary, where two pieces in flight hide
// those misses, the barriers cost more (220 us from 193).
template <bool SHARE>
__global__ __launch_bounds__(kGramRaggedWaves* kWave) __attribute__((amdgpu_waves_per_eu(3, 3))) void
k_gram_rpass(const GramProb<float>* __restrict__ probs, const GramGroup* __restrict__ groups,
             int split, int first) {
  const GramGroup g = groups[blockIdx.x];
  const GramProb<float> p = probs[g.id];
  if (!p.st->done) gram_pass<float, 1, kGramRaggedWaves, SHARE>(p, g.group, split, first);
}

template <int NT, int CPT, bool ONE>
__device__ inline void gram_rsteps(const GramProb<float>& p, const GramBounds& bd, int first,
                                   const mp_trace& t, v4f* lds, void* sh) {
  StepShared<float, NT, CPT>& s = *static_cast<StepShared<float, NT, CPT>*>(sh);
  const long long cap = p.st->max_iters;
  if (threadIdx.x < NT)
    gram_steps<float, NT, CPT, true, false, NT, ONE>(p, bd, cap, first, t, lds, s);
  else
    gram_steps<float, NT, CPT, false, false, NT, ONE>(p, bd, cap, first, t, lds, s);
}

// C1, C2: correlations per thread for problems of at most NT * C1 atoms and
// for the others.
template <int NT, int C1, int C2, bool ONE>
__global__ __launch_bounds__(NT + 2 * kWave) void k_gram_rsteps(
    const GramProb<float>* __restrict__ probs, const RInst* __restrict__ inst,
    const int* __restrict__ order, float* __restrict__ X, const GramBounds* __restrict__ bounds,
    mp_trace tr, int* again, int first) {
  extern __shared__ v4f lds[];
  __shared__ __attribute__((aligned(16))) char sh[sizeof(StepShared<float, NT, C2>)];
  static_assert(C1 <= C2, "the larger share's LDS holds the smaller's");
  const int id = order[blockIdx.x];
  GramProb<float> p = probs[id];
  if (p.st->done) return;
  p.x = X + inst[id].x_off;
  mp_trace t = tr;
  if (t.idx) t.idx += id * tr.cap;
  if (t.coef) t.coef += id * tr.cap;
  if (t.rr) t.rr += id * tr.cap;
  if (t.r) t.r += id * tr.cap * tr.ldr;
  const GramBounds bd = bounds[id];
  if (p.mp == NT * C1) gram_rsteps<NT, C1, ONE>(p, bd, first, t, lds, sh);
  else gram_rsteps<NT, C2, ONE>(p, bd, first, t, lds, sh);
  if (threadIdx.x == 0 && !p.st->done)
    (void)__hip_atomic_fetch_or(again, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

GramBounds gram_bounds_one(int64_t n, double max_norm) {
  GramBounds b = gram_bounds(n, max_norm, false);
  b.dot = static_cast<float>(dot_roundings(n, 1) / 16777216.0 * max_norm * 1.01);
  return b;
}

int64_t gram_ragged_stride(int64_t max_ld, int64_t max_m, int64_t m) {
  if (max_m <= 4096 && max_ld <= 4096) return m <= 1024 ? 1024 : 4096;
  return m <= 8192 ? 8192 : 32768;
}

int gram_ragged_groups(int64_t tiles, int num_cus) {
  int split = 1;
  while (split < kGramRaggedWaves && tiles * split / kGramRaggedWaves < 3 * num_cus) split *= 2;
  return kGramRaggedWaves / split;
}

hipError_t launch_gram_rinit(const GramRagged& g, const float* Y, float* X, const long long* caps,
                             long long cap_all, double eps, hipStream_t s) {
  k_gram_rinit<<<dim3(g.count), dim3(256), 0, s>>>(g.probs, g.inst, Y, X, caps, cap_all, eps);
  return hipGetLastError();
}

// Every problem's residual into the packed R.
__global__ __launch_bounds__(256) void k_gram_rcopy(const GramProb<float>* __restrict__ probs,
                                                    const RInst* __restrict__ inst,
                                                    float* __restrict__ R) {
  const GramProb<float> p = probs[blockIdx.x];
  float* r = R + inst[blockIdx.x].y_off;
  for (int64_t i = threadIdx.x; i < p.n; i += 256) r[i] = p.r[i];
}

hipError_t launch_gram_rcopy(const GramProb<float>* probs, const RInst* inst, int count, float* R,
                             hipStream_t s) {
  k_gram_rcopy<<<dim3(count), dim3(256), 0, s>>>(probs, inst, R);
  return hipGetLastError();
}

template <int NT, int C1, int C2, bool ONE>
static hipError_t launch_rsteps_t(const GramRagged& g, float* X, mp_trace tr, int par, int first,
                                  hipStream_t s) {
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_gram_rsteps<NT, C1, C2, ONE>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kStepLds);
  if (attr != hipSuccess) return attr;
  k_gram_rsteps<NT, C1, C2, ONE>
      <<<dim3(g.count), dim3(NT + 2 * kWave), static_cast<size_t>(g.lds), s>>>(
          g.probs, g.inst, g.order, X, g.bounds, tr, g.again + par, first);
  return hipGetLastError();
}

hipError_t launch_gram_rround(const GramRagged& g, float* X, long long round, mp_trace tr,
                              hipStream_t s) {
  if (g.lds > kStepLds) return hipErrorInvalidValue;
  const int par = static_cast<int>(round & 1), first = round == 0 ? 1 : 0;
  const unsigned packs = static_cast<unsigned>((g.max_ld * (kRhs / 4) + 1023) / 1024);
  k_gram_rpack<<<dim3(packs, g.count), dim3(256), 0, s>>>(g.probs, g.again, par, first);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 block(kGramRaggedWaves * kWave);
  if (g.split == 1)
    k_gram_rpass<true><<<dim3(g.ngroups), block, 0, s>>>(g.probs, g.groups, g.split, first);
  else
    k_gram_rpass<false><<<dim3(g.ngroups), block, 0, s>>>(g.probs, g.groups, g.split, first);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (g.small)
    return g.one ? launch_rsteps_t<256, 4, 16, true>(g, X, tr, par, first, s)
                 : launch_rsteps_t<256, 4, 16, false>(g, X, tr, par, first, s);
  return g.one ? launch_rsteps_t<512, 16, 64, true>(g, X, tr, par, first, s)
               : launch_rsteps_t<512, 16, 64, false>(g, X, tr, par, first, s);
}

}  // namespace mp
