// The decode on carried correlations (k_gram.h): the pass and the steps.
#include <algorithm>

#include "k_common.h"
#include "k_gram.h"
#include "k_key2.h"

namespace mp {

// ---------------------------------------------------------------------------
// The pass: [c~ | g_req] = Psi^T [r | psi_req], 16 atoms x 16 right-hand sides
// per wave on v_mfma_f32_16x16x4_f32.
//
// Bound by the dictionary's bytes, so its reads are whole 256-byte pieces of
// a column (16 lanes each).  The matrix operand wants lane l to hold atom
// l % 16 at rows 4 (l / 16) of a 16-row step, where no two neighbouring lanes
// share a column: read straight from memory that is one cache access per
// lane, 64 per load, and the pass ran at 4.0 TB/s on the L1's access rate
// (N = 8192, M = 32768: 266 us).  Each wave therefore turns its 16 atoms x 64
// rows over in 4 KB of LDS of its own (no barriers; float4 f of atom a at
// position f ^ a of its row, so that neither side meets bank conflicts),
// with the next pieces (8 KB) in flight in registers.  The right-hand sides
// are laid out in operand order by k_gram_pack and come from L2.
//
// Each 16-atom tile's rows are split over `split` waves of the workgroup, so
// that a short dictionary still gives every CU waves; their sums meet in LDS
// in a fixed order.  Two FP32 chains (even and odd steps) are cut every
// 2 kPassRows rows and the cuts are summed in FP64, which keeps the rounding
// bound of the products at that of a kChain-term sum.
template <typename T>
struct Vec16 {
  typedef v4f type;
};
template <>
struct Vec16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};
// 16 bytes of a column as floats.
__device__ inline void put_floats(float* p, const v4f& v) { *reinterpret_cast<v4f*>(p) = v; }
__device__ inline void put_floats(float* p, const Vec16<double>::type& v) {
  typedef float v2f __attribute__((ext_vector_type(2)));
  *reinterpret_cast<v2f*>(p) = v2f{static_cast<float>(v.x), static_cast<float>(v.y)};
}

constexpr int kPassThreads = 512;
constexpr int kPassWaves = kPassThreads / kWave;
constexpr int kPassRows = 64;           // rows of a piece: 4 steps of 16
constexpr int kChain = kPassRows;       // rows summed in one FP32 chain, at most

// The right-hand sides in operand order: float4 s * 64 + 16 q + i holds rows
// 16 s + 4 q .. + 3 of right-hand side i (r, the wanted columns, then zeros).
// The first pass also clears the slot map.
template <typename T>
__global__ __launch_bounds__(256) void k_gram_pack(GramProb<T> p, int first) {
  if (p.st->done) return;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t all = static_cast<int64_t>(gridDim.x) * 256;
  const int nreq = first ? 0 : p.ctl->nreq;
  for (int64_t e = t; e < p.ld * 4; e += all) {
    const int i = static_cast<int>(e % 16);
    const int64_t row4 = e / 64 * 4 + e % 64 / 16;  // float4 of the column
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
__global__ __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_gram_pass(
    GramProb<T> p, int split, int first) {
  constexpr int NL = kPassRows * 16 * sizeof(T) / 16 / kWave;  // 16-byte loads of a piece
  constexpr int LPA = kWave / (16 / NL);                        // lanes of a load per atom
  constexpr int D = sizeof(T) == 4 ? 2 : 1;  // pieces in flight: 8 KB per wave
  typedef typename Vec16<T>::type vec;
  if (p.st->done) return;
  __shared__ v4f turn[kPassWaves][16 * 16];  // then the split sums
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int tiles = kPassWaves / split;  // per workgroup
  const int part = wave % split;
  const int64_t m0 = (static_cast<int64_t>(blockIdx.x) * tiles + wave / split) * 16;
  const int i = lane % 16, q = lane / 16;
  const int nreq = first ? 0 : p.ctl->nreq;
  double tot[4] = {0.0, 0.0, 0.0, 0.0};
  if (m0 < p.m) {
    // load j of a piece: atoms j 64 / LPA + lane / LPA, 16 bytes lane % LPA
    const vec* a[NL];
    int put[NL];  // in floats
    const int li = lane % LPA;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int at = j * (kWave / LPA) + lane / LPA;
      const int64_t atom = m0 + at < p.m ? m0 + at : p.m - 1;
      a[j] = reinterpret_cast<const vec*>(p.psi + atom * p.ld) + li;
      const int f = li * (16 / static_cast<int>(sizeof(T)));  // first row of the 16 bytes
      put[j] = 4 * (at * 16 + ((f / 4) ^ at)) + f % 4;
    }
    const v4f* b = reinterpret_cast<const v4f*>(p.rhs) + lane;
    v4f* my = turn[wave];
    const int pieces = static_cast<int>(p.ld / kPassRows);
    const int k0 = pieces * part / split, k1 = pieces * (part + 1) / split;
    v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
    vec va[D][NL];
    v4f vb[D][4];
    auto load = [&](vec(&x)[NL], v4f(&y)[4], int k) {
      const int kk = k < k1 ? k : k1 - 1;  // past the end: read again, not used
#pragma unroll
      for (int j = 0; j < NL; ++j) x[j] = __builtin_nontemporal_load(a[j] + LPA * kk);
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = b[(4 * kk + j) * 64];
    };
    auto use = [&](vec(&x)[NL], v4f(&y)[4], int next) {
#pragma unroll
      for (int j = 0; j < NL; ++j) put_floats(reinterpret_cast<float*>(my) + put[j], x[j]);
      v4f rb[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) rb[j] = y[j];
      __builtin_amdgcn_wave_barrier();
      load(x, y, next);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const v4f xa = my[i * 16 + ((4 * s + q) ^ i)];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[s & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[e], rb[s][e], acc[s & 1], 0, 0, 0);
      }
      __builtin_amdgcn_wave_barrier();
    };
    auto flush = [&]() {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        tot[e] += static_cast<double>(acc[0][e]) + static_cast<double>(acc[1][e]);
        acc[0][e] = acc[1][e] = 0.0f;
      }
    };
    if (k0 < k1) {
#pragma unroll
      for (int d = 0; d < D; ++d) load(va[d], vb[d], k0 + d);
      for (int k = k0; k < k1; k += D)
#pragma unroll
        for (int d = 0; d < D; ++d)
          if (k + d < k1) {
            use(va[d], vb[d], k + d + D);
            if (d == D - 1 || k + d + 1 >= k1) flush();
          }
    }
  }
  __syncthreads();
  double(*red)[4][kWave] = reinterpret_cast<double(*)[4][kWave]>(&turn[0][0]);
#pragma unroll
  for (int e = 0; e < 4; ++e) red[wave][e][lane] = tot[e];
  __syncthreads();
  if (part != 0 || m0 >= p.m) return;
  for (int w = 1; w < split; ++w)
#pragma unroll
    for (int e = 0; e < 4; ++e) tot[e] += red[wave + w][e][lane];
  // this lane: right-hand side i of atoms m0 + 4 q .. + 3 (zero past the last)
  const int64_t base = m0 + 4 * q;
  v4f o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = base + e < p.m ? static_cast<float>(tot[e]) : 0.0f;
  if (i == 0)
    *reinterpret_cast<v4f*>(p.c + base) = o;
  else if (i <= nreq)
    *reinterpret_cast<v4f*>(p.g + static_cast<int64_t>(p.ctl->slot0 + i - 1) * p.mp + base) = o;
}

template <typename T>
hipError_t launch_gram_pass(const GramProb<T>& p, int num_cus, bool first, hipStream_t s) {
  const int64_t packs = p.ld * 4 / 256;  // ld is a multiple of 64
  k_gram_pack<T><<<dim3(static_cast<unsigned>(packs)), dim3(256), 0, s>>>(p, first ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tiles = (p.m + 15) / 16;
  // the fewest row splits that give two workgroups per CU
  int split = 1;
  while (split < kPassWaves && tiles * split / kPassWaves < 2 * num_cus) split *= 2;
  const int per = kPassWaves / split;
  k_gram_pass<T><<<dim3(static_cast<unsigned>((tiles + per - 1) / per)), dim3(kPassThreads), 0, s>>>(
      p, split, first ? 1 : 0);
  return hipGetLastError();
}

template hipError_t launch_gram_pass<float>(const GramProb<float>&, int, bool, hipStream_t);
template hipError_t launch_gram_pass<double>(const GramProb<double>&, int, bool, hipStream_t);

// The bounds (u = 2^-24): a product of the pass is a chain of at most kChain
// terms, rounded once more to FP32 (and, from an FP64 dictionary, both
// operands rounded to FP32 first); dot_column_f32 is two lane chains of
// ld / 128 terms, then 7 additions (in FP64 its rounding is far below the
// rest).  Each is at most (terms + additions) u sum |a b| <= (...) u ||a||
// ||b||; a step adds r's rounding (u ||r'|| against a unit column), c~'s own
// (u |c~|) and that of the coefficient (u |c|, in col).
GramBounds gram_bounds(int64_t n, double max_norm, bool f64) {
  const double u = 1.0 / 16777216.0, nn = static_cast<double>(n + 64);
  const double slack = 1.01;
  const double prod = (std::min<double>(nn, kChain) + 7) * u * slack;
  GramBounds b;
  b.pass = static_cast<float>(prod * max_norm);
  b.col = static_cast<float>(prod * max_norm * max_norm);
  b.step = static_cast<float>(2.1 * u * max_norm * slack);
  b.dot = static_cast<float>((f64 ? 0.1 : nn / 128 + 10) * u * max_norm * slack);
  return b;
}

// ---------------------------------------------------------------------------
// The steps: one workgroup of NT data threads, each with CPT of the carried
// correlations in registers (float4s t + NT u of c~), and two more waves that
// run the product's two lane chains; r and the slot map in LDS.  A step is a chain of dependent latencies, not of bytes: the largest
// |c~| (registers, DPP, LDS), the list of atoms within the band (almost
// always one), then one round trip to memory for everything the step needs
// (the column for the product and the update, its Gram column, x~_idx, all
// requested together), the product's two lane chains, and the update; three
// workgroup barriers in all.  The chains have waves of their own so that no
// wave holds both a chain's column and a share of c~ and its Gram column in
// registers, and none requests its Gram column late.
//
// Order of the sums: the product is dot_column_f32's (two lane chains, added
// per lane, wave_sum); ||r||^2 is block_sum<1024>'s over per-thread sums
// (float4 i belongs to thread i mod 1024 of a 1024-thread workgroup: here to
// wave i / 64 mod 16 in that numbering, and a wave of this kernel plays
// 1024 / NT of those in turn).
constexpr int kStepChain = 16; // 16-byte chunks of a chain's column in flight per lane

// Row-wise maximum of a non-negative float: afterwards every lane of a
// 16-lane row holds the row's maximum.
__device__ inline float row_max(float v) {
  v = __builtin_fmaxf(v, dpp_f32<kDppQuadSwap1>(v));
  v = __builtin_fmaxf(v, dpp_f32<kDppQuadSwap2>(v));
  v = __builtin_fmaxf(v, dpp_f32<kDppRowRor4>(v));
  return __builtin_fmaxf(v, dpp_f32<kDppRowRor8>(v));
}
__device__ inline float lane_f32(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ inline float wave_max_f32(float v) {
  v = row_max(v);
  return __builtin_fmaxf(__builtin_fmaxf(lane_f32(v, 0), lane_f32(v, 16)),
                         __builtin_fmaxf(lane_f32(v, 32), lane_f32(v, 48)));
}

// acc += <a, b> over 16 bytes, in the order of the stepping forms' products.
__device__ inline void fma_chunk(const v4f& a, const v4f& b, float& acc) {
  acc = __builtin_fmaf(a.x, b.x, acc);
  acc = __builtin_fmaf(a.y, b.y, acc);
  acc = __builtin_fmaf(a.z, b.z, acc);
  acc = __builtin_fmaf(a.w, b.w, acc);
}
typedef Vec16<double>::type v2dd;
__device__ inline void fma_chunk(const v2dd& a, const v2dd& b, double& acc) {
  acc = __builtin_fma(a.x, b.x, acc);
  acc = __builtin_fma(a.y, b.y, acc);
}
// r - c psi over 16 bytes, and the sum of squares added to s (the stepping
// forms' order).
__device__ inline v4f update_chunk(float c, const v4f& a, const v4f& r, double& s) {
  v4f o;
  o.x = __builtin_fmaf(-c, a.x, r.x);
  o.y = __builtin_fmaf(-c, a.y, r.y);
  o.z = __builtin_fmaf(-c, a.z, r.z);
  o.w = __builtin_fmaf(-c, a.w, r.w);
  s += static_cast<double>(o.x) * o.x + static_cast<double>(o.y) * o.y +
       (static_cast<double>(o.z) * o.z + static_cast<double>(o.w) * o.w);
  return o;
}
__device__ inline v2dd update_chunk(double c, const v2dd& a, const v2dd& r, double& s) {
  v2dd o;
  o.x = __builtin_fma(-c, a.x, r.x);
  o.y = __builtin_fma(-c, a.y, r.y);
  s = __builtin_fma(o.x, o.x, s);
  s = __builtin_fma(o.y, o.y, s);
  return o;
}

// dot_column_f32 / dot_column_f64 (the same chains, so the same result) with
// few loads in flight, for a kernel whose registers hold the correlations.
template <typename T, typename V>
__device__ inline T dot_column_narrow(const V* __restrict__ p, const V* __restrict__ r, int ldu,
                                      int lane) {
  const int h0 = ldu / 2;
  T acc_a = 0, acc_b = 0;
#pragma unroll 2
  for (int i = lane; i < h0; i += kWave) {
    const V a = p[i], b = p[h0 + i];
    fma_chunk(a, r[i], acc_a);
    fma_chunk(b, r[h0 + i], acc_b);
  }
  return wave_sum(acc_a + acc_b);
}

// max(m, |v|) over the four elements.
__device__ inline float max_abs4(float m, const v4f& v) {
  return __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(m, __builtin_fabsf(v.x)),
                                         __builtin_fmaxf(__builtin_fabsf(v.y),
                                                         __builtin_fabsf(v.z))),
                         __builtin_fabsf(v.w));
}

// LDS of the steps kernel beside r, the column and the slot map.
template <typename T, int NT, int CPT>
struct StepShared {
  static constexpr int W = NT / kWave;
  double red[16];
  Key2 keys[kGramMaxCand];
  v4f spread[W][CPT / 4];
  float wmax[16];
  T chain[2][kWave];
  int n[2];
  int cand[kGramMaxCand];
  int want[(kGramReq + W - 1) / W * W];
};

// The kernel's program for the data waves (DATA) and for the two chain waves:
// one source, so that both take every barrier and every decision alike, and
// two copies, so that the chain waves' registers hold no correlations.
template <typename T, int NT, int CPT, bool DATA>
__device__ void gram_steps(const GramProb<T>& p, const GramBounds& bd, long long max_iters,
                           int first, const typename GramTrace<T>::type& tr,
                           typename Vec16<T>::type* r_lds, StepShared<T, NT, CPT>& sh) {
  typedef typename Vec16<T>::type V16;
  constexpr int E = 16 / sizeof(T);
  // the slot map is in LDS beside r and the column where there is room (FP32)
  constexpr bool map_lds = sizeof(T) == 4;
  constexpr int W = NT / kWave;    // data waves; waves W and W + 1 run the chains
  constexpr int V = 1024 / NT;     // 1024-thread waves each data wave plays
  constexpr int NA = NT + 2 * kWave;
  constexpr int C4 = CPT / 4;
  constexpr int TOP = (kGramReq + W - 1) / W;  // columns each wave proposes
  DevState* st = p.st;
  V16* s_col = r_lds + p.ld / E;
  uint16_t* s_map = map_lds ? reinterpret_cast<uint16_t*>(s_col + p.ld / E) : p.map;
  float* s_wmax = sh.wmax;
  double* s_red = sh.red;
  T(*s_chain)[kWave] = sh.chain;
  int* s_n = sh.n;
  int* s_cand = sh.cand;
  Key2* s_keys = sh.keys;
  int* s_want = sh.want;
  v4f(*s_spread)[CPT / 4] = sh.spread;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int tid = static_cast<int>(threadIdx.x);
  const int ldu = static_cast<int>(p.ld / E), h0 = ldu / 2;
  const int m = static_cast<int>(p.m);
  constexpr bool data = DATA;

  // this launch's state: the correlations into registers, r and the map into LDS
  v4f cv[C4];
  if constexpr (data) {
#pragma unroll
    for (int u = 0; u < C4; ++u) cv[u] = reinterpret_cast<const v4f*>(p.c)[tid + NT * u];
  } else {
#pragma unroll
    for (int u = 0; u < C4; ++u) cv[u] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  long long t = st->t;
  double rr = st->rr;
  const double thr = st->thr;
  int used = first ? 0 : p.ctl->used;
  for (int i = tid; i < ldu; i += NA) r_lds[i] = reinterpret_cast<const V16*>(p.r)[i];
  if constexpr (map_lds)
    for (int i = tid; i < m; i += NA) s_map[i] = p.map[i];
  if (tid < 16) {
    s_wmax[tid] = 0.0f;
    s_red[tid] = 0.0;
  }
  if (tid < 2) s_n[tid] = 0;
  float lm = 0.0f;
#pragma unroll
  for (int u = 0; u < C4; ++u)
    lm = max_abs4(lm, cv[u]);
  float wm = wave_max_f32(lm);
  __syncthreads();
  if (data && lane == 0) s_wmax[wave] = wm;
  __syncthreads();

  float rn = static_cast<float>(__builtin_sqrt(rr));
  float err = bd.pass * rn;
  bool fresh = true;       // c~ straight from a pass
  int stop = -1;           // MP_STOP_* once the run is over
  bool bail = false;
  int par = 0;
  int idx = -1;            // the atom of the last step, if its Gram column is missing
  for (;;) {
    // ---- the shortlist: atoms within the band of the largest |c~| ----------
    const float cmax = row_max(s_wmax[lane % 16]);
    const float band = 2.002f * (err + bd.dot * rn);
    if (!(band <= 0.125f * cmax) || !(rr > 1e-48) || !(rr < 1e60)) {
      bail = fresh;  // no band narrow enough even on fresh products
      break;
    }
    const float tau = cmax - band;
    if constexpr (data) {
      // a lane that holds one spreads its correlations over the wave (LDS)
      for (unsigned long long lanes = __ballot(lm >= tau); lanes != 0; lanes &= lanes - 1) {
        const int l = __builtin_ctzll(lanes);
        if (lane == l) {
#pragma unroll
          for (int u = 0; u < C4; ++u) s_spread[wave][u] = cv[u];
        }
        __builtin_amdgcn_wave_barrier();
        const float v = lane < CPT ? reinterpret_cast<const float*>(s_spread[wave])[lane] : 0.0f;
        __builtin_amdgcn_wave_barrier();
        if (lane < CPT && __builtin_fabsf(v) >= tau) {
          const int pos = atomicAdd(&s_n[par], 1);
          if (pos < kGramMaxCand)
            s_cand[pos] = 4 * (wave * kWave + l + NT * (lane / 4)) + lane % 4;
        }
      }
    }
    __syncthreads();
    const int nc = __builtin_amdgcn_readfirstlane(s_n[par]);
    if (nc > kGramMaxCand) {
      bail = fresh;
      break;
    }
    if (tid == 0) s_n[par ^ 1] = 0;
    par ^= 1;

    // ---- the winner (largest FP32 |c|, smallest index) and its coefficient --
    int win;
    T c = 0;
    if (nc > 1) {
      for (int q = wave; q < nc; q += W + 2) {
        const int a = s_cand[q];
        const T v = dot_column_narrow<T>(
            reinterpret_cast<const V16*>(p.psi + static_cast<int64_t>(a) * p.ld), r_lds, ldu,
            lane);
        if (lane == 0) s_keys[q] = make_key2(static_cast<double>(v), a);
      }
      __syncthreads();
      const Key2 best = wave_max_key2(lane < nc ? s_keys[lane] : Key2{0, 0});
      win = key2_index(best);
      c = static_cast<T>(key2_value(best));
    } else {
      win = s_cand[0];
    }
    win = __builtin_amdgcn_readfirstlane(win);
    // every request of the step at once
    const V16* col = reinterpret_cast<const V16*>(p.psi + static_cast<int64_t>(win) * p.ld);
    const unsigned slot = static_cast<unsigned>(
        __builtin_amdgcn_readfirstlane(static_cast<int>(s_map[win])));
    const bool have = slot != kGramNone;
    T x_old = 0;
    v4f g[C4];
    if constexpr (data) {
      const v4f* gp =
          reinterpret_cast<const v4f*>(p.g + static_cast<int64_t>(have ? slot : 0u) * p.mp);
#pragma unroll
      for (int u = 0; u < C4; ++u) g[u] = gp[tid + NT * u];
    } else {
      // wave W + h: half h of the column into LDS for the update, and its
      // lane chain of the product
      if (tid == NT) x_old = p.x[win];
      const int off = wave == W ? 0 : h0;
      T acc = 0;
      for (int base = lane; base < h0; base += kStepChain * kWave) {
        V16 ch[kStepChain];
#pragma unroll
        for (int u = 0; u < kStepChain; ++u) {
          const int i = base + kWave * u;
          ch[u] = col[off + (i < h0 ? i : h0 - 1)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kStepChain; ++u) {
          const int i = base + kWave * u;
          if (i < h0) {
            s_col[off + i] = ch[u];
            fma_chunk(ch[u], r_lds[off + i], acc);
          }
        }
      }
      s_chain[wave - W][lane] = acc;
    }
    __syncthreads();
    if (nc == 1) c = wave_sum(s_chain[0][lane] + s_chain[1][lane]);
    if (c == 0) {
      stop = MP_STOP_STALLED;
      break;
    }

    // ---- the update: r, ||r||^2, x~, the carried correlations ---------------
    if constexpr (data) {
      double sq[V];
#pragma unroll
      for (int v = 0; v < V; ++v) sq[v] = 0.0;
      for (int i0 = tid; i0 < ldu; i0 += NT * V)
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int i = i0 + NT * v;
          if (i < ldu) r_lds[i] = update_chunk(c, s_col[i], r_lds[i], sq[v]);
        }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double sv = wave_sum(sq[v]);
        if (lane == 0) s_red[wave + W * v] = sv;
      }
      if (have) {
        const float cf = static_cast<float>(c);
        lm = 0.0f;
#pragma unroll
        for (int u = 0; u < C4; ++u) {
#pragma unroll
          for (int e = 0; e < 4; ++e) cv[u][e] = __builtin_fmaf(-cf, g[u][e], cv[u][e]);
          lm = max_abs4(lm, cv[u]);
        }
        wm = wave_max_f32(lm);
        if (lane == 0) s_wmax[wave] = wm;
      }
    }
    __syncthreads();
    rr = wave_sum(lane < 16 ? s_red[lane] : 0.0);
    if (tr.r && t < tr.cap) {  // the residual's trace entry, if asked for
      T* rt = tr.r + t * tr.ldr;
      const T* rs = reinterpret_cast<const T*>(r_lds);
#pragma unroll 1
      for (int64_t i = tid; i < p.n; i += NA) rt[i] = rs[i];
    }
    if (tid == NT) {
      p.x[win] = x_old + c;
      if (t < tr.cap) {
        if (tr.idx) tr.idx[t] = win;
        if (tr.coef) tr.coef[t] = c;
        if (tr.rr) tr.rr[t] = rr;
      }
    }
    ++t;
    rn = static_cast<float>(__builtin_sqrt(rr));
    err += __builtin_fabsf(static_cast<float>(c)) * bd.col + bd.step * rn;
    fresh = false;
    if (!(rr > thr)) {
      stop = MP_STOP_CONVERGED;
      break;
    }
    if (t >= max_iters) {
      stop = MP_STOP_MAX_ITERS;
      break;
    }
    if (!have) {
      idx = win;
      break;
    }
  }

  // ---- out: r and the state; unless the run is over, the next pass's list ---
  __syncthreads();
  for (int i = tid; i < ldu; i += NA) reinterpret_cast<V16*>(p.r)[i] = r_lds[i];
  if (tid == 0) {
    st->t = t;
    st->rr = rr;
    if (stop >= 0 || bail) {
      st->reason = stop;
      st->done = 1;
      st->pad[0] = bail ? 1 : 0;
    }
  }
  if (stop >= 0 || bail) return;
  // the missing column first, then each wave's best atoms without one
  // (cv: |c~| of this thread's atoms without a Gram column, -1 for the rest)
#pragma unroll
  for (int u = 0; u < C4; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int atom = 4 * (tid + NT * u) + e;
      const bool open = data && atom < m && atom != idx && s_map[atom] == kGramNone;
      cv[u][e] = open ? __builtin_fabsf(cv[u][e]) : -1.0f;
    }
  for (int k = 0; k < TOP; ++k) {
    float best = -1.0f;
    int at = 0;
#pragma unroll
    for (int u = 0; u < C4; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (cv[u][e] > best) {
          best = cv[u][e];
          at = 4 * u + e;
        }
    const uint64_t key = best >= 0.0f ? make_key(best, 4 * (tid + NT * (at / 4)) + at % 4) : 0ull;
    const uint64_t w = wave_max(key);
    if (w != 0 && w == key) {  // one lane: keys differ by their atom
#pragma unroll
      for (int u = 0; u < C4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (at == 4 * u + e) cv[u][e] = -1.0f;
    }
    if (data && lane == 0) s_want[k * W + wave] = w != 0 ? key_index(w) : -1;
  }
  __syncthreads();
  // a full cache starts over
  const bool reset = used + kGramReq > p.slots;
  if (reset) {
    used = 0;
    for (int i = tid; i < m; i += NA) p.map[i] = static_cast<uint16_t>(kGramNone);
    __syncthreads();
  }
  if (tid == 0) {
    GramCtl* ctl = p.ctl;
    int nreq = 0;
    if (idx >= 0) ctl->req[nreq++] = idx;
    for (int k = 0; k < W * TOP && nreq < kGramReq; ++k)
      if (s_want[k] >= 0) ctl->req[nreq++] = s_want[k];
    for (int k = 0; k < nreq; ++k) p.map[ctl->req[k]] = static_cast<uint16_t>(used + k);
    ctl->nreq = nreq;
    ctl->slot0 = used;
    ctl->used = used + nreq;
    ctl->err = err;
  }
}

template <typename T, int NT, int CPT>
__global__ __launch_bounds__(NT + 2 * kWave) void k_gram_steps(
    GramProb<T> p, GramBounds bd, long long max_iters, int first,
    typename GramTrace<T>::type tr) {
  extern __shared__ v4f lds[];
  typename Vec16<T>::type* r_lds = reinterpret_cast<typename Vec16<T>::type*>(lds);
  __shared__ StepShared<T, NT, CPT> sh;
  if (p.st->done) return;
  if (threadIdx.x < NT) gram_steps<T, NT, CPT, true>(p, bd, max_iters, first, tr, r_lds, sh);
  else gram_steps<T, NT, CPT, false>(p, bd, max_iters, first, tr, r_lds, sh);
}

constexpr int64_t kStepLds = 150 * 1024;  // r, a column and (FP32) the slot map, at most

static int64_t step_lds(int64_t ld, int64_t m, int esize) {
  return 2 * ld * esize + (esize == 4 ? 2 * m : 0);
}

// The smallest workgroup that holds the correlations: fewer waves make the
// reductions and barriers of a step shorter.  Columns above 4096 rows take
// 512 threads, so that no thread updates more than a few chunks of r.
GramShape gram_shape(int64_t ld, int64_t m, int esize) {
  const GramShape shapes[] = {{256, 4}, {256, 16}, {512, 16}, {512, 32}, {512, 64}};
  if (step_lds(ld, m, esize) > kStepLds) return GramShape{0, 0};
  for (const GramShape& s : shapes)
    if (m <= static_cast<int64_t>(s.threads) * s.per_thread &&
        (ld * esize <= 16384 || s.threads == 512))
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
  if (sh.threads == 512 && sh.per_thread == 64)
    return launch_steps_t<T, 512, 64>(p, b, max_iters, first, tr, s);
  return hipErrorInvalidValue;
}
template hipError_t launch_gram_steps<float>(const GramProb<float>&, const GramShape&,
                                             const GramBounds&, long long, bool, mp_trace,
                                             hipStream_t);
template hipError_t launch_gram_steps<double>(const GramProb<double>&, const GramShape&,
                                              const GramBounds&, long long, bool, mp_trace_f64,
                                              hipStream_t);

}  // namespace mp
