// The decode on carried correlations (k_gram.h): the pass and the steps.
#include <algorithm>

#include "k_common.h"
#include "k_gram.h"

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
// with the next two pieces in flight in registers.  The right-hand sides
// are laid out in operand order by k_gram_pack and come from L2.
//
// Each 16-atom tile's rows are split over `split` waves of the workgroup, so
// that a short dictionary still gives every CU waves; their sums meet in LDS
// in a fixed order.  Two FP32 chains (even and odd steps) are cut every
// 2 kPassRows rows and the cuts are summed in FP64, which keeps the rounding
// bound of the products at that of a kChain-term sum.
constexpr int kPassThreads = 512;
constexpr int kPassWaves = kPassThreads / kWave;
constexpr int kPassRows = 64;           // rows of a piece: 4 steps of 16
constexpr int kChain = kPassRows;       // rows summed in one FP32 chain, at most

// The right-hand sides in operand order: float4 s * 64 + 16 q + i holds rows
// 16 s + 4 q .. + 3 of right-hand side i (r, the wanted columns, then zeros).
// The first pass also clears the slot map.
__global__ __launch_bounds__(256) void k_gram_pack(GramProb p, int first) {
  if (p.st->done) return;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t all = static_cast<int64_t>(gridDim.x) * 256;
  const int nreq = first ? 0 : p.ctl->nreq;
  for (int64_t e = t; e < p.ld * 4; e += all) {
    const int i = static_cast<int>(e % 16);
    const int64_t row4 = e / 64 * 4 + e % 64 / 16;  // float4 of the column
    v4f v = v4f{0.f, 0.f, 0.f, 0.f};
    if (i <= nreq) {
      const float* src = i == 0 ? p.r : p.psi + static_cast<int64_t>(p.ctl->req[i - 1]) * p.ld;
      v = reinterpret_cast<const v4f*>(src)[row4];
    }
    reinterpret_cast<v4f*>(p.rhs)[e] = v;
  }
  if (first)
    for (int64_t e = t; e < p.m; e += all) p.map[e] = static_cast<uint16_t>(kGramNone);
}

__global__ __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(4))) void k_gram_pass(GramProb p, int split, int first) {
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
    // load j of a piece: atoms 4 j + q, float4 i of their 16
    const v4f* a[4];
    int put[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int at = 4 * j + q;
      const int64_t atom = m0 + at < p.m ? m0 + at : p.m - 1;
      a[j] = reinterpret_cast<const v4f*>(p.psi + atom * p.ld) + i;
      put[j] = at * 16 + (i ^ at);
    }
    const v4f* b = reinterpret_cast<const v4f*>(p.rhs) + lane;
    v4f* my = turn[wave];
    const int pieces = static_cast<int>(p.ld / kPassRows);
    const int k0 = pieces * part / split, k1 = pieces * (part + 1) / split;
    v4f acc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
    v4f va[2][4], vb[2][4];
    auto load = [&](v4f(&x)[4], v4f(&y)[4], int k) {
      const int kk = k < k1 ? k : k1 - 1;  // past the end: read again, not used
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = __builtin_nontemporal_load(a[j] + 16 * kk);
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = b[(4 * kk + j) * 64];
    };
    auto use = [&](v4f(&x)[4], v4f(&y)[4], int next) {
#pragma unroll
      for (int j = 0; j < 4; ++j) my[put[j]] = x[j];
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
      load(va[0], vb[0], k0);
      load(va[1], vb[1], k0 + 1);
      int k = k0;
      for (; k + 1 < k1; k += 2) {
        use(va[0], vb[0], k + 2);
        use(va[1], vb[1], k + 3);
        flush();
      }
      if (k < k1) {
        use(va[0], vb[0], k1);
        flush();
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

hipError_t launch_gram_pass(const GramProb& p, int num_cus, bool first, hipStream_t s) {
  const int64_t packs = p.ld * 4 / 256;  // ld is a multiple of 64
  k_gram_pack<<<dim3(static_cast<unsigned>(packs)), dim3(256), 0, s>>>(p, first ? 1 : 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t tiles = (p.m + 15) / 16;
  // the fewest row splits that give two workgroups per CU
  int split = 1;
  while (split < kPassWaves && tiles * split / kPassWaves < 2 * num_cus) split *= 2;
  const int per = kPassWaves / split;
  k_gram_pass<<<dim3(static_cast<unsigned>((tiles + per - 1) / per)), dim3(kPassThreads), 0, s>>>(
      p, split, first ? 1 : 0);
  return hipGetLastError();
}

// The bounds (u = 2^-24): a product of the pass is a chain of at most kChain
// terms, rounded once more to FP32; dot_column_f32 is two
// lane chains of ld / 128 terms, then 7 additions.  Each is at most
// (terms + additions) u sum |a b| <= (...) u ||a|| ||b||; a step adds r's
// rounding (u ||r'|| against a unit column) and c~'s own (u |c~|).
GramBounds gram_bounds(int64_t n, double max_norm) {
  const double u = 1.0 / 16777216.0, nn = static_cast<double>(n + 64);
  const double slack = 1.01;
  const double prod = (std::min<double>(nn, kChain) + 4) * u * slack;
  GramBounds b;
  b.pass = static_cast<float>(prod * max_norm);
  b.col = static_cast<float>(prod * max_norm * max_norm);
  b.step = static_cast<float>(2.1 * u * max_norm * slack);
  b.dot = static_cast<float>((nn / 128 + 10) * u * max_norm * slack);
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
constexpr int kStepLd4 = 4;    // float4s of a column per data thread, at most
constexpr int kStepChain = 16; // float4s of a chain's column in flight per lane

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

// dot_column_f32 (the same chains, so the same result) with fewer loads in
// flight, for a kernel whose registers hold the carried correlations.
__device__ inline float dot_column_narrow(const v4f* __restrict__ p,
                                          const v4f* __restrict__ r, int ld4, int lane) {
  const int h0 = ld4 / 2;
  float acc_a = 0.0f, acc_b = 0.0f;
  int i = lane;
  while (i + kWave * 1 < h0) dot_block2<2, false>(p, r, h0, i, acc_a, acc_b);
  if (i < h0) dot_block2<1, false>(p, r, h0, i, acc_a, acc_b);
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
template <int NT, int CPT>
struct StepShared {
  static constexpr int W = NT / kWave;
  double red[16];
  uint64_t keys[kGramMaxCand];
  v4f spread[W][CPT / 4];
  float wmax[16];
  float chain[2][kWave];
  int n[2];
  int cand[kGramMaxCand];
  int want[(kGramReq + W - 1) / W * W];
};

// The kernel's program for the data waves (DATA) and for the two chain waves:
// one source, so that both take every barrier and every decision alike, and
// two copies, so that the chain waves' registers hold no correlations.
template <int NT, int CPT, bool DATA>
__device__ void gram_steps(const GramProb& p, const GramBounds& bd, long long max_iters, int first,
                           const mp_trace& tr, v4f* r_lds, StepShared<NT, CPT>& sh) {
  constexpr int W = NT / kWave;    // data waves; waves W and W + 1 run the chains
  constexpr int V = 1024 / NT;     // 1024-thread waves each data wave plays
  constexpr int NA = NT + 2 * kWave;
  constexpr int C4 = CPT / 4;
  constexpr int TOP = (kGramReq + W - 1) / W;  // columns each wave proposes
  DevState* st = p.st;
  v4f* s_col = r_lds + p.ld / 4;
  uint16_t* s_map = reinterpret_cast<uint16_t*>(s_col + p.ld / 4);
  float* s_wmax = sh.wmax;
  double* s_red = sh.red;
  float(*s_chain)[kWave] = sh.chain;
  int* s_n = sh.n;
  int* s_cand = sh.cand;
  uint64_t* s_keys = sh.keys;
  int* s_want = sh.want;
  v4f(*s_spread)[CPT / 4] = sh.spread;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int tid = static_cast<int>(threadIdx.x);
  const int ld4 = static_cast<int>(p.ld / 4), h0 = ld4 / 2;
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
  for (int i = tid; i < ld4; i += NA) r_lds[i] = reinterpret_cast<const v4f*>(p.r)[i];
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
    float c = 0.0f;
    if (nc > 1) {
      for (int q = wave; q < nc; q += W + 2) {
        const int a = s_cand[q];
        const float v = dot_column_narrow(
            reinterpret_cast<const v4f*>(p.psi + static_cast<int64_t>(a) * p.ld), r_lds, ld4,
            lane);
        if (lane == 0) s_keys[q] = make_key(v, a);
      }
      __syncthreads();
      const uint64_t best = wave_max(lane < nc ? s_keys[lane] : 0ull);
      win = key_index(best);
      c = key_value(best);
    } else {
      win = s_cand[0];
    }
    win = __builtin_amdgcn_readfirstlane(win);
    // every request of the step at once
    const v4f* col = reinterpret_cast<const v4f*>(p.psi + static_cast<int64_t>(win) * p.ld);
    const unsigned slot = static_cast<unsigned>(
        __builtin_amdgcn_readfirstlane(static_cast<int>(s_map[win])));
    const bool have = slot != kGramNone;
    float x_old = 0.0f;
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
      float acc = 0.0f;
      for (int base = lane; base < h0; base += kStepChain * kWave) {
        v4f ch[kStepChain];
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
            const v4f b = r_lds[off + i];
            s_col[off + i] = ch[u];
            acc = __builtin_fmaf(ch[u].x, b.x, acc);
            acc = __builtin_fmaf(ch[u].y, b.y, acc);
            acc = __builtin_fmaf(ch[u].z, b.z, acc);
            acc = __builtin_fmaf(ch[u].w, b.w, acc);
          }
        }
      }
      s_chain[wave - W][lane] = acc;
    }
    __syncthreads();
    if (nc == 1) c = wave_sum(s_chain[0][lane] + s_chain[1][lane]);
    if (c == 0.0f) {
      stop = MP_STOP_STALLED;
      break;
    }

    // ---- the update: r, ||r||^2, x~, the carried correlations ---------------
    if constexpr (data) {
      double sq[V];
#pragma unroll
      for (int v = 0; v < V; ++v) sq[v] = 0.0;
#pragma unroll
      for (int u = 0; u < kStepLd4; ++u) {
        const int i = tid + NT * u;
        if (i < ld4) {
          const v4f rv = r_lds[i], a = s_col[i];
          v4f o;
          o.x = __builtin_fmaf(-c, a.x, rv.x);
          o.y = __builtin_fmaf(-c, a.y, rv.y);
          o.z = __builtin_fmaf(-c, a.z, rv.z);
          o.w = __builtin_fmaf(-c, a.w, rv.w);
          r_lds[i] = o;
          sq[u % V] += static_cast<double>(o.x) * o.x + static_cast<double>(o.y) * o.y +
                       (static_cast<double>(o.z) * o.z + static_cast<double>(o.w) * o.w);
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const double sv = wave_sum(sq[v]);
        if (lane == 0) s_red[wave + W * v] = sv;
      }
      if (have) {
        lm = 0.0f;
#pragma unroll
        for (int u = 0; u < C4; ++u) {
#pragma unroll
          for (int e = 0; e < 4; ++e) cv[u][e] = __builtin_fmaf(-c, g[u][e], cv[u][e]);
          lm = max_abs4(lm, cv[u]);
        }
        wm = wave_max_f32(lm);
        if (lane == 0) s_wmax[wave] = wm;
      }
    }
    __syncthreads();
    rr = wave_sum(lane < 16 ? s_red[lane] : 0.0);
    if (tr.r && t < tr.cap) {  // the residual's trace entry, if asked for
      float* rt = tr.r + t * tr.ldr;
#pragma unroll 1
      for (int i = tid; i < ld4; i += NA) trace_rows4(rt, i, p.n, r_lds[i]);
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
    err += __builtin_fabsf(c) * bd.col + bd.step * rn;
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
  for (int i = tid; i < ld4; i += NA) reinterpret_cast<v4f*>(p.r)[i] = r_lds[i];
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

template <int NT, int CPT>
__global__ __launch_bounds__(NT + 2 * kWave) void k_gram_steps(GramProb p, GramBounds bd,
                                                               long long max_iters, int first,
                                                               mp_trace tr) {
  extern __shared__ v4f r_lds[];
  __shared__ StepShared<NT, CPT> sh;
  if (p.st->done) return;
  if (threadIdx.x < NT) gram_steps<NT, CPT, true>(p, bd, max_iters, first, tr, r_lds, sh);
  else gram_steps<NT, CPT, false>(p, bd, max_iters, first, tr, r_lds, sh);
}

// The smallest workgroup that holds the correlations: fewer waves make the
// reductions and barriers of a step shorter; a column takes at most kStepLd4
// float4s per thread.
GramShape gram_shape(int64_t ld, int64_t m) {
  const GramShape shapes[] = {{256, 4}, {256, 16}, {512, 16}, {512, 32}, {512, 64}};
  for (const GramShape& s : shapes)
    if (m <= static_cast<int64_t>(s.threads) * s.per_thread && ld <= 4 * kStepLd4 * s.threads &&
        ld <= 8192)
      return s;
  return GramShape{0, 0};
}

template <int NT, int CPT>
static hipError_t launch_steps_t(const GramProb& p, const GramBounds& b, long long max_iters,
                                 bool first, mp_trace tr, hipStream_t s) {
  constexpr int kMax = 2 * 8192 * 4 + NT * CPT * 2;  // r, a column and the slot map
  static const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(k_gram_steps<NT, CPT>),
                          hipFuncAttributeMaxDynamicSharedMemorySize, kMax);
  if (attr != hipSuccess) return attr;
  const size_t lds = static_cast<size_t>(p.ld) * 8 + static_cast<size_t>(p.m) * 2;
  k_gram_steps<NT, CPT><<<dim3(1), dim3(NT + 2 * kWave), lds, s>>>(p, b, max_iters,
                                                             first ? 1 : 0, tr);
  return hipGetLastError();
}

hipError_t launch_gram_steps(const GramProb& p, const GramShape& sh, const GramBounds& b,
                             long long max_iters, bool first, mp_trace tr, hipStream_t s) {
  if (sh.threads == 256 && sh.per_thread == 4)
    return launch_steps_t<256, 4>(p, b, max_iters, first, tr, s);
  if (sh.threads == 256 && sh.per_thread == 16)
    return launch_steps_t<256, 16>(p, b, max_iters, first, tr, s);
  if (sh.threads == 512 && sh.per_thread == 16)
    return launch_steps_t<512, 16>(p, b, max_iters, first, tr, s);
  if (sh.threads == 512 && sh.per_thread == 32)
    return launch_steps_t<512, 32>(p, b, max_iters, first, tr, s);
  if (sh.threads == 512 && sh.per_thread == 64)
    return launch_steps_t<512, 64>(p, b, max_iters, first, tr, s);
  return hipErrorInvalidValue;
}

}  // namespace mp
