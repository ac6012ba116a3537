// The MP steps on carried correlations (k_gram.h), for one signal by one
// workgroup: the device code shared by the kernels that run it.
#pragma once

#include "k_common.h"
#include "k_gram.h"
#include "k_key2.h"

namespace mp {

template <typename T>
struct Vec16 {
  typedef v4f type;
};
template <>
struct Vec16<double> {
  typedef double type __attribute__((ext_vector_type(2)));
};

// ---------------------------------------------------------------------------
// The steps: one workgroup of NT data threads, each with CPT of the carried
// correlations in registers (float4s t + NT u of c~), and two more waves that
// run the product's two lane chains; r and the slot map in LDS.  A step is a
// chain of dependent latencies, not of bytes: the largest |c~| (registers, DPP, LDS), the list of atoms within the band (almost
// always one), then one round trip to memory for everything the step needs
// (the column for the product and the update, its Gram column, x~_idx, all
// requested together), the product's two lane chains, and the update; three
// workgroup barriers in all.  The chains have waves of their own so that no
// wave holds both a chain's column and a share of c~ and its Gram column in
// registers, and none requests its Gram column late.
//
// Order of the sums: the product is dot_column_f32's (two lane chains, added
// per lane, wave_sum); ||r||^2 is block_sum<VN>'s over per-thread sums (16-byte
// chunk i belongs to thread i mod VN of a VN-thread workgroup, the one of the
// form whose results these are: here to wave i / 64 mod (VN / 64) in that
// numbering, and a wave of this kernel plays VN / NT of those in turn).
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
// 2 S loads in flight.  ONE: one chain over the whole column, the ragged FP32
// form's product.
template <typename T, bool ONE, int S, typename V>
__device__ inline T dot_column_narrow(const V* __restrict__ p, const V* __restrict__ r, int ldu,
                                      int lane) {
  T acc_a = 0, acc_b = 0;
  constexpr int U = ONE ? 2 * S : S;
  const int len = ONE ? ldu : ldu / 2;
  const V* pb = p + len;
  const V* rb = r + len;
  for (int base = lane; base < len; base += U * kWave) {
    V a[U], b[ONE ? 1 : U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + kWave * u;
      const int at = i < len ? i : len - 1;
      a[u] = p[at];
      if constexpr (!ONE) b[u] = pb[at];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = base + kWave * u;
      if (i < len) {
        fma_chunk(a[u], r[i], acc_a);
        if constexpr (!ONE) fma_chunk(b[u], rb[i], acc_b);
      }
    }
  }
  return wave_sum(acc_a + acc_b);
}

// sqrt(rr) from above, for the bounds: two instructions (v_rsq_f64 is good to
// 2^-26) where the FP64 square root is a chain of 25.
__device__ inline float norm_above(double rr) {
  return 1.000001f * static_cast<float>(rr * __builtin_amdgcn_rsq(rr));
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
  uint64_t want[kWave];
};

// The kernel's program for the data waves (DATA) and for the two chain waves:
// one source, so that both take every barrier and every decision alike, and
// two copies, so that the chain waves' registers hold no correlations.
// FULL: p.g holds every atom's Gram column (no slot map; the decode leaves
// only at its stop or to have the correlations renewed).  VN: threads of the
// workgroup whose order ||r||^2 is summed in.  ONE: the product is one lane
// chain over the whole column (wave W runs it).
template <typename T, int NT, int CPT, bool DATA, bool FULL, int VN, bool ONE>
__device__ void gram_steps(const GramProb<T>& p, const GramBounds& bd, long long max_iters,
                           int first, const typename GramTrace<T>::type& tr,
                           typename Vec16<T>::type* r_lds, StepShared<T, NT, CPT>& sh) {
  typedef typename Vec16<T>::type V16;
  constexpr int E = 16 / sizeof(T);
  // the slot map is in LDS beside r and the column where there is room (FP32)
  constexpr bool map_lds = !FULL && sizeof(T) == 4;
  constexpr int W = NT / kWave;    // data waves; waves W and W + 1 run the chains
  constexpr int NR = NT > 512 ? 512 : NT;  // threads that update r
  constexpr int V = VN / NR;       // waves of that workgroup each of their waves plays
  constexpr int NA = NT + 2 * kWave;
  constexpr int C4 = CPT / 4;
  constexpr int TOP = kWave / W < 10 ? kWave / W : 10;  // columns each wave proposes
  DevState* st = p.st;
  V16* s_col = r_lds + p.ld / E;
  uint16_t* s_map = map_lds ? reinterpret_cast<uint16_t*>(s_col + p.ld / E) : p.map;
  float* s_wmax = sh.wmax;
  double* s_red = sh.red;
  T(*s_chain)[kWave] = sh.chain;
  int* s_n = sh.n;
  int* s_cand = sh.cand;
  Key2* s_keys = sh.keys;
  uint64_t* s_want = sh.want;
  v4f(*s_spread)[CPT / 4] = sh.spread;
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
  const int tid = static_cast<int>(threadIdx.x);
  const int ldu = static_cast<int>(p.ld / E), h0 = ldu / 2;
  const int m = static_cast<int>(p.m);
  constexpr bool data = DATA;

  // (the last correlations of a share that is not all of c~)
  auto held = [&](int u) {
    return NT <= 512 || u + 1 < C4 || 4 * (tid + NT * u) < static_cast<int>(p.mp);
  };

  // this launch's state: the correlations into registers, r and the map into LDS
  v4f cv[C4];
  if constexpr (data) {
#pragma unroll
    for (int u = 0; u < C4; ++u)
      cv[u] = held(u) ? reinterpret_cast<const v4f*>(p.c)[tid + NT * u]
                      : v4f{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int u = 0; u < C4; ++u) cv[u] = v4f{0.f, 0.f, 0.f, 0.f};
  }
  long long t = st->t;
  double rr = st->rr;
  const double thr = st->thr;
  int used = FULL || first ? 0 : p.ctl->used;
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

  float rn = norm_above(rr);
  float err = bd.pass * rn;
  bool fresh = true;       // c~ straight from a pass
  int stop = -1;           // MP_STOP_* once the run is over
  bool bail = false;
  int par = 0;
  int idx = -1;            // the atom of the last step, if its Gram column is missing
  for (;;) {
    // ---- the shortlist: atoms within the band of the largest |c~| ----------
    const float cmax = row_max(s_wmax[lane % 16]);
    if (!fresh) err += bd.carry * cmax;  // c~'s own rounding in the last step
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
      // the chain waves, which have the registers for 16 loads in flight, take
      // the first two (4 loads in flight in any wave: 18,000 clocks at
      // N = 8192, on a quarter of the steps)
      for (int q = data ? wave + 2 : wave - W; q < nc; q += W + 2) {
        const int a = s_cand[q];
        const T v = dot_column_narrow<T, ONE, DATA ? 2 : 8>(
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
    const unsigned slot =
        FULL ? static_cast<unsigned>(win)
             : static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(s_map[win])));
    const bool have = FULL || slot != kGramNone;
    T x_old = 0;
    v4f g[C4];
    if constexpr (data) {
      const v4f* gp =
          reinterpret_cast<const v4f*>(p.g + static_cast<int64_t>(have ? slot : 0u) * p.mp);
#pragma unroll
      for (int u = 0; u < C4; ++u)
        g[u] = held(u) ? gp[tid + NT * u] : v4f{0.f, 0.f, 0.f, 0.f};
    } else {
      // wave W + h: half h of the column into LDS for the update, and its
      // lane chain of the product
      const int off = wave == W ? 0 : (ONE ? ldu : h0);
      const int len = ONE ? ldu - off : h0;
      T acc = 0;
      for (int base = lane; base < len; base += kStepChain * kWave) {
        V16 ch[kStepChain];
#pragma unroll
        for (int u = 0; u < kStepChain; ++u) {
          const int i = base + kWave * u;
          ch[u] = col[off + (i < len ? i : len - 1)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < kStepChain; ++u) {
          const int i = base + kWave * u;
          if (i < len) {
            s_col[off + i] = ch[u];
            fma_chunk(ch[u], r_lds[off + i], acc);
          }
        }
      }
      // x~_idx for the update's end; requested before the column's loop it is
      // waited for ahead of that loop, a round trip a step
      x_old = p.x[win];
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
      if (wave < NR / kWave) {
        double sq[V];
#pragma unroll
        for (int v = 0; v < V; ++v) sq[v] = 0.0;
        for (int i0 = tid; i0 < ldu; i0 += NR * V)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const int i = i0 + NR * v;
            if (i < ldu) r_lds[i] = update_chunk(c, s_col[i], r_lds[i], sq[v]);
          }
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const double sv = wave_sum(sq[v]);
          if (lane == 0) s_red[wave + NR / kWave * v] = sv;
        }
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
    rn = norm_above(rr);
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
  if (FULL || stop >= 0 || bail) return;
  // the missing column first, then the largest of each wave's best atoms
  // without one
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
    if (data && lane == 0) s_want[k * W + wave] = w;
  }
  __syncthreads();
  // a cache that is nearly full starts over; before that it takes what fits.
  // A pass that only renews the correlations adds columns while there is
  // plenty of room: late in a decode they would push out those in use.
  const bool add = idx >= 0 || p.slots - used >= 4 * kGramReq;
  const bool reset = add && used + kGramReq / 4 > p.slots;
  if (reset) {
    used = 0;
    for (int i = tid; i < m; i += NA) p.map[i] = static_cast<uint16_t>(kGramNone);
    __syncthreads();
  }
  if (wave == 0) {  // the proposals by rank
    GramCtl* ctl = p.ctl;
    const int base = idx >= 0 ? 1 : 0;
    const int room = p.slots - used < kGramReq ? p.slots - used : kGramReq;
    const uint64_t key = add && lane < W * TOP ? s_want[lane] : 0;
    int rank = 0;
    for (int k = 0; k < W * TOP; ++k) rank += s_want[k] > key;
    if (key != 0 && base + rank < room) {
      ctl->req[base + rank] = key_index(key);
      p.map[key_index(key)] = static_cast<uint16_t>(used + base + rank);
    }
    const int found = base + static_cast<int>(__popcll(__ballot(key != 0)));
    if (lane == 0) {
      if (idx >= 0) {
        ctl->req[0] = idx;
        p.map[idx] = static_cast<uint16_t>(used);
      }
      const int nreq = found < room ? found : room;
      ctl->nreq = nreq;
      ctl->slot0 = used;
      ctl->used = used + nreq;
    }
  }
}

}  // namespace mp
