// Host side of libmp.so: argument checking, context ownership, the iteration
// driver, and the C ABI declared in include/mp.h.
#include <math.h>
#include <cmath>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <climits>
#include <string>
#include <vector>

#include "k_gram.h"
#include "k_sign_gram.h"
#include "mp_internal.h"

namespace {

thread_local std::string g_create_error;

constexpr int64_t kMaxN = 16384;          // the residual is staged whole in LDS
constexpr int64_t kMaxSignN = 16384;      // two 16-byte chunks of a column per lane
constexpr int64_t kMaxRaggedN = 8192;     // per-instance residual in LDS, 32 KB
constexpr int kMaxRaggedSplit = 4096;     // instances cut into parts, at most
constexpr int kRaggedDefaultSplit = 3;    // parts of an instance, at most, unless configured
constexpr int64_t kLdAlign = 64;          // padded column length (floats): 256 B aligned
constexpr int kMaxChunk = 64;             // iterations enqueued per host check
constexpr double kNormTol = 1e-4;
// Caps are cut to this (no decode gets there), so that the host's counts of
// launches and rounds, small multiples of the cap, do not overflow.
constexpr long long kMaxCap = LLONG_MAX / 8;
long long step_cap(const mp_opts* opts) {
  return std::min<long long>(opts->max_iters, kMaxCap);
}

mp_status fail(mp_ctx* ctx, mp_status s, const std::string& msg) {
  if (ctx) ctx->err = msg;
  else g_create_error = msg;
  return s;
}

#define HIP_TRY(ctx, expr)                                                            \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess)                                                             \
      return fail((ctx), MP_EDEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

int64_t round_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

void free_batched(mp_ctx* c) {
  (void)hipFree(c->b_r32);
  (void)hipFree(c->b_rq);
  (void)hipFree(c->b_slots);
  (void)hipFree(c->b_act);
  (void)hipFree(c->b_state);
  (void)hipFree(c->b_partials);
  (void)hipFree(c->b_keep);
  (void)hipFree(c->b_tcap);
  if (c->h_slots) (void)hipHostFree(c->h_slots);
  if (c->h_bstate) (void)hipHostFree(c->h_bstate);
  c->b_r32 = nullptr;
  c->b_rq = nullptr;
  c->b_slots = nullptr;
  c->b_act = nullptr;
  c->b_state = nullptr;
  c->b_partials = nullptr;
  c->b_keep = nullptr;
  c->b_tcap = nullptr;
  c->h_slots = nullptr;
  c->h_bstate = nullptr;
  c->bcap = 0;
}

void free_ragged(mp_ctx* c) {
  (void)hipFree(c->r_psi32);
  (void)hipFree(c->r_psib);
  (void)hipFree(c->r_inst);
  (void)hipFree(c->r_items);
  (void)hipFree(c->r_slots);
  if (c->h_rq) (void)hipHostFree(c->h_rq);
  (void)hipFree(c->r_caps);
  (void)hipFree(c->r_res);
  (void)hipFree(c->r_queue);
  if (c->h_rres) (void)hipHostFree(c->h_rres);
  if (c->r_graph) (void)hipGraphExecDestroy(c->r_graph);
  if (c->r_cap_stream) (void)hipStreamDestroy(c->r_cap_stream);
}

void free_omp_carry(mp_ctx* c) {
  mp::OmpBufs& b = c->omp;
  (void)hipFree(b.oc);
  (void)hipFree(b.c);
  (void)hipFree(b.p);
  (void)hipFree(b.w15);
  (void)hipFree(b.rhs);
  (void)hipFree(b.hr);
  (void)hipFree(b.hq);
  (void)hipFree(b.dpart);
  (void)hipFree(b.tops);
  b.oc = nullptr;
  b.c = b.p = b.w15 = b.rhs = b.hr = b.hq = nullptr;
  b.dpart = nullptr;
  b.tops = nullptr;
}

void free_omp(mp_ctx* c) {
  mp::OmpBufs& b = c->omp;
  (void)hipFree(b.q);
  (void)hipFree(b.rmat);
  (void)hipFree(b.z);
  (void)hipFree(b.sel);
  (void)hipFree(b.in_s);
  (void)hipFree(b.w);
  (void)hipFree(b.h1);
  (void)hipFree(b.h2);
  (void)hipFree(b.hp);
  (void)hipFree(b.part);
  (void)hipFree(b.os);
  free_omp_carry(c);
  b = mp::OmpBufs{};
}

void free_sign_gram(mp_ctx* c) {
  mp::SignGram& b = c->sign_gram;
  (void)hipFree(b.carry);
  (void)hipFree(b.pos);
  (void)hipFree(b.g);
  (void)hipFree(b.h);
  (void)hipFree(b.parts);
  b = mp::SignGram{};
}

void free_gram(mp_ctx* c) {
  (void)hipFree(c->gram_c);
  (void)hipFree(c->gram_g);
  (void)hipFree(c->gram_map);
  (void)hipFree(c->gram_rhs);
  (void)hipFree(c->gram_ctl);
  c->gram_c = nullptr;
  c->gram_g = nullptr;
  c->gram_map = nullptr;
  c->gram_rhs = nullptr;
  c->gram_ctl = nullptr;
  c->gram_slots = 0;
}

void free_gram_batch(mp_ctx* c) {
  (void)hipFree(c->gram_bc);
  (void)hipFree(c->gram_br);
  (void)hipFree(c->gram_bst);
  (void)hipFree(c->gram_again);
  (void)hipFree(c->gram_btcap);
  if (c->gram_hbst) (void)hipHostFree(c->gram_hbst);
  if (c->gram_hagain) (void)hipHostFree(c->gram_hagain);
  c->gram_bc = nullptr;
  c->gram_br = nullptr;
  c->gram_bst = nullptr;
  c->gram_again = nullptr;
  c->gram_btcap = nullptr;
  c->gram_hbst = nullptr;
  c->gram_hagain = nullptr;
  c->gram_bcap = 0;
}

void free_gram_ragged(mp_ctx* c) {
  (void)hipFree(c->gram_rmem);
  if (c->gram_hrmem) (void)hipHostFree(c->gram_hrmem);
  for (hipEvent_t& e : c->gram_rev) {
    if (e) (void)hipEventDestroy(e);
    e = nullptr;
  }
  c->gram_rmem = c->gram_hrmem = nullptr;
}

void free_ctx(mp_ctx* c) {
  if (!c) return;
  free_gram(c);
  free_sign_gram(c);
  free_gram_ragged(c);
  free_gram_batch(c);
  (void)hipFree(c->gram_full);
  free_batched(c);
  free_ragged(c);
  free_omp(c);
  (void)hipFree(c->psibt);
  (void)hipFree(c->psi32);
  (void)hipFree(c->psi64);
  (void)hipFree(c->r64_work);
  (void)hipFree(c->psiq);
  (void)hipFree(c->psis);
  (void)hipFree(c->sign_c64);
  (void)hipFree(c->sign_r64);
  (void)hipFree(c->sign_rrp);
  (void)hipFree(c->sign_slots);
  (void)hipFree(c->small_slots);
  (void)hipFree(c->scales);
  (void)hipFree(c->r_work);
  (void)hipFree(c->st);
  (void)hipFree(c->partials);
  (void)hipFree(c->bal);
  if (c->async_pending && c->async_ev) (void)hipEventSynchronize(c->async_ev);
  if (c->async_ev) (void)hipEventDestroy(c->async_ev);
  if (c->h_st) (void)hipHostFree(c->h_st);
  for (hipEvent_t e : c->done_ev)
    if (e) (void)hipEventDestroy(e);
  for (hipEvent_t e : c->ev) (void)hipEventDestroy(e);
  delete c;
}

// The current device, if it is a gfx950 this library was built for.
mp_status open_device(int& dev, hipDeviceProp_t& prop) {
  int count = 0;
  if (hipGetDeviceCount(&count) != hipSuccess || count < 1)
    return fail(nullptr, MP_EDEVICE, "no HIP device");
  HIP_TRY(nullptr, hipGetDevice(&dev));
  HIP_TRY(nullptr, hipGetDeviceProperties(&prop, dev));
  if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(nullptr, MP_EUNSUPPORTED, std::string("device is ") + prop.gcnArchName +
                                              ", this library is built for gfx950");
  return MP_OK;
}

// The largest column norm of the FP64 squared norms.
double largest_norm(const std::vector<double>& norm2) {
  double v = 0.0;
  for (double q : norm2) v = std::max(v, q);
  return std::sqrt(v);
}

// Eq. 4 on the FP64 squared column norms: finite always, 1 within kNormTol
// unless MP_SKIP_NORM_CHECK.  Returns MP_OK or the status with `msg` set.
mp_status check_norms(const std::vector<double>& norm2, uint32_t flags, std::string& msg) {
  for (size_t j = 0; j < norm2.size(); ++j) {
    if (!isfinite(norm2[j])) {
      char buf[96];
      snprintf(buf, sizeof buf, "column %lld holds NaN or Inf", static_cast<long long>(j));
      msg = buf;
      return MP_ENONFINITE;
    }
    if (!(flags & MP_SKIP_NORM_CHECK) && fabs(sqrt(norm2[j]) - 1.0) > kNormTol) {
      char buf[128];
      snprintf(buf, sizeof buf, "column %lld has norm %.9g (must be 1 within 1e-4)",
               static_cast<long long>(j), sqrt(norm2[j]));
      msg = buf;
      return MP_ENOTNORM;
    }
  }
  return MP_OK;
}

// The trace's residual rows: ldr must cover the longest residual it receives.
template <class T>
mp_status check_trace(mp_ctx* c, const T* trace, int64_t rows) {
  if (!trace) return MP_OK;
  if (trace->cap < 0) return fail(c, MP_EINVAL, "trace cap must be >= 0");
  if (trace->r && trace->ldr < rows)
    return fail(c, MP_EINVAL, "trace ldr must be >= the residual length");
  return MP_OK;
}

// A context with a stream-ordered decode not yet collected takes no other
// decode (its device state and the host mirror belong to that decode).
mp_status check_not_pending(mp_ctx* c) {
  if (c->async_pending)
    return fail(c, MP_EINVAL, "a stream-ordered decode is pending: collect it with mp_solve_result");
  return MP_OK;
}

mp_status check_opts(mp_ctx* c, const mp_opts* opts,
                     uint32_t allowed = MP_SOLVE_STEP_LAUNCHES) {
  if (mp_status ps = check_not_pending(c); ps != MP_OK) return ps;
  if (!(opts->eps >= 0.0) || !isfinite(opts->eps))
    return fail(c, MP_EINVAL, "eps must be finite and >= 0");
  if (opts->max_iters < 0) return fail(c, MP_EINVAL, "max_iters must be >= 0");
  if (opts->flags & ~allowed) return fail(c, MP_EINVAL, "unknown opts.flags");
  if (opts->rescore_k < 0 || opts->rescore_k > 8)
    return fail(c, MP_EINVAL, "rescore_k must be in 0..8");
  return MP_OK;
}

// The pinned host mirror of the device state (entry 0) and the two slots
// run_iterations copies each chunk's state into (entries 1, 2), with the
// events that mark those copies: made once per context, so that a decode
// allocates nothing.
bool make_host_state(mp_ctx* c) {
  if (hipHostMalloc(&c->h_st, 3 * sizeof(mp::DevState), hipHostMallocDefault) != hipSuccess) {
    c->h_st = nullptr;
    return false;
  }
  for (hipEvent_t& e : c->done_ev)
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
      e = nullptr;
      return false;
    }
  if (hipEventCreateWithFlags(&c->async_ev, hipEventDisableTiming) != hipSuccess) {
    c->async_ev = nullptr;
    return false;
  }
  return true;
}

// Length of the next chunk of launches.  Doubling from 4 up to kMaxChunk
// while the run is young; once two chunk-end states are known, the
// remaining steps are estimated from the decay of ||r||^2 between them
// (ln rr falls about linearly once MP settles) and the chunk is cut to what
// that estimate still needs beyond the launches already in flight, plus a
// margin: launches issued past the stop return at once but still cost a
// dispatch each, which dominates short decodes.  Returns 0 when the
// launches in flight should cover the estimate (the caller then waits).
int next_chunk(int doubling, long long issued, const mp::DevState* a, const mp::DevState* b) {
  const double thr = b ? b->thr : 0.0;
  if (!a || !b || b->done || b->t <= a->t || !(b->rr > thr) || !(a->rr > b->rr) ||
      !(thr > 0.0))
    return doubling;
  const double rate = (std::log(a->rr) - std::log(b->rr)) / static_cast<double>(b->t - a->t);
  const double rem = std::log(b->rr / thr) / rate;  // steps still needed after b
  const long long ahead = issued - (b->t + 1);         // launches in flight past b
  const double want = std::ceil(rem * 1.25) + 2.0 - static_cast<double>(ahead);
  if (want <= 0.0) return 0;
  return static_cast<int>(std::min<double>(want, doubling));
}

// The single-signal iteration driver: after init (state already copied to
// c->h_st), enqueue chunks of iterations with `enqueue(e0, e1)` (record e0,
// when not null, before the iteration's launch and e1 after it); the kernels
// stop doing work once the device state says the run is over.  Two chunks
// stay in flight: after enqueuing chunk k the host waits for the state copy
// that follows chunk k-1.
//
// Timing, with profiling on.  `windowed` (one kernel launch per iteration):
// each chunk is cut from its start into windows of prof_every consecutive
// launches (at most a chunk), timed by one event before the window's first
// launch and one after its last, so the launches inside run as untimed ones
// do and the average per launch includes the gaps between them.  Otherwise
// (OMP: several kernels per iteration, `enqueue` brackets the selection
// launch) every prof_every-th iteration is timed on its own.  Only launches
// that performed an iteration are counted: a window, all its launches.
// t0: steps the decode has behind it (the state's t counts from there).
template <typename Enqueue>
mp_status run_iterations(mp_ctx* c, long long T, hipStream_t s, bool windowed, Enqueue enqueue,
                         bool known_running = false, const mp::DevState* dst = nullptr,
                         long long t0 = 0) {
  if (!dst) dst = c->st;
  c->prof_ms = 0.0;
  c->prof_launches = 0;
  long long issued = 0;
  int chunk = 4;
  hipEvent_t* done_ev = c->done_ev;
  mp::DevState* h_slot = c->h_st + 1;
  // the last two chunk-end states read back (for the chunk-length estimate)
  mp::DevState hist[2];
  int nhist = 0;
  long long slot_base[2] = {0, 0};
  int slot_len[2] = {0, 0};
  mp_status status = MP_OK;
  // Launch j of a decode ran its correlation pass unless the run had stopped
  // by then.  A run that stops after t steps stops in launch t+1 in the
  // one-bit form; in the others in launch t (converged or out of steps: step
  // t applied, no pass) or t+1 (no usable winner).  Only launches that ran a
  // pass are timed.
  auto account = [&](int k) {
    if (!c->profiling) return;
    const mp::DevState& sl = h_slot[k];
    const bool late = c->storage == MP_SIGN1 ||
                      (sl.reason != MP_STOP_CONVERGED && sl.reason != MP_STOP_MAX_ITERS);
    const long long stop_launch = sl.done ? sl.t - t0 + (late ? 1 : 0) : LLONG_MAX;
    const int w = windowed ? std::min(c->prof_every, kMaxChunk) : 1;
    for (int j = 0; j + w <= slot_len[k]; j += w) {
      if (slot_base[k] + j + w > stop_launch) break;
      if (!windowed && (slot_base[k] + j) % c->prof_every != 0) continue;
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, c->ev[(k * kMaxChunk + j) * 2],
                              c->ev[(k * kMaxChunk + j) * 2 + 1]) == hipSuccess) {
        c->prof_ms += ms;
        c->prof_launches += w;
      }
    }
  };
  bool finished = !known_running && c->h_st->done != 0;
  int next = 0;      // slot the next chunk goes to
  int inflight = 0;  // chunks enqueued but not yet waited for
  while (!finished && status == MP_OK) {
    while (inflight < 2 && issued < T && status == MP_OK) {
      const int k = next;
      int want = next_chunk(chunk, t0 + issued, nhist == 2 ? &hist[0] : nullptr,
                            nhist >= 1 ? &hist[nhist - 1] : nullptr);
      if (want == 0) {
        if (inflight > 0) break;  // wait for what is in flight
        want = 2;
      }
      const int len = static_cast<int>(std::min<long long>(want, T - issued));
      const int w = windowed ? std::min(c->prof_every, kMaxChunk) : 1;
      for (int j = 0; j < len; ++j) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        const int j0 = j - j % w;  // first launch of j's window
        if (c->profiling && j0 + w <= len &&
            (windowed || (issued + j) % c->prof_every == 0)) {
          if (j == j0) e0 = c->ev[(k * kMaxChunk + j0) * 2];
          if (j == j0 + w - 1) e1 = c->ev[(k * kMaxChunk + j0) * 2 + 1];
        }
        hipError_t e = enqueue(e0, e1);
        if (e != hipSuccess) {
          status = fail(c, MP_EDEVICE, std::string("launch: ") + hipGetErrorString(e));
          break;
        }
      }
      if (status != MP_OK) break;
      slot_base[k] = issued;
      slot_len[k] = len;
      issued += len;
      hipError_t e = hipMemcpyAsync(&h_slot[k], dst, sizeof(mp::DevState),
                                    hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipEventRecord(done_ev[k], s);
      if (e != hipSuccess) {
        status = fail(c, MP_EDEVICE, std::string("state copy: ") + hipGetErrorString(e));
        break;
      }
      ++inflight;
      next ^= 1;
      chunk = std::min(chunk * 2, kMaxChunk);
    }
    if (status != MP_OK || inflight == 0) break;
    const int old = inflight == 2 ? next : (next ^ 1);  // the older chunk in flight
    hipError_t e = hipEventSynchronize(done_ev[old]);
    if (e != hipSuccess) {
      status = fail(c, MP_EDEVICE, std::string("sync: ") + hipGetErrorString(e));
      break;
    }
    --inflight;
    account(old);
    if (h_slot[old].done) finished = true;
    if (nhist == 2) hist[0] = hist[1];
    hist[nhist == 2 ? 1 : nhist] = h_slot[old];
    if (nhist < 2) ++nhist;
  }
  // drain the chunk still in flight (its launches return at once)
  if (hipStreamSynchronize(s) != hipSuccess && status == MP_OK)
    status = fail(c, MP_EDEVICE, "stream synchronize failed");
  return status;
}

// Device buffers of one carried single-signal decode (FP32, BF16, FP8): the
// context's own (mp_solve) or carved from the library's static scratch
// (mp_solve_noalloc).
struct CarriedBufs {
  mp::DevState* st;  // the decode's state
  float* r_work;     // 2 x ld floats: r_k in half k mod 2 (padding rows written 0)
  uint64_t* keys;    // 2 x grid x kLpTopK key slots
  mp::BalState* bal; // column shares and pass timings (any contents: a balance hint only)
};

mp_status finish_result(mp_ctx* c, mp_result* res);

// The carried decode: launch k takes step k (k >= 1) and runs pass k+1, so T
// steps take T+1 launches; r ends in the half the state names.  The kernels
// read the stop threshold from the device state, so the host starts
// launching without waiting for the init kernel (launches after a stop, zero
// input included, return at once).  At the end one small kernel copies r out
// of the half the state names, and the state comes back with one wait.
// Allocates nothing: every buffer is in `b`, the context (pinned state slots
// and events made at its creation) or the caller's arguments.
//
// Stream-ordered (MP_SOLVE_ASYNC): the same launches, all T+1 of them
// enqueued at once (the host does not read the state), then the state copy
// into the host mirror and the context's event; mp_solve_result waits for it.
mp_status enqueue_result(mp_ctx* c, const mp::DevState* st, hipStream_t s, int persistent) {
  HIP_TRY(c, hipMemcpyAsync(c->h_st, st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipEventRecord(c->async_ev, s));
  c->async_pending = true;
  c->async_persistent = persistent;
  return MP_OK;
}

// Buffers that only make a decode faster take at most an eighth of the memory
// that is free, so that what a program sets up beside them still fits.
bool room_for(size_t bytes) {
  size_t free = 0, total = 0;
  if (hipMemGetInfo(&free, &total) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return bytes <= free / 8;
}

// Whether a cap leaves carried correlations their start: a decode pays for two
// passes with all right-hand sides before it gains, and takes its steps, if it
// is allowed only a few, sooner in the form with a launch each.  Carried and
// that form, us, N x M of 1024 x 4096, 4096 x 16384 and 8192 x 32768:
//   FP32  cap 3: 124 66, 221 182, 490 532    cap 4: 135 104, 222 264, 493 729
//   FP64  cap 2: 138 89, 296 238, 766 706    cap 3: 142 102, 298 323, 764 1027
//   BF16  cap 4: 127 114, 226 191, 486 436   cap 6: 136 131, 233 248, 499 617
//   FP8   cap 6: 125 130, 229 196, 493 377   cap 8: 138 151, 236 235, 507 476
//   OMP   cap 3 (96 MiB, 256 MiB, 1 GiB): 288 187, 331 261, 632 617
//         cap 4: 303 223, 352 323, 644 799
bool cap_pays(mp_dtype storage, long long cap) {
  const int few = storage == MP_F64 ? 2 : storage == MP_BF16 ? 4 : storage == MP_FP8_E4M3 ? 6 : 3;
  return cap > few;
}

// The buffers of the decode on carried correlations, made by the first
// decode that takes it: Gram columns for at most a quarter of the
// dictionary's bytes (n / 4 columns; a decode of K atoms needs little more
// than K of them, and MP recovers K well below n / 4), at least 256.
// Returns false where the form does not apply (size, column norms that are
// not near 1) or the memory is not there: the decode then takes one launch
// per step.
bool ensure_gram(mp_ctx* c, hipStream_t s) {
  if (!c->carried_on) return false;
  if (c->gram_tried) return c->gram_slots > 0;
  c->gram_tried = true;
  const mp::GramShape sh = mp::gram_shape(c->ld, c->m, c->storage == MP_F64 ? 8 : 4);
  if (sh.threads == 0 || !(c->max_norm > 0.99) || !(c->max_norm < 1.01)) return false;
  c->gram_mp = mp::gram_stride(sh);
  const int64_t want = std::max<int64_t>(256, c->n / 4);
  const int64_t slots = round_up(std::min<int64_t>(want, c->m) + mp::kGramReq, 16);
  const size_t row = static_cast<size_t>(c->gram_mp) * sizeof(float);
  if (!room_for(row * static_cast<size_t>(slots)) ||
      hipMalloc(&c->gram_c, row) != hipSuccess ||
      hipMalloc(&c->gram_g, row * static_cast<size_t>(slots)) != hipSuccess ||
      hipMalloc(&c->gram_map, sizeof(uint16_t) * static_cast<size_t>(c->m)) != hipSuccess ||
      hipMalloc(&c->gram_rhs, sizeof(float) * (mp::kGramReq + 1) * static_cast<size_t>(c->ld)) !=
          hipSuccess ||
      hipMalloc(&c->gram_ctl, sizeof(mp::GramCtl)) != hipSuccess ||
      // entries past m stay zero (the pass writes the tiles of m)
      hipMemsetAsync(c->gram_c, 0, row, s) != hipSuccess ||
      hipMemsetAsync(c->gram_g, 0, row * static_cast<size_t>(slots), s) != hipSuccess) {
    (void)hipGetLastError();
    free_gram(c);
    return false;
  }
  c->gram_slots = static_cast<int>(slots);
  return true;
}

// The decode on carried correlations (k_gram.h), after the init kernel: pairs
// of a pass and the steps it allows, the host keeping two pairs in flight.
// `gave_up` is set when the device asks for the stepping form instead (no
// shortlist narrow enough, or norms outside the bounds' range): the t0 steps
// taken stand, and that form goes on from them (the state runs again, r is in
// half t0 mod 2).
template <typename T>
mp_status solve_gram(mp_ctx* c, const T* psi, T* r_work, T* x, const mp_opts* opts,
                     const typename mp::GramTrace<T>::type& tr, hipStream_t s, bool& gave_up,
                     long long& t0) {
  const mp::GramShape sh = mp::gram_shape(c->ld, c->m, sizeof(T));
  const mp::GramBounds bounds = mp::gram_bounds(c->n, c->max_norm, sizeof(T) == 8);
  const mp::GramProb<T> p{psi, c->ld, c->n, c->m, c->gram_mp, c->gram_c, c->gram_g, c->gram_map,
                          c->gram_slots, c->gram_rhs, r_work, x, c->st,
                          static_cast<mp::GramCtl*>(c->gram_ctl)};
  gave_up = false;
  const bool timed = c->profiling;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  // a pair takes at least one step, unless it only renews the correlations,
  // which the next one then follows with a step
  const long long cap = step_cap(opts), most = 2 * cap + 2;
  long long issued = 0, seen = 0;
  bool over = cap <= 0;
  while (!over && seen < most) {
    while (issued < most && issued - seen < 2) {
      HIP_TRY(c, mp::launch_gram_pass(p, c->num_cus, issued == 0, s));
      HIP_TRY(c, mp::launch_gram_steps(p, sh, bounds, cap, issued == 0, tr, s));
      const int k = static_cast<int>(issued & 1);
      HIP_TRY(c, hipMemcpyAsync(&c->h_st[1 + k], c->st, sizeof(mp::DevState),
                                hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipEventRecord(c->done_ev[k], s));
      ++issued;
    }
    const int k = static_cast<int>(seen & 1);
    HIP_TRY(c, hipEventSynchronize(c->done_ev[k]));
    ++seen;
    over = c->h_st[1 + k].done != 0;
    gave_up = c->h_st[1 + k].pad[0] != 0;
    t0 = c->h_st[1 + k].t;
  }
  if (!over && cap > 0) gave_up = true;  // (not reached: unfinished is never a result)
  c->carried_steps = t0;
  if (gave_up) {
    HIP_TRY(c, mp::launch_resume<T>(c->st, r_work, c->ld, static_cast<int>(t0 & 1), s));
    return MP_OK;
  }
  if (timed) {
    // the decode's time on the device over the steps it took
    HIP_TRY(c, hipEventRecord(c->ev[1], s));
    HIP_TRY(c, hipEventSynchronize(c->ev[1]));
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      const mp::DevState& d = c->h_st[1 + static_cast<int>((seen - 1) & 1)];
      c->prof_ms = ms;
      c->prof_launches = seen > 0 && d.t > 0 ? d.t : 1;
    }
  }
  return MP_OK;
}

// Whether the Gram columns of all atoms (m^2 floats, rounded up) suit the
// context: norms near 1, M <= 16384, and their memory in proportion, at most
// 64 MiB (M = 4096) or 8 times the dictionary's (M = 8 N).
bool gram_full_suits(const mp_ctx* c) {
  const mp::GramShape sh = mp::gram_shape(c->ld, c->m, 4);
  const int64_t bytes = 4 * mp::gram_stride(sh) * c->m;
  return c->carried_on && sh.threads != 0 && c->m <= 16384 && c->max_norm > 0.99 &&
         c->max_norm < 1.01 && bytes <= std::max<int64_t>(int64_t{64} << 20, 8 * 4 * c->ld * c->m);
}

// What making them costs, us: the symmetric product's 2 m^2 n / 2 operations at
// the 70 TFLOP/s that it reaches with the allocation (N = 2048, M = 8192: 1.9 ms;
// N = 4096, M = 16384: 11.5 ms).
double gram_full_us(const mp_ctx* c) {
  return static_cast<double>(c->m) * static_cast<double>(c->m) * static_cast<double>(c->ld) / 70e6;
}

// What B signals gain on them by every step of the longest, us, against a round
// of products (rounds of 64 steps less 16, and carried: 500 x 1000, 500 signals
// 15.1 and 2.4; 2048 x 8192, 2 signals 17.3 and 2.6, 256 signals 32 and 3.0; 4096 x
// 16384, 4 signals 35.4 and 3.9).
double gram_gain_us(const mp_ctx* c, int64_t B) {
  const double elems = static_cast<double>(c->m) * static_cast<double>(c->ld);
  return 9.0 + 0.33e-6 * elems + 3.3e-9 * elems * static_cast<double>(B);
}

// The Gram columns of all atoms, made once per context, with one signal's c~
// and flags behind them; false where they are not there.
bool make_gram_full(mp_ctx* c, hipStream_t s) {
  if (c->gram_full || c->gram_full_tried) return c->gram_full != nullptr;
  c->gram_full_tried = true;
  const int64_t stride = mp::gram_stride(mp::gram_shape(c->ld, c->m, 4));
  const size_t bytes = sizeof(float) * static_cast<size_t>(stride) * static_cast<size_t>(c->m);
  const size_t one = sizeof(float) * static_cast<size_t>(stride);
  if (!room_for(bytes + one) || hipMalloc(&c->gram_full, bytes + one + 2 * sizeof(int)) != hipSuccess) {
    (void)hipGetLastError();
    c->gram_full = nullptr;
    return false;
  }
  c->gram_full_mp = stride;
  c->gram_sc = c->gram_full + static_cast<size_t>(stride) * static_cast<size_t>(c->m);
  c->gram_sagain = reinterpret_cast<int*>(c->gram_sc + stride);
  if (hipMemsetAsync(stride != c->m ? c->gram_full : c->gram_sc, 0,
                     stride != c->m ? bytes + one : one, s) != hipSuccess ||
      mp::launch_gram_full(c->psi32, c->ld, c->m, c->gram_full, stride, c->num_cus, s) !=
          hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(c->gram_full);
    c->gram_full = nullptr;
    return false;
  }
  return true;
}

// Whether a batched decode of at most tmax steps takes the carried
// correlations, with the buffers for B signals if so.  The Gram columns are
// made where a decode of N / 16 steps (of the cap, if that is lower) would pay for
// them, or once the rounds of this context's decodes have cost as much more as
// they would have saved (gram_owed): a context that decodes a few short batches
// never makes columns that cost more than all of them.
bool ensure_gram_batch(mp_ctx* c, int64_t B, long long tmax, hipStream_t s) {
  if (!gram_full_suits(c)) return false;
  const double likely = std::min<double>(static_cast<double>(tmax), std::max<double>(2.0, c->n / 16.0));
  if (!c->gram_full && gram_full_us(c) > std::max(gram_gain_us(c, B) * likely, c->gram_owed))
    return false;
  if (!make_gram_full(c, s)) return false;
  if (B <= c->gram_bcap) return true;
  free_gram_batch(c);
  const size_t b = static_cast<size_t>(B);
  const size_t cbytes = sizeof(float) * static_cast<size_t>(c->gram_full_mp) * b;
  if (!room_for(cbytes + sizeof(float) * static_cast<size_t>(c->ld) * b) ||
      hipMalloc(&c->gram_bc, cbytes) != hipSuccess ||
      hipMalloc(&c->gram_br, sizeof(float) * static_cast<size_t>(c->ld) * b) != hipSuccess ||
      hipMalloc(&c->gram_bst, sizeof(mp::DevState) * b) != hipSuccess ||
      hipMalloc(&c->gram_again, 2 * sizeof(int)) != hipSuccess ||
      hipMalloc(&c->gram_btcap, sizeof(long long) * b) != hipSuccess ||
      hipHostMalloc(&c->gram_hbst, sizeof(mp::DevState) * b, hipHostMallocDefault) !=
          hipSuccess ||
      hipHostMalloc(&c->gram_hagain, 4 * sizeof(int), hipHostMallocDefault) != hipSuccess ||
      hipMemsetAsync(c->gram_bc, 0, cbytes, s) != hipSuccess) {
    (void)hipGetLastError();
    free_gram_batch(c);
    return false;
  }
  c->gram_bcap = B;
  return true;
}

// One signal of a small dictionary on every atom's Gram column (as the batched
// decode holds them, made by the first decode): no passes, so a decode is the
// products Psi^T y, then the steps in one workgroup, and again each time the
// carried correlations have lost too many digits.  `used` false: not taken, or
// handed on after t0 steps, which stand.
//
// The one launch that holds the dictionary in LDS (k_f32_small) costs 30 us
// and 5 a step (its exchange between workgroups), this 43 and 2.4, so low caps
// stay there.  Decodes of K atoms under a cap of 20 K, to ||r|| of 1e-6 ||y|| and of
// 0.04 ||y||, here and in that launch, us: M = 192, K = 4: 92 and 150, 51 and 55; M =
// 1024, K = 4: 86 and 93, 61 and 55; K = 5: 95 and 114, 59 and 60; K = 8: 138 and
// 206, 70 and 84.  (A decode that takes a few steps of a large cap is slower here:
// N = 256, M = 1024, 1 step 45 and 36, 5 steps 63 and 56, 12 steps 78 and 90.)  The
// Gram columns are made where they cost at most 0.065 us a step of the cap (4 us
// at N = 256, M = 1024).
mp_status solve_small_full(mp_ctx* c, float* r_work, float* x, float* r, const mp_opts* opts,
                           const mp_trace& tr, hipStream_t s, bool& used, long long& t0) {
  used = false;
  const long long least = c->m <= 512 ? 64 : 96;
  const mp::GramShape sh = mp::gram_shape(c->ld, c->m, 4);
  if (opts->max_iters < least || sh.threads * sh.per_thread > 8192 || !gram_full_suits(c) ||
      (!c->gram_full && gram_full_us(c) > 0.065 * static_cast<double>(opts->max_iters)) ||
      !make_gram_full(c, s))
    return MP_OK;
  const mp::GramBounds bounds = mp::gram_bounds_full(c->n, c->max_norm);
  const mp::GramBatch b{c->psi32, c->ld, c->n, c->m, c->gram_full_mp, c->gram_full, c->gram_sc,
                        r_work, x, c->m, c->st};
  const bool timed = c->profiling;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  // every round takes a step (or gives up); two are all that most decodes need,
  // and one brings ||r|| down by three decades
  int rounds = opts->eps >= 1e-3 ? 1 : 2;
  const long long most = step_cap(opts) + 1;
  long long issued = 0;
  do {
    for (int k = 0; k < rounds && issued < most; ++k, ++issued)
      HIP_TRY(c, mp::launch_gram_bround(b, sh, bounds, 1, c->num_cus, issued, c->gram_sagain,
                                        true, tr, s));
    if (timed) HIP_TRY(c, hipEventRecord(c->ev[1], s));
    if (r) HIP_TRY(c, mp::launch_copy_selected(r_work, c->ld, c->n, c->st, r, s));
    HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    rounds = 2;
  } while (!c->h_st->done && issued < most);
  used = c->h_st->done && !c->h_st->pad[0];
  c->carried_steps = c->h_st->t;
  if (!used) {
    t0 = c->h_st->t;
    HIP_TRY(c, mp::launch_resume<float>(c->st, r_work, c->ld, 0, s));
    return MP_OK;
  }
  if (timed) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = c->h_st->t > 0 ? c->h_st->t : 1;
    }
  }
  return MP_OK;
}

mp_status solve_carried(mp_ctx* c, const float* y, float* x, float* r, const mp_opts* opts,
                        mp_result* res, const mp_trace& tr, hipStream_t s, const CarriedBufs& b,
                        bool allow_one_launch, bool allow_gram) {
  const bool async = (opts->flags & MP_SOLVE_ASYNC) != 0;
  long long t0 = 0;  // steps taken on carried correlations before another form goes on
  HIP_TRY(c, mp::launch_init(y, c->n, c->ld, x, c->m, b.r_work, b.st, opts->eps,
                             step_cap(opts), s));
  if (allow_one_launch && c->storage == MP_F32 && c->small.grid > 0 &&
      !(opts->flags & MP_SOLVE_STEP_LAUNCHES)) {
    // (MP_SMALL_SPIN_LIMIT limits the waits of the one launch, which only it has)
    if (allow_gram && !async && opts->max_iters > 0 && !getenv("MP_SMALL_SPIN_LIMIT")) {
      bool used = false;
      const mp_status fs = solve_small_full(c, b.r_work, x, r, opts, tr, s, used, t0);
      if (fs != MP_OK) return fs;
      if (used) {
        const mp_status rs = finish_result(c, res);
        if (rs == MP_OK && res) res->persistent = 1;
        return rs;
      }
    }
    // the whole decode in one launch, every share of the dictionary in LDS:
    // a new tag epoch for every decode (never 0 mod the epoch range: the
    // zeroed words match no step); when it wraps, clear the words so that
    // none left from a decode that many decodes ago can match
    c->small_epoch = c->small_epoch % (mp::small_epoch_mod() - 1) + 1;
    if (c->small_epoch == 1)
      HIP_TRY(c, hipMemsetAsync(c->small_slots, 0,
                                sizeof(unsigned long long) * mp::small_slot_words(), s));
    const bool timed = c->profiling && !async;
    if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
    HIP_TRY(c, mp::launch_f32_small(c->psi32, c->ld, c->n, c->m, b.r_work, c->small,
                                    c->small_slots, c->small_epoch, t0, step_cap(opts), x, b.st, tr,
                                    s));
    if (timed) HIP_TRY(c, hipEventRecord(c->ev[1], s));
    if (r) HIP_TRY(c, mp::launch_copy_selected(b.r_work, c->ld, c->n, b.st, r, s));
    if (async) return enqueue_result(c, b.st, s, 1);
    HIP_TRY(c, hipMemcpyAsync(c->h_st, b.st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    if (c->profiling) {
      // the launch time per step it took (each with a pass)
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
        c->prof_ms = ms;
        c->prof_launches = c->h_st->t > t0 ? c->h_st->t - t0 : 1;
      }
    }
    const mp_status fs = finish_result(c, res);
    if (fs == MP_OK && res) res->persistent = 1;
    return fs;
  }
  // the reduced-precision forms keep the FP32 columns too: with all 8
  // candidates re-scored (the default) the atom they select is the FP32
  // form's, which the carried correlations give without a pass per step
  // (N = 8192, M = 32768, K = 256: BF16 8.1 ms from 89.0, FP8 7.4 from 42.1)
  if (allow_gram && (c->storage == MP_F32 || c->rescore_k == mp::kLpTopK) && !async &&
      !(opts->flags & MP_SOLVE_STEP_LAUNCHES) && cap_pays(c->storage, opts->max_iters) &&
      ensure_gram(c, s)) {
    bool gave_up = false;
    const mp_status gs = solve_gram<float>(c, c->psi32, b.r_work, x, opts, tr, s, gave_up, t0);
    if (gs != MP_OK) return gs;
    if (!gave_up) {
      if (r) HIP_TRY(c, mp::launch_copy_selected(b.r_work, c->ld, c->n, b.st, r, s));
      HIP_TRY(c, hipMemcpyAsync(c->h_st, b.st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipStreamSynchronize(s));
      return finish_result(c, res);
    }
  }
  long long k = t0;
  const long long T = step_cap(opts);
  auto step = [&](hipEvent_t e0, hipEvent_t e1) {
    hipError_t e;
    if (e0 && (e = hipEventRecord(e0, s)) != hipSuccess) return e;
    if (c->storage == MP_F32)
      e = mp::launch_mp_step_f32(c->psi32, c->ld, c->n, c->m, b.r_work, c->geom, b.keys, b.bal,
                                 k, t0, T, x, b.st, tr, s);
    else
      e = mp::launch_mp_step_lp(c->storage, c->psiq, c->scales, c->psi32, c->ld, c->n, c->m,
                                b.r_work, c->geom, c->rescore_k, b.keys, k, t0, T, x, b.st, tr,
                                s);
    ++k;
    if (e != hipSuccess) return e;
    if (e1 && (e = hipEventRecord(e1, s)) != hipSuccess) return e;
    return hipSuccess;
  };
  if (async) {
    const long long launches = T > 0 ? T + 1 : 0;
    for (long long j = 0; j < launches; ++j) {
      const hipError_t e = step(nullptr, nullptr);
      if (e != hipSuccess) return fail(c, MP_EDEVICE, std::string("launch: ") + hipGetErrorString(e));
    }
    if (r) HIP_TRY(c, mp::launch_copy_selected(b.r_work, c->ld, c->n, b.st, r, s));
    return enqueue_result(c, b.st, s, 0);
  }
  const mp_status st = run_iterations(c, T > 0 ? T - t0 + 1 : 0, s, true, step,
                                      /*known_running=*/true, b.st, t0);
  if (st != MP_OK) return st;
  if (r) HIP_TRY(c, mp::launch_copy_selected(b.r_work, c->ld, c->n, b.st, r, s));
  HIP_TRY(c, hipMemcpyAsync(c->h_st, b.st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  const mp_status fs = finish_result(c, res);
  if (fs == MP_OK && res) res->persistent = 0;
  return fs;
}

// Final state of a single-signal decode into `res`, with the internal stop
// reasons mapped to errors.
mp_status finish_result(mp_ctx* c, mp_result* res) {
  const mp::DevState& d = *c->h_st;
  if (d.fail)
    return fail(c, MP_EDEVICE, "a wait of the persistent one-bit decode gave up");
  if (d.reason == mp::kStopNonFinite) return fail(c, MP_ENONFINITE, "y holds NaN or Inf");
  if (d.reason == mp::kStopInternal)
    return fail(c, MP_EDEVICE,
                "internal error: a selected index fell outside the dictionary");
  if (res) {
    res->iters = d.t;
    res->yy = d.yy;
    res->rr = d.rr;
    res->stop_reason = d.reason;
    res->persistent = 0;
  }
  return MP_OK;
}

// The batched decode on carried correlations.  `handed_on`: the signals that
// need the rounds of products to go on from the steps they have taken.
mp_status solve_gram_batch(mp_ctx* c, const float* Y, int64_t ldy, int64_t B, float* X,
                           int64_t ldx, const mp_opts* opts, const int64_t* max_iters_b,
                           const mp_trace& tr, hipStream_t s, int64_t& handed_on) {
  handed_on = 0;
  const mp::GramShape sh = mp::gram_shape(c->ld, c->m, 4);
  const mp::GramBounds bounds = mp::gram_bounds_full(c->n, c->max_norm);
  if (max_iters_b)
    HIP_TRY(c, hipMemcpyAsync(c->gram_btcap, max_iters_b, sizeof(long long) * B,
                              hipMemcpyHostToDevice, s));
  const bool timed = c->profiling;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  HIP_TRY(c, mp::launch_gram_binit(Y, ldy, c->n, c->ld, X, ldx, c->m, c->gram_br, c->gram_bst,
                                   max_iters_b ? c->gram_btcap : nullptr, opts->max_iters,
                                   opts->eps, static_cast<int>(B), s));
  const mp::GramBatch b{c->psi32, c->ld, c->n, c->m, c->gram_full_mp, c->gram_full, c->gram_bc,
                        c->gram_br, X, ldx, c->gram_bst};
  // rounds until no signal goes on, two in flight; every round takes each
  // running signal at least one step on (or it gives up)
  long long issued = 0, seen = 0;
  bool over = false;
  while (!over) {
    while (issued - seen < 2) {
      HIP_TRY(c, mp::launch_gram_bround(b, sh, bounds, static_cast<int>(B), c->num_cus, issued,
                                        c->gram_again, false, tr, s));
      const int k = static_cast<int>(issued & 1);
      HIP_TRY(c, hipMemcpyAsync(c->gram_hagain + 2 * k, c->gram_again, 2 * sizeof(int),
                                hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipEventRecord(c->done_ev[k], s));
      ++issued;
    }
    const int k = static_cast<int>(seen & 1);
    HIP_TRY(c, hipEventSynchronize(c->done_ev[k]));
    over = c->gram_hagain[2 * k + k] == 0;
    ++seen;
  }
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[1], s));
  HIP_TRY(c, hipMemcpyAsync(c->gram_hbst, c->gram_bst, sizeof(mp::DevState) * B,
                            hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  long long most = 0;
  for (int64_t j = 0; j < B; ++j) {
    handed_on += c->gram_hbst[j].pad[0] != 0;
    most = std::max(most, c->gram_hbst[j].t);
  }
  c->carried_steps = most;
  if (timed) {
    // the decode's time on the device over the steps of its longest signal
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = most > 0 ? most : 1;
    }
  }
  return MP_OK;
}

// The problems, Gram columns and buffers of the ragged decode on carried
// correlations, made with the context.  Gram columns per problem:
// max(64, n / 4) and five passes' (a cache that starts over costs more passes:
// 17 rounds against 11 for 512 problems); in all at most the dictionaries'
// bytes and 128 MiB (many tiny problems, whose rounding up would dominate, keep the
// persistent launch, as do problems past the steps kernel's limits, and a
// context whose memory does not reach).  So do FP32 sets of dictionaries that
// the launch's passes take in a few microseconds a step, several short columns
// side by side in a wave (whole decodes, carried and that launch with its
// default and its best shape, us: 64 x 256, 16 problems 233, 133, 118; 64 x
// 2048 267, 240, 179; 128 x 512 320, 281, 231; 128 x 1024 335, 475, 333, 128
// problems 540, 912, 649; 192 x 768 415, 937, 712; BF16, 64 x 256 241, 280, 253).
void make_gram_ragged(mp_ctx* c, hipStream_t s) {
  if (!(c->max_norm > 0.99) || !(c->max_norm < 1.01) || c->r_count > 65535) return;
  const size_t count = static_cast<size_t>(c->r_count);
  const int64_t max_m = *std::max_element(c->r_m.begin(), c->r_m.end());
  if (max_m > 32768) return;
  int64_t lds = 0, work = 0, gcols = 0, maps = 0, tiles = 0, dict = 0;
  std::vector<int64_t> stride(count), slots(count);
  bool quick = c->storage == MP_F32;  // passes of a few microseconds
  for (size_t i = 0; i < count; ++i) {
    const int64_t ld = round_up(c->r_n[i], kLdAlign), m = c->r_m[i];
    quick = quick && ld <= 128 && m * (ld / 64) * (ld / 64) <= 2048;
    stride[i] = mp::gram_ragged_stride(c->r_max_ld, max_m, m);
    slots[i] = round_up(
        std::min<int64_t>(std::max<int64_t>(64, c->r_n[i] / 4) + 4 * mp::kGramReq, m) +
            mp::kGramReq, 16);
    lds = std::max(lds, 8 * ld + 2 * m);
    work += stride[i] + (mp::kGramReq + 2) * ld;
    gcols += slots[i] * stride[i];
    maps += round_up(m, 8);
    tiles += (m + mp::kGramTile - 1) / mp::kGramTile;
    dict += ld * m;
  }
  if (quick || lds > 150 * 1024 || gcols > dict + (int64_t{1} << 25)) return;
  const int per = mp::gram_ragged_groups(tiles, c->num_cus);
  std::vector<mp::GramGroup> groups;
  for (int id : c->r_order) {
    const int64_t t = (c->r_m[id] + mp::kGramTile - 1) / mp::kGramTile;
    for (int64_t k = 0; k * per < t; ++k)
      groups.push_back(mp::GramGroup{id, static_cast<int>(k)});
  }
  // one allocation, cut into pieces on 256-byte lines
  size_t total = 0;
  auto piece = [&total](size_t bytes) {
    const size_t at = total;
    total += (bytes + 255) / 256 * 256;
    return at;
  };
  const size_t o_work = piece(sizeof(float) * work), o_g = piece(sizeof(float) * gcols);
  const size_t zeroed = total;  // entries past a problem's atoms stay zero
  const size_t o_probs = piece(sizeof(mp::GramProb<float>) * count),
               o_bounds = piece(sizeof(mp::GramBounds) * count),
               o_order = piece(sizeof(int) * count),
               o_groups = piece(sizeof(mp::GramGroup) * groups.size()),
               o_map = piece(sizeof(uint16_t) * maps),
               o_ctl = piece(sizeof(mp::GramCtl) * count),
               o_st = piece(sizeof(mp::DevState) * count), o_again = piece(2 * sizeof(int));
  auto make = [&]() {
    if (!room_for(total) || hipMalloc(&c->gram_rmem, total) != hipSuccess) return false;
    if (hipHostMalloc(&c->gram_hrmem, sizeof(mp::DevState) * count + 4 * sizeof(int),
                      hipHostMallocDefault) != hipSuccess)
      return false;
    for (hipEvent_t& e : c->gram_rev)
      if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
        e = nullptr;
        return false;
      }
    char* mem = static_cast<char*>(c->gram_rmem);
    c->gram_rprobs = mem + o_probs;
    c->gram_rbounds = mem + o_bounds;
    c->gram_rorder = reinterpret_cast<int*>(mem + o_order);
    c->gram_rgroups = mem + o_groups;
    c->gram_rst = reinterpret_cast<mp::DevState*>(mem + o_st);
    c->gram_ragain = reinterpret_cast<int*>(mem + o_again);
    c->gram_hrst = static_cast<mp::DevState*>(c->gram_hrmem);
    c->gram_hragain = reinterpret_cast<int*>(c->gram_hrst + count);
    std::vector<mp::GramProb<float>> probs(count);
    std::vector<mp::GramBounds> bounds(count);
    float *w = reinterpret_cast<float*>(mem + o_work), *g = reinterpret_cast<float*>(mem + o_g);
    uint16_t* map = reinterpret_cast<uint16_t*>(mem + o_map);
    for (size_t i = 0; i < count; ++i) {
      const int64_t ld = round_up(c->r_n[i], kLdAlign);
      mp::GramProb<float>& p = probs[i];
      p.psi = c->r_psi32 + c->r_psi_off[i];
      p.ld = ld;
      p.n = c->r_n[i];
      p.m = c->r_m[i];
      p.mp = stride[i];
      p.c = w;
      p.rhs = w + stride[i];
      p.r = p.rhs + (mp::kGramReq + 1) * ld;
      w += stride[i] + (mp::kGramReq + 2) * ld;
      p.g = g;
      g += slots[i] * stride[i];
      p.slots = static_cast<int>(slots[i]);
      p.map = map;
      map += round_up(p.m, 8);
      p.x = nullptr;
      p.st = c->gram_rst + i;
      p.ctl = reinterpret_cast<mp::GramCtl*>(mem + o_ctl) + i;
      bounds[i] = c->storage == MP_BF16 ? mp::gram_bounds(p.n, c->max_norm, false)
                                        : mp::gram_bounds_one(p.n, c->max_norm);
    }
    return hipMemsetAsync(mem, 0, zeroed, s) == hipSuccess &&
           hipMemcpyAsync(c->gram_rprobs, probs.data(), sizeof(probs[0]) * count,
                          hipMemcpyHostToDevice, s) == hipSuccess &&
           hipMemcpyAsync(c->gram_rbounds, bounds.data(), sizeof(bounds[0]) * count,
                          hipMemcpyHostToDevice, s) == hipSuccess &&
           hipMemcpyAsync(c->gram_rorder, c->r_order.data(), sizeof(int) * count,
                          hipMemcpyHostToDevice, s) == hipSuccess &&
           hipMemcpyAsync(c->gram_rgroups, groups.data(), sizeof(groups[0]) * groups.size(),
                          hipMemcpyHostToDevice, s) == hipSuccess &&
           hipStreamSynchronize(s) == hipSuccess;
  };
  if (!make()) {
    (void)hipGetLastError();
    free_gram_ragged(c);
    return;
  }
  c->gram_rngroups = static_cast<int>(groups.size());
  c->gram_rsplit = mp::kGramRaggedWaves / per;
  c->gram_rlds = lds;
  c->gram_rsmall = max_m <= 4096 && c->r_max_ld <= 4096;
}

// The ragged decode on carried correlations.  `gave_up`: some problem needs
// the persistent launch to go on from the steps it has taken.
mp_status solve_gram_ragged(mp_ctx* c, const float* Y, float* X, const mp_opts* opts,
                            float* R, const long long* caps, const mp_trace& tr, hipStream_t s,
                            bool& gave_up) {
  gave_up = false;
  const mp::GramRagged g{static_cast<const mp::GramProb<float>*>(c->gram_rprobs),
                         c->r_inst,
                         static_cast<const mp::GramBounds*>(c->gram_rbounds),
                         c->gram_rorder,
                         static_cast<const mp::GramGroup*>(c->gram_rgroups),
                         c->gram_ragain,
                         static_cast<int>(c->r_count),
                         c->gram_rngroups,
                         c->gram_rsplit,
                         c->r_max_ld,
                         c->gram_rlds,
                         c->gram_rsmall,
                         c->storage == MP_F32};
  const bool timed = c->profiling;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  HIP_TRY(c, mp::launch_gram_rinit(g, Y, X, caps, opts->max_iters, opts->eps, s));
  long long issued = 0, seen = 0;
  bool over = false;
  while (!over) {
    while (issued - seen < 2) {
      HIP_TRY(c, mp::launch_gram_rround(g, X, issued, tr, s));
      const int k = static_cast<int>(issued & 1);
      HIP_TRY(c, hipMemcpyAsync(c->gram_hragain + 2 * k, c->gram_ragain, 2 * sizeof(int),
                                hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipEventRecord(c->gram_rev[k], s));
      ++issued;
    }
    const int k = static_cast<int>(seen & 1);
    HIP_TRY(c, hipEventSynchronize(c->gram_rev[k]));
    over = c->gram_hragain[2 * k + k] == 0;
    ++seen;
  }
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[1], s));
  if (R) HIP_TRY(c, mp::launch_gram_rcopy(g.probs, c->r_inst, g.count, R, s));
  HIP_TRY(c, hipMemcpyAsync(c->gram_hrst, c->gram_rst, sizeof(mp::DevState) * c->r_count,
                            hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  for (int64_t i = 0; i < c->r_count; ++i) {
    gave_up |= c->gram_hrst[i].pad[0] != 0;
    c->carried_steps = std::max<int64_t>(c->carried_steps, c->gram_hrst[i].t);
  }
  if (timed) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = 1;
    }
  }
  return MP_OK;
}

// Results of a batched decode: one entry per signal and the call's status.
template <class State>
mp_status batched_results(mp_ctx* c, const State* slots, int64_t B, mp_result* res,
                          const char* bad_y = "a column of Y holds NaN or Inf") {
  bool nonfinite = false, internal = false;
  for (int64_t b = 0; b < B; ++b) {
    const State& d = slots[b];
    nonfinite |= d.reason == mp::kStopNonFinite;
    internal |= d.reason == mp::kStopInternal;
    if (res) {
      res[b].iters = d.t;
      res[b].yy = d.yy;
      res[b].rr = d.rr;
      res[b].stop_reason = d.reason;
      res[b].persistent = 0;
    }
  }
  if (internal)
    return fail(c, MP_EDEVICE, "internal error: a selected index fell outside the dictionary");
  if (nonfinite) return fail(c, MP_ENONFINITE, bad_y);
  return MP_OK;
}

}  // namespace

extern "C" {

const char* mp_status_str(mp_status s) {
  switch (s) {
    case MP_OK: return "MP_OK";
    case MP_EINVAL: return "MP_EINVAL";
    case MP_ENOTNORM: return "MP_ENOTNORM";
    case MP_ENONFINITE: return "MP_ENONFINITE";
    case MP_ENOMEM: return "MP_ENOMEM";
    case MP_EDEVICE: return "MP_EDEVICE";
    case MP_EUNSUPPORTED: return "MP_EUNSUPPORTED";
  }
  return "MP_UNKNOWN";
}

const char* mp_last_error(const mp_ctx* ctx) {
  return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

mp_status mp_create(mp_ctx** out, const float* psi, int64_t n, int64_t m, int64_t ld,
                    mp_dtype storage, uint32_t flags, void* stream) {
  g_create_error.clear();
  if (!out) return fail(nullptr, MP_EINVAL, "out is NULL");
  *out = nullptr;
  if (!psi) return fail(nullptr, MP_EINVAL, "psi is NULL");
  if (n < 1 || m < 1) return fail(nullptr, MP_EINVAL, "n and m must be >= 1");
  if (ld < n) return fail(nullptr, MP_EINVAL, "ld must be >= n");
  if (n > kMaxN) return fail(nullptr, MP_EINVAL, "n exceeds 16384");
  if (m >= (int64_t{1} << 31)) return fail(nullptr, MP_EINVAL, "m must be < 2^31");
  if (flags & ~MP_SKIP_NORM_CHECK) return fail(nullptr, MP_EINVAL, "unknown flags");
  if (storage == MP_F64)
    return fail(nullptr, MP_EINVAL, "an FP64 dictionary is taken by mp_create_f64");
  if (storage == MP_SIGN1)
    return fail(nullptr, MP_EINVAL, "a sign-bit dictionary is taken by mp_create_signs");
  if (storage != MP_F32 && storage != MP_BF16 && storage != MP_FP8_E4M3)
    return fail(nullptr, MP_EINVAL, "unknown storage type");
  int dev = 0;
  hipDeviceProp_t prop;
  if (mp_status ds = open_device(dev, prop); ds != MP_OK) return ds;
  hipStream_t s = static_cast<hipStream_t>(stream);

  mp_ctx* c = new mp_ctx();
  c->device = dev;
  c->num_cus = prop.multiProcessorCount;
  c->n = n;
  c->m = m;
  c->ld = round_up(n, kLdAlign);
  c->storage = storage;
  c->geom = mp::corr_f32_geometry(m, c->num_cus);

  auto bail = [&](mp_status st, const std::string& msg) {
    free_ctx(c);
    return fail(nullptr, st, msg);
  };
  const size_t psi_bytes = static_cast<size_t>(c->ld) * static_cast<size_t>(m) * sizeof(float);
  if (hipMalloc(&c->psi32, psi_bytes) != hipSuccess) return bail(MP_ENOMEM, "dictionary copy");
  // r and the published keys in two halves (the reduced-precision decode
  // alternates between them by launch parity)
  if (hipMalloc(&c->r_work, 2 * c->ld * sizeof(float)) != hipSuccess)
    return bail(MP_ENOMEM, "r");
  if (hipMalloc(&c->st, sizeof(mp::DevState)) != hipSuccess) return bail(MP_ENOMEM, "state");
  if (c->geom.grid * mp::kLpTopK > 2 * 1024)
    return bail(MP_EUNSUPPORTED, "more correlation workgroups than the key slots hold");
  const size_t nkeys = 2 * static_cast<size_t>(c->geom.grid) * mp::kLpTopK;
  if (hipMalloc(&c->partials, sizeof(uint64_t) * nkeys) != hipSuccess)
    return bail(MP_ENOMEM, "partials");
  if (hipMalloc(&c->bal, sizeof(mp::BalState)) != hipSuccess) return bail(MP_ENOMEM, "shares");
  if (!make_host_state(c)) return bail(MP_ENOMEM, "pinned state");
  // the one-launch decode of small FP32 dictionaries (every share in LDS)
  if (storage == MP_F32) {
    c->small = mp::small_geometry(c->ld, m, c->num_cus);
    if (c->small.grid > 0) {
      const size_t bytes = sizeof(unsigned long long) * mp::small_slot_words();
      if (hipMalloc(&c->small_slots, bytes) != hipSuccess) return bail(MP_ENOMEM, "step records");
      if (hipMemsetAsync(c->small_slots, 0, bytes, s) != hipSuccess)
        return bail(MP_EDEVICE, "step records");
    }
  }
  // set-up of mp_solve_noalloc's scratch on this device (the entry point
  // looks it up itself if this fails)
  {
    void* scratch_ptr = nullptr;
    (void)mp::noalloc_scratch(dev, &scratch_ptr);
  }

  hipError_t e = hipMemsetAsync(c->psi32, 0, psi_bytes, s);
  if (e == hipSuccess)
    e = hipMemcpy2DAsync(c->psi32, c->ld * sizeof(float), psi, ld * sizeof(float),
                         n * sizeof(float), m, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = hipMemsetAsync(c->r_work, 0, 2 * c->ld * sizeof(float), s);
  if (e == hipSuccess) e = hipMemsetAsync(c->partials, 0, sizeof(uint64_t) * nkeys, s);
  if (e == hipSuccess) e = hipMemsetAsync(c->bal, 0, sizeof(mp::BalState), s);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("copy: ") + hipGetErrorString(e));

  // Column norms in FP64 (eq. 4): finiteness always, unit norm unless skipped.
  double* d_norm2 = nullptr;
  if (hipMalloc(&d_norm2, sizeof(double) * m) != hipSuccess) return bail(MP_ENOMEM, "norms");
  std::vector<double> norm2(static_cast<size_t>(m));
  e = mp::launch_norms(c->psi32, c->ld, n, m, d_norm2, nullptr, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(norm2.data(), d_norm2, sizeof(double) * m, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(d_norm2);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("norms: ") + hipGetErrorString(e));
  {
    std::string msg;
    const mp_status ns = check_norms(norm2, flags, msg);
    if (ns != MP_OK) return bail(ns, msg);
    c->max_norm = largest_norm(norm2);
  }
  // Reduced-precision copy the correlation pass streams (same padded layout).
  if (storage == MP_BF16 || storage == MP_FP8_E4M3) {
    const size_t esize = storage == MP_BF16 ? 2 : 1;
    const size_t qbytes = static_cast<size_t>(c->ld) * static_cast<size_t>(m) * esize;
    if (hipMalloc(&c->psiq, qbytes) != hipSuccess) return bail(MP_ENOMEM, "reduced copy");
    if (storage == MP_BF16) {
      e = mp::launch_quant_bf16(c->psi32, c->ld, m, static_cast<uint16_t*>(c->psiq), s);
    } else {
      if (hipMalloc(&c->scales, sizeof(float) * m) != hipSuccess)
        return bail(MP_ENOMEM, "scales");
      e = mp::launch_quant_fp8(c->psi32, c->ld, m, static_cast<uint8_t*>(c->psiq), c->scales, s);
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return bail(MP_EDEVICE, std::string("quantise: ") + hipGetErrorString(e));
  }
  *out = c;
  return MP_OK;
}

void mp_destroy(mp_ctx* ctx) { free_ctx(ctx); }

mp_status mp_set_profiling(mp_ctx* ctx, int every) {
  if (!ctx) return MP_EINVAL;
  if (every < 0) return fail(ctx, MP_EINVAL, "every must be >= 0");
  if (every > 0 && ctx->ev.empty()) {
    ctx->ev.resize(2 * 2 * kMaxChunk, nullptr);
    for (hipEvent_t& e : ctx->ev) HIP_TRY(ctx, hipEventCreate(&e));
  }
  ctx->profiling = every > 0;
  ctx->prof_every = every > 0 ? every : 1;
  return MP_OK;
}

mp_status mp_kernel_time(const mp_ctx* ctx, double* avg_ms, int64_t* launches) {
  if (!ctx || !avg_ms || !launches) return MP_EINVAL;
  *launches = ctx->prof_launches;
  *avg_ms = ctx->prof_launches ? ctx->prof_ms / static_cast<double>(ctx->prof_launches) : 0.0;
  return MP_OK;
}

mp_status mp_set_carried(mp_ctx* ctx, int on) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  mp_ctx* c = ctx;
  if (on != 0 && on != 1) return fail(c, MP_EINVAL, "on must be 0 or 1");
  if (mp_status ps = check_not_pending(c); ps != MP_OK) return ps;
  HIP_TRY(c, hipSetDevice(c->device));
  if (c->carried_on == (on != 0)) return MP_OK;
  c->carried_on = on != 0;
  if (on) {
    if (c->ragged) make_gram_ragged(c, nullptr);
    return MP_OK;
  }
  free_gram(c);
  free_sign_gram(c);
  free_omp_carry(c);
  free_gram_batch(c);
  free_gram_ragged(c);
  (void)hipFree(c->gram_full);
  c->gram_full = nullptr;
  c->gram_tried = c->gram_full_tried = false;
  return MP_OK;
}

mp_status mp_carried_steps(const mp_ctx* ctx, int64_t* steps) {
  if (!ctx || !steps) return MP_EINVAL;
  *steps = ctx->carried_steps;
  return MP_OK;
}

mp_status mp_get_storage(const mp_ctx* ctx, void* codes, float* scales, void* stream) {
  if (!ctx || !codes) return MP_EINVAL;
  mp_ctx* c = const_cast<mp_ctx*>(ctx);
  if (c->ragged) return fail(c, MP_EINVAL, "not available for a ragged context");
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (c->storage == MP_F64) {
    HIP_TRY(c, hipMemcpy2DAsync(codes, c->n * sizeof(double), c->psi64, c->ld * sizeof(double),
                                c->n * sizeof(double), c->m, hipMemcpyDeviceToDevice, s));
  } else if (c->storage == MP_SIGN1) {
    const size_t w = static_cast<size_t>((c->n + 31) / 32) * sizeof(uint32_t);
    HIP_TRY(c, hipMemcpy2DAsync(codes, w, c->psis, c->sign_ws * sizeof(uint32_t), w, c->m,
                                hipMemcpyDeviceToDevice, s));
  } else if (c->storage == MP_F32) {
    HIP_TRY(c, hipMemcpy2DAsync(codes, c->n * sizeof(float), c->psi32, c->ld * sizeof(float),
                                c->n * sizeof(float), c->m, hipMemcpyDeviceToDevice, s));
  } else {
    const size_t esize = c->storage == MP_BF16 ? 2 : 1;
    HIP_TRY(c, hipMemcpy2DAsync(codes, c->n * esize, c->psiq, c->ld * esize, c->n * esize, c->m,
                                hipMemcpyDeviceToDevice, s));
    if (c->storage == MP_FP8_E4M3 && scales)
      HIP_TRY(c, hipMemcpyAsync(scales, c->scales, sizeof(float) * c->m, hipMemcpyDeviceToDevice,
                                s));
  }
  HIP_TRY(c, hipStreamSynchronize(s));
  return MP_OK;
}

// The buffers of the one-bit decode in batches of steps; false where it does
// not apply (more rows of r per workgroup of the stepping form than a replay
// holds: M below N / 16) or the memory is not there.
static bool ensure_sign_gram(mp_ctx* c) {
  mp::SignGram& b = c->sign_gram;
  if (!c->carried_on) return false;
  if (b.tried) return b.carry != nullptr;
  const size_t grid = static_cast<size_t>(c->geom.grid);
  b.tried = true;
  if ((c->ld + c->geom.grid - 1) / c->geom.grid > 64 * mp::kSignRows) return false;
  const size_t act = mp::kSignActive;
  if (!room_for(sizeof(short) * act * static_cast<size_t>(mp::sign_gram_stride(c->m))) ||
      hipMalloc(&b.carry, sizeof(mp::SignCarry)) != hipSuccess ||
      hipMalloc(&b.pos, sizeof(unsigned short) * static_cast<size_t>(c->m)) != hipSuccess ||
      hipMalloc(&b.g, sizeof(short) * act * static_cast<size_t>(mp::sign_gram_stride(c->m))) !=
          hipSuccess ||
      hipMalloc(&b.h, sizeof(short) * act * act) != hipSuccess ||
      hipMalloc(&b.parts, sizeof(double) * mp::kSignSteps * grid) != hipSuccess) {
    (void)hipGetLastError();
    free_sign_gram(c);
    b.tried = true;
    return false;
  }
  return true;
}

// The one-bit decode in batches of steps (k_sign_gram.hip), in chunks of
// rounds: one round at first, which is all that a short decode needs, then up
// to kRounds with two chunks in flight (a readback leaves the device idle for
// 10 us, a round after the stop costs 18).  `over`: it reached its stop.
// Otherwise the rounds brought too few steps (more atoms near the largest
// |c| than a round can add and name, in an order that names the wrong ones; a
// round costs about 60 us, a step of the persistent launch 7 to 10): t0 steps
// stand, and c64, r64, x~ and the state are as of them.  The state as last seen
// is left in *c->h_st; r (not null) is copied with the first chunks, and
// `r_done` says that it was the last one, so that nothing is left to wait for.
static mp_status solve_sign_gram(mp_ctx* c, float* x, float* r, long long T, const mp_trace& tr,
                                 hipStream_t s, bool& over, long long& t0, bool& r_done) {
  constexpr int kRounds = 4, kSlowRounds = 8, kSlowSteps = 4;
  const bool timed = c->profiling;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  HIP_TRY(c, mp::launch_sgram_init(c->sign_gram, c->m, s));
  long long issued = 0, seen = 0;
  long long total = 0, upto[2] = {0, 0};     // rounds enqueued; up to a chunk's end
  long long mark_rounds = 0, mark_t = 0;     // where the rate of steps was last looked at
  bool slow = false;
  over = false;
  auto round = [&](bool first) {
    return mp::launch_sgram_round(c->psis, c->sign_ws, c->n, c->m, c->ld, c->sign_c64, c->sign_r64,
                                  c->r_work, c->geom, c->sign_gram, first, T, x, c->st, tr, s);
  };
  HIP_TRY(c, round(true));
  while (!over && (!slow || issued > seen)) {
    while (!slow && issued - seen < (seen < 2 ? 1 : 2)) {
      const int rounds = static_cast<int>(std::min<long long>(issued + 1, kRounds));
      for (int k = 0; k < rounds; ++k) HIP_TRY(c, round(false));
      const int k = static_cast<int>(issued & 1);
      if (r && issued < 2)
        HIP_TRY(c, hipMemcpyAsync(r, c->r_work, c->n * sizeof(float), hipMemcpyDeviceToDevice, s));
      HIP_TRY(c, hipMemcpyAsync(&c->h_st[1 + k], c->st, sizeof(mp::DevState),
                                hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipEventRecord(c->done_ev[k], s));
      total += rounds;
      upto[k] = total;
      ++issued;
    }
    const int k = static_cast<int>(seen & 1);
    HIP_TRY(c, hipEventSynchronize(c->done_ev[k]));
    ++seen;
    over = c->h_st[1 + k].done != 0;
    t0 = c->h_st[1 + k].t;
    const long long rounds = upto[k] - mark_rounds;
    if (rounds >= kSlowRounds) {
      slow = slow || t0 - mark_t < kSlowSteps * rounds;
      mark_rounds = upto[k];
      mark_t = t0;
    }
  }
  *c->h_st = c->h_st[1 + static_cast<int>((seen - 1) & 1)];
  r_done = over && seen <= 2;  // (one chunk in flight until then)
  c->carried_steps = t0;
  if (timed) {
    HIP_TRY(c, hipEventRecord(c->ev[1], s));
    HIP_TRY(c, hipEventSynchronize(c->ev[1]));
  }
  return MP_OK;
}

mp_status mp_solve(mp_ctx* ctx, const float* y, float* x, float* r, const mp_opts* opts,
                   mp_result* res, const mp_trace* trace, void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  if (ctx->ragged) return fail(ctx, MP_EINVAL, "a ragged context is decoded with mp_solve_ragged");
  if (ctx->storage == MP_F64)
    return fail(ctx, MP_EINVAL, "an MP_F64 context is decoded with mp_solve_f64");
  if (!y || !x || !opts) return fail(ctx, MP_EINVAL, "y, x and opts must not be NULL");
  if (mp_status os = check_opts(ctx, opts, MP_SOLVE_STEP_LAUNCHES | MP_SOLVE_ASYNC); os != MP_OK)
    return os;
  if (opts->flags & MP_SOLVE_ASYNC) {
    if (ctx->storage == MP_SIGN1)
      return fail(ctx, MP_EINVAL, "stream-ordered decodes need MP_F32, MP_BF16 or MP_FP8_E4M3");
    if (res) return fail(ctx, MP_EINVAL, "a stream-ordered decode takes res = NULL");
  }
  mp_trace tr{};
  if (mp_status ts = check_trace(ctx, trace, ctx->n); ts != MP_OK) return ts;
  if (trace) tr = *trace;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  mp_ctx* c = ctx;
  c->carried_steps = 0;
  c->rescore_k = opts->rescore_k == 0 ? mp::kLpTopK : opts->rescore_k;
  c->prof_ms = 0.0;
  c->prof_launches = 0;
  bool persistent = false;  // the one-bit decode took no launch per step
  long long timed_from = 0;  // steps before the launch the profiling events bracket

  if (c->storage != MP_SIGN1)
    return solve_carried(c, y, x, r, opts, res, tr, s,
                         CarriedBufs{c->st, c->r_work, c->partials, c->bal}, true, true);

  HIP_TRY(c, mp::launch_init(y, c->n, c->ld, x, c->m, c->r_work, c->st, opts->eps,
                             step_cap(opts), s));
  bool r_done = false;  // r and the state are there already
  {
    const long long T = step_cap(opts);
    const bool stepwise = (opts->flags & MP_SOLVE_STEP_LAUNCHES) != 0;
    long long t0 = 0;    // steps behind the launches below
    // batches of steps, unless the caller asks for one launch per step or
    // limits the waits of the persistent launch, which only that has.  A cap
    // of a few steps takes the persistent launch where it fits: it costs 75 us
    // and 7 a step at N = 48 .. 64, the batches 110 and 1.
    const bool batches = !stepwise && (T > 64 || !c->sign_persist) &&
                         !getenv("MP_SIGN_SPIN_LIMIT") && ensure_sign_gram(c);
    if (!batches) {
      // the host passes on the threshold, and launches nothing after a stop
      HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipStreamSynchronize(s));
    }
    // c(0) = Psi^T y and r = y in FP64; launch k runs the stop test for the
    // k-1 steps taken and takes step k, so T steps take T+2 launches
    if (batches || !c->h_st->done)
      HIP_TRY(c, mp::launch_sign_c0(c->psis, c->sign_ws, c->n, c->m, y, c->ld, c->sign_c64,
                                    c->sign_r64, s));
    if (batches) {
      const mp_status gs = solve_sign_gram(c, x, r, T, tr, s, persistent, t0, r_done);
      if (gs != MP_OK) return gs;
      // (a decode that the init kernel ended took none of the forms)
      if (persistent && c->h_st->t == 0 && c->h_st->reason != MP_STOP_STALLED) persistent = false;
    }
    const double thr = c->h_st->thr;
    // otherwise the whole decode, or what the batches left of it, as one
    // persistent launch when it fits; a launch the device refuses falls back to
    // stepping
    if (!persistent && c->sign_persist && !stepwise && !c->h_st->done) {
      if (c->profiling) HIP_TRY(c, hipEventRecord(c->ev[0], s));
      // a new tag epoch for every decode (never 0 mod kSignEpochMod: the
      // zeroed words match no step); when it wraps, clear the words so that
      // none left from a decode that many decodes ago can match
      c->sign_epoch = c->sign_epoch % (mp::kSignEpochMod - 1) + 1;
      if (c->sign_epoch == 1)
        HIP_TRY(c, hipMemsetAsync(c->sign_slots, 0,
                                  sizeof(unsigned long long) * mp::kSignSlotWords * 2 *
                                      static_cast<size_t>(c->geom.grid),
                                  s));
      timed_from = t0;
      const hipError_t e = mp::launch_sign_persist(
          c->psis, c->sign_ws, c->n, c->m, c->ld, c->sign_c64, c->sign_r64, c->r_work, c->geom,
          c->sign_slots, c->sign_epoch, t0, T, thr, x, c->st, tr, s);
      if (e == hipSuccess) {
        persistent = true;
        if (c->profiling) HIP_TRY(c, hipEventRecord(c->ev[1], s));
      } else {
        (void)hipGetLastError();
      }
    }
    long long k = 0;
    const mp_status st = persistent ? MP_OK :
        run_iterations(c, T > 0 ? T - t0 + 2 : 0, s, true, [&](hipEvent_t e0, hipEvent_t e1) {
      hipError_t e;
      if (e0 && (e = hipEventRecord(e0, s)) != hipSuccess) return e;
      e = mp::launch_mp_step_sign(c->psis, c->sign_ws, c->n, c->m, c->ld, c->sign_c64,
                                  c->sign_r64, c->r_work, c->sign_rrp, c->geom, c->partials, k, t0,
                                  T, thr, x, c->st, tr, s);
      ++k;
      if (e != hipSuccess) return e;
      if (e1 && (e = hipEventRecord(e1, s)) != hipSuccess) return e;
      return hipSuccess;
    }, false, nullptr, t0);
    if (st != MP_OK) return st;
  }

  if (!r_done) {
    // the one-bit form keeps its FP32 r in the first n floats of r_work
    if (r)
      HIP_TRY(c, hipMemcpyAsync(r, c->r_work, c->n * sizeof(float), hipMemcpyDeviceToDevice, s));
    HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
  }
  if (persistent && c->profiling) {
    // the persistent launch runs t + 2 steps (step j of it does what launch
    // j of the stepping form does): the launch time over the steps
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = c->h_st->t - timed_from + 2;
    }
  }
  const mp_status fs = finish_result(c, res);
  if (fs == MP_OK && res) res->persistent = persistent ? 1 : 0;
  return fs;
}

mp_status mp_solve_noalloc(mp_ctx* ctx, const float* y, float* x, float* r, const mp_opts* opts,
                           mp_result* res, const mp_trace* trace, void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  mp_ctx* c = ctx;
  if (c->ragged || !(c->storage == MP_F32 || c->storage == MP_BF16 ||
                     c->storage == MP_FP8_E4M3))
    return fail(c, MP_EINVAL,
                "mp_solve_noalloc decodes MP_F32, MP_BF16 and MP_FP8_E4M3 contexts of mp_create");
  if (!y || !x || !opts) return fail(c, MP_EINVAL, "y, x and opts must not be NULL");
  if (mp_status os = check_opts(c, opts, MP_SOLVE_STEP_LAUNCHES | MP_SOLVE_ASYNC); os != MP_OK)
    return os;
  if ((opts->flags & MP_SOLVE_ASYNC) && res)
    return fail(c, MP_EINVAL, "a stream-ordered decode takes res = NULL");
  if (mp_status ts = check_trace(c, trace, c->n); ts != MP_OK) return ts;
  if (c->ld > mp::kNoAllocMaxLd)
    return fail(c, MP_EINVAL, "N exceeds the static scratch (at most 16384 rows)");
  if (2 * static_cast<int64_t>(c->geom.grid) * mp::kLpTopK > mp::kNoAllocMaxKeys)
    return fail(c, MP_EINVAL, "more correlation workgroups than the static scratch holds");
  mp_trace tr{};
  if (trace) tr = *trace;
  HIP_TRY(c, hipSetDevice(c->device));
  void* base = nullptr;
  HIP_TRY(c, mp::noalloc_scratch(c->device, &base));
  unsigned char* b = static_cast<unsigned char*>(base);
  c->carried_steps = 0;
  c->rescore_k = opts->rescore_k == 0 ? mp::kLpTopK : opts->rescore_k;
  c->prof_ms = 0.0;
  c->prof_launches = 0;
  return solve_carried(c, y, x, r, opts, res, tr, static_cast<hipStream_t>(stream),
                       CarriedBufs{reinterpret_cast<mp::DevState*>(b),
                                   reinterpret_cast<float*>(b + mp::kNoAllocR),
                                   reinterpret_cast<uint64_t*>(b + mp::kNoAllocKeys),
                                   reinterpret_cast<mp::BalState*>(b + mp::kNoAllocBal)},
                       false, false);
}

mp_status mp_solve_result(mp_ctx* ctx, mp_result* res) {
  if (!ctx) return MP_EINVAL;
  mp_ctx* c = ctx;
  if (!c->async_pending) return fail(c, MP_EINVAL, "no stream-ordered decode is pending");
  c->err.clear();
  HIP_TRY(c, hipSetDevice(c->device));
  c->async_pending = false;
  HIP_TRY(c, hipEventSynchronize(c->async_ev));
  const mp_status fs = finish_result(c, res);
  if (fs == MP_OK && res) res->persistent = c->async_persistent;
  return fs;
}

// Dictionaries below this many bytes select by a pass every step, which then
// costs no more than the launches that carrying adds (decodes of 16, 64 and 128
// atoms by carried correlations and by passes, ms: N = 2048, M = 8192, 64 MiB:
// 5.32 and 5.21 at 128; M = 12288, 96 MiB: 0.84 and 1.37, 3.06 and 3.52, 5.8 and
// 7.0; N = 4096, M = 8192, 128 MiB: 1.09 and 1.43, 3.1 and 4.0).  Short decodes
// come to the same: 1, 2, 4 and 8 atoms at 96 MiB 0.16 and 0.29, 0.29 and 0.29,
// 0.32 and 0.30, 0.48 and 0.61; only two atoms of a large dictionary, a pass
// each either way, cost more (1 GiB: 0.65 and 0.55).
constexpr int64_t kOmpCarryBytes = int64_t{96} << 20;

static mp_status ensure_omp(mp_ctx* c, int64_t tq) {
  mp::OmpBufs& b = c->omp;
  if (b.tq >= tq) return MP_OK;
  free_omp(c);
  const size_t ld = static_cast<size_t>(c->ld), t = static_cast<size_t>(tq);
  bool ok = hipMalloc(&b.q, sizeof(float) * t * ld) == hipSuccess &&
            hipMalloc(&b.rmat, sizeof(float) * t * t) == hipSuccess &&
            hipMalloc(&b.z, sizeof(double) * t) == hipSuccess &&
            hipMalloc(&b.sel, sizeof(int) * t) == hipSuccess &&
            hipMalloc(&b.in_s, static_cast<size_t>(c->m)) == hipSuccess &&
            hipMalloc(&b.w, sizeof(float) * ld) == hipSuccess &&
            hipMalloc(&b.h1, sizeof(float) * t) == hipSuccess &&
            hipMalloc(&b.h2, sizeof(float) * t) == hipSuccess &&
            hipMalloc(&b.hp, sizeof(float) * t * mp::kOmpProjSlices) == hipSuccess &&
            hipMalloc(&b.part, sizeof(double) * (ld / 64)) == hipSuccess &&
            hipMalloc(&b.os, sizeof(mp::OmpState)) == hipSuccess;
  if (!ok) {
    free_omp(c);
    return fail(c, MP_ENOMEM, "OMP work buffers");
  }
  b.tq = tq;
  return MP_OK;
}

// Whether OMP's selection takes the carried correlations, and their buffers if
// so.  They save the pass of all steps but one in fifteen or more and cost two
// launches more a step and five more a pass.
// Without them (column norms not near 1, no memory) every step selects by a
// pass.
static bool ensure_omp_carry(mp_ctx* c) {
  mp::OmpBufs& b = c->omp;
  if (!c->carried_on || c->ld * c->m * 4 < kOmpCarryBytes || !(c->max_norm > 0.99) ||
      !(c->max_norm < 1.01))
    return false;
  if (b.oc) return true;
  const size_t ld = static_cast<size_t>(c->ld), req = mp::kGramReq;
  b.mp = round_up(c->m, mp::kGramTile);
  b.ldh = round_up(b.tq, mp::kGramTile);
  const size_t stride = static_cast<size_t>(b.mp), ldh = static_cast<size_t>(b.ldh);
  if (!room_for(sizeof(float) * (stride + ldh + 2 * ld) * (req + 1)) ||
      hipMalloc(&b.oc, sizeof(mp::OmpCarry)) != hipSuccess ||
      hipMalloc(&b.c, sizeof(float) * stride) != hipSuccess ||
      hipMalloc(&b.p, sizeof(float) * stride * req) != hipSuccess ||
      hipMalloc(&b.w15, sizeof(float) * ld * req) != hipSuccess ||
      hipMalloc(&b.rhs, sizeof(float) * ld * (req + 1)) != hipSuccess ||
      hipMalloc(&b.hr, sizeof(float) * ldh) != hipSuccess ||
      hipMalloc(&b.hq, sizeof(float) * ldh * req) != hipSuccess ||
      hipMalloc(&b.dpart, sizeof(double) * (ld / 64)) != hipSuccess ||
      hipMalloc(&b.tops, sizeof(uint64_t) * static_cast<size_t>(mp::omp_tops(c->m))) !=
          hipSuccess) {
    (void)hipGetLastError();
    free_omp_carry(c);
    return false;
  }
  return true;
}

// The OMP decode on carried correlations (k_omp_gram.hip), after the init
// kernel: rounds of a block (which returns at once while the current one
// lasts) and some steps (which return at once while they wait for a block),
// enqueued in chunks.  A block lasts fifteen to twenty steps: with kOmpSlots steps
// a round the launches that return at once come to about 3 us a step.  The
// first chunk is one round of one step (its block has no candidates yet), the
// second one of three, the third one, each looked at before the next is
// enqueued, so that a decode of a few atoms does not wait for launches past its
// stop (3 us each); then two chunks in flight, soon of kOmpRounds.  `gave_up`:
// as in solve_gram, after `known` steps.
static mp_status solve_omp_gram(mp_ctx* c, const mp_trace& tr, long long T, hipStream_t s,
                                bool& gave_up, long long& known) {
  constexpr int kOmpSlots = 4, kOmpRounds = 2;
  mp::OmpBufs& b = c->omp;
  const mp::GramBounds bounds = mp::gram_bounds(c->n, c->max_norm, false);
  const bool timed = c->profiling;
  gave_up = false;
  if (timed) HIP_TRY(c, hipEventRecord(c->ev[0], s));
  HIP_TRY(c, mp::launch_omp_carry_init(b, s));
  // every two rounds take a step: a block is followed by one unless it renewed
  // the correlations, and then the next one is
  const long long most = 2 * T + 2;
  long long rounds = 0, steps = 0, upto[2] = {0, 0};  // enqueued; steps up to a chunk's end
  long long issued = 0, seen = 0, bound = 0;
  bool over = T <= 0;
  while (!over && (rounds < most || issued > seen)) {
    while (rounds < most && issued - seen < (seen < 3 ? 1 : 2)) {
      const int slots = issued == 0 ? 1 : issued == 1 ? 3 : kOmpSlots;
      for (int round = 0; round < (issued < 5 ? 1 : kOmpRounds); ++round, ++rounds) {
        HIP_TRY(c, mp::launch_omp_block(c->psi32, c->ld, c->n, c->m, c->r_work, b, c->st, bound,
                                        c->num_cus, s));
        for (int k = 0; k < slots; ++k, ++steps) {
          HIP_TRY(c, mp::launch_omp_pick(c->psi32, c->ld, c->m, c->r_work, b, bounds, k == 0,
                                         tr.coef != nullptr, c->st, s));
          HIP_TRY(c, mp::launch_omp_fit(c->psi32, c->ld, c->n, c->r_work, c->st, b, bound, true,
                                        tr, s));
          bound = std::min(bound + 1, T);
        }
      }
      const int k = static_cast<int>(issued & 1);
      HIP_TRY(c, hipMemcpyAsync(&c->h_st[1 + k], c->st, sizeof(mp::DevState),
                                hipMemcpyDeviceToHost, s));
      HIP_TRY(c, hipEventRecord(c->done_ev[k], s));
      upto[k] = steps;
      ++issued;
    }
    const int k = static_cast<int>(seen & 1);
    HIP_TRY(c, hipEventSynchronize(c->done_ev[k]));
    ++seen;
    over = c->h_st[1 + k].done != 0;
    gave_up = c->h_st[1 + k].pad[0] != 0;
    known = c->h_st[1 + k].t;
    // directions there can be once the chunks in flight are done
    bound = std::min(known + steps - upto[k], T);
  }
  if (!over) gave_up = true;
  c->carried_steps = known;
  if (gave_up) {
    HIP_TRY(c, mp::launch_resume<float>(c->st, c->r_work, c->ld, 0, s));
    return MP_OK;
  }
  if (timed) {
    // the decode's time on the device over the steps it took
    HIP_TRY(c, hipEventRecord(c->ev[1], s));
    HIP_TRY(c, hipEventSynchronize(c->ev[1]));
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, c->ev[0], c->ev[1]) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = known > 0 ? known : 1;
    }
  }
  return MP_OK;
}

mp_status mp_solve_omp(mp_ctx* ctx, const float* y, float* x, float* r, const mp_opts* opts,
                       mp_result* res, const mp_trace* trace, void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  if (ctx->ragged || ctx->storage != MP_F32)
    return fail(ctx, MP_EINVAL, "mp_solve_omp needs an MP_F32 context from mp_create");
  if (!y || !x || !opts) return fail(ctx, MP_EINVAL, "y, x and opts must not be NULL");
  if (mp_status os = check_opts(ctx, opts, MP_SOLVE_STEP_LAUNCHES | MP_SOLVE_ASYNC); os != MP_OK)
    return os;
  if (opts->flags & MP_SOLVE_ASYNC) {
    if (ctx->storage == MP_SIGN1)
      return fail(ctx, MP_EINVAL, "stream-ordered decodes need MP_F32, MP_BF16 or MP_FP8_E4M3");
    if (res) return fail(ctx, MP_EINVAL, "a stream-ordered decode takes res = NULL");
  }
  mp_trace tr{};
  if (mp_status ts = check_trace(ctx, trace, ctx->n); ts != MP_OK) return ts;
  if (trace) tr = *trace;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  mp_ctx* c = ctx;
  c->carried_steps = 0;
  // at most min(T, N) atoms: beyond N the selected atoms span the whole space
  const long long T = std::min<long long>(opts->max_iters, c->n);
  if (mp_status bs = ensure_omp(c, std::max<long long>(T, 1)); bs != MP_OK) return bs;
  mp::OmpBufs& b = c->omp;
  HIP_TRY(c, hipMemsetAsync(b.in_s, 0, static_cast<size_t>(c->m), s));
  HIP_TRY(c, mp::launch_init(y, c->n, c->ld, x, c->m, c->r_work, c->st, opts->eps, T, s));
  bool stepping = true;
  long long it = 0;  // iterations behind or enqueued: a bound on the atoms selected
  if (!(opts->flags & MP_SOLVE_STEP_LAUNCHES) && cap_pays(MP_F32, T) && ensure_omp_carry(c)) {
    const mp_status gs = solve_omp_gram(c, tr, T, s, stepping, it);
    if (gs != MP_OK) return gs;
  }
  if (stepping) {
    HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
    HIP_TRY(c, hipStreamSynchronize(s));
    const long long t0 = it;
    const mp_status st = run_iterations(c, T - t0, s, false, [&](hipEvent_t e0, hipEvent_t e1) {
      hipError_t e = mp::launch_omp_select(c->psi32, c->ld, c->m, c->r_work, c->geom, c->partials,
                                           c->st, b, s, e0, e1);
      if (e == hipSuccess)
        e = mp::launch_omp_fit(c->psi32, c->ld, c->n, c->r_work, c->st, b, it, false, tr, s);
      ++it;
      return e;
    }, false, nullptr, t0);
    if (st != MP_OK) return st;
  }
  HIP_TRY(c, mp::launch_omp_solve(b, c->st, x, s));
  HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
  if (r)
    HIP_TRY(c, hipMemcpyAsync(r, c->r_work, c->n * sizeof(float), hipMemcpyDeviceToDevice, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  return finish_result(c, res);
}

mp_status mp_create_f64(mp_ctx** out, const double* psi, int64_t n, int64_t m, int64_t ld,
                        uint32_t flags, void* stream) {
  g_create_error.clear();
  if (!out) return fail(nullptr, MP_EINVAL, "out is NULL");
  *out = nullptr;
  if (!psi) return fail(nullptr, MP_EINVAL, "psi is NULL");
  if (n < 1 || m < 1) return fail(nullptr, MP_EINVAL, "n and m must be >= 1");
  if (ld < n) return fail(nullptr, MP_EINVAL, "ld must be >= n");
  if (n > kMaxN) return fail(nullptr, MP_EINVAL, "n exceeds 16384");
  if (m >= (int64_t{1} << 31)) return fail(nullptr, MP_EINVAL, "m must be < 2^31");
  if (flags & ~MP_SKIP_NORM_CHECK) return fail(nullptr, MP_EINVAL, "unknown flags");
  int dev = 0;
  hipDeviceProp_t prop;
  if (mp_status ds = open_device(dev, prop); ds != MP_OK) return ds;
  hipStream_t s = static_cast<hipStream_t>(stream);

  mp_ctx* c = new mp_ctx();
  c->device = dev;
  c->num_cus = prop.multiProcessorCount;
  c->n = n;
  c->m = m;
  c->ld = round_up(n, kLdAlign);
  c->storage = MP_F64;
  c->geom = mp::corr_f32_geometry(m, c->num_cus);  // same workgroup layout as FP32

  auto bail = [&](mp_status st, const std::string& msg) {
    free_ctx(c);
    return fail(nullptr, st, msg);
  };
  const size_t psi_bytes = static_cast<size_t>(c->ld) * static_cast<size_t>(m) * sizeof(double);
  if (hipMalloc(&c->psi64, psi_bytes) != hipSuccess) return bail(MP_ENOMEM, "dictionary copy");
  // r in two halves that alternate by launch parity
  if (hipMalloc(&c->r64_work, 2 * c->ld * sizeof(double)) != hipSuccess)
    return bail(MP_ENOMEM, "r");
  if (hipMalloc(&c->st, sizeof(mp::DevState)) != hipSuccess) return bail(MP_ENOMEM, "state");
  if (c->geom.grid * 2 > 2 * 1024)
    return bail(MP_EUNSUPPORTED, "more correlation workgroups than the key slots hold");
  // two words per workgroup, in two halves that alternate by launch parity
  const size_t nkeys = static_cast<size_t>(c->geom.grid) * 4;
  if (hipMalloc(&c->partials, sizeof(uint64_t) * nkeys) != hipSuccess)
    return bail(MP_ENOMEM, "partials");
  if (hipMalloc(&c->bal, sizeof(mp::BalState)) != hipSuccess) return bail(MP_ENOMEM, "shares");
  if (!make_host_state(c)) return bail(MP_ENOMEM, "pinned state");

  hipError_t e = hipMemsetAsync(c->psi64, 0, psi_bytes, s);
  if (e == hipSuccess)
    e = hipMemcpy2DAsync(c->psi64, c->ld * sizeof(double), psi, ld * sizeof(double),
                         n * sizeof(double), m, hipMemcpyDeviceToDevice, s);
  if (e == hipSuccess) e = hipMemsetAsync(c->r64_work, 0, 2 * c->ld * sizeof(double), s);
  if (e == hipSuccess) e = hipMemsetAsync(c->bal, 0, sizeof(mp::BalState), s);
  if (e == hipSuccess) e = hipMemsetAsync(c->partials, 0, sizeof(uint64_t) * nkeys, s);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("copy: ") + hipGetErrorString(e));

  double* d_norm2 = nullptr;
  if (hipMalloc(&d_norm2, sizeof(double) * m) != hipSuccess) return bail(MP_ENOMEM, "norms");
  std::vector<double> norm2(static_cast<size_t>(m));
  e = mp::launch_norms_f64(c->psi64, c->ld, n, m, d_norm2, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(norm2.data(), d_norm2, sizeof(double) * m, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(d_norm2);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("norms: ") + hipGetErrorString(e));
  {
    std::string msg;
    const mp_status ns = check_norms(norm2, flags, msg);
    if (ns != MP_OK) return bail(ns, msg);
    c->max_norm = largest_norm(norm2);
  }
  *out = c;
  return MP_OK;
}

mp_status mp_create_signs(mp_ctx** out, const uint32_t* signs, int64_t n, int64_t m, int64_t ldw,
                          uint32_t flags, void* stream) {
  g_create_error.clear();
  if (!out) return fail(nullptr, MP_EINVAL, "out is NULL");
  *out = nullptr;
  if (!signs) return fail(nullptr, MP_EINVAL, "signs is NULL");
  if (n < 1 || m < 1) return fail(nullptr, MP_EINVAL, "n and m must be >= 1");
  if (n > kMaxSignN) return fail(nullptr, MP_EINVAL, "n exceeds 16384");
  if (ldw < (n + 31) / 32) return fail(nullptr, MP_EINVAL, "ldw must be >= ceil(n / 32)");
  if (m >= (int64_t{1} << 31)) return fail(nullptr, MP_EINVAL, "m must be < 2^31");
  if (flags & ~MP_SKIP_NORM_CHECK) return fail(nullptr, MP_EINVAL, "unknown flags");
  int dev = 0;
  hipDeviceProp_t prop;
  if (mp_status ds = open_device(dev, prop); ds != MP_OK) return ds;
  hipStream_t s = static_cast<hipStream_t>(stream);

  mp_ctx* c = new mp_ctx();
  c->device = dev;
  c->num_cus = prop.multiProcessorCount;
  c->n = n;
  c->m = m;
  c->ld = round_up(n, kLdAlign);
  c->storage = MP_SIGN1;
  c->sign_ws = round_up((n + 31) / 32, 4);
  c->geom = mp::sign_geometry(n, m, c->num_cus);

  auto bail = [&](mp_status st, const std::string& msg) {
    free_ctx(c);
    return fail(nullptr, st, msg);
  };
  const size_t words = static_cast<size_t>(m) * static_cast<size_t>(c->sign_ws);
  if (hipMalloc(&c->psis, words * sizeof(uint32_t)) != hipSuccess)
    return bail(MP_ENOMEM, "sign-bit copy");
  if (hipMalloc(&c->sign_c64, sizeof(double) * m) != hipSuccess)
    return bail(MP_ENOMEM, "correlations");
  if (hipMalloc(&c->sign_r64, sizeof(double) * c->ld) != hipSuccess) return bail(MP_ENOMEM, "r");
  if (hipMalloc(&c->r_work, c->ld * sizeof(float)) != hipSuccess) return bail(MP_ENOMEM, "r");
  if (hipMalloc(&c->st, sizeof(mp::DevState)) != hipSuccess) return bail(MP_ENOMEM, "state");
  if (c->geom.grid > 1024)
    return bail(MP_EUNSUPPORTED, "more correlation workgroups than the key slots hold");
  // pair keys, one per workgroup, in two halves alternating by launch parity
  const size_t nkeys = 4 * static_cast<size_t>(c->geom.grid);
  if (hipMalloc(&c->partials, sizeof(uint64_t) * nkeys) != hipSuccess)
    return bail(MP_ENOMEM, "partials");
  if (hipMalloc(&c->sign_rrp, sizeof(double) * 2 * c->geom.grid) != hipSuccess)
    return bail(MP_ENOMEM, "partial norms");
  // the persistent decode (bits in LDS): one workgroup per CU, all resident
  c->sign_persist = mp::sign_persist_fits(n, m, c->ld, c->sign_ws, c->geom, c->num_cus) &&
                    mp::sign_persist_resident(n, c->sign_ws, c->geom, c->num_cus);
  const size_t slot_bytes =
      sizeof(unsigned long long) * mp::kSignSlotWords * 2 * static_cast<size_t>(c->geom.grid);
  if (hipMalloc(&c->sign_slots, slot_bytes) != hipSuccess)
    return bail(MP_ENOMEM, "step records");
  if (!make_host_state(c)) return bail(MP_ENOMEM, "pinned state");
  hipError_t e = mp::launch_copy_signs(signs, ldw, n, m, c->sign_ws, c->psis, s);
  if (e == hipSuccess) e = hipMemsetAsync(c->r_work, 0, c->ld * sizeof(float), s);
  if (e == hipSuccess) e = hipMemsetAsync(c->partials, 0, sizeof(uint64_t) * nkeys, s);
  if (e == hipSuccess)
    e = hipMemsetAsync(c->sign_slots, 0, slot_bytes, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("copy: ") + hipGetErrorString(e));
  *out = c;
  return MP_OK;
}

mp_status mp_solve_f64(mp_ctx* ctx, const double* y, double* x, double* r, const mp_opts* opts,
                       mp_result* res, const mp_trace_f64* trace, void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  if (ctx->ragged || ctx->storage != MP_F64)
    return fail(ctx, MP_EINVAL, "mp_solve_f64 needs a context from mp_create_f64");
  if (!y || !x || !opts) return fail(ctx, MP_EINVAL, "y, x and opts must not be NULL");
  if (mp_status os = check_opts(ctx, opts); os != MP_OK) return os;
  mp_trace_f64 tr{};
  if (mp_status ts = check_trace(ctx, trace, ctx->n); ts != MP_OK) return ts;
  if (trace) tr = *trace;
  HIP_TRY(ctx, hipSetDevice(ctx->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  mp_ctx* c = ctx;
  c->carried_steps = 0;

  HIP_TRY(c, mp::launch_init_f64(y, c->n, c->ld, x, c->m, c->r64_work, c->st, opts->eps,
                                 step_cap(opts), s));
  HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  bool carried = false;  // decoded on carried correlations (r is in half 0)
  long long t0 = 0;      // steps taken on them before the stepping form goes on
  if (!(opts->flags & MP_SOLVE_STEP_LAUNCHES) && !c->h_st->done &&
      cap_pays(MP_F64, opts->max_iters) && ensure_gram(c, s)) {
    bool gave_up = false;
    const mp_status gs =
        solve_gram<double>(c, c->psi64, c->r64_work, x, opts, tr, s, gave_up, t0);
    if (gs != MP_OK) return gs;
    carried = !gave_up;
  }
  // launch k takes step k (k >= 1) and runs pass k+1: T steps take T+1
  // launches; r ends in the half the state names
  long long k = t0;
  const long long T = step_cap(opts);
  const double thr = c->h_st->thr;
  const mp_status st = carried ? MP_OK : run_iterations(c, T > 0 ? T - t0 + 1 : 0, s, true, [&](hipEvent_t e0, hipEvent_t e1) {
    hipError_t e;
    if (e0 && (e = hipEventRecord(e0, s)) != hipSuccess) return e;
    e = mp::launch_mp_step_f64(c->psi64, c->ld, c->n, c->m, c->r64_work, c->geom, c->partials,
                               c->bal, k, t0, T, thr, x, c->st, tr, s);
    ++k;
    if (e != hipSuccess) return e;
    if (e1 && (e = hipEventRecord(e1, s)) != hipSuccess) return e;
    return hipSuccess;
  }, false, nullptr, t0);
  if (st != MP_OK) return st;

  HIP_TRY(c, hipMemcpyAsync(c->h_st, c->st, sizeof(mp::DevState), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (r)
    HIP_TRY(c, hipMemcpyAsync(r, c->r64_work + (c->h_st->r_sel ? c->ld : 0),
                              c->n * sizeof(double), hipMemcpyDeviceToDevice, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  return finish_result(c, res);
}


// Make sure the context has a BF16 copy for the batched product and buffers
// for `B` signals.
static mp_status ensure_batched(mp_ctx* c, int64_t B, hipStream_t s) {
  if (!c->psibt) {
    const size_t bytes =
        static_cast<size_t>(c->ld) * static_cast<size_t>(round_up(c->m, 16)) * 2;
    if (hipMalloc(&c->psibt, bytes) != hipSuccess) return fail(c, MP_ENOMEM, "BF16 tiles");
    HIP_TRY(c, mp::launch_tile_bf16(c->psi32, c->ld, c->m, c->psibt, s));
  }
  if (B <= c->bcap) return MP_OK;
  free_batched(c);
  const int64_t cap = B;
  const int mtiles = mp::bcorr_mtiles(c->m, mp::kBTileMinAtoms);  // the most lists of a tiling
  const size_t ldb = static_cast<size_t>(c->ld);
  c->ldq = c->ld + 32;
  bool ok = hipMalloc(&c->b_r32, sizeof(float) * ldb * cap) == hipSuccess &&
            hipMalloc(&c->b_rq, sizeof(uint16_t) * static_cast<size_t>(c->ldq) * cap) ==
                hipSuccess &&
            hipMalloc(&c->b_slots, sizeof(mp::BSlot) * cap) == hipSuccess &&
            hipMalloc(&c->b_act, sizeof(int) * 2 * cap) == hipSuccess &&
            hipMalloc(&c->b_state, sizeof(mp::BState)) == hipSuccess &&
            hipMalloc(&c->b_partials, sizeof(uint64_t) * cap * mtiles * 8) == hipSuccess &&
            hipMalloc(&c->b_keep, sizeof(int) * 4 * cap) == hipSuccess &&
            hipMalloc(&c->b_tcap, sizeof(long long) * cap) == hipSuccess &&
            hipHostMalloc(&c->h_slots, sizeof(mp::BSlot) * cap, hipHostMallocDefault) ==
                hipSuccess &&
            hipHostMalloc(&c->h_bstate, 2 * sizeof(mp::BState), hipHostMallocDefault) ==
                hipSuccess;
  if (!ok) {
    free_batched(c);
    return fail(c, MP_ENOMEM, "batched work buffers");
  }
  HIP_TRY(c, hipMemsetAsync(c->b_keep, 0, sizeof(int) * 4 * cap, s));
  HIP_TRY(c, hipMemsetAsync(c->b_state, 0, sizeof(mp::BState), s));
  c->bcap = cap;
  return MP_OK;
}

mp_status mp_solve_batched(mp_ctx* ctx, const float* Y, int64_t ldy, int64_t B, float* X,
                           int64_t ldx, float* R, int64_t ldr, const mp_opts* opts,
                           const int64_t* max_iters_b, mp_result* res, const mp_trace* trace,
                           void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  mp_ctx* c = ctx;
  if (c->ragged) return fail(c, MP_EINVAL, "a ragged context is decoded with mp_solve_ragged");
  if (c->storage == MP_F64 || c->storage == MP_SIGN1)
    return fail(c, MP_EINVAL, "batched decoding needs an FP32, BF16 or FP8 context");
  if (mp_status ps = check_not_pending(c); ps != MP_OK) return ps;
  if (B < 0) return fail(c, MP_EINVAL, "B must be >= 0");
  if (B == 0) return MP_OK;
  if (B >= (int64_t{1} << 31) / 2) return fail(c, MP_EINVAL, "B too large");
  if (!Y || !X || !opts) return fail(c, MP_EINVAL, "Y, X and opts must not be NULL");
  if (ldy < c->n || ldx < c->m || (R && ldr < c->n))
    return fail(c, MP_EINVAL, "leading dimensions must be >= the column lengths");
  if (!(opts->eps >= 0.0) || !isfinite(opts->eps))
    return fail(c, MP_EINVAL, "eps must be finite and >= 0");
  if (opts->max_iters < 0) return fail(c, MP_EINVAL, "max_iters must be >= 0");
  if (opts->flags != 0) return fail(c, MP_EINVAL, "opts.flags must be 0");
  if (opts->rescore_k < 0 || opts->rescore_k > 8)
    return fail(c, MP_EINVAL, "rescore_k must be in 0..8");
  long long tmax = opts->max_iters;
  if (max_iters_b) {
    tmax = 0;
    for (int64_t b = 0; b < B; ++b) {
      if (max_iters_b[b] < 0) return fail(c, MP_EINVAL, "max_iters_b entries must be >= 0");
      tmax = std::max<long long>(tmax, max_iters_b[b]);
    }
  }
  mp_trace tr{};
  if (mp_status ts = check_trace(c, trace, c->n); ts != MP_OK) return ts;
  if (trace) tr = *trace;
  HIP_TRY(c, hipSetDevice(c->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  c->carried_steps = 0;
  const int rk = opts->rescore_k == 0 ? mp::kLpTopK : opts->rescore_k;
  c->prof_ms = 0.0;
  c->prof_launches = 0;
  // with all 8 candidates re-scored the atom selected is the FP32 argmax,
  // which the carried correlations give without a product per round
  int64_t left = B;  // signals the rounds decode, or go on with
  if (rk == mp::kLpTopK && tmax > 1 && ensure_gram_batch(c, B, tmax, s)) {
    const mp_status gs = solve_gram_batch(c, Y, ldy, B, X, ldx, opts, max_iters_b, tr, s, left);
    if (gs != MP_OK) return gs;
    if (left == 0) {
      if (R) {
        HIP_TRY(c, hipMemcpy2DAsync(R, ldr * sizeof(float), c->gram_br, c->ld * sizeof(float),
                                    c->n * sizeof(float), B, hipMemcpyDeviceToDevice, s));
        HIP_TRY(c, hipStreamSynchronize(s));
      }
      return batched_results(c, c->gram_hbst, B, res);
    }
    c->prof_ms = 0.0;
    c->prof_launches = 0;
    if (mp_status st = ensure_batched(c, B, s); st != MP_OK) return st;
    HIP_TRY(c, mp::launch_bresume(c->gram_bst, c->gram_br, c->ld, c->b_r32, c->b_rq, c->ldq,
                                  c->b_slots, static_cast<int>(B), c->b_act, c->b_keep, c->bcap,
                                  c->b_state, s));
  } else {
    if (mp_status st = ensure_batched(c, B, s); st != MP_OK) return st;
    if (max_iters_b)
      HIP_TRY(c, hipMemcpyAsync(c->b_tcap, max_iters_b, sizeof(long long) * B,
                                hipMemcpyHostToDevice, s));
    HIP_TRY(c, mp::launch_binit(Y, ldy, c->n, c->ld, X, ldx, c->m, c->b_r32, c->b_rq, c->ldq,
                                c->b_slots, max_iters_b ? c->b_tcap : nullptr, opts->max_iters,
                                opts->eps, static_cast<int>(B), c->b_act, c->b_keep, c->bcap,
                                c->b_state, s));
  }

  // Rounds in chunks, two chunks in flight; the kernels stop doing work once
  // the active list is empty.  No signal runs more than tmax rounds.
  hipEvent_t done_ev[2] = {nullptr, nullptr};
  HIP_TRY(c, hipEventCreateWithFlags(&done_ev[0], hipEventDisableTiming));
  HIP_TRY(c, hipEventCreateWithFlags(&done_ev[1], hipEventDisableTiming));
  long long issued = 0;
  int chunk = 4, next = 0, inflight = 0;
  long long slot_base[2] = {0, 0};
  int slot_len[2] = {0, 0};
  bool finished = false;
  mp_status status = MP_OK;
  // upper bound on the active count used to size each round's grids: all
  // left at first, then the count read back after each completed chunk
  int nact_hint = static_cast<int>(left);
  auto account = [&](int k, int n_after) {
    if (!c->profiling) return;
    (void)n_after;
    for (int j = 0; j < slot_len[k]; ++j) {
      if ((slot_base[k] + j) % c->prof_every != 0) continue;
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, c->ev[(k * kMaxChunk + j) * 2],
                              c->ev[(k * kMaxChunk + j) * 2 + 1]) == hipSuccess) {
        c->prof_ms += ms;
        c->prof_launches += 1;
      }
    }
  };
  while (!finished && status == MP_OK) {
    while (inflight < 2 && issued < tmax && status == MP_OK) {
      const int k = next;
      const int len = static_cast<int>(std::min<long long>(chunk, tmax - issued));
      for (int j = 0; j < len; ++j) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (c->profiling && (issued + j) % c->prof_every == 0) {
          e0 = c->ev[(k * kMaxChunk + j) * 2];
          e1 = c->ev[(k * kMaxChunk + j) * 2 + 1];
        }
        hipError_t e = mp::launch_bround(c->psibt, c->psi32, c->ld, c->n, c->m, c->b_r32,
                                         c->b_rq, c->ldq, X, ldx, c->b_slots, c->b_act,
                                         c->b_keep, c->bcap, c->b_state, c->b_partials,
                                         issued + j, nact_hint, c->b_cfg, c->num_cus, rk, tr, s,
                                         e0, e1);
        if (e != hipSuccess) {
          status = fail(c, MP_EDEVICE, std::string("launch: ") + hipGetErrorString(e));
          break;
        }
      }
      if (status != MP_OK) break;
      slot_base[k] = issued;
      slot_len[k] = len;
      issued += len;
      hipError_t e = hipMemcpyAsync(&c->h_bstate[k], c->b_state, sizeof(mp::BState),
                                    hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipEventRecord(done_ev[k], s);
      if (e != hipSuccess) {
        status = fail(c, MP_EDEVICE, std::string("state copy: ") + hipGetErrorString(e));
        break;
      }
      ++inflight;
      next ^= 1;
      chunk = std::min(chunk * 2, kMaxChunk);
    }
    if (status != MP_OK || inflight == 0) break;
    const int old = inflight == 2 ? next : (next ^ 1);
    hipError_t e = hipEventSynchronize(done_ev[old]);
    if (e != hipSuccess) {
      status = fail(c, MP_EDEVICE, std::string("sync: ") + hipGetErrorString(e));
      break;
    }
    --inflight;
    // the length of the list the chunk's last round r left for round r+1
    // (the signals still running after round r-1): an upper bound for every
    // later round, zero once all have stopped
    const mp::BState& hb = c->h_bstate[old];
    const long long r_last = slot_base[old] + slot_len[old] - 1;
    const int n_after = hb.n_active[(r_last + 1) & 1];
    account(old, n_after);
    // rounds already in flight were sized with the older hint, which is also
    // an upper bound; the count never increases
    nact_hint = std::min(nact_hint, n_after);
    if (n_after == 0) finished = true;
  }
  if (hipStreamSynchronize(s) != hipSuccess && status == MP_OK)
    status = fail(c, MP_EDEVICE, "stream synchronize failed");
  (void)hipEventDestroy(done_ev[0]);
  (void)hipEventDestroy(done_ev[1]);
  if (status != MP_OK) return status;

  if (R)
    HIP_TRY(c, hipMemcpy2DAsync(R, ldr * sizeof(float), c->b_r32, c->ld * sizeof(float),
                                c->n * sizeof(float), B, hipMemcpyDeviceToDevice, s));
  HIP_TRY(c, hipMemcpyAsync(c->h_slots, c->b_slots, sizeof(mp::BSlot) * B, hipMemcpyDeviceToHost,
                            s));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (rk == mp::kLpTopK && tmax > 1 && !c->gram_full && gram_full_suits(c)) {
    // what the Gram columns would have saved this call, which may take them
    long long longest = 0;
    for (int64_t b = 0; b < B; ++b) longest = std::max(longest, c->h_slots[b].t);
    c->gram_owed += gram_gain_us(c, B) * static_cast<double>(longest);
  }
  return batched_results(c, c->h_slots, B, res);
}


// ---------------------------------------------------------------------------
// Many independent instances

mp_status mp_create_ragged(mp_ctx** out, const mp_instance* inst, int64_t count, mp_dtype storage,
                           uint32_t flags, void* stream) {
  g_create_error.clear();
  if (!out) return fail(nullptr, MP_EINVAL, "out is NULL");
  *out = nullptr;
  if (!inst) return fail(nullptr, MP_EINVAL, "inst is NULL");
  if (count < 1 || count >= (int64_t{1} << 30)) return fail(nullptr, MP_EINVAL, "bad count");
  if (flags & ~MP_SKIP_NORM_CHECK) return fail(nullptr, MP_EINVAL, "unknown flags");
  if (storage != MP_F32 && storage != MP_BF16) {
    if (storage == MP_FP8_E4M3)
      return fail(nullptr, MP_EUNSUPPORTED, "ragged instances support MP_F32 and MP_BF16");
    return fail(nullptr, MP_EINVAL, "unknown storage type");
  }
  for (int64_t i = 0; i < count; ++i) {
    const mp_instance& d = inst[i];
    char buf[96];
    snprintf(buf, sizeof buf, "instance %lld: ", static_cast<long long>(i));
    if (!d.psi) return fail(nullptr, MP_EINVAL, std::string(buf) + "psi is NULL");
    if (d.n < 1 || d.m < 1) return fail(nullptr, MP_EINVAL, std::string(buf) + "n, m must be >= 1");
    if (d.ld < d.n) return fail(nullptr, MP_EINVAL, std::string(buf) + "ld must be >= n");
    if (d.n > kMaxRaggedN) return fail(nullptr, MP_EINVAL, std::string(buf) + "n exceeds 8192");
    if (d.m >= (int64_t{1} << 31)) return fail(nullptr, MP_EINVAL, std::string(buf) + "m too large");
  }
  int dev = 0, ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1)
    return fail(nullptr, MP_EDEVICE, "no HIP device");
  HIP_TRY(nullptr, hipGetDevice(&dev));
  hipDeviceProp_t prop;
  HIP_TRY(nullptr, hipGetDeviceProperties(&prop, dev));
  if (strncmp(prop.gcnArchName, "gfx950", 6) != 0)
    return fail(nullptr, MP_EUNSUPPORTED, std::string("device is ") + prop.gcnArchName +
                                              ", this library is built for gfx950");
  hipStream_t s = static_cast<hipStream_t>(stream);
  mp_ctx* c = new mp_ctx();
  c->device = dev;
  c->num_cus = prop.multiProcessorCount;
  c->storage = storage;
  c->ragged = true;
  c->r_count = count;
  // the untuned shape: the tuner's choice on the 512-instance mix of
  // N in {128, ..., 1024} (one 1024-thread workgroup per CU, the largest
  // instances in three parts)
  c->r_cfg = storage == MP_BF16 ? mp::RConfig{1024, 2, 2, kRaggedDefaultSplit}
                                : mp::RConfig{1024, 1, 2, kRaggedDefaultSplit};
  auto bail = [&](mp_status st, const std::string& msg) {
    free_ctx(c);
    return fail(nullptr, st, msg);
  };
  // packed layout of the copies, descriptors, and the work order
  std::vector<mp::RInst> desc(static_cast<size_t>(count));
  std::vector<int64_t> psi_off(static_cast<size_t>(count));
  int64_t elems = 0, yo = 0, xo = 0, msum = 0;
  c->r_n.resize(count);
  c->r_m.resize(count);
  for (int64_t i = 0; i < count; ++i) {
    const int64_t ld = round_up(inst[i].n, kLdAlign);
    psi_off[i] = elems;
    desc[i].n = inst[i].n;
    desc[i].m = inst[i].m;
    desc[i].ld = ld;
    desc[i].y_off = yo;
    desc[i].x_off = xo;
    elems += ld * inst[i].m;
    yo += inst[i].n;
    xo += inst[i].m;
    msum += inst[i].m;
    c->r_max_ld = std::max(c->r_max_ld, ld);
    c->r_n[i] = inst[i].n;
    c->r_m[i] = inst[i].m;
  }
  c->r_sum_n = yo;
  c->r_sum_m = xo;
  if (hipMalloc(&c->r_psi32, sizeof(float) * elems) != hipSuccess)
    return bail(MP_ENOMEM, "dictionary copies");
  if (storage == MP_BF16 && hipMalloc(&c->r_psib, sizeof(uint16_t) * elems) != hipSuccess)
    return bail(MP_ENOMEM, "BF16 copies");
  const int64_t max_split = std::min<int64_t>(count, kMaxRaggedSplit);
  if (hipMalloc(&c->r_inst, sizeof(mp::RInst) * count) != hipSuccess ||
      hipMalloc(&c->r_items, sizeof(mp::RItem) * count * mp::kRaggedMaxParts) != hipSuccess ||
      hipMalloc(&c->r_slots, sizeof(unsigned long long) * max_split * 2 * mp::kRaggedMaxParts *
                                 mp::kRaggedRecWords) != hipSuccess ||
      hipHostMalloc(&c->h_rq, sizeof(mp::RQueue), hipHostMallocDefault) != hipSuccess ||
      hipMalloc(&c->r_caps, sizeof(long long) * count) != hipSuccess ||
      hipMalloc(&c->r_res, sizeof(mp::RResult) * count) != hipSuccess ||
      hipMalloc(&c->r_queue, sizeof(mp::RQueue)) != hipSuccess ||
      hipHostMalloc(&c->h_rres, sizeof(mp::RResult) * count, hipHostMallocDefault) != hipSuccess)
    return bail(MP_ENOMEM, "ragged buffers");
  if (hipStreamCreateWithFlags(&c->r_cap_stream, hipStreamNonBlocking) != hipSuccess)
    return bail(MP_EDEVICE, "capture stream");
  hipError_t e = hipMemsetAsync(c->r_psi32, 0, sizeof(float) * elems, s);
  for (int64_t i = 0; i < count && e == hipSuccess; ++i)
    e = hipMemcpy2DAsync(c->r_psi32 + psi_off[i], desc[i].ld * sizeof(float), inst[i].psi,
                         inst[i].ld * sizeof(float), inst[i].n * sizeof(float), inst[i].m,
                         hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("copy: ") + hipGetErrorString(e));
  // column norms of every instance (eq. 4)
  double* d_norm2 = nullptr;
  if (hipMalloc(&d_norm2, sizeof(double) * msum) != hipSuccess) return bail(MP_ENOMEM, "norms");
  std::vector<double> norm2(static_cast<size_t>(msum));
  int64_t mo = 0;
  for (int64_t i = 0; i < count && e == hipSuccess; ++i) {
    e = mp::launch_norms(c->r_psi32 + psi_off[i], desc[i].ld, desc[i].n, desc[i].m,
                         d_norm2 + mo, nullptr, s);
    mo += desc[i].m;
  }
  if (e == hipSuccess)
    e = hipMemcpyAsync(norm2.data(), d_norm2, sizeof(double) * msum, hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(d_norm2);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("norms: ") + hipGetErrorString(e));
  mo = 0;
  for (int64_t i = 0; i < count; ++i) {
    for (int64_t j = 0; j < desc[i].m; ++j) {
      const double v = norm2[mo + j];
      char buf[128];
      if (!isfinite(v)) {
        snprintf(buf, sizeof buf, "instance %lld column %lld holds NaN or Inf",
                 static_cast<long long>(i), static_cast<long long>(j));
        return bail(MP_ENONFINITE, buf);
      }
      if (!(flags & MP_SKIP_NORM_CHECK) && fabs(sqrt(v) - 1.0) > kNormTol) {
        snprintf(buf, sizeof buf, "instance %lld column %lld has norm %.9g",
                 static_cast<long long>(i), static_cast<long long>(j), sqrt(v));
        return bail(MP_ENOTNORM, buf);
      }
    }
    mo += desc[i].m;
  }
  if (storage == MP_BF16) {
    // padding rows are zero and quantise to zero: one pass over everything
    e = mp::launch_quant_bf16(c->r_psi32, elems, 1, c->r_psib, s);
    if (e != hipSuccess) return bail(MP_EDEVICE, "quantise");
  }
  c->max_norm = largest_norm(norm2);
  c->r_psi_off = psi_off;
  for (int64_t i = 0; i < count; ++i) {
    desc[i].psi32 = c->r_psi32 + psi_off[i];
    desc[i].psib = storage == MP_BF16 ? c->r_psib + psi_off[i] : nullptr;
  }
  // most work first (iterations grow with n, a pass costs n * m); the work
  // list itself is built per launch shape (ragged_items)
  c->r_est.resize(count);
  for (int64_t i = 0; i < count; ++i)
    c->r_est[i] = static_cast<double>(desc[i].n) * desc[i].n * desc[i].m;
  c->r_order.resize(count);
  for (int64_t i = 0; i < count; ++i) c->r_order[i] = static_cast<int>(i);
  std::stable_sort(c->r_order.begin(), c->r_order.end(),
                   [&](int a1, int b1) { return c->r_est[a1] > c->r_est[b1]; });
  e = hipMemcpyAsync(c->r_inst, desc.data(), sizeof(mp::RInst) * count, hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return bail(MP_EDEVICE, std::string("upload: ") + hipGetErrorString(e));
  make_gram_ragged(c, s);
  *out = c;
  return MP_OK;
}

mp_status mp_batched_set_config(mp_ctx* ctx, const mp_batched_config* cfg) {
  if (!ctx || !cfg) return MP_EINVAL;
  if (ctx->ragged || ctx->storage == MP_F64 || ctx->storage == MP_SIGN1)
    return fail(ctx, MP_EINVAL, "batched decoding needs an FP32, BF16 or FP8 context");
  if (cfg->atoms128_above < 0 || cfg->atoms64_above < 0 || cfg->atoms32_above < 0)
    return fail(ctx, MP_EINVAL, "the active counts must be >= 0");
  ctx->b_cfg = mp::BConfig{cfg->atoms128_above, cfg->atoms64_above, cfg->atoms32_above};
  return MP_OK;
}

mp_status mp_batched_get_config(const mp_ctx* ctx, mp_batched_config* cfg) {
  if (!ctx || !cfg || ctx->ragged) return MP_EINVAL;
  cfg->atoms128_above = ctx->b_cfg.atoms128_above;
  cfg->atoms64_above = ctx->b_cfg.atoms64_above;
  cfg->atoms32_above = ctx->b_cfg.atoms32_above;
  return MP_OK;
}

mp_status mp_ragged_set_config(mp_ctx* ctx, const mp_ragged_config* cfg) {
  if (!ctx || !cfg) return MP_EINVAL;
  if (!ctx->ragged) return fail(ctx, MP_EINVAL, "not a ragged context");
  mp::RConfig cf{cfg->threads, cfg->cols_per_wave, cfg->wgs_per_cu,
                 cfg->split == 0 ? kRaggedDefaultSplit : cfg->split};
  if (!mp::ragged_config_valid(cf, ctx->storage == MP_BF16))
    return fail(ctx, MP_EINVAL, "threads must be 256/512/1024, cols_per_wave 1/2/4, "
                                "wgs_per_cu 1..8, split 0..8");
  ctx->r_cfg = cf;
  return MP_OK;
}

mp_status mp_ragged_get_config(const mp_ctx* ctx, mp_ragged_config* cfg) {
  if (!ctx || !cfg || !ctx->ragged) return MP_EINVAL;
  cfg->threads = ctx->r_cfg.threads;
  cfg->cols_per_wave = ctx->r_cfg.cols_per_wave;
  cfg->wgs_per_cu = ctx->r_cfg.wgs_per_cu;
  cfg->split = ctx->r_cfg.split;
  return MP_OK;
}

// The work list for the current launch shape: instances most work first; an
// instance whose work exceeds the average per workgroup of the grid is cut
// into parts (at most cfg.split, each a share of its columns; at most
// kMaxRaggedSplit instances are cut), consecutive in the list.
static mp_status ragged_items(mp_ctx* c, int grid, hipStream_t s) {
  if (c->r_nitems > 0 && memcmp(&c->r_items_cfg, &c->r_cfg, sizeof(mp::RConfig)) == 0)
    return MP_OK;
  double total = 0.0;
  for (double w : c->r_est) total += w;
  const double target = total / std::max(grid, 1);
  std::vector<mp::RItem> items;
  items.reserve(c->r_count * 2);
  int nslots = 0;
  for (int id : c->r_order) {
    int parts = 1;
    if (c->r_cfg.split > 1 && nslots < kMaxRaggedSplit && target > 0.0) {
      const double want = std::ceil(c->r_est[id] / target);
      parts = static_cast<int>(std::min<double>(want, c->r_cfg.split));
      parts = std::max(1, std::min<int>(parts, static_cast<int>(c->r_m[id])));
    }
    const int slot = parts > 1 ? nslots++ : -1;
    for (int p = 0; p < parts; ++p) items.push_back(mp::RItem{id, p, parts, slot});
  }
  HIP_TRY(c, hipMemcpyAsync(c->r_items, items.data(), sizeof(mp::RItem) * items.size(),
                            hipMemcpyHostToDevice, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  c->r_nitems = static_cast<int>(items.size());
  c->r_nslots = nslots;
  c->r_items_cfg = c->r_cfg;
  return MP_OK;
}

mp_status mp_solve_ragged(mp_ctx* ctx, const float* Y, float* X, float* R, const mp_opts* opts,
                          const int64_t* max_iters, mp_result* res, const mp_trace* trace,
                          void* stream) {
  if (!ctx) return MP_EINVAL;
  ctx->err.clear();
  mp_ctx* c = ctx;
  if (!c->ragged) return fail(c, MP_EINVAL, "not a ragged context (use mp_create_ragged)");
  if (!Y || !X || !opts) return fail(c, MP_EINVAL, "Y, X and opts must not be NULL");
  if (!(opts->eps >= 0.0) || !isfinite(opts->eps))
    return fail(c, MP_EINVAL, "eps must be finite and >= 0");
  if (opts->max_iters < 0) return fail(c, MP_EINVAL, "max_iters must be >= 0");
  if (opts->flags != 0) return fail(c, MP_EINVAL, "opts.flags must be 0");
  if (opts->rescore_k < 0 || opts->rescore_k > 8)
    return fail(c, MP_EINVAL, "rescore_k must be in 0..8");
  if (max_iters)
    for (int64_t i = 0; i < c->r_count; ++i)
      if (max_iters[i] < 0) return fail(c, MP_EINVAL, "max_iters entries must be >= 0");
  mp_trace tr{};
  const int64_t max_n = *std::max_element(c->r_n.begin(), c->r_n.end());
  if (mp_status ts = check_trace(c, trace, max_n); ts != MP_OK) return ts;
  if (trace) tr = *trace;
  HIP_TRY(c, hipSetDevice(c->device));
  hipStream_t s = static_cast<hipStream_t>(stream);
  c->carried_steps = 0;
  const bool lp = c->storage == MP_BF16;
  const int rk = opts->rescore_k == 0 ? mp::kLpTopK : opts->rescore_k;
  const long long* caps = max_iters ? c->r_caps : nullptr;
  if (max_iters)
    HIP_TRY(c, hipMemcpyAsync(c->r_caps, max_iters, sizeof(long long) * c->r_count,
                              hipMemcpyHostToDevice, s));
  // MP_RAGGED_SPIN_LIMIT limits the waits of the persistent launch, so it
  // selects that launch
  const mp::GramProb<float>* from = nullptr;  // problems handed on to it
  if ((!lp || rk == mp::kLpTopK) && !getenv("MP_RAGGED_SPIN_LIMIT") && c->gram_rmem) {
    c->prof_ms = 0.0;
    c->prof_launches = 0;
    bool gave_up = false;
    const mp_status gs = solve_gram_ragged(c, Y, X, opts, R, caps, tr, s, gave_up);
    if (gs != MP_OK) return gs;
    if (!gave_up)
      return batched_results(c, c->gram_hrst, c->r_count, res, "an instance's y holds NaN or Inf");
    from = static_cast<const mp::GramProb<float>*>(c->gram_rprobs);
  }
  int grid = c->num_cus * c->r_cfg.wgs_per_cu;
  if (mp_status is = ragged_items(c, grid, s); is != MP_OK) return is;
  if (grid > c->r_nitems) grid = c->r_nitems;
  const size_t lds = static_cast<size_t>(c->r_max_ld) * sizeof(float);
  // polls per wait between the parts of an instance before the solve fails;
  // MP_RAGGED_SPIN_LIMIT (a non-negative integer; 0 gives up at the first
  // wait) overrides it, so that tests can drive the failure path
  long long spin_limit = 1ll << 22;
  if (const char* env = getenv("MP_RAGGED_SPIN_LIMIT")) {
    char* end = nullptr;
    const long long v = strtoll(env, &end, 10);
    if (end != env && v >= 0) spin_limit = v;
  }

  // (re)capture the solve as a graph when its arguments change
  struct Key {
    const void *y, *x, *r, *caps, *ti, *tc, *trr, *tres, *from;
    double eps;
    long long cap_all, tcap, tldr, spin;
    int rk, threads, cc, grid, split, nitems, nslots, pad;
  } key{Y, X, R, caps, tr.idx, tr.coef, tr.rr, tr.r, from, opts->eps, opts->max_iters, tr.cap, tr.ldr,
        spin_limit, rk, c->r_cfg.threads, c->r_cfg.cols_per_wave, grid, c->r_cfg.split,
        c->r_nitems, c->r_nslots, 0};
  const unsigned char* kb = reinterpret_cast<const unsigned char*>(&key);
  std::vector<unsigned char> kv(kb, kb + sizeof key);
  if (!c->r_graph || kv != c->r_graph_key) {
    if (c->r_graph) {
      (void)hipGraphExecDestroy(c->r_graph);
      c->r_graph = nullptr;
    }
    HIP_TRY(c, hipStreamBeginCapture(c->r_cap_stream, hipStreamCaptureModeThreadLocal));
    hipError_t le = mp::launch_ragged(c->r_cfg, lp, grid, lds, c->r_inst, c->r_items,
                                      c->r_nitems, Y, X, R, caps, opts->max_iters, opts->eps,
                                      rk, c->r_res, c->r_queue, c->r_slots, c->r_nslots,
                                      spin_limit, from, tr, c->r_cap_stream);
    hipGraph_t g = nullptr;
    hipError_t ee = hipStreamEndCapture(c->r_cap_stream, &g);
    if (le != hipSuccess || ee != hipSuccess) {
      if (g) (void)hipGraphDestroy(g);
      return fail(c, MP_EDEVICE, std::string("capture: ") +
                                     hipGetErrorString(le != hipSuccess ? le : ee));
    }
    hipError_t ie = hipGraphInstantiate(&c->r_graph, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (ie != hipSuccess) {
      c->r_graph = nullptr;
      return fail(c, MP_EDEVICE, std::string("instantiate: ") + hipGetErrorString(ie));
    }
    c->r_graph_key = kv;
  }
  c->prof_ms = 0.0;
  c->prof_launches = 0;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (c->profiling) {
    e0 = c->ev[0];
    e1 = c->ev[1];
    HIP_TRY(c, hipEventRecord(e0, s));
  }
  HIP_TRY(c, hipGraphLaunch(c->r_graph, s));
  if (e1) HIP_TRY(c, hipEventRecord(e1, s));
  HIP_TRY(c, hipMemcpyAsync(c->h_rres, c->r_res, sizeof(mp::RResult) * c->r_count,
                            hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipMemcpyAsync(c->h_rq, c->r_queue, sizeof(mp::RQueue), hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (e1) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, e0, e1) == hipSuccess) {
      c->prof_ms = ms;
      c->prof_launches = 1;
    }
  }
  bool nonfinite = false, internal = false;
  for (int64_t i = 0; i < c->r_count; ++i) {
    mp::RResult d = c->h_rres[i];
    if (from && c->gram_hrst[i].pad[0] == 0) {  // decoded before the launch
      const mp::DevState& g = c->gram_hrst[i];
      d = mp::RResult{g.t, g.yy, g.rr, g.reason, 0};
    }
    nonfinite |= d.reason == mp::kStopNonFinite;
    internal |= d.reason == mp::kStopInternal;
    if (res) {
      res[i].iters = d.t;
      res[i].yy = d.yy;
      res[i].rr = d.rr;
      res[i].stop_reason = d.reason;
      res[i].persistent = 0;
    }
  }
  if (c->h_rq->fail)
    return fail(c, MP_EDEVICE, "a wait between the parts of an instance gave up");
  if (internal)
    return fail(c, MP_EDEVICE, "internal error: a selected index fell outside the dictionary");
  if (nonfinite) return fail(c, MP_ENONFINITE, "an instance's y holds NaN or Inf");
  return MP_OK;
}

}  // extern "C"
