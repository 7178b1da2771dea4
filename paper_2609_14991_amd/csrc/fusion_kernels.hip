// The C ABI entry points fusion_step / fusion_run and their several-LM forms:
// argument checks, the choice of kernel and launch shape, the exchange memory.
// The kernels are in fusion_device.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "fusion_shapes.h"

namespace fusion {

static thread_local std::string t_err;

int set_error(int code, const std::string &msg) {
  t_err = msg;
  return code;
}

int hip_error(hipError_t e, const char *what) {
  return set_error(FUSION_E_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

namespace {

__device__ int g_status;

// Beam exchange memory of fusion_run_lms_noalloc, one copy per GPU, held until
// the process ends.  Host code never passes this name to a kernel: it is a
// host-side stand-in, not a device address.  The device address comes from
// hipGetSymbolAddress (static_scratch below) and is what the kernels receive.
constexpr size_t kStaticScratchBytes = FUSION_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned long long scratch[kStaticScratchBytes / sizeof(unsigned long long)];

__global__ void zero_ints(int *p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

// ---------------------------------------------------------------------------
// launch
// ---------------------------------------------------------------------------
// lanes per hypothesis and 4-token strips per lane for a vocabulary
Shape shape_for(int V) {
  if (V <= 256) return {64, 1, 256};
  if (V <= 1024) return {256, 1, 1024};
  if (V <= 4096) return {1024, 1, 4096};
  return {1024, 2, 8192};
}

// the kernel of a shape (each shape and LM count is compiled in a file of its own);
// two LMs are compiled for vocabularies up to 4096 (two LMs at 8192 need more LDS
// than a workgroup has)
KernelFn pick(const Shape &sh, int km, bool al, int mode, int n_lm) {
  if (n_lm == 2) {
    if (sh.W == 64) return pick_w64_2lm(km, al, mode);
    if (sh.W == 256) return pick_w256_2lm(km, al, mode);
    return sh.NC == 1 ? pick_w1024_2lm(km, al, mode) : nullptr;
  }
  if (sh.W == 64) return pick_w64(km, al, mode);
  if (sh.W == 256) return pick_w256(km, al, mode);
  return sh.NC == 1 ? pick_w1024(km, al, mode) : pick_w1024x2(km, al, mode);
}

// dynamic LDS of a launch: per LM the dense row and the arc entries, the first
// LM's context row (rows of at most 4096 tokens), the phrase entries, with one LM
// the phrase entry values (rows of at most 4096 tokens), the phrase side tables
// and per LM the top-level next states
size_t dyn_lds_bytes(int Vp, int n_lm) {
  return (size_t)Vp * (12 * n_lm + 4 + (Vp <= 4096 ? 4 : 0) + (n_lm == 1 && Vp <= 4096 ? 4 : 0)) +
         (size_t)4 * (kAux * (2 + n_lm) + 4);
}

struct DeviceInfo {
  int lds_per_block = 0, cus = 0;
  int *status = nullptr;  // device address of g_status
  bool ok = false;
};

DeviceInfo device_info() {
  static std::mutex mu;
  static DeviceInfo cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return {};
  std::lock_guard<std::mutex> lk(mu);
  if (!cache[dev].ok) {
    int v = 0, c = 0;
    if (hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess) return {};
    if (hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return {};
    void *st = nullptr;
    if (hipGetSymbolAddress(&st, HIP_SYMBOL(g_status)) != hipSuccess) return {};
    cache[dev].status = static_cast<int *>(st);
    cache[dev].lds_per_block = v;
    cache[dev].cus = c;
    cache[dev].ok = true;
  }
  return cache[dev];
}

// The device address of this GPU's static scratch array, looked up once per
// device (with that device current) and kept; nullptr after a failed lookup.
int static_scratch(unsigned long long **out) {
  static std::mutex mu;
  static unsigned long long *ptr[64] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_error(e, "hipGetDevice");
  if (dev < 0 || dev >= 64) return set_error(FUSION_E_UNSUPPORTED, "device index beyond 63");
  std::lock_guard<std::mutex> lk(mu);
  if (!ptr[dev]) {
    void *a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_error(e, "hipGetSymbolAddress(scratch)");
    ptr[dev] = reinterpret_cast<unsigned long long *>(a);
  }
  *out = ptr[dev];
  return FUSION_OK;
}

// Per device and kernel: its static LDS, resident workgroups per CU at the
// launch's dynamic LDS, and whether that dynamic LDS has been granted; looked up
// once (the dynamic LDS of a kernel is fixed by its template shape)
struct KernelInfo {
  const void *fn = nullptr;
  int dev = -1;
  size_t static_lds = 0;
  int per_cu = 0;
};

int kernel_info(KernelFn fn, int W, size_t dyn, int lds_per_block, KernelInfo *out) {
  static std::mutex mu;
  static std::vector<KernelInfo> cache;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_error(e, "hipGetDevice");
  const void *f = reinterpret_cast<const void *>(fn);
  std::lock_guard<std::mutex> lk(mu);
  for (const KernelInfo &ki : cache)
    if (ki.fn == f && ki.dev == dev) {
      *out = ki;
      return FUSION_OK;
    }
  KernelInfo ki;
  ki.fn = f;
  ki.dev = dev;
  hipFuncAttributes attr;
  e = hipFuncGetAttributes(&attr, f);
  if (e != hipSuccess) return hip_error(e, "hipFuncGetAttributes");
  ki.static_lds = attr.sharedSizeBytes;
  if (dyn + ki.static_lds > (size_t)lds_per_block)
    return set_error(FUSION_E_UNSUPPORTED, "vocabulary too large for the device's LDS");
  e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn);
  if (e != hipSuccess) return hip_error(e, "hipFuncSetAttribute");
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&ki.per_cu, f, W, dyn);
  if (e != hipSuccess) return hip_error(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
  cache.push_back(ki);
  *out = ki;
  return FUSION_OK;
}

// fixed: caller-provided exchange memory of fixed_words 64-bit words (no
// allocation); nullptr: the exchange is allocated stream-ordered per call.
// keep_exchange: the call continues a frame loop whose earlier calls used the
// same exchange with p.t_base counting their frames, so its records need no
// reset (only when one launch holds every stream; otherwise it is reset anyway)
int launch(Params &p, int n_hyp, hipStream_t stream, unsigned long long *fixed = nullptr, size_t fixed_words = 0,
           bool keep_exchange = false) {
  const Shape sh = shape_for(p.V);
  const int km = p.k <= 1 ? 1 : p.k <= 4 ? 4 : 8;
  const bool al = (p.V % 4 == 0) && ((uintptr_t)p.logits % 16 == 0) && (!p.fused || (uintptr_t)p.fused % 16 == 0);
  const int mode = p.step_mode ? kModeStep : p.B == 1 ? kModeGreedy : p.B * p.k > 64 ? (p.recombine ? kModeBeamRCWide : kModeBeamWide)
                                                             : (p.recombine ? kModeBeamRC : kModeBeam);
  KernelFn fn = pick(sh, km, al, mode, p.n_lm);
  if (!fn) return set_error(FUSION_E_UNSUPPORTED, "two LMs need V <= 4096");
  const DeviceInfo di = device_info();
  if (!di.ok) return set_error(FUSION_E_HIP, "cannot query the device");
  p.status = di.status;
  const size_t dyn = dyn_lds_bytes(sh.Vp, p.n_lm);
  KernelInfo ki;
  int rc0 = kernel_info(fn, sh.W, dyn, di.lds_per_block, &ki);
  if (rc0 != FUSION_OK) return rc0;
  hipError_t e = hipSuccess;
  p.s_off = 0;
  p.xcd_map = 0;
  if (p.B == 1 || p.step_mode) {
    hipLaunchKernelGGL(fn, dim3(n_hyp), dim3(sh.W), dyn, stream, p);
    e = hipGetLastError();
    return e == hipSuccess ? FUSION_OK : hip_error(e, "fusion kernel launch");
  }
  // beam: a stream's workgroups meet every frame.  They take their slots from
  // arrival counters (see the kernel), which keeps a launch free of deadlock
  // even when other work holds part of the device, provided the incomplete
  // streams (one per blockIdx class, at most 8 x (B - 1) workgroups) cannot
  // fill it.  A launch holds no more streams than fit at once, so that no
  // workgroup waits at a rendezvous for a sibling that has yet to start behind
  // whole streams (the wait is bounded); further streams run in further launches
  const long resident = (long)ki.per_cu * di.cus;
  if (resident <= 8L * (p.B - 1)) return set_error(FUSION_E_UNSUPPORTED, "a beam does not fit on the device");
  // exchange records: 2 buffers x B x k candidates x (3 + n_lm (+1 recombining)) words per
  // stream, then the 8 arrival counters (4 words)
  const size_t stream_words = (size_t)2 * p.B * p.k * (3 + p.n_lm + (p.recombine ? 1 : 0));
  constexpr size_t kTicketWords = 4;
  // 8 or more streams are dealt over the 8 blockIdx classes, i.e. XCDs, whatever
  // their number: a class short of a stream has B workgroups that exit at once.  An
  // XCD must then hold its share of the streams.  (Rounding a launch down to
  // whole multiples of 8 streams split 23 streams of 8 slots, two LMs, 2,500
  // tokens into launches of 16 and 7: 2.20 ms instead of 1.13 ms for 60
  // frames.)  Fewer streams are spread over the whole device: by class, a single
  // stream would always be XCD 0's, several calls at once would share that XCD
  // while the others idle, and n calls of B slots whose incomplete streams fill it
  // (n (B - 1) of its slots) would hold each other off until the rendezvous
  // times out.  Spread, such calls have the device's room.  Measured over 60
  // frames, 1 to 7 streams: 2 to 4 slots 0-4 % slower spread, 8 slots -2 to 4 %, 16
  // slots 1-5 % faster.
  const long per_xcd = resident / 8;
  const bool by_xcd = per_xcd >= p.B;
  int s_batch = (int)std::min<long>(p.S, by_xcd ? 8 * (per_xcd / p.B) : resident / p.B);
  if (fixed) {
    if (stream_words + kTicketWords > fixed_words)
      return set_error(FUSION_E_UNSUPPORTED, "one stream's beam exchange exceeds the static scratch");
    s_batch = (int)std::min<size_t>((size_t)s_batch, (fixed_words - kTicketWords) / stream_words);
  }
  const size_t xwords = (size_t)s_batch * stream_words + kTicketWords;
  void *xbuf = fixed;
  if (!fixed) {
    e = hipMallocAsync(&xbuf, xwords * sizeof(unsigned long long), stream);
    if (e != hipSuccess) return hip_error(e, "hipMallocAsync");
  }
  p.xchg = reinterpret_cast<unsigned long long *>(xbuf);
  p.tickets = reinterpret_cast<unsigned *>(p.xchg + (size_t)s_batch * stream_words);
  int rc = FUSION_OK;
  for (int s0 = 0; s0 < p.S && rc == FUSION_OK; s0 += s_batch) {
    const int ns = std::min(s_batch, p.S - s0);
    // tag 0 (no frame uses it) everywhere and the counters at 0, so that neither
    // uninitialised memory nor an earlier batch's records can pass for the
    // current frame's (a frame loop that keeps the exchange relies on its
    // global frame numbers and on the counters resetting themselves)
    if (!(keep_exchange && s_batch >= p.S)) {
      const int n_ints = (int)(xwords * 2);
      hipLaunchKernelGGL(zero_ints, dim3(std::min(64, (n_ints + 255) / 256)), dim3(256), 0, stream,
                         reinterpret_cast<int *>(xbuf), n_ints);
      e = hipGetLastError();
      if (e != hipSuccess) {
        rc = hip_error(e, "exchange reset launch");
        break;
      }
    }
    Params q = p;
    q.s_off = s0;
    q.n_str = ns;
    q.xcd_map = by_xcd && ns >= 8 ? 1 : 0;
    hipLaunchKernelGGL(fn, dim3((q.xcd_map ? (ns + 7) / 8 * 8 : ns) * p.B), dim3(sh.W), dyn, stream, q);
    e = hipGetLastError();
    if (e != hipSuccess) rc = hip_error(e, "fusion kernel launch");
  }
  if (!fixed) {
    hipError_t e2 = hipFreeAsync(xbuf, stream);
    if (rc == FUSION_OK && e2 != hipSuccess) rc = hip_error(e2, "hipFreeAsync");
  }
  return rc;
}

int check_common(const NgramTables *const *lms, const float *alphas, int32_t n_lm, const BoostTrie *trie,
                 const float *logits, int32_t V, int32_t k, int32_t blank_id, int32_t blank_mode, float beta,
                 bool need_logits = true) {
  if (n_lm < 1 || n_lm > FUSION_MAX_LMS) return set_error(FUSION_E_ARG, "n_lm out of range");
  if (!lms || !alphas) return set_error(FUSION_E_ARG, "NULL LM list or weights");
  for (int i = 0; i < n_lm; ++i) {
    if (!lms[i]) return set_error(FUSION_E_ARG, "NULL n-gram tables");
    if (V != lms[i]->dev.V) return set_error(FUSION_E_ARG, "V does not match the n-gram tables");
    if (blank_id != lms[i]->dev.blank) return set_error(FUSION_E_ARG, "blank_id does not match the n-gram tables");
    if (!std::isfinite(alphas[i])) return set_error(FUSION_E_ARG, "non-finite fusion weight");
  }
  if (need_logits && !logits) return set_error(FUSION_E_ARG, "NULL logits");
  if (trie && (trie->dev.V != V || trie->dev.blank != blank_id))
    return set_error(FUSION_E_ARG, "phrase tree built for another vocabulary or blank");
  if (k < 1 || k > FUSION_MAX_K || k > V) return set_error(FUSION_E_ARG, "k out of range");
  if (blank_mode != FUSION_BLANK_AM && blank_mode != FUSION_BLANK_COMPETE) return set_error(FUSION_E_ARG, "unknown blank_mode");
  if (blank_mode == FUSION_BLANK_AM && k != 1) return set_error(FUSION_E_ARG, "FUSION_BLANK_AM needs k == 1");
  if (!std::isfinite(beta)) return set_error(FUSION_E_ARG, "non-finite fusion weight");
  return FUSION_OK;
}

Params make_params(const NgramTables *const *lms, const float *alphas, int32_t n_lm, const BoostTrie *trie) {
  Params p;
  std::memset(&p, 0, sizeof p);
  for (int i = 0; i < n_lm; ++i) {
    p.lm[i] = lms[i]->dev;
    p.lam[i] = alphas[i];
  }
  p.n_lm = n_lm;
  if (trie) p.tr = trie->dev;
  p.has_trie = trie != nullptr;
  return p;
}

int step_impl(const NgramTables *const *lms, const float *alphas, int32_t n_lm, const BoostTrie *trie,
              const float *logits, const int32_t *lm_state, const int32_t *boost_state, int32_t H, int32_t V,
              float beta, int32_t blank_id, int32_t k, int32_t blank_mode, float *fused, int32_t *tokens,
              float *scores, int32_t *next_lm, int32_t *next_boost, hipStream_t stream) {
  int rc = check_common(lms, alphas, n_lm, trie, logits, V, k, blank_id, blank_mode, beta, H != 0);
  if (rc != FUSION_OK) return rc;
  if (H < 0 || H > (1 << 24)) return set_error(FUSION_E_ARG, "H out of range");
  if (H == 0) return FUSION_OK;  // no hypotheses: no buffer is read or written
  if (!lm_state || !tokens || !scores || !next_lm || !next_boost || (trie && !boost_state))
    return set_error(FUSION_E_ARG, "NULL state or output buffer");
  Params p = make_params(lms, alphas, n_lm, trie);
  p.logits = logits;
  p.lm_state = const_cast<int32_t *>(lm_state);
  p.boost_state = const_cast<int32_t *>(boost_state);
  p.tokens = tokens;
  p.scores = scores;
  p.next_lm = next_lm;
  p.next_boost = next_boost;
  p.fused = fused;
  p.T = 1;
  p.S = H;
  p.B = 1;
  p.V = V;
  p.k = k;
  p.blank = blank_id;
  p.mode = blank_mode;
  p.step_mode = 1;
  p.beta = beta;
  return launch(p, H, stream);
}

int run_impl(const NgramTables *const *lms, const float *alphas, int32_t n_lm, const BoostTrie *trie,
             const float *logits, int32_t T, int32_t S, int32_t B, int32_t V, int32_t k, float beta,
             int32_t blank_id, int32_t blank_mode, int32_t *lm_state, int32_t *boost_state, double *hyp_score,
             int32_t *tokens, int32_t *parents, float *fused, int64_t *traffic, int32_t flags, uint64_t *hist,
             hipStream_t stream, bool no_alloc = false, unsigned long long *xbuf = nullptr, size_t xbuf_words = 0,
             int32_t t_base = 0) {
  int rc = check_common(lms, alphas, n_lm, trie, logits, V, k, blank_id, blank_mode, beta, T != 0 && S != 0);
  if (rc != FUSION_OK) return rc;
  if (T < 0 || S < 0 || B < 1 || B > FUSION_MAX_BEAM) return set_error(FUSION_E_ARG, "T, S or B out of range");
  if ((int64_t)S * B > (1 << 24)) return set_error(FUSION_E_ARG, "too many hypotheses");
  if (B == 1 && k != 1) return set_error(FUSION_E_ARG, "greedy decoding (B == 1) needs k == 1");
  if (B > 1 && blank_mode != FUSION_BLANK_COMPETE) return set_error(FUSION_E_ARG, "beam decoding needs FUSION_BLANK_COMPETE");
  if (flags & ~FUSION_RUN_RECOMBINE) return set_error(FUSION_E_ARG, "unknown flags");
  if (T == 0 || S == 0) return FUSION_OK;  // nothing to decode: no buffer is read or written
  if (!lm_state || !tokens || (trie && !boost_state)) return set_error(FUSION_E_ARG, "NULL state or output buffer");
  if (B > 1 && (!hyp_score || !parents)) return set_error(FUSION_E_ARG, "beam decoding needs hyp_score and parents");
  Params p = make_params(lms, alphas, n_lm, trie);
  p.logits = logits;
  p.lm_state = lm_state;
  p.boost_state = boost_state;
  p.hyp_score = hyp_score;
  p.tokens = tokens;
  p.parents = parents;
  p.fused = fused;
  p.traffic = traffic;
  p.T = T;
  p.S = S;
  p.B = B;
  p.V = V;
  p.k = k;
  p.blank = blank_id;
  p.mode = blank_mode;
  p.step_mode = 0;
  p.beta = beta;
  p.recombine = (flags & FUSION_RUN_RECOMBINE) && B > 1;
  p.hist = p.recombine ? reinterpret_cast<unsigned long long *>(hist) : nullptr;
  p.t_base = t_base;
  if (B == 1 && T == 1 && !traffic) {
    // One greedy frame is a step with its states in place.  In mode A the frame loop
    // would look through the frame for blank and then begin it again; a step
    // decides blank by the way.  (It has no byte count.)  Kernel time of one frame in
    // mode A, half of the frames blank, 64 streams: 128 tokens 9.4 us in a frame
    // loop, 6.6 as a step; 1024: 8.6, 6.8; 4096: 9.9, 7.7; 8190: 12.2, 10.1.  (A
    // single stream whose one frame is blank's: 4.8 and 5.7 at 1024 tokens)
    p.step_mode = 1;
    p.next_lm = lm_state;
    p.next_boost = trie ? boost_state : nullptr;
  }
  if (xbuf) return launch(p, S * B, stream, xbuf, xbuf_words, t_base > 0);
  if (no_alloc) {
    unsigned long long *xs = nullptr;
    rc = static_scratch(&xs);
    if (rc != FUSION_OK) return rc;
    return launch(p, S * B, stream, xs, kStaticScratchBytes / sizeof(unsigned long long));
  }
  return launch(p, S * B, stream);
}

}  // namespace
}  // namespace fusion

using namespace fusion;

extern "C" const char *fusion_last_error(void) { return t_err.c_str(); }

extern "C" int fusion_device_status(hipStream_t stream, int32_t *code) {
  if (!code) return set_error(FUSION_E_ARG, "NULL code");
  hipError_t e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return hip_error(e, "hipStreamSynchronize");
  int v = 0;
  e = hipMemcpyFromSymbol(&v, HIP_SYMBOL(g_status), sizeof(int), 0, hipMemcpyDeviceToHost);
  if (e != hipSuccess) return hip_error(e, "hipMemcpyFromSymbol");
  int zero = 0;
  e = hipMemcpyToSymbol(HIP_SYMBOL(g_status), &zero, sizeof(int), 0, hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_error(e, "hipMemcpyToSymbol");
  int32_t end_bits = 0;
  const int rc = end_status_take(&end_bits);
  if (rc != FUSION_OK) return rc;
  *code = v | end_bits;
  return FUSION_OK;
}

extern "C" int fusion_step(const NgramTables *lm, const BoostTrie *trie, const float *logits,
                           const int32_t *lm_state, const int32_t *boost_state, int32_t H, int32_t V,
                           float lambda, float beta, int32_t blank_id, int32_t k, int32_t blank_mode,
                           float *fused, int32_t *tokens, float *scores, int32_t *next_lm,
                           int32_t *next_boost, hipStream_t stream) {
  return step_impl(&lm, &lambda, 1, trie, logits, lm_state, boost_state, H, V, beta, blank_id, k, blank_mode,
                   fused, tokens, scores, next_lm, next_boost, stream);
}

extern "C" int fusion_step_lms(const NgramTables *const *lms, const float *alphas, int32_t n_lm,
                               const BoostTrie *trie, const float *logits, const int32_t *lm_state,
                               const int32_t *boost_state, int32_t H, int32_t V, float beta, int32_t blank_id,
                               int32_t k, int32_t blank_mode, float *fused, int32_t *tokens, float *scores,
                               int32_t *next_lm, int32_t *next_boost, hipStream_t stream) {
  return step_impl(lms, alphas, n_lm, trie, logits, lm_state, boost_state, H, V, beta, blank_id, k, blank_mode,
                   fused, tokens, scores, next_lm, next_boost, stream);
}

extern "C" int fusion_run(const NgramTables *lm, const BoostTrie *trie, const float *logits, int32_t T,
                          int32_t S, int32_t B, int32_t V, int32_t k, float lambda, float beta,
                          int32_t blank_id, int32_t blank_mode, int32_t *lm_state, int32_t *boost_state,
                          double *hyp_score, int32_t *tokens, int32_t *parents, float *fused,
                          int64_t *traffic, hipStream_t stream) {
  return run_impl(&lm, &lambda, 1, trie, logits, T, S, B, V, k, beta, blank_id, blank_mode, lm_state,
                  boost_state, hyp_score, tokens, parents, fused, traffic, 0, nullptr, stream);
}

extern "C" int fusion_run_lms(const NgramTables *const *lms, const float *alphas, int32_t n_lm,
                              const BoostTrie *trie, const float *logits, int32_t T, int32_t S, int32_t B,
                              int32_t V, int32_t k, float beta, int32_t blank_id, int32_t blank_mode,
                              int32_t *lm_state, int32_t *boost_state, double *hyp_score, int32_t *tokens,
                              int32_t *parents, float *fused, int64_t *traffic, int32_t flags,
                              uint64_t *hist, hipStream_t stream) {
  return run_impl(lms, alphas, n_lm, trie, logits, T, S, B, V, k, beta, blank_id, blank_mode, lm_state,
                  boost_state, hyp_score, tokens, parents, fused, traffic, flags, hist, stream);
}

extern "C" int fusion_run_lms_noalloc(const NgramTables *const *lms, const float *alphas, int32_t n_lm,
                                      const BoostTrie *trie, const float *logits, int32_t T, int32_t S,
                                      int32_t B, int32_t V, int32_t k, float beta, int32_t blank_id,
                                      int32_t blank_mode, int32_t *lm_state, int32_t *boost_state,
                                      double *hyp_score, int32_t *tokens, int32_t *parents, float *fused,
                                      int64_t *traffic, int32_t flags, uint64_t *hist, hipStream_t stream) {
  return run_impl(lms, alphas, n_lm, trie, logits, T, S, B, V, k, beta, blank_id, blank_mode, lm_state,
                  boost_state, hyp_score, tokens, parents, fused, traffic, flags, hist, stream, true);
}

extern "C" int fusion_run_projected(const NgramTables *const *lms, const float *alphas, int32_t n_lm,
                                    const BoostTrie *trie, const uint16_t *A, const uint16_t *W, const float *bias,
                                    int32_t K, float *logits, int32_t chunk, int32_t T, int32_t S, int32_t B,
                                    int32_t V, int32_t k,
                                    float beta, int32_t blank_id, int32_t blank_mode, int32_t *lm_state,
                                    int32_t *boost_state, double *hyp_score, int32_t *tokens, int32_t *parents,
                                    int32_t flags, uint64_t *hist, hipStream_t stream) {
  int rc = check_common(lms, alphas, n_lm, trie, nullptr, V, k, blank_id, blank_mode, beta, false);
  if (rc != FUSION_OK) return rc;
  if (T < 0 || S < 0 || B < 1 || B > FUSION_MAX_BEAM) return set_error(FUSION_E_ARG, "T, S or B out of range");
  if ((int64_t)S * B > (1 << 24)) return set_error(FUSION_E_ARG, "too many hypotheses");
  if (chunk < 1) return set_error(FUSION_E_ARG, "chunk must be at least 1");
  if (T == 0 || S == 0) return FUSION_OK;
  if (!A || !W || !logits) return set_error(FUSION_E_ARG, "NULL joint states, weight or logits workspace");
  const int64_t H = (int64_t)S * B;
  const int32_t C = std::min(chunk, T);
  if ((int64_t)C * H > INT32_MAX) return set_error(FUSION_E_ARG, "chunk * H exceeds the projection's row count");
  // the beam's exchange records, allocated once for all chunks (every stream at once)
  unsigned long long *xbuf = nullptr;
  size_t xwords = 0;
  if (B > 1) {
    // every stream's records and the arrival counters (4 words)
    xwords = (size_t)S * 2 * B * k * (3 + n_lm + ((flags & FUSION_RUN_RECOMBINE) ? 1 : 0)) + 4;
    hipError_t e = hipMallocAsync(reinterpret_cast<void **>(&xbuf), xwords * sizeof(unsigned long long), stream);
    if (e != hipSuccess) return hip_error(e, "hipMallocAsync");
  }
  for (int32_t t = 0; t < T && rc == FUSION_OK; t += C) {
    const int32_t n = std::min(C, T - t);
    // the chunk's logits of all H hypotheses from their joint hidden states
    rc = joint_project(A + (size_t)t * H * K, W, bias, (int32_t)(n * H), V, K, logits, stream);
    if (rc != FUSION_OK) break;
    rc = run_impl(lms, alphas, n_lm, trie, logits, n, S, B, V, k, beta, blank_id, blank_mode, lm_state, boost_state,
                  hyp_score, tokens + (size_t)t * H, parents ? parents + (size_t)t * H : nullptr, nullptr, nullptr,
                  flags, hist, stream, false, xbuf, xwords, t);
  }
  if (xbuf) {
    const hipError_t e = hipFreeAsync(xbuf, stream);
    if (rc == FUSION_OK && e != hipSuccess) rc = hip_error(e, "hipFreeAsync");
  }
  return rc;
}
