// The fusion kernel for gfx950: Eq. (1) of the paper (Sec. III-C) with greedy or
// top-k selection and a frame-synchronous beam.  Its launches and the C ABI entry
// points are in fusion_kernels.hip; each compiled shape is a file of its own
// (fusion_w*.hip).
//
// Work mapping.  One workgroup per hypothesis (W = 64, 256 or 1024 lanes),
// so a 64 x 4 beam keeps all 256 CUs busy.  Lane g owns the tokens
// y = (c * W + g) * 4 + j (j < 4, c < NC): every logits row read is a
// coalesced 16-byte strip per lane held in registers; the level-1 dense LM row
// goes straight from HBM into the workgroup's LDS row (global_load_lds), where
// the arcs of the longer contexts are then scattered.
//
// Per frame and hypothesis, the method's steps in order:
//   1  one load brings the state record (the whole backoff chain: backoffs and
//      arc ranges of every context level) and the phrase node; the logits row
//      and the dense row are issued alongside;
//   2  one load brings the arcs of all levels (flattened) and the phrase
//      transitions of the state; meanwhile the row statistics are reduced
//      (online max / sum-exp, raw argmax);
//   3  the arcs are scattered into LDS level by level, each summed with the
//      backoffs above its level (the addition order of the backoff
//      recursion), and the phrase transitions with their entry values;
//   4  key = (x + lambda*lm) + beta*boost per owned token, top-k per lane, per
//      wave (shuffles) and per hypothesis; each candidate carries where its
//      next LM / phrase state comes from, so no further lookup is needed;
//   5  beam: the B workgroups of a stream publish their candidates as tagged
//      records, poll for all of the stream's, and each ranks the B*k (fp64 running
//      score) to take its own new hypothesis.
// No MFMA: ~10 flops per score over gathered data.
#pragma once

#include <hip/hip_runtime.h>

#include <climits>
#include <cmath>

#include "fusion_shapes.h"

namespace fusion {

namespace {

constexpr int kMaxWaves = 16;
constexpr int kMaxLevels = FUSION_MAX_ORDER;  // context levels 1..N-1 <= 5
constexpr int kRecW = 16;                     // words read per state record: record_stride(FUSION_MAX_ORDER)
constexpr int kSpinLimit = 1 << 21;           // bounded wait at the beam rendezvous (polls, each waiting
                                              // for its loads: about a second)

static __device__ __align__(64) int32_t g_zero_words[16];  // never written: the record and node of "no state"


// The kernel's argument block (its one argument, a Params, at offset 0) through an
// address the compiler cannot see through: a field read from it is read where it
// is used.  For pointers that only rare paths of the frame loop need; read as
// plain arguments, they are hoisted out of the loop and hold scalar registers
// across it (pushing other values into spill slots)
__device__ __forceinline__ const __attribute__((address_space(4))) Params &args_here() {
  const __attribute__((address_space(4))) char *kb =
      (const __attribute__((address_space(4))) char *)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(kb));
  return *(const __attribute__((address_space(4))) Params *)kb;
}
__device__ __forceinline__ bool before(float ka, int ya, float kb, int yb) {
  return ka > kb || (ka == kb && ya < yb);
}
__device__ __forceinline__ float as_float(int v) { return __int_as_float(v); }
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
// the splitmix64 finalizer: a 64-bit mix for the beam's history hashes
__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
// log(exp(a) + exp(b)) in fp64.  Not inlined: the merges that call it are rare,
// and inlined, the constants of its exp and log1p would stay in vector
// registers across the whole frame loop of the recombining kernel
__device__ __attribute__((noinline)) double log_add(double a, double b) {
  const double m = a > b ? a : b, d = a > b ? b - a : a - b;
  return m + log1p(exp(d));
}
__device__ __forceinline__ unsigned long long umin64(unsigned long long a, unsigned long long b) {
  return a < b ? a : b;
}

// raw buffer access to one V-wide row: a 4-SGPR descriptor and a per-lane
// byte offset; reads past the row return 0
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t row_rsrc(const float *base, int n) {
  // every field uniform (a descriptor the compiler cannot prove uniform costs a
  // readfirstlane loop around each access)
  const unsigned long long v = reinterpret_cast<unsigned long long>(base);
  const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)v);
  const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(v >> 32));
  float *ub = reinterpret_cast<float *>(((unsigned long long)hi << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, __builtin_amdgcn_readfirstlane(n * 4), 0x00020000);
}
__device__ __forceinline__ float4 row_load4(rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}
__device__ __forceinline__ float row_load1(rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
__device__ __forceinline__ void row_store4(rsrc_t r, float4 v, int voff, int soff) {
  typedef int v4i __attribute__((ext_vector_type(4)));
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v), r, voff, soff, 0);
}
__device__ __forceinline__ void row_store1(rsrc_t r, float v, int voff, int soff) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), r, voff, soff, 0);
}
typedef __attribute__((address_space(3))) void *lds_ptr_t;

// record words: [0] c_1 | m << 16, [1] state id, [2 + 3(L-2) + {0,1,2}] = (bo, first arc, arcs) of level L
__device__ __forceinline__ constexpr int rec_bo_word(int L) { return 2 + 3 * (L - 2); }
__device__ __forceinline__ constexpr int rec_beg_word(int L) { return 3 + 3 * (L - 2); }
__device__ __forceinline__ constexpr int rec_cnt_word(int L) { return 4 + 3 * (L - 2); }
// the record word naming the chain's context row (record_ctx_word)
__device__ __forceinline__ constexpr int rec_ctx_word(int N) { return 2 + 3 * (N > 2 ? N - 2 : 0); }

// ---- wave-level reductions with DPP moves (no LDS) ------------------------------
// rows of 16 lanes: quad_perm [1,0,3,2], quad_perm [2,3,0,1], row_half_mirror,
// row_mirror; then row_bcast:15 (rows 1, 3) and row_bcast:31 (rows 2, 3) carry
// the row results to lane 63
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_f(float ident, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(ident), __float_as_int(v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp_f<0xB1, 0xF>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x4E, 0xF>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x141, 0xF>(-INFINITY, v));
  return fmaxf(v, dpp_f<0x140, 0xF>(-INFINITY, v));
}
__device__ __forceinline__ float row_sum(float v) {
  v = v + dpp_f<0xB1, 0xF>(0.0f, v);
  v = v + dpp_f<0x4E, 0xF>(0.0f, v);
  v = v + dpp_f<0x141, 0xF>(0.0f, v);
  return v + dpp_f<0x140, 0xF>(0.0f, v);
}
// uniform maximum over the wave (-0 and +0 may come out either way)
__device__ __forceinline__ float wave_max_f(float v) {
  v = row_max(v);
  v = fmaxf(v, dpp_f<0x142, 0xA>(-INFINITY, v));
  v = fmaxf(v, dpp_f<0x143, 0xC>(-INFINITY, v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// uniform sum over the wave
__device__ __forceinline__ float wave_sum(float v) {
  v = row_sum(v);
  v = v + dpp_f<0x142, 0xA>(0.0f, v);
  v = v + dpp_f<0x143, 0xC>(0.0f, v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
// order-preserving map of non-NaN floats onto int32 (x + 0.0 first folds -0
// into +0, so equal floats map to equal ints); an involution
__device__ __forceinline__ int ord_key(float x) {
  const int b = __float_as_int(x + 0.0f);
  return b ^ ((b >> 31) & 0x7FFFFFFF);
}
__device__ __forceinline__ float key_of(int i) { return __int_as_float(i ^ ((i >> 31) & 0x7FFFFFFF)); }
// (order-preserving key image, token id) as one unsigned 64-bit value, larger
// for a higher key and, at equal keys, for a lower id
__device__ __forceinline__ unsigned long long sel_order(int key, int y) {
  return ((unsigned long long)((uint32_t)key ^ 0x80000000u) << 32) | (unsigned long long)(~(uint32_t)y);
}
// the key of a composite's upper half
__device__ __forceinline__ int sel_key(int hi) { return (int)((uint32_t)hi ^ 0x80000000u); }
// uniform maximum of an int over the wave (identity INT_MIN)
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(INT_MIN, v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ int wave_max_i(int v) {
  v = max(v, dpp_i<0xB1, 0xF>(v));
  v = max(v, dpp_i<0x4E, 0xF>(v));
  v = max(v, dpp_i<0x141, 0xF>(v));
  v = max(v, dpp_i<0x140, 0xF>(v));
  v = max(v, dpp_i<0x142, 0xA>(v));
  v = max(v, dpp_i<0x143, 0xC>(v));
  return __builtin_amdgcn_readlane(v, 63);
}
// e^x through the hardware base-2 exponential (about 1e-6 relative error near
// the arguments used here, x <= 0)
__device__ __forceinline__ float exp_fast(float x) { return __builtin_amdgcn_exp2f(x * 1.4426950408889634f); }

// every lane of each 16-lane row ends with the row's best (key desc, id asc)
template <int CTRL>
__device__ __forceinline__ void dpp_best(float &k, int &y) {
  const float k2 = dpp_f<CTRL, 0xF>(-INFINITY, k);
  const int y2 = __builtin_amdgcn_update_dpp(INT_MAX, y, CTRL, 0xF, 0xF, false);
  if (before(k2, y2, k, y)) {
    k = k2;
    y = y2;
  }
}
__device__ __forceinline__ void row_best(float &k, int &y) {
  dpp_best<0xB1>(k, y);
  dpp_best<0x4E>(k, y);
  dpp_best<0x141>(k, y);
  dpp_best<0x140>(k, y);
}

// Barrier for data exchanged through LDS alone: waits for this wave's LDS
// operations but not for its vector-memory loads in flight (the next frame's
// logits).  __syncthreads would wait for those too (its release fence waits for
// every outstanding vector-memory operation).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Orders a wave's own LDS writes before its later LDS reads by other lanes (one
// wave's LDS operations complete in order; this keeps the compiler to it)
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
// The lane (below n <= 64) whose total has rank b, totals descending, lower lanes
// first among equals; -1 if fewer than b + 1 lanes hold a total.  tot: every lane's
// total in LDS (NaN: none), mine: this lane's.  Counting the totals ahead needs 16-byte
// LDS reads and one compare each; equal totals show as a rank that no lane or
// several lanes hold
__device__ __forceinline__ int slot_holder(const double *tot, double mine, int n, int lane, int b) {
  int gt = 0;
  for (int q0 = 0; q0 < n; q0 += 16) {
    double tv[16];
#pragma unroll
    for (int q = 0; q < 16; q += 2) {
      const double2 d = *reinterpret_cast<const double2 *>(&tot[q0 + q]);
      tv[q] = d.x;
      tv[q + 1] = d.y;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) gt += (int)(tv[q] > mine);
  }
  const bool live = lane < n && mine == mine;
  unsigned long long hold = __ballot(live && gt == b);
  if (hold == 0ull && __popcll(__ballot(live)) > b) {
    int r = gt;
#pragma unroll 1
    for (int j = 0; j < n; ++j) r += (int)(tot[j] == mine && j < lane);
    hold = __ballot(live && r == b);
  }
  return hold ? __ffsll((long long)hold) - 1 : -1;
}
constexpr int kHashSlots = 512;
// Beam recombination among n <= 64 Q candidates, Q per lane (lane, lane + 64, ..):
// candidates of equal history hash merge into the first of them in candidate
// order, whose total becomes the log-sum of theirs folded in that order; the
// others' totals become NaN.  hash: this lane's (Q = 1; with Q > 1 they are in hh
// already).  The first of each history is found through an LDS table: every candidate
// lowers its hash's slot to its own index; those whose slot went to another
// history try again with other bits of their hashes.  (Comparing all pairs took
// n steps of several instructions on one wave.)  Then each round folds the next
// member of every history at once
template <int Q>
__device__ __forceinline__ void merge_equal(double (&t)[Q], unsigned long long hash, int n, int lane, double *tot,
                                            unsigned long long *hh, int *tab) {
  const double none = __longlong_as_double(0x7FF8000000000000ll);
  unsigned long long hq[Q];
  int first[Q];
  bool todo[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int i = q * 64 + lane;
    todo[q] = t[q] == t[q];  // only candidates below n hold a total
    hq[q] = Q == 1 ? hash : (todo[q] ? hh[i] : 0ull);
    if (Q == 1) hh[i] = hash;
    if (i < n) tot[i] = t[q];
    first[q] = i;
  }
  for (int shift = 0;; shift += 9) {
    unsigned long long open = 0ull;
#pragma unroll
    for (int q = 0; q < Q; ++q) open |= __ballot(todo[q]);
    if (open == 0ull) break;
#pragma unroll
    for (int e = 0; e < kHashSlots; e += 256) *reinterpret_cast<int4 *>(&tab[e + lane * 4]) = make_int4(INT_MAX, INT_MAX, INT_MAX, INT_MAX);
    wave_lds_sync();
    int sl[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      // (once the hash's upper bits are used up, bits of a multiple of it.  The search ends
      // whatever the bits: in each round the least open candidate of every slot finds
      // itself there)
      sl[q] = (int)((shift < 45 ? hq[q] >> shift : hq[q] * 0x9E3779B97F4A7C15ull >> (shift % 50)) & (kHashSlots - 1));
      if (todo[q]) atomicMin(&tab[sl[q]], q * 64 + lane);
    }
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      if (todo[q]) {
        const int f = tab[sl[q]];
        if (hh[f] == hq[q]) {
          first[q] = f;
          todo[q] = false;
        }
      }
    }
    wave_lds_sync();
  }
  // members other than the first, next in order
  bool member[Q];
  unsigned long long left = 0ull;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    member[q] = first[q] != q * 64 + lane;
    left |= __ballot(member[q]);
  }
  if (left == 0ull) return;
  bool lead[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) lead[q] = !member[q] && t[q] == t[q];
  bool gone[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) gone[q] = member[q];
  while (left) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (lead[q]) tab[q * 64 + lane] = INT_MAX;
    wave_lds_sync();
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (member[q]) atomicMin(&tab[first[q]], q * 64 + lane);
    wave_lds_sync();
    left = 0ull;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int nx = lead[q] ? tab[q * 64 + lane] : INT_MAX;
      if (__ballot(nx != INT_MAX)) {
        if (nx != INT_MAX) t[q] = log_add(t[q], tot[nx]);
      }
      if (member[q] && tab[first[q]] == q * 64 + lane) member[q] = false;
      left |= __ballot(member[q]);
    }
    wave_lds_sync();
  }
#pragma unroll
  for (int q = 0; q < Q; ++q)
    if (gone[q]) t[q] = none;
}

// hypothesis state carried between frames (LDS, written by one lane)
template <int NL>
struct HypState {
  // per LM: where the next state comes from (an id; -1: reached from c1p by
  // token y; -(r + 2): reached from the context of context row r by token y),
  // the parent's c_1, the last token of the context (-1: from the record), the
  // id of the state scored this frame
  int lmsrc[NL], c1p[NL], c1[NL], cur_lm[NL];
  int qsrc, y, fl;  // phrase source, token; flags 1 alive, 2 invalid
  int cur_q;        // phrase state scored this frame
  double S;         // running beam score
  unsigned long long hist;  // 48-bit hash of the history (initial states, emitted tokens): recombination
};


template <int W, int NC, int KM, bool AL, int MODE, int NL>
__global__ void __launch_bounds__(W, W == 64 ? 1 : 4) fusion_kernel(Params p) {
  constexpr int NW = W / 64;
  constexpr int Vp = NC * 4 * W;
  constexpr int kUA = W >= 1024 ? 1 : 4;  // arcs per lane fetched in the second hop
  constexpr int kUD = W >= 1024 ? 1 : 2;  // phrase transitions per lane fetched in the second hop
  constexpr bool CTX = NC == 1;  // context rows used (an 8192-wide row pair would not fit the LDS)
  extern __shared__ __align__(16) unsigned char dyn[];
  // LDS rows, one entry per token: per LM, the dense level-1 row and the winning
  // explicit arc (stamp << 48 | level << 45 | offset << 32 | value bits, kept by
  // an atomic max, so the highest level wins whatever the order of the writes);
  // the phrase transition overriding the root's (stamp << 16 | transition + 1).
  // The stamp is the number of rows assembled so far: entries of earlier rows
  // compare lower and read as absent, so nothing is cleared per frame.  Row NL of
  // lmval holds the first LM's context row when its state has one: the LM row of
  // the deepest context of the chain with many successors, already resolved
  // through every level up to that context
  // With one LM the phrase term reads erow: per token the entry value E of the
  // phrase state after it, the root's unless this frame's phrase state
  // overrides the token.  Each lane puts its tokens back to the root's values
  // right after reading them, and the scatter writes the overrides; a frame that
  // keeps its rows finds them through ptag instead.
  constexpr bool ER = NL == 1 && NC == 1;  // (8192-wide rows: no room in the LDS)
  constexpr int kRows = NL + (CTX ? 1 : 0);
  float *lmval = reinterpret_cast<float *>(dyn);                                                  // [kRows][Vp]
  unsigned long long *arcw = reinterpret_cast<unsigned long long *>(dyn + 4 * kRows * Vp);        // [NL][Vp]
  uint32_t *ptag = reinterpret_cast<uint32_t *>(dyn + (4 * kRows + 8 * NL) * Vp);
  float *erow = reinterpret_cast<float *>(dyn + (4 * kRows + 8 * NL + 4) * Vp);                   // [Vp] if ER
  float *sE = reinterpret_cast<float *>(dyn + (4 * kRows + 8 * NL + 4 + (ER ? 4 : 0)) * Vp);  // sE[j + 1]: entry value of transition j
  int *sDT = reinterpret_cast<int *>(sE + kAux + 4);
  int *sTN = sDT + kAux;  // [NL][kAux]
  __shared__ float s_pm[kMaxWaves], s_ps[kMaxWaves];
  __shared__ int s_paid[kMaxWaves];
  __shared__ float s_lse;  // the current frame's log-sum-exp of the logits row
  __shared__ int s_am;     // and the lowest id holding its maximum
  __shared__ int s_nstat;  // waves done with the next frame's strip statistics
  __shared__ unsigned s_emit[2];  // greedy: which of 64 frames blank does not take
  // greedy: each wave's best, (key image, token, first LM's source, phrase source) and the
  // second LM's source; frames alternate between two buffers
  __shared__ __align__(16) int4 s_best[2][MODE == kModeGreedy ? kMaxWaves : 1];
  __shared__ int s_best1[2][MODE == kModeGreedy ? kMaxWaves : 1];
  __shared__ int w_key[kMaxWaves][KM];  // order-preserving images of the keys (ord_key)
  __shared__ int w_y[kMaxWaves][KM];
  // the best keys of 16 groups of lanes, and the hypothesis' listed entries
  // (compacted) and top K, all as sel_order composites (KM > 1)
  __shared__ __align__(16) int s_wmax[16];
  __shared__ __align__(16) unsigned long long s_sel[16];
  __shared__ unsigned long long s_win[KM];
  __shared__ HypState<NL> hs;
  // beam rendezvous staging (wave 0): candidate records (the second LM's source
  // and c_1 in s_xb), parent flags, totals
  constexpr bool RCM = MODE == kModeBeamRC || MODE == kModeBeamRCWide;
  constexpr int kCand = MODE == kModeBeamWide || MODE == kModeBeamRCWide ? FUSION_MAX_BEAM * FUSION_MAX_K : 64;
  constexpr int kStaged = kCand > 64 ? kCand : 1;
  __shared__ int4 s_xa[kStaged];
  __shared__ int2 s_xb[NL > 1 ? kStaged : 1];
  __shared__ int s_xf[kStaged];
  __shared__ __align__(16) double s_tot[kCand];
  // recombination: history hash after each candidate, the table that groups them
  __shared__ unsigned long long s_hh[RCM ? kCand : 1];
  __shared__ __align__(16) int s_tab[RCM ? kHashSlots : 4];
  __shared__ int s_surv[64];  // beams of more than 64 candidates: those left to rank
  __shared__ long long s_sbase[NL][kMaxLevels];  // state id of arc index i of level L < N-1: s_sbase[L] + i
  __shared__ int s_lbeg[NL][kMaxLevels];  // first arc of each level of the current state
  __shared__ int s_cfg[2];  // V, blank: re-read each frame so per-token masks stay inside the loop
  __shared__ int s_ticket;  // beam: this workgroup's arrival ticket
  __shared__ unsigned long long s_bytes, s_steps;

  const LMDevice *lms = p.lm;
  const TrieDevice &tr = p.tr;
  const int g = threadIdx.x;
  // this lane's entries of the arc and phrase rows back to 0 (absent)
  auto clear_rows = [&]() {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int y0 = (c * W + g) * 4;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        *reinterpret_cast<uint4 *>(arcw + i * Vp + y0) = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4 *>(arcw + i * Vp + y0 + 2) = make_uint4(0u, 0u, 0u, 0u);
      }
      *reinterpret_cast<uint4 *>(ptag + y0) = make_uint4(0u, 0u, 0u, 0u);
    }
  };
  const int wave = g >> 6;
  const int lane = g & 63;
  constexpr bool BEAM = MODE >= kModeBeam;
  constexpr bool RC = RCM;
  constexpr bool WIDE = MODE == kModeBeamWide || MODE == kModeBeamRCWide;  // more than 64 candidates a stream
  constexpr bool GR = MODE == kModeGreedy;
  const int B = BEAM ? p.B : 1, K = GR ? 1 : p.k;
  int Nl[NL], RSl[NL];  // order and record stride of each LM
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    Nl[i] = lms[i].N;
    RSl[i] = lms[i].rec_stride;
  }
  // workgroup -> (stream, hypothesis); with xcd_map the B workgroups of a stream
  // share blockIdx mod 8, i.e. one XCD and its L2, for the per-frame exchange.
  // A beam takes its index r within that class from an arrival counter: the
  // workgroups that have started always hold the first tickets of each class,
  // so every stream but the last one started in a class is complete and runs
  // to its end, freeing room for the rest.  The beam therefore needs no
  // co-residency guarantee (no cooperative launch), only room for the
  // incomplete streams beside one complete one (checked at launch)
  int sl, b;
  {
    const int x = blockIdx.x;
    int r = p.xcd_map ? x >> 3 : x;
    if constexpr (BEAM) {
      const int n_cls = p.xcd_map ? (int)(gridDim.x >> 3) : (int)gridDim.x;
      if (g == 0) {
        unsigned *ctr = p.tickets + (p.xcd_map ? (x & 7) : 0);
        const int tk = (int)atomicAdd(ctr, 1u);
        // the class's last ticket leaves the counter at 0 for the next launch
        if (tk == n_cls - 1) atomicExch(ctr, 0u);
        s_ticket = tk;
      }
      __syncthreads();
      r = s_ticket;
      if (r >= n_cls) {  // counters not reset since an earlier launch: no slot for this workgroup
        if (g == 0) atomicOr(p.status, FUSION_STATUS_SYNC_TIMEOUT);
        return;
      }
    }
    if (p.xcd_map) {
      sl = (x & 7) + 8 * (r / B);
      b = r % B;
      if (sl >= p.n_str) return;  // the last tickets of a class with one stream fewer than the others
    } else {
      sl = r / B;
      b = r % B;
    }
  }
  const int s = sl + p.s_off;
  const int H = p.S * B;
  const int h = s * B + b;

  // ---- prologue ------------------------------------------------------------------
  // Steps and greedy launches hold the hypothesis state in scalar registers.  A step
  // reads it in every wave, ahead of everything else: it is little more than its
  // dependent loads, so its logits are fetched beside the state, their statistics
  // are reduced while the record is on its way and combined while the arcs are
  // (256 x 4096, k = 4: 10.2 us before, 9.1 with the frame compiled as straight
  // code; 777 x 1001, k = 8, fused rows: 12.2 and 10.3)
  constexpr bool STEP = MODE == kModeStep;
  int st_src[NL], st_c1p[NL], st_c1[NL], st_q = 0, st_y = -1, st_fl = 0, st_par = 0;
  bool st_same = false;  // greedy: blank was emitted: the state of the frame before, whose rows in LDS still hold
  if constexpr (STEP) {
    if (p.has_trie) st_q = p.boost_state[h];
#pragma unroll
    for (int i = 0; i < NL; ++i) st_src[i] = p.lm_state[(int64_t)i * H + h];  // [n_lm][H]
  }
  if (g < kMaxLevels) {
#pragma unroll
    for (int i = 0; i < NL; ++i)
      s_sbase[i][g] = (g >= 2 && g + 1 <= Nl[i] - 1) ? lms[i].off[g + 1] - lms[i].arc_base[g] : 0;
  }
  if (g == 0) {
    s_cfg[0] = p.V;
    s_cfg[1] = p.blank;
    s_bytes = 0;
    s_steps = 0;
    s_nstat = 0;
  }
  if (!STEP && g == 0) {
    const int V = p.V, blank = p.blank;
    const int q = p.has_trie ? p.boost_state[h] : 0;
    const double sc = BEAM ? p.hyp_score[h] : 0.0;
    bool ok_lm = true;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int sig = p.lm_state[(int64_t)i * H + h];  // [n_lm][H]
      const bool ok_i = sig >= 0 && sig < lms[i].n_states && sig != blank && (sig != V + 1 || lms[i].eos_ok);
      ok_lm = ok_lm && ok_i;
      hs.lmsrc[i] = sig;
      hs.c1p[i] = -1;
      // c_1, the last token of the state: the state itself below V + 2, else
      // from its record (so that every frame knows c_1 before its record arrives)
      hs.c1[i] = !ok_i ? -1 : sig < V + 2 ? sig : (lms[i].rec[(int64_t)(sig - V - 2) * lms[i].rec_stride] & 0xFFFF);
      hs.cur_lm[i] = sig;
    }
    const bool ok_q = !p.has_trie || (q >= 0 && q < tr.n_nodes);
    const bool alive = !BEAM || sc > -INFINITY;
    hs.qsrc = q;
    hs.y = -1;
    hs.fl = (alive ? 1 : 0) | ((ok_lm && ok_q) ? 0 : 2);
    hs.cur_q = q;
    hs.S = sc;
    if constexpr (RC) {
      // the history carried from an earlier call, else one that starts at the
      // slot's initial states (never 0, which marks the start of a stream)
      unsigned long long hh = p.hist ? (p.hist[h] & ((1ull << 48) - 1)) : 0ull;
      if (hh == 0ull) {
        hh = mix64(0x243F6A8885A308D3ull ^ (unsigned long long)(unsigned)q);
#pragma unroll
        for (int i = 0; i < NL; ++i) hh = mix64(hh ^ ((unsigned long long)(unsigned)hs.lmsrc[i] << (8 * i + 1)));
        hh &= (1ull << 48) - 1;
        hh = hh ? hh : 1ull;
      }
      hs.hist = hh;
    }
    if (alive && !(ok_lm && ok_q))
      atomicOr(p.status, (ok_lm ? 0 : FUSION_STATUS_BAD_LM_STATE) | (ok_q ? 0 : FUSION_STATUS_BAD_BOOST_STATE));
  }
  // logits strip of this lane, raw (masked per frame): frame t+1's strip is
  // fetched during frame t, so it is in registers when t+1 begins
  const int voff = g * 16;
  // Rows that are not whole 16-byte strips (AL false: V % 4 != 0, or a base off 16
  // bytes) are read in 16-byte strips all the same, from 4-byte aligned addresses:
  // four loads a strip kept the address units busy for longer than the memory
  // (32 greedy streams of 8190
  // tokens: 584 us for 120 frames before, 540 after; a step of 777 x 1001 with its
  // fused rows, which leave in strips too: 13.9 and 13.6).  A strip that would pass the row's end reads the row's last four
  // tokens, and strip_of shifts them into place.  Only the smallest shape, where
  // rows may be shorter than a strip, reads single tokens
  constexpr bool SHIFT = !AL && W > 64;
  float xraw[NC][4];
  float xraw0[NC][4];  // a beam's wave 1: wave 0's strip too, for its row statistics
  auto fetch_strip = [&](const rsrc_t &xr, float (&dst)[NC][4], int off) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      if (AL) {
        const float4 xx = row_load4(xr, off, c * W * 16);
        dst[c][0] = xx.x; dst[c][1] = xx.y; dst[c][2] = xx.z; dst[c][3] = xx.w;
      } else if (SHIFT) {
        const float4 xx = row_load4(xr, min(off + c * W * 16, p.V * 4 - 16), 0);
        dst[c][0] = xx.x; dst[c][1] = xx.y; dst[c][2] = xx.z; dst[c][3] = xx.w;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[c][j] = row_load1(xr, off + 4 * j, c * W * 16);
      }
    }
  };
  // lane's strip c of wave sw's as fetched, its V % 4 last tokens in the row's last strip in place
  auto strip_of = [&](const float (&xs)[NC][4], int c, int sw, int V, float (&x)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) x[j] = xs[c][j];
    if constexpr (SHIFT) {
      const int r = V & 3, at = (V >> 2) - (c * W + sw * 64);  // the lane holding the row's last strip (uniform)
      if (r != 0 && at >= 0 && at < 64) {
        const bool last = lane == at;
        if (r == 1) {
          x[0] = last ? x[3] : x[0];
        } else if (r == 2) {
          x[0] = last ? x[2] : x[0];
          x[1] = last ? x[3] : x[1];
        } else {
          x[0] = last ? x[1] : x[0];
          x[1] = last ? x[2] : x[1];
          x[2] = last ? x[3] : x[2];
        }
      }
    }
  };
  // the logits row of this hypothesis at the frame being fetched; it advances by
  // one frame (H rows) per fetch and stays on the last frame
  const int64_t xstride = (int64_t)H * p.V;
  // Greedy mode A: a frame whose raw argmax is blank emits blank whatever the LM and
  // the phrases say and changes no state, so the frame loop passes it over (unless
  // fused rows or the byte count need its scores).  Which frames those are depends
  // on the logits alone: 64 frames at a time are looked through ahead of the loop,
  // each wave reading whole rows, several in flight.  The row statistics then serve
  // no purpose (a greedy decision compares keys) and are left out too.  It pays at
  // every width and share of blank from two frames on, also where blank is rare,
  // since the rows then come from the caches and the frames need no statistics.
  // Kernel us with and without it, 64 streams, 3 % and 90 % of the frames blank:
  // 150 frames of 128 tokens 426 / 475 and 111 / 321, of 1024 465 / 629 and 96 / 432,
  // of 8190 821 / 973 and 224 / 736; 13 frames of 1024 47 / 60 and 17 / 44; 2 frames
  // of 1024 12.2 / 13.3 and 9.1 / 12.0, of 128 12.3 / 12.1 and 10.9 / 11.1 (its worst:
  // 3 % at 128 tokens).  One frame is a step
  const bool pass_blank = GR && p.mode == FUSION_BLANK_AM && !p.fused && !p.traffic && p.V >= 4;
  const bool stats = !GR || p.fused != nullptr || (p.mode == FUSION_BLANK_AM && !pass_blank);
  // the frame decoded next, from t on, among the 64 from t0 that s_emit describes;
  // past them the first frame of the next 64
  auto next_frame = [&](int t, int t0) -> int {
    const unsigned long long bits =
        ((unsigned long long)(unsigned)uni((int)s_emit[1]) << 32) | (unsigned)uni((int)s_emit[0]);
    const unsigned long long left = t - t0 < 64 ? bits >> (t - t0) : 0ull;
    return left != 0ull ? t + __ffsll((long long)left) - 1 : t0 + 64;
  };
  auto scan_frames = [&](int t0) {
    constexpr int kRow = NC * NW;                            // 16-byte loads per lane of a row
    constexpr int kFly = 8;                                  // of them in flight
    constexpr int kLoads = kRow < kFly ? kRow : kFly, kParts = kRow / kLoads, kRowsAt = kFly / kLoads;
    // (opaque to the compiler: as loop invariants, the strips' offsets and the lane masks
    // of blank would be held, and spilled, across the frame loop: 140 scalar registers
    // spilled, 66 so; 64 streams x 500 frames, 1024 tokens: 1655 us before, 1565 so,
    // with 8 loads in flight instead of 16, which spilled vector registers)
    int V = p.V, blank = p.blank;
    asm volatile("" : "+s"(V), "+s"(blank));
    const int n = min(64, p.T - t0);
    lds_barrier();  // every wave has read the last block's bits
    if (g < 2) s_emit[g] = 0u;
    lds_barrier();
    for (int f0 = wave * kRowsAt; f0 < n; f0 += NW * kRowsAt) {
      float top[kRowsAt], low[kRowsAt];  // this lane's highest logit, and the highest of ids below blank
      const float *row[kRowsAt];
#pragma unroll
      for (int r = 0; r < kRowsAt; ++r) {
        row[r] = p.logits + ((int64_t)(t0 + min(f0 + r, n - 1)) * H + h) * V;
        top[r] = low[r] = -INFINITY;
      }
#pragma unroll 1
      for (int part = 0; part < kParts; ++part) {
        float4 v[kRowsAt][kLoads];
#pragma unroll
        for (int r = 0; r < kRowsAt; ++r) {
          const rsrc_t xr = row_rsrc(row[r], V);
#pragma unroll
          for (int c = 0; c < kLoads; ++c)
            // a strip past the row's end reads the row's last four tokens again
            v[r][c] = row_load4(xr, min(((part * kLoads + c) * 64 + lane) * 4, V - 4) * 4, 0);
        }
#pragma unroll
        for (int r = 0; r < kRowsAt; ++r)
#pragma unroll
          for (int c = 0; c < kLoads; ++c) {
            const float4 x = v[r][c];
            top[r] = fmaxf(top[r], fmaxf(fmaxf(x.x, x.y), fmaxf(x.z, x.w)));
            if (blank > 0) {  // uniform
              const int y0 = min(((part * kLoads + c) * 64 + lane) * 4, V - 4);
              low[r] = fmaxf(low[r], y0 < blank ? x.x : -INFINITY);
              low[r] = fmaxf(low[r], y0 + 1 < blank ? x.y : -INFINITY);
              low[r] = fmaxf(low[r], y0 + 2 < blank ? x.z : -INFINITY);
              low[r] = fmaxf(low[r], y0 + 3 < blank ? x.w : -INFINITY);
            }
          }
      }
#pragma unroll
      for (int r = 0; r < kRowsAt; ++r) {
        const int f = f0 + r;
        const float xb = row[r][blank];
        // blank takes the frame if nothing is above it and no lower id equals it
        const bool emits = !(xb > -INFINITY) || __ballot(top[r] > xb || low[r] >= xb) != 0ull;
        if (f < n && lane == 0) {
          if (emits) atomicOr(&s_emit[f >> 5], 1u << (f & 31));
          else p.tokens[(int64_t)(t0 + f) * H + h] = blank;
        }
      }
    }
    lds_barrier();
  };
  const float *xrow = p.logits + (int64_t)h * p.V;
  auto fetch_logits = [&]() {
    const rsrc_t xr = row_rsrc(xrow, p.V);
    fetch_strip(xr, xraw, voff);
    if (NW > 1 && BEAM && wave == 1) fetch_strip(xr, xraw0, lane * 16);
  };
  float rE[NC][4];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int y0 = (c * W + g) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) rE[c][j] = (p.has_trie && y0 + j < p.V) ? tr.root_E[y0 + j] : 0.0f;
  }
  if (STEP) fetch_logits();
  clear_rows();
  if (ER) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      *reinterpret_cast<float4 *>(erow + (c * W + g) * 4) = make_float4(rE[c][0], rE[c][1], rE[c][2], rE[c][3]);
  }
  if constexpr (STEP) {
    const int V = p.V, blank = p.blank;
    st_q = uni(st_q);
    bool ok_lm = true;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int sig = st_src[i] = uni(st_src[i]);
      const bool ok_i = sig >= 0 && sig < lms[i].n_states && sig != blank && (sig != V + 1 || lms[i].eos_ok);
      ok_lm = ok_lm && ok_i;
      st_c1p[i] = -1;
      st_c1[i] = ok_i && sig < V + 2 ? sig : -1;  // of a longer state, from its record
    }
    const bool ok_q = !p.has_trie || (st_q >= 0 && st_q < tr.n_nodes);
    st_fl = 1 | ((ok_lm && ok_q) ? 0 : 2);
    if (g == 0) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        hs.cur_lm[i] = st_src[i];
      }
      hs.cur_q = st_q;
      if (st_fl & 2)
        atomicOr(p.status, (ok_lm ? 0 : FUSION_STATUS_BAD_LM_STATE) | (ok_q ? 0 : FUSION_STATUS_BAD_BOOST_STATE));
    }
  }
  if (!STEP) {
    __syncthreads();
    fetch_logits();
  }
  if constexpr (GR) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      st_src[i] = uni(hs.lmsrc[i]);
      st_c1p[i] = uni(hs.c1p[i]);
      st_c1[i] = uni(hs.c1[i]);
    }
    st_q = uni(hs.qsrc);
    st_y = uni(hs.y);
    st_fl = uni(hs.fl);
  }
  // row statistics of the logits of strip sw (the 64-lane strip of wave sw) held
  // in xs: strip max, sum of exp below it, lowest id holding the max (only the
  // acoustic blank decision needs it).  They depend on the logits alone, so a beam
  // computes those of frame t+1 in frame t in the waves that are idle while wave 0
  // ends the frame (wave 1 takes wave 0's strip), frame 0's here; a step and a greedy
  // frame compute theirs in the shadow of the record's load
  auto row_stats = [&](const float (&xs)[NC][4], int sw, int V) {
    float xv[NC][4];  // tokens >= V: -inf
    float lmx = -INFINITY;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      strip_of(xs, c, sw, V, xv[c]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        xv[c][j] = (c * W + sw * 64 + lane) * 4 + j < V ? xv[c][j] : -INFINITY;
        lmx = fmaxf(lmx, xv[c][j]);
      }
    }
    const float mw = wave_max_f(lmx);
    float lsum = 0.0f;
    if (mw > -INFINITY) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) lsum += (xv[c][j] > -INFINITY) ? exp_fast(xv[c][j] - mw) : 0.0f;
    }
    const float ssum = wave_sum(lsum);
    int aid = INT_MAX;
    if (p.mode == FUSION_BLANK_AM && mw > -INFINITY) {
#pragma unroll
      for (int c = NC - 1; c >= 0; --c) {
        unsigned long long mj[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) mj[j] = __ballot(xv[c][j] == mw && (c * W + sw * 64 + lane) * 4 + j < V);
        const unsigned long long any = mj[0] | mj[1] | mj[2] | mj[3];
        if (any) {
          const int src = __ffsll((long long)any) - 1;
          int jj = 3;
#pragma unroll
          for (int j = 2; j >= 0; --j) jj = ((mj[j] >> src) & 1ull) ? j : jj;
          aid = (c * W + sw * 64 + src) * 4 + jj;
        }
      }
    }
    if (lane == 0) {
      s_pm[sw] = mw;
      s_ps[sw] = ssum;
      s_paid[sw] = aid;
    }
  };
  // the strip statistics of all NW waves combined into s_lse / s_am (one wave)
  auto combine_stats = [&]() {
    const bool wl = lane < NW;
    const float pm = wl ? s_pm[lane] : -INFINITY;
    const float M = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(row_max(pm)), 0));
    const float term = (wl && pm > -INFINITY) ? s_ps[lane] * exp_fast(pm - M) : 0.0f;
    const float lse = M + logf(__int_as_float(__builtin_amdgcn_readlane(__float_as_int(row_sum(term)), 0)));
    float ak = pm;
    int ay = wl ? s_paid[lane] : INT_MAX;
    row_best(ak, ay);
    if (lane == 0) {
      s_lse = lse;
      s_am = ay;
    }
  };
  // a V-wide fp32 row straight from HBM into an LDS row (this wave's strips)
  auto load_row = [&](const float *drow, float *row, int V) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int wbase = c * W + wave * 64;  // first 4-token strip of this wave
      // (of a row that is not whole strips, the last strip reads up to 12 bytes past it:
      // the next row, or the pad behind the table)
      const int y0 = (wbase + lane) * 4;
      __builtin_amdgcn_global_load_lds(drow + (y0 < V ? y0 : 0), (lds_ptr_t)(row + wbase * 4), 16, 0, 0);
    }
  };
  // (the last of the n waves to come here combines)
  auto combine_last = [&](int n) {
    int done = 0;
    if (lane == 0) done = __hip_atomic_fetch_add(&s_nstat, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP);
    if (uni(done) == n - 1) {
      combine_stats();
      if (lane == 0) s_nstat = 0;
    }
  };
  if (BEAM || (GR && NW == 1 && stats)) {
    row_stats(xraw, wave, p.V);
    __syncthreads();
    if (wave == NW - 1) combine_stats();
    __syncthreads();
  }

  bool aborted = false;  // after one failed rendezvous this workgroup stops waiting
  int gen = 0;           // rows assembled so far (the LDS entries' stamp)
  int tn;                // the frame decoded after this one
  int blk = -1;          // greedy: the 64 frames s_emit describes
  // (a step is one frame, known as such to the compiler: as a loop it held every
  // table pointer and lane mask in scalar registers across the frame, spilling a hundred)
  for (int t = 0; STEP ? t < 1 : t < p.T; t = tn) {
    if (GR && pass_blank && (t >> 6) != blk) {
      blk = t >> 6;
      scan_frames(blk << 6);
      tn = next_frame(t, blk << 6);
      xrow = p.logits + ((int64_t)min(tn, p.T - 1) * H + h) * p.V;
      fetch_logits();
      if (tn != t) continue;
    }
    int V = p.V, blank = p.blank;
    if (GR) asm volatile("" : "+s"(V), "+s"(blank));  // (as s_cfg)
    if (BEAM) {
      V = uni(s_cfg[0]);
      blank = uni(s_cfg[1]);
    }
    const int fl = !BEAM ? st_fl : uni(hs.fl);
    const bool act = (fl & 1) != 0;
    const bool inv = act && (fl & 2) != 0;
    const bool ok = act && !inv;
    // A greedy hypothesis that emitted blank keeps its state, and so the rows in LDS:
    // neither the second memory round trip nor the scatter is needed (32 streams of
    // 8190 tokens, blank competing, half of the frames blank: 5.9 us a frame before,
    // 4.6 after).  A beam slot rarely keeps its state: its next hypothesis comes
    // from any slot, and the test cost the 64 x 4 beam 3 %
    const bool keep = GR && (!ok || st_same);
    if (!keep) {
      ++gen;
      // stamps repeat after 2^14 rows: the entries are cleared before they would
      // (the previous frame's last reads of them precede its final barrier)
      if (gen > 0x4000) {
        gen = 1;
        clear_rows();
        __syncthreads();
      }
    }
    const uint32_t stamp = (uint32_t)gen;
    const int qsrc = !BEAM ? st_q : uni(hs.qsrc), yin = !BEAM ? st_y : uni(hs.y);
    int lmsrc[NL], c1[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      lmsrc[i] = !BEAM ? st_src[i] : uni(hs.lmsrc[i]);
      c1[i] = !BEAM ? st_c1[i] : uni(hs.c1[i]);
    }
    // ---- hop 1: state records, phrase node, dense level-1 rows ------------------
    const int32_t *rp[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      rp[i] = nullptr;
      if (ok) {
        if (lmsrc[i] < -1) rp[i] = lms[i].ctx_rec + ((int64_t)(-lmsrc[i] - 2) * V + yin) * RSl[i];
        else if (lmsrc[i] < 0) rp[i] = lms[i].rec_dense + ((int64_t)(!BEAM ? st_c1p[i] : uni(hs.c1p[i])) * V + yin) * RSl[i];
        else if (lmsrc[i] >= V + 2) rp[i] = lms[i].rec + (int64_t)(lmsrc[i] - V - 2) * RSl[i];
      }
    }
    const int4 *np = nullptr;
    if (ok && p.has_trie) np = qsrc < 0 ? tr.root_node + yin : tr.node + qsrc;
    const int64_t rowoff = ((int64_t)t * H + h) * V;
    // this frame's logits (fetched during the previous frame); waited for here,
    // before this frame's loads are issued
    float xv[NC][4];
    auto take_strip = [&]() {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        strip_of(xraw, c, wave, V, xv[c]);
#pragma unroll
        for (int j = 0; j < 4; ++j) xv[c][j] = (act && (c * W + g) * 4 + j < V) ? xv[c][j] : -INFINITY;
      }
    };
    if (!STEP) {
#pragma unroll
      for (int c = 0; c < NC; ++c) asm volatile("" ::"v"(xraw[c][0]), "v"(xraw[c][1]), "v"(xraw[c][2]), "v"(xraw[c][3]));
      take_strip();
    }
    // the state records and the phrase node with scalar loads (uniform addresses):
    // kRecW words per record (the record arrays carry a tail pad so that reading
    // past a short record stays inside them); "no record" / "no node" read the
    // zero words
    int rec[NL][kRecW];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const __attribute__((address_space(4))) int32_t *r =
          (const __attribute__((address_space(4))) int32_t *)(rp[i] ? rp[i] : g_zero_words);
#pragma unroll
      for (int w = 0; w < kRecW; ++w) rec[i][w] = r[w];
    }
    const __attribute__((address_space(4))) int32_t *nq =
        (const __attribute__((address_space(4))) int32_t *)(np ? reinterpret_cast<const int32_t *>(np) : g_zero_words);
    const int node[4] = {nq[0], nq[1], nq[2], nq[3]};
    if (!keep && !STEP) {
      // the level-1 dense rows straight into LDS: only the records are waited for
      // before the second hop
#pragma unroll
      for (int i = 0; i < NL; ++i) load_row(lms[i].dense + (int64_t)(ok ? c1[i] : 0) * V, lmval + i * Vp, V);
    }
    if (STEP) {
      row_stats(xraw, wave, V);
      take_strip();
      __builtin_amdgcn_sched_barrier(0);  // the record is waited for after this, not before
    } else if (GR && NW > 1 && stats) {
      // a greedy frame's own, under the latency of its records.  (As work that the
      // waves did after the last frame's selection they delayed the next frame: 64 streams
      // of 100 frames with their fused rows, blank competing, 4096 tokens: 478 us,
      // 415 so; 1024: 394, 359; 8190: 671, 620; mode A at 4096: 492, 435)
      row_stats(xraw, wave, V);
      combine_last(NW);
    } else if (NW == 1 && t > 0 && stats) {  // a single wave has no idle helper
      row_stats(xraw, 0, V);
      combine_stats();
    }
    // ---- decode the records ---------------------------------------------------------
    const float phiq = as_float(node[0]);
    const int dbeg = node[1];
    const int dcnt = node[2];
    const int qid = np ? node[3] : qsrc;
    // per LM: order m of the state, its id; backoffs, first arcs and arc counts of
    // levels 2..m.  The first LM's context row (level D >= 2 of the chain, row r)
    // replaces the levels up to D: only the arcs of the levels above D are fetched
    // (lcnt 0 for the others).  Further LMs fetch the arcs of every level
    int m[NL], sid[NL], total_arcs[NL], Dc = 0, crow = 0;
    float bo[NL][kMaxLevels];
    int lcnt[NL][kMaxLevels], lbeg[NL][kMaxLevels];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      m[i] = rp[i] ? (rec[i][0] >> 16) : 1;
      sid[i] = rp[i] ? rec[i][1] : lmsrc[i];
      int Di = 0;
      if (CTX && i == 0 && rp[0]) {
        const int n0 = Nl[0];
        const int cw = n0 == 3 ? rec[0][rec_ctx_word(3)] : n0 == 4 ? rec[0][rec_ctx_word(4)]
                     : n0 == 5 ? rec[0][rec_ctx_word(5)] : n0 == 6 ? rec[0][rec_ctx_word(6)] : 0;
        Dc = Di = (int)((unsigned)cw >> 28);
        crow = cw & 0x0FFFFFFF;
      }
      total_arcs[i] = 0;
      // levels above m are absent: backoff 0 and no arcs (their record words
      // hold zeros or, at level N, the context-row word)
#pragma unroll
      for (int L = 2; L < kMaxLevels; ++L) {
        const bool lv = L <= m[i];
        bo[i][L] = lv ? as_float(rec[i][rec_bo_word(L)]) : 0.0f;
        lcnt[i][L] = (lv && L > Di) ? rec[i][rec_cnt_word(L)] : 0;
        lbeg[i][L] = lv ? rec[i][rec_beg_word(L)] : 0;
        total_arcs[i] += lcnt[i][L];
      }
    }
    if (!keep) {
      if (STEP) {
        // (a state below V + 2 is its own c_1; the first LM's context row takes the place
        // of the dense row)
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          if (rp[i]) c1[i] = rec[i][0] & 0xFFFF;
          if (ok && !(CTX && i == 0 && Dc >= 2)) load_row(lms[i].dense + (int64_t)c1[i] * V, lmval + i * Vp, V);
        }
      }
      if (CTX && ok && Dc >= 2) load_row(lms[0].ctx_lm + (int64_t)crow * V, lmval + NL * Vp, V);
      // ---- hop 2: first arcs of levels 2..m (flattened) and first phrase transitions --
      int2 ab[NL][kUA];
      int at[NL][kUA], tn[NL][kUA];  // at = level << 16 | offset within the level
#pragma unroll
      for (int i = 0; i < NL; ++i) {
#pragma unroll
        for (int u = 0; u < kUA; ++u) {
          int f = u * W + g;
          ab[i][u] = make_int2(INT_MAX, 0);
          at[i][u] = 0;
          tn[i][u] = 0;
          // the level of flattened arc f against the (uniform) starts of the levels:
          // the last level that starts at or before f; then f's offset within it
          int L = 2, bL = lbeg[i][2], fo = f, e = 0;
#pragma unroll
          for (int L2 = 3; L2 < kMaxLevels; ++L2) {
            e += lcnt[i][L2 - 1];  // first flattened index of level L2
            const bool past = f >= e && L2 <= m[i];
            L = past ? L2 : L;
            bL = past ? lbeg[i][L2] : bL;
            fo = past ? f - e : fo;
          }
          f = fo;
          if (u * W + g < total_arcs[i]) {
            at[i][u] = (L << 16) | f;
            ab[i][u] = lms[i].arcs[bL + f];
            if (L == Nl[i] - 1 && f < kAux) tn[i][u] = lms[i].top_next[bL + f - lms[i].arc_base[Nl[i] - 1]];
          }
        }
      }
      int4 dd[kUD];
#pragma unroll
      for (int u = 0; u < kUD; ++u) {
        const int j = u * W + g;
        dd[u] = make_int4(INT_MAX, 0, 0, 0);
        if (j < dcnt) dd[u] = tr.delta[dbeg + j];
      }
      if (ok && g == 0) {
        if (!GR) hs.cur_q = qid;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          if (!GR) {
            hs.cur_lm[i] = sid[i];
            hs.c1[i] = c1[i];
          }
#pragma unroll
          for (int L = 2; L < kMaxLevels; ++L) s_lbeg[i][L] = lbeg[i][L];
        }
      }
      // ---- scatter (no ordering between levels: see arcw) ----------------------------
      // an arc of level L is stored summed with the backoffs of levels L+1.., the
      // addition order of the backoff recursion
      auto put_arc = [&](int i, int L, int j, int2 a, int tnext) {
        const int y = a.x;
        if (y < V) {
          float v = as_float(a.y);
#pragma unroll
          for (int L2 = 3; L2 < kMaxLevels; ++L2) {
            if (L2 > m[i]) break;  // uniform: the levels above m back off by nothing
            v = v + (L2 > L ? bo[i][L2] : 0.0f);
          }
          const uint32_t tag = (stamp << 16) | (uint32_t)((L << 13) | j);
          __hip_atomic_fetch_max(arcw + i * Vp + y, ((unsigned long long)tag << 32) | (unsigned long long)__float_as_uint(v),
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          if (L == Nl[i] - 1 && j < kAux) sTN[i * kAux + j] = tnext;
        }
      };
      if (STEP) {
        // the rows are cleared and the waves' statistics are there
        lds_barrier();
        if (wave == NW - 1) combine_stats();
      }
      if (ok) {
#pragma unroll
        for (int u = 0; u < kUD; ++u) {
          const int j = u * W + g;
          if (j < dcnt) {
            ptag[dd[u].x] = (stamp << 16) | (uint32_t)(j + 1);
            if (ER) erow[dd[u].x] = as_float(dd[u].z);
            if (j < kAux) {
              sE[j + 1] = as_float(dd[u].z);
              sDT[j] = dd[u].y;
            }
          }
        }
        for (int j = kUD * W + g; j < dcnt; j += W) {
          const int4 e = tr.delta[dbeg + j];
          ptag[e.x] = (stamp << 16) | (uint32_t)(j + 1);
          if (ER) erow[e.x] = as_float(e.z);
          if (j < kAux) {
            sE[j + 1] = as_float(e.z);
            sDT[j] = e.y;
          }
        }
#pragma unroll
        for (int i = 0; i < NL; ++i)
#pragma unroll
          for (int u = 0; u < kUA; ++u)
            if (at[i][u] != 0) put_arc(i, at[i][u] >> 16, at[i][u] & 0xFFFF, ab[i][u], tn[i][u]);
        // arcs beyond the first kUA * W of the flattened levels
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int N = Nl[i];
          int covered = kUA * W;
#pragma unroll
          for (int L = 2; L < kMaxLevels; ++L) {
            if (L > m[i]) break;  // uniform
            const int bL = lbeg[i][L], cL = lcnt[i][L];
            const int done = min(cL, max(0, covered));
            covered -= cL;
            const int2 *A = lms[i].arcs + bL;
            for (int j0 = done; j0 < cL; j0 += 4 * W) {
              int2 a4[4];
              int t4[4];
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const int j = j0 + u * W + g;
                a4[u] = j < cL ? A[j] : make_int2(INT_MAX, 0);
                t4[u] = (L == N - 1 && j < cL && j < kAux) ? lms[i].top_next[bL + j - lms[i].arc_base[N - 1]] : 0;
              }
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const int j = j0 + u * W + g;
                if (j < cL) put_arc(i, L, j, a4[u], t4[u]);
              }
            }
          }
        }
      }
      __builtin_amdgcn_s_waitcnt(0);  // the dense rows have landed in LDS
      __syncthreads();
    }
    if (GR && NW > 1 && keep && stats) lds_barrier();  // (else the rows' barrier)
    // ---- the row statistics of this frame ---------------------------------------------
    // the log-sum-exp is needed by wave 0 (selected scores, beam totals) and, for
    // fused rows, by every wave; the acoustic argmax (mode A) by every wave
    const float lse = __int_as_float(uni(__float_as_int(s_lse)));
    const int am = uni(s_am);
    // ---- keys and the fused row ------------------------------------------------------
    // (frames that the acoustic argmax gives to blank never get here when they are
    // passed over)
    const bool blank_only = inv || (p.mode == FUSION_BLANK_AM && !pass_blank && am == blank);
    const bool want_keys = ok && (!blank_only || p.fused);
    const bool compete = p.mode == FUSION_BLANK_COMPETE;
    const bool write_fused = p.fused != nullptr && ok;
    float kk[NC][4];
    bool cd[NC][4];  // token (c, j) of this lane is a candidate
    // which tokens compete this frame (uniform): blank in blank-only frames or
    // when it competes, the others unless the frame is blank-only
    const bool take_blank = act & (blank_only | compete);
    const bool take_other = act & !blank_only;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int y0 = (c * W + g) * 4;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        // bitwise logic on lane masks: no per-token branches
        const int y = y0 + j;
        const bool is_blank = y == blank;
        cd[c][j] = (y < V) & ((is_blank & take_blank) | (!is_blank & take_other));
        kk[c][j] = xv[c][j];
      }
      if (want_keys) {
        uint32_t aw[NL][4], av[NL][4];  // tag and value halves of the arc entries
        float lv[NL][4];                // dense rows
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const uint4 a01 = *reinterpret_cast<const uint4 *>(arcw + i * Vp + y0);
          const uint4 a23 = *reinterpret_cast<const uint4 *>(arcw + i * Vp + y0 + 2);
          const float4 l4 = *reinterpret_cast<const float4 *>(lmval + (CTX && i == 0 && Dc >= 2 ? NL : i) * Vp + y0);
          aw[i][0] = a01.y; aw[i][1] = a01.w; aw[i][2] = a23.y; aw[i][3] = a23.w;
          av[i][0] = a01.x; av[i][1] = a01.z; av[i][2] = a23.x; av[i][3] = a23.z;
          lv[i][0] = l4.x; lv[i][1] = l4.y; lv[i][2] = l4.z; lv[i][3] = l4.w;
        }
        float eh[4];
        uint32_t hi[4];
        const bool use_row = ER && !keep;  // uniform
        if (use_row) {
          const float4 ev4 = *reinterpret_cast<const float4 *>(erow + y0);
          eh[0] = ev4.x; eh[1] = ev4.y; eh[2] = ev4.z; eh[3] = ev4.w;
          // this lane's entry values back to the root's for the next rows
          *reinterpret_cast<float4 *>(erow + y0) = make_float4(rE[c][0], rE[c][1], rE[c][2], rE[c][3]);
        } else {
          // transition + 1 of this frame's phrase entry, 0 if none
          const uint4 p4 = *reinterpret_cast<const uint4 *>(ptag + y0);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const uint32_t pw = j == 0 ? p4.x : j == 1 ? p4.y : j == 2 ? p4.z : p4.w;
            hi[j] = (pw >> 16) == stamp ? (pw & 0xFFFFu) : 0u;
          }
          // the phrase entry values: the LDS copy of the state's first kAux transitions
          // (read for every token, index 0 when unused, so that no per-token branch
          // guards the read), the delta table beyond them only for a state with more
#pragma unroll
          for (int j = 0; j < 4; ++j) eh[j] = sE[min((int)hi[j], kAux)];
          asm volatile("" ::"v"(eh[0]), "v"(eh[1]), "v"(eh[2]), "v"(eh[3]));
          if (dcnt > kAux) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              if (hi[j] > (uint32_t)kAux) eh[j] = as_float(tr.delta[dbeg + (int)hi[j] - 1].z);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) eh[j] = hi[j] ? eh[j] : rE[c][j];
        }
        // per LM, the dense row (the first LM's context row when it has one) plus
        // the backoffs of the levels above it up to m, in increasing order (the
        // levels above m back off by 0)
        float dres[NL][4];
#pragma unroll
        for (int i = 0; i < NL; ++i) {
#pragma unroll
          for (int j = 0; j < 4; ++j) dres[i][j] = lv[i][j];
          const int from = (CTX && i == 0 && Dc >= 2) ? Dc + 1 : 2;
#pragma unroll
          for (int L2 = 2; L2 < kMaxLevels; ++L2) {
            if (L2 > m[i]) break;  // uniform
            if (L2 >= from) {
#pragma unroll
              for (int j = 0; j < 4; ++j) dres[i][j] = dres[i][j] + bo[i][L2];
            }
          }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int y = y0 + j;
          const float x = xv[c][j];
          // the LM terms in model order: u = (x + a_1 lm_1) + a_2 lm_2 ..., each LM
          // its winning arc of this frame if there is one, else its backed-off
          // dense row
          float u = x;
#pragma unroll
          for (int i = 0; i < NL; ++i) {
            const float lmv = (aw[i][j] >> 16) == stamp ? __uint_as_float(av[i][j]) : dres[i][j];
            const float a1 = p.lam[i] * lmv;
            u = u + a1;
          }
          // phrases: the transition's entry value if this state overrides y, else the
          // root's (with no phrase tree both are 0 and so is phi)
          const float bst = eh[j] - phiq;
          const float a3 = p.beta * ((ER || p.has_trie) ? bst : 0.0f);
          kk[c][j] = (y == blank) ? x : u + a3;
        }
      } else if (GR && ER && !keep) {
        // a frame given to blank without its keys: the overrides it scattered go all
        // the same (the frames that keep these rows find them through ptag)
        *reinterpret_cast<float4 *>(erow + y0) = make_float4(rE[c][0], rE[c][1], rE[c][2], rE[c][3]);
      }
      if (write_fused && y0 < V) {
        const rsrc_t fr = row_rsrc(args_here().fused + rowoff, V);
        if (AL || y0 + 3 < V) {
          row_store4(fr, make_float4(kk[c][0] - lse, kk[c][1] - lse, kk[c][2] - lse, kk[c][3] - lse), voff, c * W * 16);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (y0 + j < V) row_store1(fr, kk[c][j] - lse, voff + 4 * j, c * W * 16);
        }
      }
    }
    // the next frame's logits strip: fetched here, in a compute-bound phase, rather
    // than beside the frame-start loads, whose burst sets the start of the frame.
    // Unconditional (the last frame fetches its own row again): a conditional
    // fetch would make the compiler wait for it where the branches join
    tn = GR && pass_blank ? next_frame(t + 1, blk << 6) : t + 1;
    if (!STEP && tn < p.T) xrow += (int64_t)(tn - t) * xstride;
    if (!STEP) fetch_logits();
    // ---- the wave's top-k: per round the wave maximum of the remaining keys, then
    // the lowest id holding it (ties to the lowest id).  Keys compete as
    // order-preserving ints; tokens that are not candidates or are already taken
    // hold INT_MIN, below every key including -inf (a key that is the all-ones NaN
    // maps there too: such a token is no candidate).  The per-round work stays in
    // the vector units (the scalar unit is shared by all the waves of the CU):
    // each lane finds its own first token holding the maximum, the compare mask
    // is the ballot, the winning lane removes its token, and lane r keeps round
    // r's entry until the list is written at the end.
    {
      int sk[NC][4];
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int o = ord_key(kk[c][j]);
          sk[c][j] = cd[c][j] ? o : INT_MIN;
        }
      // With K > 1 the rounds below run only in a wave that holds more than K
      // keys at or above tau, the K-th largest of 16 maxima, one of every 64, 16 or
      // 4 lanes (1024, 256, 64 lanes): those maxima are K distinct tokens with keys
      // >= tau, so no key below tau is among the hypothesis' top K.  (With one
      // maximum per wave the bound of a 256-lane hypothesis was the lowest of four
      // maxima, and there was none for k = 8:
      // a step of 777 x 1001 with k = 8 took 13.6 us, 12.2 so.)  A wave with at most K such keys writes
      // them straight into its list (any order: the hypothesis' top-k ranks
      // by key, then id).
      bool listed = false;
      if constexpr (KM > 1) {
        int lb = INT_MIN;
#pragma unroll
        for (int c = 0; c < NC; ++c) lb = max(lb, max(max(sk[c][0], sk[c][1]), max(sk[c][2], sk[c][3])));
        int mw = lb, group = wave;
        if constexpr (NW == 16) {
          mw = wave_max_i(mw);
        } else {
          static_assert(NW == 4 || NW == 1, "16 groups of lanes");
          mw = max(mw, dpp_i<0xB1, 0xF>(mw));
          mw = max(mw, dpp_i<0x4E, 0xF>(mw));
          if (NW == 4) {
            mw = max(mw, dpp_i<0x141, 0xF>(mw));
            mw = max(mw, dpp_i<0x140, 0xF>(mw));
          }
          group = g / (W / 16);
        }
        // (the group in the low bits makes the maxima distinct; tau, with them
        // cleared, can only be lower, which keeps it a valid bound)
        if (lane % (W / 16 < 64 ? W / 16 : 64) == 0) s_wmax[group] = (mw & ~15) | (15 - group);
        lds_barrier();
        // the K-th largest: lane l < 16 counts those ahead of maximum l and the lane
        // of rank K-1 holds it
        const int mine = s_wmax[lane & 15];
        int r = 0;
#pragma unroll
        for (int w2 = 0; w2 < 16; w2 += 4) {
          const int4 d = *reinterpret_cast<const int4 *>(&s_wmax[w2]);
          r += (int)(d.x > mine) + (int)(d.y > mine) + (int)(d.z > mine) + (int)(d.w > mine);
        }
        const unsigned long long at = __ballot(lane < 16 && r == K - 1);
        const int tau = __builtin_amdgcn_readlane(mine, __ffsll((long long)at) - 1) & ~15;
        // survivors: keys >= tau, never a non-candidate (INT_MIN; every real key,
        // -inf included, maps above it)
        const int thr = max(tau, INT_MIN + 1);
        unsigned long long sb[NC][4];
        int n = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            sb[c][j] = __ballot(sk[c][j] >= thr);
            n += __popcll(sb[c][j]);
          }
        if (n <= K) {
          int base = 0;
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              if (sk[c][j] >= thr) {
                const int slot = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(sb[c][j] >> 32),
                                                                  __builtin_amdgcn_mbcnt_lo((uint32_t)sb[c][j], 0u));
                w_key[wave][slot] = sk[c][j];
                w_y[wave][slot] = (c * W + wave * 64 + lane) * 4 + j;
              }
              base += __popcll(sb[c][j]);
            }
          if (lane >= n && lane < K) {
            w_key[wave][lane] = INT_MIN;
            w_y[wave][lane] = INT_MAX;
          }
          listed = true;
        } else {
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int j = 0; j < 4; ++j) sk[c][j] = sk[c][j] >= thr ? sk[c][j] : INT_MIN;
        }
      }
      int rk = INT_MIN, ry = INT_MAX;  // lane r: entry r of the wave's list (greedy: every lane holds the one)
      for (int r = 0; r < (listed ? 0 : K); ++r) {
        int lbc[NC];
        int lb = INT_MIN;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          lbc[c] = max(max(sk[c][0], sk[c][1]), max(sk[c][2], sk[c][3]));
          lb = max(lb, lbc[c]);
        }
        const int M = wave_max_i(lb);
        if (M == INT_MIN) break;
        // lowest strip, then lowest lane, then lowest position holding M
        int src = -1, wc = 0;
#pragma unroll
        for (int c = NC - 1; c >= 0; --c) {
          const unsigned long long has = __ballot(lbc[c] == M);
          if (has) {
            src = __ffsll((long long)has) - 1;
            wc = c;
          }
        }
        int jm = 3;  // this lane's first position holding M in strip wc
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (c == wc) {
            jm = sk[c][2] == M ? 2 : jm;
            jm = sk[c][1] == M ? 1 : jm;
            jm = sk[c][0] == M ? 0 : jm;
          }
        const int wy = (wc * W + wave * 64 + src) * 4 + __builtin_amdgcn_readlane(jm, src);
        if constexpr (GR) {
          rk = M;
          ry = wy;
          break;
        }
        const int kill = lane == src ? wc * 4 + jm : -1;
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int j = 0; j < 4; ++j) sk[c][j] = kill == c * 4 + j ? INT_MIN : sk[c][j];
        rk = lane == r ? M : rk;
        ry = lane == r ? wy : ry;
      }
      if constexpr (GR) {
        // the state after this wave's best token (see HypState)
        int cl[NL], cq = qid;
#pragma unroll
        for (int i = 0; i < NL; ++i) cl[i] = sid[i];
        if (ry != INT_MAX && ry != blank) {  // uniform
          uint32_t aw[NL];
#pragma unroll
          for (int i = 0; i < NL; ++i) aw[i] = (uint32_t)(arcw[i * Vp + ry] >> 32);
          const uint32_t pw = ptag[ry];
          const int hi = uni((pw >> 16) == stamp ? (int)(pw & 0xFFFFu) : 0);
#pragma unroll
          for (int i = 0; i < NL; ++i) {
            const int lo = uni((aw[i] >> 16) == stamp ? (int)(aw[i] & 0xFFFFu) : 0);
            cl[i] = (CTX && i == 0 && Dc >= 2) ? -(crow + 2) : -1;
            if (lo) {
              const int L = lo >> 13, jj = lo & 0x1FFF, N = Nl[i];
              cl[i] = L < N - 1 ? (int)(s_sbase[i][L] + s_lbeg[i][L] + jj)
                    : jj < kAux ? sTN[i * kAux + jj]
                                : lms[i].top_next[s_lbeg[i][L] + jj - lms[i].arc_base[N - 1]];
            }
          }
          cq = !p.has_trie ? 0 : hi == 0 ? -1 : hi <= kAux ? sDT[hi - 1] : tr.delta[dbeg + hi - 1].y;
        }
        if (lane == 0) {
          s_best[st_par][wave] = make_int4(rk, ry, cl[0], cq);
          if constexpr (NL > 1) s_best1[st_par][wave] = cl[1];
        }
      } else if (!listed && lane < K) {
        w_key[wave][lane] = rk;
        w_y[wave][lane] = ry;
      }
    }
    if (p.traffic && act && g == 0) {
      // the frame's algorithmic bytes: the logits row; per LM the level-1 row and,
      // for every level of the state's chain, its arc list (at most a row) and
      // 12 bytes of record, plus 8 for a chain of two or more levels; the phrase
      // node and its delta list.  Recomputed here from the frame's sources, which
      // the hypothesis state holds until the install, so that the decode keeps
      // no value alive for a count that only the counting launch takes
      const __attribute__((address_space(4))) Params &pk = args_here();
      unsigned long long by = 4ull * V;
      if (ok) {
        const unsigned long long row = 4ull * V;
        const int y = hs.y;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const int rs = pk.lm[i].rec_stride;
          by += umin64(8ull * (unsigned long long)pk.lm[i].cnt1[hs.c1[i]], row);
          const int src = hs.lmsrc[i];
          const int32_t *r = src < -1  ? pk.lm[i].ctx_rec + ((int64_t)(-src - 2) * V + y) * rs
                             : src < 0 ? pk.lm[i].rec_dense + ((int64_t)hs.c1p[i] * V + y) * rs
                             : src >= V + 2 ? pk.lm[i].rec + (int64_t)(src - V - 2) * rs
                                            : nullptr;
          const int mi = r ? (r[0] >> 16) : 1;
          for (int L = 2; L < kMaxLevels; ++L)
            if (L <= mi) by += umin64(8ull * (unsigned long long)(unsigned)r[rec_cnt_word(L)], row) + 12ull;
          if (mi >= 2) by += 8ull;
        }
        if (pk.has_trie) {
          const int q = hs.qsrc;
          const int4 nd = q < 0 ? pk.tr.root_node[y] : pk.tr.node[q];
          by += 16ull + 16ull * (unsigned long long)nd.z;
        }
      }
      by += BEAM ? 8ull : 4ull;
      if (p.fused) by += 4ull * V;
      s_bytes += by;
      s_steps += 1ull;
    }
    lds_barrier();
    // a beam's next frame's row statistics, by the waves other than wave 0 (ahead of the
    // frame's end, off wave 0's path)
    if (BEAM && NW > 1 && wave != 0 && tn < p.T) {
      row_stats(xraw, wave, V);
      if (wave == 1) row_stats(xraw0, 0, V);
      combine_last(NW - 1);
    }
    if constexpr (GR) {
      // ---- greedy: the best of the waves' bests, in every wave ------------------------
      // Each wave resolved its own best token's next state while it still could read
      // the LDS rows; after one barrier every wave picks the winner, with no wave-0
      // phase that the others wait for and no second barrier (64 streams of 500
      // frames, 1024 tokens: 3.75 us a frame before, 3.3 after; 285 streams of 63:
      // 180 us before, 158 after; 8190 tokens: no change)
      int4 bw = make_int4(INT_MIN, INT_MAX, 0, 0);
      int b1 = 0;
      if (lane < NW) {
        bw = s_best[st_par][lane];
        if constexpr (NL > 1) b1 = s_best1[st_par][lane];
      }
      const int M = wave_max_i(bw.x);
      unsigned long long top = __ballot(bw.x == M && lane < NW);
      if constexpr (NC > 1) {
        // equal keys: the lowest id, which with several strips per lane may be any wave's
        if (top & (top - 1)) {
          const int ym = ~wave_max_i(bw.x == M ? ~bw.y : INT_MIN);
          top = __ballot(bw.x == M && bw.y == ym && lane < NW);
        }
      }
      const int from = __ffsll((long long)top) - 1;
      // (every competing key the all-ones NaN, as in a row of 0xFF bytes: no wave has a
      // candidate, each left the state as it is, and the frame goes to blank)
      const int yw = __builtin_amdgcn_readlane(bw.y, from);
      const int cy = yw != INT_MAX ? yw : blank;
      st_q = __builtin_amdgcn_readlane(bw.w, from);
      st_same = cy == blank;
      st_y = cy;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        st_src[i] = i == 0 ? __builtin_amdgcn_readlane(bw.z, from) : __builtin_amdgcn_readlane(b1, from);
        st_c1p[i] = c1[i];
        st_c1[i] = cy != blank ? cy : c1[i];
      }
      st_par ^= 1;
      if (g == 0) {
        // for the byte count and the final state
        p.tokens[(int64_t)t * H + h] = cy;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          hs.lmsrc[i] = st_src[i];
          hs.c1p[i] = st_c1p[i];
          hs.c1[i] = st_c1[i];
        }
        hs.qsrc = st_q;
        hs.y = cy;
      }
      continue;
    }
    // ---- the hypothesis' top-k (wave 0): the K-entry lists of the NW waves spread
    // over the lanes (entry j of wave w is element e = j*NW + w, lane e % 64, slot
    // e / 64); K rounds of a wave maximum, ties to the lowest id -------------------
    if (wave == 0) {
      constexpr int kSlots = (NW * KM + 63) / 64;
      int ek[kSlots], ey[kSlots];
#pragma unroll
      for (int q = 0; q < kSlots; ++q) {
        const int e = q * 64 + lane;
        const int w = e % NW, j = e / NW;
        ey[q] = j < K ? w_y[w][j] : INT_MAX;
        ek[q] = (j < K && ey[q] != INT_MAX) ? w_key[w][j] : INT_MIN;
      }
      // candidate j ends in lane j
      int ck = INT_MIN, cy = INT_MAX;
      bool picked = false;
      if constexpr (KM > 1) {
        // at most 16 listed entries (the usual case after the wave-level
        // narrowing): compact them into LDS, let each count the entries ahead
        // of it (key desc, then id asc) in registers, and place it by that rank
        unsigned long long vb[kSlots];
        int n = 0;
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
          vb[q] = __ballot(ek[q] != INT_MIN);
          n += __popcll(vb[q]);
        }
        if (n <= 16) {
          // an entry is ahead of another exactly when its composite is larger;
          // padding (0) is never ahead of a listed entry (every key is above INT_MIN)
          int base = 0;
#pragma unroll
          for (int q = 0; q < kSlots; ++q) {
            const int pos = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(vb[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vb[q], 0u));
            if (ek[q] != INT_MIN) s_sel[pos] = sel_order(ek[q], ey[q]);
            base += __popcll(vb[q]);
          }
          if (lane >= n && lane < 16) s_sel[lane] = 0ull;
          // one wave: its LDS operations complete in order
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          unsigned long long cv[16];
#pragma unroll
          for (int q = 0; q < 16; q += 2) {
            const ulonglong2 d = *reinterpret_cast<const ulonglong2 *>(&s_sel[q]);
            cv[q] = d.x;
            cv[q + 1] = d.y;
          }
          const unsigned long long me = s_sel[lane & 15];
          int r = 0;
#pragma unroll
          for (int q = 0; q < 16; ++q) r += (int)(cv[q] > me);
          if (lane < n && r < K) s_win[r] = me;
          asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
          const int nk = min(n, K);
          const unsigned long long wv = s_win[lane < nk ? lane : 0];
          if (lane < nk) {
            ck = sel_key((int)(wv >> 32));
            cy = (int)~(uint32_t)wv;
          }
          picked = true;
        }
      }
      for (int j = 0; j < (picked ? 0 : K); ++j) {
        int v = ek[0];
#pragma unroll
        for (int q = 1; q < kSlots; ++q) v = max(v, ek[q]);
        const int M = wave_max_i(v);
        if (M == INT_MIN) break;
        int by = INT_MAX, bl = 0, bq = 0;
#pragma unroll
        for (int q = 0; q < kSlots; ++q) {
          for (unsigned long long own = __ballot(ek[q] == M); own; own &= own - 1) {
            const int l = __ffsll((long long)own) - 1;
            const int yl = __builtin_amdgcn_readlane(ey[q], l);
            if (yl < by) {
              by = yl;
              bl = l;
              bq = q;
            }
          }
        }
        if (lane == j) {
          ck = M;
          cy = by;
        }
#pragma unroll
        for (int q = 0; q < kSlots; ++q)
          if (q == bq && lane == bl) ek[q] = INT_MIN;
      }
      // each candidate lane resolves where its next state comes from (see HypState)
      const float cf = cy != INT_MAX ? key_of(ck) - lse : -INFINITY;
      int cl[NL], cq = qid;
#pragma unroll
      for (int i = 0; i < NL; ++i) cl[i] = sid[i];
      if (cy != INT_MAX && cy != blank) {
        // the token's LDS entries of this frame: per LM the winner's level /
        // offset, the phrase transition
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          const uint32_t aw = (uint32_t)(arcw[i * Vp + cy] >> 32);
          const uint32_t lo = (aw >> 16) == stamp ? (aw & 0xFFFFu) : 0u;
          // -1: the state after (c_1, y) (rec_dense); -(r + 2): the state after
          // (context of row r, y) (ctx_rec)
          cl[i] = (CTX && i == 0 && Dc >= 2) ? -(crow + 2) : -1;
          if (lo) {
            const int L = (int)(lo >> 13), jj = (int)(lo & 0x1FFFu), N = Nl[i];
            const int bL = s_lbeg[i][L];
            cl[i] = L < N - 1 ? (int)(s_sbase[i][L] + bL + jj)
                              : (jj < kAux ? sTN[i * kAux + jj] : lms[i].top_next[bL + jj - lms[i].arc_base[N - 1]]);
          }
        }
        const uint32_t pw = ptag[cy];
        const uint32_t hi = (pw >> 16) == stamp ? (pw & 0xFFFFu) : 0u;
        cq = -1;
        if (hi) {
          // LDS copy for the first kAux transitions, the table beyond; the table is
          // read through a global-space pointer so the two loads stay distinct
          // (a merged load would take the slower generic-address path)
          const int4 __attribute__((address_space(1))) *gdelta =
              (const int4 __attribute__((address_space(1))) *)tr.delta;
          cq = (int)hi - 1 < kAux ? sDT[hi - 1] : gdelta[dbeg + (int)hi - 1].y;
        }
        if (!p.has_trie) cq = 0;
      }
      if (MODE == kModeStep) {
        if (lane < K) {
          const int64_t o = (int64_t)h * K + lane;
          // (a one-frame greedy call has no scores, and no phrase states without a tree)
          if (cy == INT_MAX) {
            p.tokens[o] = p.scores ? -1 : blank;
            if (p.scores) p.scores[o] = -INFINITY;
#pragma unroll
            for (int i = 0; i < NL; ++i) p.next_lm[(int64_t)i * H * K + o] = hs.cur_lm[i];  // [n_lm][H][k]
            if (p.next_boost) p.next_boost[o] = hs.cur_q;
          } else {
            int q = cq;
#pragma unroll
            for (int i = 0; i < NL; ++i) {
              int l = cl[i];
              if (!inv && l < -1) l = lms[i].ctx_rec[((int64_t)(-l - 2) * V + cy) * RSl[i] + 1];
              else if (!inv && l < 0) l = lms[i].rec_dense[((int64_t)hs.c1[i] * V + cy) * RSl[i] + 1];
              p.next_lm[(int64_t)i * H * K + o] = l;
            }
            if (!inv && q < 0) q = tr.root_node[cy].w;
            p.tokens[o] = cy;
            if (p.scores) p.scores[o] = cf;
            if (p.next_boost) p.next_boost[o] = q;
          }
        }
      } else if constexpr (BEAM) {
        // ---- beam: publish this hypothesis' candidates, meet the stream, rank all ----
        // A candidate record is XW = 3 + NL 64-bit words (one more when recombining),
        // each carrying the frame
        // tag in its top 16 bits over 48 bits of payload: the total score S_b +
        // fused (fp64), the first LM's and the phrase source, the token, the
        // parent's c_1 (first LM) and flags, for a second LM its source and the
        // parent's c_1, and (recombination only) the hash of the history the
        // candidate reaches.  Words are written and read as relaxed agent-scope
        // atomics, so a reader that sees the current tag in all words holds the
        // whole record: polling the records is the rendezvous (no counter, no
        // fence).  Frames alternate between two buffers; a writer can be at most
        // one frame ahead of any reader of its stream, so it never overwrites a
        // buffer that is still being read.
        constexpr int XW = 3 + NL + (RC ? 1 : 0);
        // tags run 1..65535 over the global frame index (0 marks a cleared record);
        // a record left in a buffer is from two frames back, so never current
        const int tg = p.t_base + t;
        unsigned long long *xs = p.xchg + ((size_t)sl * 2 + (tg & 1)) * (size_t)B * K * XW;
        const unsigned long long tag = (unsigned long long)(tg % 65535 + 1) << 48;
        constexpr unsigned long long kPay = (1ull << 48) - 1;
        if (lane < K) {
          const bool has = act && cy != INT_MAX;
          const double tot = has ? hs.S + (double)cf : -INFINITY;
          const unsigned long long tb = (unsigned long long)__double_as_longlong(tot);
          unsigned long long w[XW];
          w[0] = (tb & kPay) | tag;
          w[1] = (tb >> 48) | ((unsigned long long)(unsigned)cl[0] << 16) | tag;
          w[2] = (unsigned long long)(unsigned)cq | ((unsigned long long)(has ? cy + 1 : 0) << 32) | tag;
          w[3] = (unsigned long long)((hs.c1[0] + 1) & 0xFFFF) | ((unsigned long long)(hs.fl & 0xFF) << 16) | tag;
          if constexpr (NL > 1)
            w[4] = (unsigned long long)(unsigned)cl[1] | ((unsigned long long)((hs.c1[1] + 1) & 0xFFFF) << 32) | tag;
          if constexpr (RC) {
            // the history after the candidate: blank emits nothing (a hash is
            // never 0, which marks the start of a stream in the carried buffer)
            const unsigned long long hist = hs.hist;
            const unsigned long long hn = mix64(hist ^ (0x632BE59BD9B4E019ull * (unsigned long long)(cy + 1))) & kPay;
            w[XW - 1] = ((!has || cy == blank) ? hist : (hn ? hn : 1ull)) | tag;
          }
#pragma unroll
          for (int q = 0; q < XW; ++q)
            __hip_atomic_store(xs + (b * K + lane) * XW + q, w[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // every workgroup of the stream ranks the same B*k candidates by (total
        // desc, parent asc, rank asc), i.e. candidate order breaks ties; slot b
        // takes rank b (NaN: no candidate, never ahead of anything)
        const int nc = B * K;
        const double kNone = __longlong_as_double(0x7FF8000000000000ll);
        const int64_t o = (int64_t)t * H + h;
        // the record of candidate i (i < nc): waits until all its words carry this
        // frame's tag; false if the wait ran out
        auto poll = [&](int i, unsigned long long (&w)[XW]) -> bool {
#pragma unroll
          for (int q = 0; q < XW; ++q) w[q] = 0ull;
          bool cur = i >= nc;
          for (int spins = 0;; ++spins) {
            if (i < nc) {
#pragma unroll
              for (int q = 0; q < XW; ++q) w[q] = __hip_atomic_load(xs + i * XW + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
              cur = true;
#pragma unroll
              for (int q = 0; q < XW; ++q) cur = cur && (w[q] & ~kPay) == tag;
            }
            if (__ballot(!cur) == 0ull || aborted) break;
            if (spins >= kSpinLimit) {
              if (lane == 0) atomicOr(p.status, FUSION_STATUS_SYNC_TIMEOUT);
              aborted = true;
              break;
            }
          }
          return cur;
        };
        // the hypothesis of this slot becomes candidate i, of record fields src0 ..
        auto install = [&](int i, double tot, int y, int src0, int c1p0, int qs, int xf, int src1, int c1p1,
                           unsigned long long hist) {
          int src[NL], c1p[NL];
          src[0] = src0;
          c1p[0] = c1p0;
          if constexpr (NL > 1) {
            src[1] = src1;
            c1p[1] = c1p1;
          }
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            hs.lmsrc[l] = src[l];
            hs.c1p[l] = c1p[l];
            hs.c1[l] = y != blank ? y : c1p[l];
          }
          hs.qsrc = qs;
          hs.y = y;
          hs.fl = 1 | (xf & 2);
          if constexpr (RC) hs.hist = hist;
          hs.S = tot;
          p.tokens[o] = y;
          p.parents[o] = i / K;
        };
        auto tot_of = [&](const unsigned long long (&w)[XW]) {
          return __longlong_as_double((long long)((w[0] & kPay) | ((w[1] & 0xFFFF) << 48)));
        };
        bool taken;  // some candidate reaches this slot
        if constexpr (!WIDE) {
          // one candidate per lane: the record stays in its lane's registers, from
          // where the winner installs it; only the totals pass through LDS
          unsigned long long w[XW];
          const bool cur = poll(lane, w);
          const int y1 = (int)((w[2] >> 32) & 0xFFFF);
          double ti = (cur && y1 != 0) ? tot_of(w) : kNone;
          if constexpr (RC) {
            double tm[1] = {ti};
            merge_equal<1>(tm, w[XW - 1] & kPay, nc, lane, s_tot, s_hh, s_tab);
            ti = tm[0];
          }
          s_tot[lane] = ti;
          wave_lds_sync();
          const int r = slot_holder(s_tot, ti, nc, lane, b);
          taken = r >= 0;
          if (lane == r)
            install(lane, ti, y1 - 1, (int)(unsigned)((w[1] >> 16) & 0xFFFFFFFFull), (int)(w[3] & 0xFFFF) - 1,
                    (int)(unsigned)(w[2] & 0xFFFFFFFFull), (int)((w[3] >> 16) & 0xFF),
                    NL > 1 ? (int)(unsigned)(w[NL > 1 ? 4 : 0] & 0xFFFFFFFFull) : 0,
                    NL > 1 ? (int)((w[NL > 1 ? 4 : 0] >> 32) & 0xFFFF) - 1 : 0, w[XW - 1] & kPay);
        } else {
          // four candidates per lane (lane, lane + 64, ..), staged in LDS
          double tq[4];
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            tq[q] = kNone;
            const int i = q * 64 + lane;
            if (q * 64 >= nc) continue;  // uniform
            unsigned long long w[XW];
            const bool cur = poll(i, w);
            if (i < nc) {
              const int y1 = (int)((w[2] >> 32) & 0xFFFF);
              s_xa[i] = make_int4(y1 - 1, (int)(unsigned)((w[1] >> 16) & 0xFFFFFFFFull),
                                  (int)(unsigned)(w[2] & 0xFFFFFFFFull), (int)(w[3] & 0xFFFF) - 1);
              s_xf[i] = (int)((w[3] >> 16) & 0xFF);
              if constexpr (NL > 1)
                s_xb[i] = make_int2((int)(unsigned)(w[4] & 0xFFFFFFFFull), (int)((w[4] >> 32) & 0xFFFF) - 1);
              if constexpr (RC) s_hh[i] = w[XW - 1] & kPay;
              if (cur && y1 != 0) tq[q] = tot_of(w);
            }
          }
          if constexpr (RC) merge_equal<4>(tq, 0ull, nc, lane, s_tot, s_hh, s_tab);
          // The best B are among the candidates at or above any bound that at least B
          // of them reach: here just below the least of the parents' best totals
          // (candidate 0 of each parent's k), which leaves little more than B.
          // Those, in candidate order, are ranked one per lane
          float least = INFINITY;
          int nv = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int i = q * 64 + lane;
            if (i < nc && i % K == 0 && tq[q] == tq[q]) least = fminf(least, (float)tq[q]);
            nv += __popcll(__ballot(tq[q] == tq[q]));
          }
          least = -wave_max_f(-least);
          const double bound = (double)(least - fabsf(least) * 1e-6f);
          unsigned long long up[4];
          int ns = 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            up[q] = __ballot(tq[q] >= bound);
            ns += __popcll(up[q]);
          }
          int wi = -1;
          if (ns <= 64 && (ns >= B || ns == nv)) {
            s_tot[lane] = kNone;
            wave_lds_sync();
            int base = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int at = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(up[q] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)up[q], 0u));
              if (tq[q] >= bound) {
                s_tot[at] = tq[q];
                s_surv[at] = q * 64 + lane;
              }
              base += __popcll(up[q]);
            }
            wave_lds_sync();
            const int r = slot_holder(s_tot, s_tot[lane], ns, lane, b);
            if (r >= 0) wi = s_surv[r];
          } else {
            // many candidates at or near one total, or few parents left: rank all
#pragma unroll
            for (int q = 0; q < 4; ++q)
              if (q * 64 + lane < nc) s_tot[q * 64 + lane] = tq[q];
            wave_lds_sync();
#pragma unroll 1
            for (int i = lane; i < nc; i += 64) {
              const double ti = s_tot[i];
              int r = ti == ti ? 0 : INT_MIN;
#pragma unroll 8
              for (int j = 0; j < nc; ++j) {
                const double tj = s_tot[j];
                r += (tj > ti || (tj == ti && j < i)) ? 1 : 0;
              }
              if (r == b) wi = i;
            }
            const unsigned long long m = __ballot(wi >= 0);
            if (m) wi = __builtin_amdgcn_readlane(wi, __ffsll((long long)m) - 1);
          }
          taken = wi >= 0;
          double tw = kNone;  // the winner's total, from its lane
#pragma unroll
          for (int q = 0; q < 4; ++q)
            if (wi == q * 64 + lane) tw = tq[q];
          if (taken && lane == (wi & 63)) {
            const int4 c = s_xa[wi];
            int2 xb = make_int2(0, 0);
            if constexpr (NL > 1) xb = s_xb[wi];
            install(wi, tw, c.x, c.y, c.w, c.z, s_xf[wi], xb.x, xb.y, RC ? s_hh[RC ? wi : 0] : 0ull);
          }
        }
        if (!taken && lane == 0) {
          // no candidate reaches this slot: the hypothesis is dead and keeps its state
#pragma unroll
          for (int i = 0; i < NL; ++i) {
            hs.lmsrc[i] = hs.cur_lm[i];
            hs.c1p[i] = -1;
          }
          hs.qsrc = hs.cur_q;
          hs.y = -1;
          hs.fl = 0;
          hs.S = -INFINITY;
          p.tokens[o] = -1;
          p.parents[o] = -1;
        }
      }
    }
    lds_barrier();
  }
  // ---- final state ----------------------------------------------------------------
  if (MODE != kModeStep && g == 0) {
    const int V = p.V;
    int nq = hs.qsrc;
    const int y = hs.y;
    // a negative source means "reached by token y" only for valid hypotheses
    // that made a transition; an invalid hypothesis keeps its raw ids
    const bool moved = (hs.fl & 2) == 0 && y >= 0 && y != p.blank;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      int nl = hs.lmsrc[i];
      if (moved && nl < -1) nl = lms[i].ctx_rec[((int64_t)(-nl - 2) * V + y) * RSl[i] + 1];
      else if (moved && nl < 0) nl = lms[i].rec_dense[((int64_t)hs.c1p[i] * V + y) * RSl[i] + 1];
      p.lm_state[(int64_t)i * H + h] = nl;
    }
    if (moved && nq < 0) nq = tr.root_node[y].w;
    if (p.has_trie) p.boost_state[h] = nq;
    if (BEAM) p.hyp_score[h] = hs.S;
    if constexpr (RC) {
      if (p.hist) p.hist[h] = hs.hist;
    }
  }
  if (p.traffic && g == 0) {
    const unsigned long long extra = (h == 0 && p.has_trie) ? 4ull * p.V * (unsigned long long)p.T : 0ull;
    atomicAdd(reinterpret_cast<unsigned long long *>(p.traffic), s_bytes + extra);
    atomicAdd(reinterpret_cast<unsigned long long *>(p.traffic) + 1, s_steps);
  }
}

// the kernel of a mode, alignment and top-k width
template <int W, int NC, int KM, bool AL, int NL>
KernelFn pick_mode(int mode) {
  if constexpr (KM == 1) {
    if (mode == kModeGreedy) return fusion_kernel<W, NC, KM, AL, kModeGreedy, NL>;
  }
  if (mode == kModeBeamRC) return fusion_kernel<W, NC, KM, AL, kModeBeamRC, NL>;
  // (more than 64 candidates need k > 1 even at the widest beam)
  if constexpr (KM > 1) {
    if (mode == kModeBeamWide) return fusion_kernel<W, NC, KM, AL, kModeBeamWide, NL>;
    if (mode == kModeBeamRCWide) return fusion_kernel<W, NC, KM, AL, kModeBeamRCWide, NL>;
  }
  return mode == kModeStep ? fusion_kernel<W, NC, KM, AL, kModeStep, NL> : fusion_kernel<W, NC, KM, AL, kModeBeam, NL>;
}
template <int W, int NC, int KM, int NL>
KernelFn pick_al(bool al, int mode) {
  return al ? pick_mode<W, NC, KM, true, NL>(mode) : pick_mode<W, NC, KM, false, NL>(mode);
}
template <int W, int NC, int NL>
KernelFn pick_k(int km, bool al, int mode) {
  return km == 1 ? pick_al<W, NC, 1, NL>(al, mode) : km == 4 ? pick_al<W, NC, 4, NL>(al, mode) : pick_al<W, NC, 8, NL>(al, mode);
}

}  // namespace
}  // namespace fusion
