// What the fusion kernel's launches (fusion_kernels.hip) and its compiled shapes
// share.  The shapes are one file each, so that they compile side by side: lanes
// per hypothesis x 4-token strips per lane, one or two LMs.
#pragma once

#include <hip/hip_runtime.h>

#include "fusion_internal.h"

namespace fusion {

struct Params {
  const float *logits;
  int32_t *lm_state;
  int32_t *boost_state;
  double *hyp_score;
  int32_t *tokens;
  int32_t *parents;
  float *fused;
  int64_t *traffic;
  float *scores;  // fusion_step outputs [H, k]; a one-frame greedy call has no scores (NULL) and
  int32_t *next_lm;     // its states in place (next_boost NULL without a phrase tree)
  int32_t *next_boost;
  unsigned long long *xchg;  // beam exchange [S][2][B][k] candidate records of 3 + n_lm (+ 1 recombining) tagged words
  unsigned long long *hist;  // recombination: [H] in/out history hashes (0: derive from the initial states) or NULL
  unsigned *tickets;         // beam: arrival counters, one per blockIdx class (8 with xcd_map, else 1)
  // t_base: the number of frames decoded by earlier calls of a frame loop that
  // keeps the exchange between calls (its records are tagged by global frame)
  // n_str: streams of this launch (beam), the first of them s_off
  int32_t T, S, B, V, k, blank, mode, has_trie, step_mode, s_off, n_str, xcd_map, n_lm, recombine, t_base;
  float lam[FUSION_MAX_LMS], beta;
  int *status;  // this GPU's status word (bits ORed in by workgroups that meet a bad state or a failed wait)
  LMDevice lm[FUSION_MAX_LMS];  // the n_lm models of Eq. (1), each with its own weight lam[i]
  TrieDevice tr;
};

typedef void (*KernelFn)(Params);

// lanes per hypothesis and 4-token strips per lane for a vocabulary
struct Shape {
  int W, NC, Vp;
};

// MODE: what a launch computes (the code of the other modes is compiled out)
// (RC: with recombination of equal histories; Wide: more than 64 candidates per
// stream, several per lane, staged in LDS: in one kernel with the others, that
// code made the 64 x 4 beam of 4096 tokens spill and run 3 % longer)
constexpr int kModeStep = 0, kModeGreedy = 1, kModeBeam = 2, kModeBeamRC = 3, kModeBeamWide = 4, kModeBeamRCWide = 5;

constexpr int kAux = 256;                     // LDS side tables: phrase transitions, top-level next states

// km: top-k width (1, 4 or 8); al: 16-byte aligned rows
KernelFn pick_w64(int km, bool al, int mode);
KernelFn pick_w256(int km, bool al, int mode);
KernelFn pick_w1024(int km, bool al, int mode);
KernelFn pick_w1024x2(int km, bool al, int mode);
KernelFn pick_w64_2lm(int km, bool al, int mode);
KernelFn pick_w256_2lm(int km, bool al, int mode);
KernelFn pick_w1024_2lm(int km, bool al, int mode);
}  // namespace fusion
