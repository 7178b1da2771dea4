// Output projection of the Transducer joint network on MFMA: the logits that
// the acoustic term of Eq. (1) (Sec. III-C) is computed from, for a batch of
// hypothesis-frames at once:
//
//   out[m, n] = sum_k A[m, k] * W[n, k] + bias[n]      (bf16 inputs, fp32 accumulate)
//
// A is [M, K] and W is [N, K], both row-major bf16 (W in the usual layout of a
// linear layer's weight), so both MFMA operands are contiguous along K.
//
// Tiling for gfx950: a workgroup of WM x WN waves computes a (16 TM WM) x
// (16 TN WN) output tile, each wave (16 TM) x (16 TN) as a TM x TN grid of
// v_mfma_f32_16x16x32_bf16 tiles.  K advances in stages of 64, NB of them in
// LDS; the operands go straight from global memory to LDS (16 bytes a lane, no
// registers, no LDS store instructions), NB - 1 stages ahead, with one barrier
// a stage that waits for the oldest stage's loads only.  A stage's rows are 128
// bytes, all LDS banks, so a fragment read (16 rows, one 16-byte chunk of each)
// would hit the same banks in every row: chunk c of row r is kept in slot
// c ^ (r % 8), which the loading lane arranges by the global chunk it picks.
// SQ_LDS_BANK_CONFLICT reads 0 (rows padded by 16 bytes: 47 % of the LDS's
// active cycles).  The MFMA operands are swapped (W rows as the tile's rows),
// so a lane ends with 4 consecutive columns of one output row.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "fusion_internal.h"

namespace fusion {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kBK = 64;                       // K per stage
constexpr int kMapNone = 0, kMap4x2 = 1, kMapRuns = 2;  // tiles to XCDs
constexpr uint32_t kOutside = 0x80000000u;    // an offset past every descriptor (operands are under 2 GiB)

__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}
// 16 bytes per lane straight into LDS (lane l lands at lds + 16 l)
__device__ __forceinline__ void load_lds(__amdgpu_buffer_rsrc_t r, unsigned char *lds, uint32_t voff, uint32_t soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)lds, 16, voff, soff, 0, 0);
}
// Barrier that also waits for this wave's LDS reads and for all but its N newest
// vector-memory operations (the loads into LDS count there, in order)
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// kWM x kWN waves, each a (16 kTM) x (16 kTN) output tile; kNB stages in LDS;
// kAux: cache policy of the output stores (see joint_project)
template <int kWM, int kWN, int kTM, int kTN, int kNB, int kAux>
__global__ void __launch_bounds__(64 * kWM * kWN, 2) joint_proj_kernel(const uint16_t *__restrict__ A,
                                                                        const uint16_t *__restrict__ W,
                                                                        const float *__restrict__ bias, int M, int N,
                                                                        int K, int n_col_tiles, int map,
                                                                        float *__restrict__ out) {
  constexpr int kRM = 16 * kTM, kRN = 16 * kTN;  // rows and columns of a wave's tile
  constexpr int kBM = kRM * kWM, kBN = kRN * kWN, kWaves = kWM * kWN;
  constexpr int kChunks = kBK / 8;               // 16-byte chunks per row and stage
  constexpr int kRowsPer = 64 / kChunks;         // rows one wave-wide load brings (1 KiB)
  constexpr int kLA = kBM / kRowsPer / kWaves, kLW = kBN / kRowsPer / kWaves, kL = kLA + kLW;  // loads per wave
  static_assert(kLA * kRowsPer * kWaves == kBM && kLW * kRowsPer * kWaves == kBN, "whole loads per wave");
  constexpr int kStage = (kBM + kBN) * kBK * 2;  // bytes of a stage
  constexpr int kSeg = kRN < 64 ? kRN : 64, kLanes = kSeg / 4, kRowsI = 64 / kLanes;  // epilogue: see there
  static_assert(kNB * kStage >= kWaves * 16 * kSeg * 4, "LDS too small for the epilogue");
  __shared__ __align__(1024) unsigned char smem[kNB * kStage];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // tile of this workgroup, which runs on XCD x = blockIdx % 8 under the hardware's
  // round-robin (see joint_project for the choice):
  // kMap4x2 (row tiles a multiple of 4, column tiles even): XCD x takes the row
  // tiles = x % 4 (mod 4) against column half x / 4, so a row band of A is fetched by
  // two XCDs instead of eight and each XCD's L2 keeps half of W.
  // kMapRuns: each XCD takes a run of consecutive tiles, column-fastest, so that a row
  // band of A is fetched by one XCD (two at a run's end) and every L2 holds W.
  // kMapNone: column-fastest over all XCDs
  int tr, tc;
  if (map == kMap4x2) {
    const int x = blockIdx.x & 7, i = blockIdx.x >> 3;
    const int half = n_col_tiles >> 1;
    tr = (i / half) * 4 + (x & 3);
    tc = (x >> 2) * half + i % half;
  } else {
    int t = blockIdx.x;
    if (map == kMapRuns) {
      const int x = t & 7, per = gridDim.x >> 3, more = gridDim.x & 7;  // the first `more` XCDs take one tile more
      t = x * per + min(x, more) + (t >> 3);
    }
    tr = t / n_col_tiles;
    tc = t % n_col_tiles;
  }
  const int bn = tc * kBN, bm = tr * kBM;
  const int wm = (wave / kWN) * kRM, wn = (wave % kWN) * kRN;

  // Load j of a stage brings rows (j * kWaves + wave) * kRowsPer .. of A (j < kLA)
  // or W to consecutive LDS: lane l lands 16 l bytes in, i.e. row l / 8, slot
  // l % 8, and fetches the chunk which that slot holds.  Rows past the operand
  // and, in a ragged last stage, chunks past K read as zeros (range check).
  const __amdgpu_buffer_rsrc_t ra = rsrc(A, (uint32_t)((int64_t)M * K * 2));
  const __amdgpu_buffer_rsrc_t rw = rsrc(W, (uint32_t)((int64_t)N * K * 2));
  const int lr = lane / kChunks, lc = (lane % kChunks) ^ (lr & 7);  // kRowsPer is 8: the row's low bits are lr
  uint32_t vo[kL];
#pragma unroll
  for (int j = 0; j < kL; ++j) {
    const int row = (j < kLA ? bm + (j * kWaves + wave) * kRowsPer : bn + ((j - kLA) * kWaves + wave) * kRowsPer) + lr;
    vo[j] = row < (j < kLA ? M : N) ? (uint32_t)(((int64_t)row * K + lc * 8) * 2) : kOutside;
  }
  auto issue = [&](int s, int buf) {
    unsigned char *base = smem + buf * kStage + wave * 1024;
    const bool ragged = (s + 1) * kBK > K && s * kBK + lc * 8 >= K;
#pragma unroll
    for (int j = 0; j < kL; ++j)
      load_lds(j < kLA ? ra : rw, base + j * kWaves * 1024, ragged ? kOutside : vo[j], s * kBK * 2);
  };

  f32x4 acc[kTM][kTN];
#pragma unroll
  for (int i = 0; i < kTM; ++i)
#pragma unroll
    for (int j = 0; j < kTN; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  const int nk = (K + kBK - 1) / kBK;
#pragma unroll
  for (int s = 0; s < kNB - 1; ++s)
    if (s < nk) issue(s, s);
  // fragment of a 16 x 32 operand tile: lane l holds row l % 16, K elements 8 * (l / 16) .. + 7
  const int fr = lane & 15, fc = lane >> 4;
  int buf = 0;
  for (int s = 0; s < nk; ++s) {
    // stage s has landed for every wave, and every wave is done reading the
    // buffer of stage s - 1, which stage s + kNB - 1 is loaded into
    if (s + kNB - 2 < nk) wait_barrier<(kNB - 2) * kL>();
    else wait_barrier<0>();
    if (s + kNB - 1 < nk) issue(s + kNB - 1, buf == 0 ? kNB - 1 : buf - 1);
    const unsigned char *pa = smem + buf * kStage, *pw = pa + kBM * kBK * 2;
#pragma unroll
    for (int ks = 0; ks < kBK / 32; ++ks) {
      bf16x8 fa[kTM], fw[kTN];
#pragma unroll
      for (int j = 0; j < kTN; ++j)
        fw[j] = *reinterpret_cast<const bf16x8 *>(pw + (wn + j * 16 + fr) * kBK * 2 + (((ks * 4 + fc) ^ (fr & 7)) * 16));
#pragma unroll
      for (int i = 0; i < kTM; ++i)
        fa[i] = *reinterpret_cast<const bf16x8 *>(pa + (wm + i * 16 + fr) * kBK * 2 + (((ks * 4 + fc) ^ (fr & 7)) * 16));
#pragma unroll
      for (int i = 0; i < kTM; ++i)
#pragma unroll
        for (int j = 0; j < kTN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[j], fa[i], acc[i][j], 0, 0, 0);
    }
    buf = buf == kNB - 1 ? 0 : buf + 1;
  }

  // Epilogue.  In the accumulator of a 16 x 16 tile lane l holds output row l %
  // 16, columns 4 * (l / 16) .. + 3.  Each 16-row slab of the wave's tile goes
  // through the wave's own LDS area (free once every wave has read the last
  // stage), chunks swizzled by the row as above, and leaves as whole row segments
  // of kSeg columns, kRowsI rows a store.  The bias is fetched before the first
  // store: a load behind stores would wait for all of them.
  float bv[kRN / kSeg][4];
#pragma unroll
  for (int sg = 0; sg < kRN / kSeg; ++sg)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = bn + wn + sg * kSeg + (lane % kLanes) * 4 + r;
      bv[sg][r] = (bias && n < N) ? bias[n] : 0.0f;
    }
  wait_barrier<0>();
  f32x4 *slab = reinterpret_cast<f32x4 *>(smem) + wave * 16 * kLanes;
  const int orow = lane / kLanes, ochunk = lane % kLanes;
#pragma unroll
  for (int i = 0; i < kTM; ++i) {
#pragma unroll
    for (int sg = 0; sg < kRN / kSeg; ++sg) {
#pragma unroll
      for (int j = 0; j < kSeg / 16; ++j)
        slab[fr * kLanes + ((j * 4 + fc) ^ (fr & (kLanes - 1)))] = acc[i][sg * (kSeg / 16) + j];
      __builtin_amdgcn_wave_barrier();
      const int n = bn + wn + sg * kSeg + ochunk * 4;
#pragma unroll
      for (int q = 0; q < 16 / kRowsI; ++q) {
        const int row = q * kRowsI + orow;
        const f32x4 x = slab[row * kLanes + (ochunk ^ (row & (kLanes - 1)))];
        i32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = __float_as_int(x[r] + bv[sg][r]);
        // a descriptor of this store's rows that exist; columns past N fall outside it
        const int m0 = bm + wm + i * 16 + q * kRowsI;
        const int rows = min(max(M - m0, 0), kRowsI);
        const __amdgpu_buffer_rsrc_t ro = rsrc(out + (int64_t)m0 * N, (uint32_t)rows * (uint32_t)N * 4u);
        const uint32_t o = ((uint32_t)orow * (uint32_t)N + (uint32_t)n) * 4u;
        __builtin_amdgcn_raw_buffer_store_b128(v, ro, n + 3 < N ? o : kOutside, 0, kAux);
        if (N % 4 != 0) {  // uniform: the row's last columns, one at a time
#pragma unroll
          for (int r = 0; r < 3; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(v[r], ro, (n + 3 >= N && n + r < N) ? o + 4 * r : kOutside, 0, kAux);
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// a launch shape of joint_proj_kernel
template <int WM_, int WN_, int TM_, int TN_, int NB_>
struct ProjCfg {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, NB = NB_;
  static constexpr int BM = 16 * TM_ * WM_, BN = 16 * TN_ * WN_;
};

}  // namespace
}  // namespace fusion

using namespace fusion;

extern "C" int joint_project(const uint16_t *A, const uint16_t *W, const float *bias, int32_t M, int32_t N,
                             int32_t K, float *out, hipStream_t stream) {
  if (M < 0 || N < 1 || K < 8) return set_error(FUSION_E_ARG, "M, N or K out of range");
  if (K % 8 != 0) return set_error(FUSION_E_UNSUPPORTED, "K must be a multiple of 8");
  if ((int64_t)M * K * 2 > 0x7FFFFFF0ll || (int64_t)N * K * 2 > 0x7FFFFFF0ll)
    return set_error(FUSION_E_UNSUPPORTED, "operand larger than 2 GiB: split the call along M");
  if (M == 0) return FUSION_OK;
  if (!A || !W || !out) return set_error(FUSION_E_ARG, "NULL operand");
  if (((uintptr_t)A | (uintptr_t)W) % 16 != 0) return set_error(FUSION_E_ARG, "A and W must be 16-byte aligned");
  constexpr ProjCfg<2, 4, 8, 4, 2> t256{};
  constexpr ProjCfg<2, 2, 4, 4, 2> t128{};
  constexpr ProjCfg<2, 2, 2, 4, 2> t64x128_3a_cu{};
  constexpr ProjCfg<2, 2, 2, 4, 3> t64x128{};
  constexpr ProjCfg<2, 2, 2, 2, 4> t64{};
  constexpr ProjCfg<2, 2, 1, 2, 4> t32{};
  constexpr int64_t kCus = 256;
  auto tiles = [&](auto cfg) -> int64_t {
    using C = decltype(cfg);
    return (int64_t)((M + C::BM - 1) / C::BM) * ((N + C::BN - 1) / C::BN);
  };
  auto go = [&](auto cfg) -> int {
    using C = decltype(cfg);
    const int nct = (N + C::BN - 1) / C::BN, nrt = (M + C::BM - 1) / C::BM;
    if (tiles(cfg) > 0x7FFFFFFFll) return set_error(FUSION_E_UNSUPPORTED, "too many tiles");
    // Tiles to XCDs: 4 x 2 where the tiles divide so; else, in a launch of more than a
    // round, in runs if W fits an L2 (up to 4 MB), has at most 32 column tiles and is
    // the smaller operand.  Not dealt at all, 128 x 128 tiles fetch every row band of A on
    // all eight XCDs: 30343 x 1024 x 248 45 us, in runs 36; 48340 x 1024 x 768 117 and 88;
    // over 190 random sizes that the rule takes 5 % (M < 2 N) to 14 % (M > 8 N) faster in
    // runs, 256 x 256 tiles 4 to 5 %.  Against 4 x 2 runs gain 7 % to lose 19 %.
    const bool by4x2 = nrt % 4 == 0 && nct % 2 == 0;
    const bool runs = tiles(t128) > kCus && M >= N && nct <= 32 && (int64_t)N * K * 2 <= 4 << 20;
    const int map = by4x2 ? kMap4x2 : runs ? kMapRuns : kMapNone;
    // Rows of whole 128-byte lines leave as streaming stores (nt with sc1: 459 us
    // for 76800 x 4096 x 640, plain 535, launches back to back); rows that share lines with their
    // neighbours are left for the L2 to merge (76800 x 1001 x 136: 91 us plain,
    // over 100 streaming)
    const dim3 grid(nct * nrt), block(64 * C::WM * C::WN);
    if (N % 32 == 0)
      hipLaunchKernelGGL((joint_proj_kernel<C::WM, C::WN, C::TM, C::TN, C::NB, 18>), grid, block, 0, stream, A, W, bias,
                         M, N, K, nct, map, out);
    else
      hipLaunchKernelGGL((joint_proj_kernel<C::WM, C::WN, C::TM, C::TN, C::NB, 0>), grid, block, 0, stream, A, W, bias,
                         M, N, K, nct, map, out);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FUSION_OK : hip_error(e, "joint projection launch");
  };
  // By the number of tiles, which decides how evenly a launch fills the 256 CUs: a
  // larger tile reads less LDS per multiply-accumulate, a smaller one fills the
  // chip.  Measured (us; tiles in brackets):
  //              256x256      128x128      64x128       64x64        32x64
  //   256x4096   19 [16]      9.6 [64]     7.5 [128]    6.2 [256]    6.1 [512]     K = 640
  //   777x2500   12 [40]      7.2 [140]    6.7 [260]    7.8 [520]    7.3 [1000]    K = 256
  //   1664x4096  21 [112]     13.3 [416]   16.7 [832]   20 [1664]    23 [3328]     K = 640
  //   3328x1001  13 [52]      8.3 [208]    7.4 [416]    8.6 [832]    9.2 [1664]    K = 136
  // 256 x 256 from a thousand tiles on, except where
  //   - half of each tile or more would lie past N: 512000 x 100 x 128 took 93 us
  //     with it, 69 with 128 x 128; x 64 x 640 188 and 151; x 200 x 640 237 and 300
  //   - K is over 640 and rows are whole lines, for fewer than 2000 tiles, where the two
  //     are level or 128 x 128 ahead (25600 x 4096: 191 and 177 at K = 704, 218 and 206
  //     at 832, 249 and 252 at 1024).  With more tiles: 76800 x 4096 508 and 545 us at
  //     704, 660 and 764 at 1024; 51200 x 4096 341 and 351, 456 and 498; 512000 x 256
  //     263 and 315, 347 and 397.  With rows that share lines, 1000 tiles do:
  //     25600 x 2500 117 and 136 at 704, 148 and 169 at 1024
  // and from 400 on where W is over 4 MB and 128 x 128 tiles cannot be dealt 4 x 2 (A
  // then goes to all XCDs, half as often): 7711 x 3968 x 648 59 us and 73, 8837 x 6784 x
  // 504 96 and 118, but 12594 x 4032 x 536 97 and 91.
  // A single column of them (N of 129 to 256) also pays as one full round, 129 to 256
  // tiles, and from 400 on: A is read once, not twice (61385 x 208 x 240 18.3 us and
  // 25.5, in runs 20.4; 188 tiles of 192 x 912 31 and 48, 35; 503 of 181 x 600 62 and 87,
  // 70; but 299 of 165 x 128 32 and 26).
  // 128 x 128 holds two workgroups a CU: 513 to 640 tiles of it leave a second
  // round nearly empty, and 64 x 128 with two stages in LDS (three a CU) is ahead:
  // 3323 x 2500 x 256 13.3 us and 17.0, 8315 x 1001 x 512 23.1 and 27.7, 3195 x 3072 x
  // 512 17.1 and 20.4; at 680 tiles the two are level.  Not for wide rows dealt 4 x 2
  // (2555 x 4096 x 640 24 and 22.8 us) or of a long K (1580 x 5635 x 560 33.8 and 31.1).
  const int64_t n256 = tiles(t256), n128 = tiles(t128);
  const bool even128 = (N + 127) / 128 % 2 == 0;
  const bool t128_4x2 = (M + 127) / 128 % 4 == 0 && even128, t64x128_4x2 = (M + 63) / 64 % 4 == 0 && even128;
  if (n256 >= 1000 && N > 128 && (K <= 640 || n256 >= 2000 || N % 32 != 0)) return go(t256);
  if (n256 >= 400 && (int64_t)N * K * 2 > 4 << 20 && !t128_4x2) return go(t256);
  if (N > 128 && N <= 256 && n256 > kCus / 2 && (n256 <= kCus || n256 >= 400)) return go(t256);
  if (n128 > 2 * kCus && n128 <= 5 * kCus / 2 && (N < 4096 || (!t64x128_4x2 && K <= 512))) return go(t64x128_3a_cu);
  if (n128 > kCus) return go(t128);
  // (the narrower tiles store 8 rows at once: their offsets need 8 rows under 2 GiB)
  if (tiles(t64x128) > kCus || N >= (1 << 25)) return go(t64x128);
  if (tiles(t64) > kCus) return go(t64);
  return go(t32);
}
