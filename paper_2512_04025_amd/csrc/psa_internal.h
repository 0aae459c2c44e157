// Host-side plan (validated, derived parameters) and the kernel launchers behind the C ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/psa.h"

namespace psa {

struct Plan {
  int B, Hq, Hkv, N, d, bq, bk, H, dtype, causal;
  float scale;
  int sq, sk, rep_mode, est_pool, alloc_mode;
  int nq, nk, group, esize;
  // element offset of level h (2..H) inside one pyramid buffer; level h is [B, Hkv, nk*(bk>>(h-1)), d]
  int64_t lvl_off[PSA_MAX_LEVELS + 2];
  int64_t pyr_elems;
  float tau[PSA_MAX_LEVELS];
  double cuts[PSA_MAX_LEVELS];  // cumulative block quotas (QUANTILE / BUDGET)
  bool krep_is_pyramid;         // representative keys are exactly pyramid level H
  bool use_mfma;                // bf16 tensor-core attention kernel applies
  int desc_pitch;               // tile descriptors per query block for the attention kernel (0: not used)
  int desc_words;               // 32-bit words per tile descriptor: one per load instruction of a 64-row tile
  // scratch layout (byte offsets, 256-aligned)
  size_t off_qrep, off_krep, off_scores, off_part, off_bmax, off_rowcnt, off_idx, off_cnt, off_desc, scratch_bytes;
};

int make_plan(const psa_params* p, Plan* out);

// LDS a workgroup may use on gfx950, and the one-time opt-in that lets a kernel ask for more than the
// default 64 KB of dynamic LDS.  The limit is raised to the hardware maximum once per kernel and
// device (never lowered again), so concurrent calls with different problem sizes cannot shrink each
// other's limit between the opt-in and the launch.  `state` is a zero-initialised per-kernel array.
constexpr size_t LDS_LIMIT = 160 * 1024;
constexpr int MAX_DEVICES = 64;
struct LdsOptIn { int done[MAX_DEVICES]; };
hipError_t allow_max_lds(const void* kernel, LdsOptIn* state);

// rows of the per-row counters written by the allocation kernel: [n_visible, c_1 .. c_H]
constexpr int ROWCNT_STRIDE = PSA_MAX_LEVELS + 1;
// per-row level counts consumed by the attention kernels: c_1 .. c_H
constexpr int CNT_STRIDE = PSA_MAX_LEVELS;

// Scores in the factored form the matrix-core importance sweep leaves behind (max pooling): per
// representative query row the softmax statistics (maximum, sum of exponentials, log2 domain) of every
// key slice, and per (representative row, key block) the largest logit.  The score of block pair
// (i, j) is 2^(max over the 8 rows r of block i of (bmax[r, j] - lse[r])).
struct FactoredScores {
  const float2* part;      // [heads][nq * 8][8 slices]
  const float* bmax;       // [heads][bm_rows][bm_pitch]
  int ksplit, bm_rows, bm_pitch;
};

// sims (nullable): also write the intra-block cosine similarities of Alg. 3, float [B*Hkv][nk][H-1]
hipError_t launch_pyramid(const Plan& pl, const void* K, const void* V, void* Kp, void* Vp, float* sims, hipStream_t s);
hipError_t launch_similarities(const Plan& pl, const void* K, float* sims, hipStream_t s);
// tau_s: host, H-1 thresholds for levels 2..H; L: uint8 [B*Hkv][nk]
hipError_t launch_level_cap(const Plan& pl, const float* sims, const float* tau_s, bool all_heads, uint8_t* L, hipStream_t s);
// Hilbert-curve token order of a T x Hg x W grid (host) and the row gather / scatter that applies it
int hilbert_order_host(int T, int Hg, int W, int32_t* perm);
hipError_t launch_permute(const Plan& pl, int heads, const void* X, const int32_t* perm, bool inverse, void* Y, hipStream_t s);
// Rk (nullable): also the keys'
hipError_t launch_representatives(const Plan& pl, const void* Q, void* Rq, const void* K, void* Rk, hipStream_t s);
// part: per (row, key slice) partial softmax statistics of the matrix-core path (Plan::off_part)
// bmax: per (representative row, key block) largest logit, kept for max pooling (Plan::off_bmax)
// factored (nullable out): when the scores can stay in factored form it is filled in, S is NOT written
// and the allocation kernel evaluates the scores itself; otherwise factored->bmax is left null and S holds the scores
hipError_t launch_importance(const Plan& pl, const void* Qrep, const void* Krep, void* part, void* bmax, float* S,
                             FactoredScores* factored, hipStream_t s);
// Scores come from S, or (factored != null) are evaluated from the factored form and, if S_out is given,
// written there as well.  rho (nullable): Eq. 9 per head.  Heads of few short rows are one workgroup, which sums up Eq. 9 itself; for all others it is a
// kernel of its own that reads rowcnt, the per-row counters [n_visible, c_1..c_H] (scratch, left alone otherwise).
// (Summing the rows' counters with atomics from the allocation kernel's 256+ workgroups per head onto a handful of addresses was measured 70 us slower than that
// 4 us kernel.)
hipError_t launch_allocate(const Plan& pl, const float* S, const FactoredScores* factored, float* S_out,
                           const uint8_t* cap, uint8_t* M, uint32_t* rowcnt, float* rho, hipStream_t s);
// Per query block its level-sorted block list and level counts and, unless desc is null or Plan::desc_pitch is 0, per
// 64-column tile of that list the source-row offsets of the tile's load instructions, level and irregularity (Plan::off_desc)
hipError_t launch_lists(const Plan& pl, const uint8_t* M, uint16_t* idx, int32_t* cnt, uint32_t* desc, hipStream_t s);
// Whether the kernels that walk a row's list make it from the level map themselves (M given, idx and cnt unused) instead of reading what
// launch_lists has made (M null): short rows, for which a launch of 4 us counts.  descriptors: the caller would get tile descriptors with the lists
// (the forward's 128-row workgroups), which save up to 10 % of the attention: there only up to 5120 tokens times rounds of the chip (512 workgroups), where
// none of 250 shapes is more than 3 % slower for it.  Attention call, us with a launch / without: 1 head x 1280 tokens 13.5 / 11.1, 40 x 1150 14.3 / 11.9, 12 x 2000
// 14.7 / 12.0, 3 x 4100 24.4 / 23.5, 4 x 5240 34.6 / 36.4, 40 x 3033 74.3 / 80.3, 1 x 12875 71.6 / 78.9, 40 x 7998 at d = 64 173 / 188.  Others, whole call: f32 2 x 1024
// 45.6 / 44.0; 32-row blocks 12 x 4000 58.5 / 52.2; gradients 8 x 745 49.7 / 47.2.
bool lists_in_kernel(const Plan& pl, bool descriptors);
// M and idx both null: dense attention (every key block at level 1)
hipError_t launch_attn_f32(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp,
                            const void* Vp, const uint8_t* M, const uint16_t* idx, const int32_t* cnt, void* O, float* lse,
                            hipStream_t s);
hipError_t launch_attn_mfma(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp,
                            const void* Vp, const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const uint32_t* desc, void* O,
                            float* lse, hipStream_t s);

// Backward of the pyramid attention.  Dr: [B*Hq*N] floats; dKp, dVp: pooled gradients of levels 1..H
// (bwd_pooled_grad_elems floats each); idx / cnt: the level-sorted block lists of launch_lists.
size_t bwd_pooled_grad_elems(const Plan& pl);
// Chunks of 32 query rows in a column of the level map, the last query block's only as far as it has rows.
inline int64_t column_chunks(const Plan& pl) {
  const int64_t full = pl.nq - 1;
  return full * ((pl.bq + 31) / 32) + (pl.N - full * pl.bq + 31) / 32;
}
hipError_t launch_attn_bwd(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                           const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const void* O, const float* lse,
                           const void* dO, float* Dr, float* dKp, float* dVp, void* dQ, void* dK, void* dV, hipStream_t s);

}  // namespace psa
