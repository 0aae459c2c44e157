// Multi-level mask assignment (Sec. 3.3.2, Alg. 2, Eq. 5-7; quantile rule of Sec. 4.4), the
// compute ratio of Eq. 9, and the per-row level-sorted block lists the attention kernels walk.
//
// alloc_kernel: one wavefront per query block.  The row of scores is turned into 64-bit keys
// (descending score, then ascending block index -> a stable descending sort), sorted with a bitonic
// network held in registers, and levels are read off the sorted order: from the fp64 inclusive
// cumulative share (Alg. 2) or from the rank against per-level quotas.
#include "psa_dev.h"
#include "psa_internal.h"

namespace psa {

struct AllocArgs {
  int N, Hq, Hkv, nq, nk, bq, bk, H, causal, mode;
  float tau[PSA_MAX_LEVELS];
  double cuts[PSA_MAX_LEVELS];
  FactoredScores fs;             // used by the FACTORED instantiation
  float* S_out;                  // FACTORED: nullable, receives the evaluated scores
};

// 0 invisible, 1 fully visible, 2 straddles the causal diagonal
__device__ __forceinline__ int block_vis(int i, int j, int bq, int bk, int N, int causal) {
  if (!causal) return 1;
  const int r0 = i * bq;
  int r1 = r0 + bq; r1 = (r1 < N ? r1 : N) - 1;
  const int c0 = j * bk;
  int c1 = c0 + bk; c1 = (c1 < N ? c1 : N) - 1;
  return c1 <= r0 ? 1 : (c0 > r1 ? 0 : 2);
}

// 32-bit pattern that sorts ASCENDING in the order of DESCENDING float value (-0 == +0)
__device__ __forceinline__ uint32_t desc_bits(float f) {
  uint32_t u = __float_as_uint(f == 0.f ? 0.f : f);
  const uint32_t asc = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return ~asc;
}
__device__ __forceinline__ float from_desc_bits(uint32_t d) {
  const uint32_t asc = ~d;
  const uint32_t u = (asc & 0x80000000u) ? (asc & 0x7fffffffu) : ~asc;
  return __uint_as_float(u);
}

// floor(a * n + 1e-3) with separately rounded product and sum (no fused multiply-add), so that the
// host-side statement of the rule gives the same integer
__device__ __forceinline__ int quota_edge(double a, int n) {
  return (int)floor(__dadd_rn(__dmul_rn(a, (double)n), 1e-3));
}

__device__ __forceinline__ double wave_incl_scan(double x, int lane) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  return x;
}

// Value of lane (l ^ m) for m = 1, 2, 4 ... 32.  Neighbours at distance 1 and 2 come through the data-parallel
// primitives of the vector unit (no LDS instruction, no wait), 4, 8 and 16 through the LDS crossbar's
// swizzle (no address register), 32 through a permute.
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v, int m) {
  switch (m) {
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, true);   // quad_perm [1,0,3,2]
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, true);   // quad_perm [2,3,0,1]
    case 4: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (4 << 10));               // and 0x1f, or 0, xor 4
    case 8: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (8 << 10));
    case 16: return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x1F | (16 << 10));
    default: return (uint32_t)__shfl_xor((int)v, 32, 64);
  }
}
__device__ __forceinline__ uint64_t lane_xor64(uint64_t v, int m) {
  return ((uint64_t)lane_xor32((uint32_t)(v >> 32), m) << 32) | lane_xor32((uint32_t)v, m);
}

// One wavefront per query block, the whole row in registers: lane l holds the KPL keys at sorted
// positions l*KPL .. l*KPL+KPL-1.  Bitonic stages whose partner distance is below KPL exchange
// registers of one lane (register numbers are compile-time); longer distances exchange the same
// register between lanes l and l ^ m.  No LDS traffic and no barrier in the sort.
// FACTORED: the scores are evaluated here from the matrix-core importance sweep's block maxima and
// softmax statistics (max pooling of Eq. 4: S_ij = 2^(max over the block's 8 rows of (largest logit - lse)))
// instead of being read from memory.  That part is plain streaming work, so the workgroup then has
// four wavefronts: all of them evaluate the row into LDS (and write it out if the caller wants the
// scores); with NW = 1 three then retire and the first sorts the row.
// NW = 4 (rows of more than 128 blocks): the row is spread over the 256 lanes of four wavefronts,
// KPL keys each; the three merge steps whose partner lane sits in another wavefront go through LDS.
// (One wavefront with 32 or 64 keys per lane needs 140+ registers: three wavefronts per SIMD, and the
// sort, a chain of short dependent steps, then runs 6.8 times longer per row than with 16 keys per lane.)
// HEAD (rows of up to 128 blocks, heads of up to HEAD_ROWS of them): one workgroup per head, a wavefront per row from the scores to the levels, and the
// compute ratio of Eq. 9 at the end: a launch less for short calls.  Whole forward, us, row per workgroup and ratio kernel -> this: 40 heads x 402
// tokens (four rows) 35.7 -> 28.3, 12 x 1000 (eight) 42.2 -> 37.4; with eight rows at most -> sixteen: 8 x 542 in 64-row blocks (nine) 39.3 -> 38.1, 12 x 2000 44.4 -> 44.0,
// float32 2 x 1024 36.7 -> 36.0.
constexpr int HEAD_ROWS = 16;
template <int KPL, bool FACTORED, int NW, bool HEAD>
__global__ __launch_bounds__(HEAD ? 64 * HEAD_ROWS : (FACTORED || NW == 4) ? 256 : 64) void alloc_kernel(const float* __restrict__ S, const uint8_t* __restrict__ cap,
                                                                    uint8_t* __restrict__ M, uint32_t* __restrict__ rowcnt, float* __restrict__ rho,
                                                                    AllocArgs a) {
  static_assert(!HEAD || NW == 1, "a wavefront per row");
  constexpr int RPW = HEAD ? HEAD_ROWS : 1;              // rows of a workgroup, each with its part of the LDS
  __shared__ int cnt_all[RPW][PSA_MAX_LEVELS + 1];
  __shared__ float lse_all[RPW][8];
  __shared__ float srow_all[RPW][FACTORED ? KPL * 64 * NW : 1];
  __shared__ int vis_all[RPW];
  const int mine = HEAD ? (int)threadIdx.x >> 6 : 0;
  int* cnt_s = cnt_all[mine];
  float *lse_s = lse_all[mine], *srow_s = srow_all[mine];
  __shared__ uint64_t xbuf[NW == 4 ? KPL * 256 : 1];
  __shared__ double wave_d[4];
  __shared__ int wave_i[4];
  constexpr int LANES = 64 * NW;
  const int lane = threadIdx.x & 63;
  const int glane = NW == 1 ? lane : (int)threadIdx.x;   // position of this lane among the sorting lanes
  const int i = HEAD ? mine : (int)blockIdx.x, hq = blockIdx.y, b = blockIdx.z;
  const int64_t head = (int64_t)b * a.Hq + hq;
  const int64_t row = head * a.nq + i;
  const float* s_row = FACTORED ? nullptr : S + row * a.nk;
  const int tid = HEAD ? lane : (int)threadIdx.x;        // among the threads that evaluate the row's scores
  constexpr int EVAL = HEAD ? 64 : 256;
  // (LDS serves one wavefront's accesses in order: a row of its own needs the fence only)
  auto row_sync = [&]() __attribute__((always_inline)) {
    if constexpr (HEAD) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
      __syncthreads();
    }
  };
  if (tid <= PSA_MAX_LEVELS) cnt_s[tid] = 0;
  if (FACTORED) {
    if (tid < 8) {      // lse of the block's 8 representative rows from the key slices' partial results
      const float2* pr = a.fs.part + ((head * a.nq + i) * 8 + tid) * 8;
      float mrow = -INFINITY, lrow = 0.f;
      for (int s2 = 0; s2 < a.fs.ksplit; ++s2) mrow = fmaxf(mrow, pr[s2].x);
      for (int s2 = 0; s2 < a.fs.ksplit; ++s2) {
        const float2 v = pr[s2];
        if (v.x != -INFINITY) lrow += v.y * __builtin_amdgcn_exp2f(v.x - mrow);
      }
      lse_s[tid] = lrow > 0.f ? mrow + __log2f(lrow) : INFINITY;   // no visible key: all scores 0
    }
    row_sync();
    const float* __restrict__ bm0 = a.fs.bmax + (head * a.fs.bm_rows + (int64_t)i * 8) * a.fs.bm_pitch;
    for (int j = tid; j < a.nk; j += EVAL) {
      float v = -INFINITY;
#pragma unroll
      for (int r = 0; r < 8; ++r) v = fmaxf(v, bm0[(int64_t)r * a.fs.bm_pitch + j] - lse_s[r]);
      const float sc = __builtin_amdgcn_exp2f(v);
      srow_s[j] = sc;
      if (a.S_out) a.S_out[row * a.nk + j] = sc;
    }
    row_sync();
    if (!HEAD && NW == 1 && tid >= 64) return;   // no workgroup barrier follows in that instantiation
  } else {
    row_sync();
  }
  uint8_t* m_row = M + row * a.nk;
  const uint8_t* cap_row = cap ? cap + ((int64_t)b * a.Hkv + hq / (a.Hq / a.Hkv)) * a.nk : nullptr;
  const bool quota = a.mode != PSA_ALLOC_THRESHOLD && a.mode != PSA_ALLOC_THRESHOLD_EXCL;
  const bool exclusive = a.mode == PSA_ALLOC_THRESHOLD_EXCL;   // Alg. 2 read with the exclusive cumulative sum

  uint64_t key[KPL];
  int n_vis = 0;
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    const int j = r * LANES + glane;   // any initial placement will do; this one reads coalesced
    uint64_t kk = ~0ull;
    if (j < a.nk) {
      const int v = block_vis(i, j, a.bq, a.bk, a.N, a.causal);
      const float sj = FACTORED ? srow_s[j] : (v != 0 ? s_row[j] : 0.f);
      if (v == 0) {
        m_row[j] = 0;
      } else {
        const uint32_t ord = (quota && v == 2) ? 0u : desc_bits(sj);
        kk = ((uint64_t)ord << 32) | (uint32_t)j;
        ++n_vis;
      }
    }
    key[r] = kk;
  }
#pragma unroll
  for (int off = 32; off; off >>= 1) n_vis += __shfl_xor(n_vis, off, 64);
  if (NW == 4) {
    if (lane == 0) wave_i[threadIdx.x >> 6] = n_vis;
    __syncthreads();
    n_vis = wave_i[0] + wave_i[1] + wave_i[2] + wave_i[3];
  }

  // bitonic sort, ascending over position glane*KPL + r
  auto in_lane = [&](uint64_t& x, uint64_t& y, bool up) {
    const bool sw = (x > y) == up;
    const uint64_t lo = sw ? y : x;
    y = sw ? x : y;
    x = lo;
  };
#pragma unroll
  for (int k = 2; k <= KPL; k <<= 1) {        // phases that stay inside a lane
#pragma unroll
    for (int jj = k >> 1; jj > 0; jj >>= 1) {
#pragma unroll
      for (int r = 0; r < KPL; ++r) {
        if (r & jj) continue;
        const bool up = k < KPL ? ((r & k) == 0) : ((glane & 1) == 0);
        in_lane(key[r], key[r | jj], up);
      }
    }
  }
#pragma unroll
  for (int kl = 2; kl <= LANES; kl <<= 1) {   // phase k = kl * KPL
    const bool up = (glane & kl) == 0;
#pragma unroll
    for (int m = kl >> 1; m > 0; m >>= 1) {   // partner lane l ^ m
      const bool keep_min = ((glane & m) == 0) == up;
      if (m >= 64) {                          // the partner is in another wavefront: through LDS
#pragma unroll
        for (int r = 0; r < KPL; ++r) xbuf[r * 256 + glane] = key[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
          const uint64_t mine = key[r];
          const uint64_t other = xbuf[r * 256 + (glane ^ m)];
          key[r] = ((mine < other) == keep_min) ? mine : other;
        }
        __syncthreads();
      } else {
#pragma unroll
        for (int r = 0; r < KPL; ++r) {
          const uint64_t mine = key[r];
          const uint64_t other = lane_xor64(mine, m);
          key[r] = ((mine < other) == keep_min) ? mine : other;
        }
      }
    }
#pragma unroll
    for (int jj = KPL >> 1; jj > 0; jj >>= 1) {
#pragma unroll
      for (int r = 0; r < KPL; ++r) {
        if (r & jj) continue;
        in_lane(key[r], key[r | jj], up);
      }
    }
  }

  const int k0 = glane * KPL;
  int e_hi[PSA_MAX_LEVELS];
  double offset = 0.0, total = 1.0;
  bool uniform = false;
  if (quota) {
    int prev = 0;
    bool none = quota_edge(a.cuts[a.H - 1], n_vis) == 0;
    for (int h = 0; h < a.H; ++h) {
      int e = none ? 1 : quota_edge(a.cuts[h], n_vis);
      e = e < prev ? prev : e;
      e = e > n_vis ? n_vis : e;
      e_hi[h] = e;
      prev = e;
    }
  } else {
    // total of the visible scores (fp64), then shares and their inclusive cumulative sum
    double part = 0.0;
#pragma unroll
    for (int r = 0; r < KPL; ++r)
      if (k0 + r < n_vis) part += (double)from_desc_bits((uint32_t)(key[r] >> 32));
    total = part;
#pragma unroll
    for (int off = 32; off; off >>= 1) total += __shfl_xor(total, off, 64);
    if (NW == 4) {
      if (lane == 0) wave_d[threadIdx.x >> 6] = total;
      __syncthreads();
      total = ((wave_d[0] + wave_d[1]) + wave_d[2]) + wave_d[3];
      __syncthreads();
    }
    uniform = !(total > 0.0);
    if (uniform) total = (double)n_vis;
    double local = 0.0;
#pragma unroll
    for (int r = 0; r < KPL; ++r)
      if (k0 + r < n_vis) local += (uniform ? 1.0 : (double)from_desc_bits((uint32_t)(key[r] >> 32))) / total;
    const double incl = wave_incl_scan(local, lane);
    offset = incl - local;
    if (NW == 4) {                            // plus the shares held by the wavefronts before this one
      if (lane == 63) wave_d[threadIdx.x >> 6] = incl;
      __syncthreads();
      for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) offset += wave_d[w];
    }
  }

  double run = 0.0;               // (the counters were cleared before the first barrier)
#pragma unroll
  for (int r = 0; r < KPL; ++r) {
    const int k = k0 + r;
    if (k < n_vis) {
      const int j = (int)(uint32_t)key[r];
      int level = 0;
      if (quota) {
        for (int h = a.H - 1; h >= 0; --h)
          if (k < e_hi[h]) level = h + 1;
      } else {
        const double share = (uniform ? 1.0 : (double)from_desc_bits((uint32_t)(key[r] >> 32))) / total;
        run += share;
        const double ehat = exclusive ? (offset + run) - share : offset + run;
        for (int h = a.H - 1; h >= 0; --h)
          if (ehat <= (double)a.tau[h]) level = h + 1;
        if (k == 0 && level == 0) level = 1;
      }
      if (block_vis(i, j, a.bq, a.bk, a.N, a.causal) == 2) level = 1;
      if (cap_row && level > 0) {
        const int cj = cap_row[j];
        level = level < cj ? level : cj;
      }
      m_row[j] = (uint8_t)level;
      atomicAdd(&cnt_s[level], 1);
    }
  }
  // the counters are complete: one wavefront is left here in either instantiation and its LDS
  // operations complete in order, so a fence is enough where the other wavefronts have retired
  if (FACTORED && NW == 1 && !HEAD) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  else row_sync();
  if constexpr (HEAD) {
    if (lane == 0) vis_all[mine] = n_vis;
    __syncthreads();
    if (rho && mine == 0) {
      // in units of 2^-(H-1): whole numbers, a row per lane
      static_assert((long long)HEAD_ROWS * KPL * 64 << (PSA_MAX_LEVELS - 1) < 1ll << 31, "32 bits hold the sum over the rows");
      int num = 0, den = lane < a.nq ? vis_all[lane & (RPW - 1)] : 0;
      for (int h = 1; h <= a.H; ++h) num += lane < a.nq ? cnt_all[lane & (RPW - 1)][h] << (a.H - h) : 0;
#pragma unroll
      for (int off = RPW / 2; off; off >>= 1) {
        num += __shfl_xor(num, off, 64);
        den += __shfl_xor(den, off, 64);
      }
      if (lane == 0) rho[head] = (float)((double)num / (double)(1 << (a.H - 1)) / (double)den);
    }
    return;
  }
  if (glane <= a.H) rowcnt[row * ROWCNT_STRIDE + lane] = lane == 0 ? (uint32_t)n_vis : (uint32_t)cnt_s[lane];
}

static hipError_t launch_rho(const Plan& pl, const uint32_t* rowcnt, float* rho, hipStream_t s);

template <int KPL, int NW>
static hipError_t launch_alloc_t(const Plan& pl, const AllocArgs& a, const float* S, const uint8_t* cap, uint8_t* M,
                                 uint32_t* rowcnt, float* rho, hipStream_t s) {
  if constexpr (NW == 1) {
    if (pl.nq <= HEAD_ROWS) {
      const dim3 heads(1, pl.Hq, pl.B);
      if (a.fs.bmax) alloc_kernel<KPL, true, 1, true><<<heads, 64 * pl.nq, 0, s>>>(S, cap, M, rowcnt, rho, a);
      else alloc_kernel<KPL, false, 1, true><<<heads, 64 * pl.nq, 0, s>>>(S, cap, M, rowcnt, rho, a);
      return hipGetLastError();
    }
  }
  dim3 grid(pl.nq, pl.Hq, pl.B);
  if (a.fs.bmax) alloc_kernel<KPL, true, NW, false><<<grid, 256, 0, s>>>(S, cap, M, rowcnt, nullptr, a);
  else alloc_kernel<KPL, false, NW, false><<<grid, 64 * NW, 0, s>>>(S, cap, M, rowcnt, nullptr, a);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess && rho ? launch_rho(pl, rowcnt, rho, s) : e;
}

hipError_t launch_allocate(const Plan& pl, const float* S, const FactoredScores* factored, float* S_out,
                           const uint8_t* cap, uint8_t* M, uint32_t* rowcnt, float* rho, hipStream_t s) {
  AllocArgs a;
  if (factored) a.fs = *factored;
  else { a.fs.part = nullptr; a.fs.bmax = nullptr; a.fs.ksplit = 0; a.fs.bm_rows = 0; a.fs.bm_pitch = 0; }
  a.S_out = factored ? S_out : nullptr;

  a.N = pl.N; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.bk = pl.bk;
  a.H = pl.H; a.causal = pl.causal; a.mode = pl.alloc_mode;
  for (int h = 0; h < PSA_MAX_LEVELS; ++h) { a.tau[h] = pl.tau[h]; a.cuts[h] = pl.cuts[h]; }
  int kpl = 1;                       // keys per lane: the row padded to a power of two >= 64
  while (64 * kpl < pl.nk) kpl <<= 1;
  switch (kpl) {
    case 1:  return launch_alloc_t<1, 1>(pl, a, S, cap, M, rowcnt, rho, s);
    case 2:  return launch_alloc_t<2, 1>(pl, a, S, cap, M, rowcnt, rho, s);
    case 4:  return launch_alloc_t<1, 4>(pl, a, S, cap, M, rowcnt, rho, s);    // from 256 keys on: four wavefronts per row
    case 8:  return launch_alloc_t<2, 4>(pl, a, S, cap, M, rowcnt, rho, s);    //   (5 us of 41 at 512 keys, 30 of 330 at 1024)
    case 16: return launch_alloc_t<4, 4>(pl, a, S, cap, M, rowcnt, rho, s);
    case 32: return launch_alloc_t<8, 4>(pl, a, S, cap, M, rowcnt, rho, s);    // 2048 keys: 256 lanes x 8
    case 64: return launch_alloc_t<16, 4>(pl, a, S, cap, M, rowcnt, rho, s);   // 4096 keys: 256 lanes x 16
    default: return hipErrorInvalidValue;   // more than PSA_MAX_NK key blocks: refused before any launch
  }
}

// Eq. 9 per (batch, head): sum_h c_h 2^-(h-1) over the visible block pairs.
__global__ __launch_bounds__(256) void rho_kernel(const uint32_t* __restrict__ rowcnt, float* __restrict__ rho,
                                                  int nq, int H) {
  __shared__ double num_s[256], den_s[256];
  const int tid = threadIdx.x;
  const uint32_t* base = rowcnt + (int64_t)blockIdx.x * nq * ROWCNT_STRIDE;
  double num = 0.0, den = 0.0;
  for (int i = tid; i < nq; i += 256) {
    const uint32_t* r = base + (int64_t)i * ROWCNT_STRIDE;
    den += (double)r[0];
    for (int h = 1; h <= H; ++h) num += (double)r[h] / (double)(1u << (h - 1));
  }
  num_s[tid] = num; den_s[tid] = den;
  __syncthreads();
  for (int off = 128; off; off >>= 1) {
    if (tid < off) { num_s[tid] += num_s[tid + off]; den_s[tid] += den_s[tid + off]; }
    __syncthreads();
  }
  if (tid == 0) rho[blockIdx.x] = (float)(num_s[0] / den_s[0]);
}

static hipError_t launch_rho(const Plan& pl, const uint32_t* rowcnt, float* rho, hipStream_t s) {
  rho_kernel<<<pl.B * pl.Hq, 256, 0, s>>>(rowcnt, rho, pl.nq, pl.H);
  return hipGetLastError();
}

// Tile descriptors for the matrix-core attention kernel (only when Plan::desc_pitch > 0).  The kept blocks of a
// level, in list order, form one stream of pooled tokens that is cut into tiles of 64; tile row r of a tile comes from
// pooled row (block id << lg_th) | (stream position & (th - 1)) of the level's array.  A tile is
// irregular when some row lies past the level's kept blocks, covers tokens past N, or (causal) is not
// visible to every query row of the block.  One word per load instruction of the kernel (rpi tile
// rows each), stored per wavefront, [row][wavefront][tile][ri]: wavefront w loads tile rows
// 16w .. 16w+15, its word k is the instruction for rows 16w + k*rpi .., and a wavefront's descriptors
// of consecutive tiles are adjacent in memory.  A word is the byte offset of the instruction's first
// source row, minus the 1024*k that the instruction offset adds, plus a constant bias that keeps it
// non-negative (the kernel's buffer descriptor starts that many bytes early).  The first word of
// each wavefront also carries level - 1 in bits 0..3 and the irregular flag in bit 4 (row offsets are
// multiples of 128 bytes).  Four null tiles (level field 15) follow the last one: the kernel
// requests tiles ahead of the one it computes (and touches one cache line further: the pitch leaves room).
struct ListArgs {
  int64_t rows;
  int N, nq, nk, bq, lg_bk, H, causal;
  int rowb, rpi, ri, words, pitch, lg_ri, lg_words;   // descriptors; pitch 0: none
  uint32_t bias;
};

// Per query block: the kept key blocks grouped by level (ascending block index inside a level), the number of blocks
// per level, and the tile descriptors.  One wavefront per query block does all three, so the descriptors read the
// list from LDS where it was just made: two kernels with the list and the counts in between took 6 + 13 us at 12
// heads x 256 query blocks x 512 key blocks and 3.3 + 3.7 at 12 x 8 x 16, this one 15 and 4.8.  NCH > 0: the row of levels is loaded once into NCH registers per
// lane (block c*64 + lane in register c), four query blocks per workgroup.  NCH = 0 (rows of more than 4096 blocks):
// the row is read again for every level, one query block per workgroup.
// DESC: descriptors are wanted; callers without them run a kernel without that code, as short as the list alone (0.3 us of 20
// to 40 for pyramid and attention on 64-row blocks x 2000 to 4000 tokens).
template <int NCH, bool DESC>
__global__ __launch_bounds__(NCH ? 256 : 64) void lists_kernel(const uint8_t* __restrict__ M, uint16_t* __restrict__ idx,
                                                               int32_t* __restrict__ cnt, uint32_t* __restrict__ desc, ListArgs a) {
  extern __shared__ uint16_t lists[];
  constexpr int WAVES = NCH ? 4 : 1;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * WAVES + wave;
  if (row >= a.rows) return;                           // (wavefronts of a workgroup do not wait for each other)
  const uint8_t* m = M + row * a.nk;
  uint16_t* out = idx + row * a.nk;
  uint16_t* lst = lists + (int64_t)wave * ((a.nk + 7) & ~7);
  int lv[NCH ? NCH : 1];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int j = c * 64 + lane;
    lv[c] = j < a.nk ? (int)m[j] : 0;
  }
  const uint64_t below = (1ull << lane) - 1ull;
  int nb_h[PSA_MAX_LEVELS];
  int pos = 0;
#pragma unroll
  for (int h = 1; h <= PSA_MAX_LEVELS; ++h) {
    int n = 0;
    if (h <= a.H) {
      auto take = [&](bool hit, int j) __attribute__((always_inline)) {
        const uint64_t mask = __ballot(hit);
        if (hit) {
          const int at = pos + n + __popcll(mask & below);
          out[at] = (uint16_t)j;
          if constexpr (DESC) lst[at] = (uint16_t)j;
        }
        n += __popcll(mask);
      };
      if constexpr (NCH > 0) {
#pragma unroll
        for (int c = 0; c < NCH; ++c) take(lv[c] == h, c * 64 + lane);
      } else {
        for (int j0 = 0; j0 < a.nk; j0 += 64) take(j0 + lane < a.nk && (int)m[j0 + lane] == h, j0 + lane);
      }
    }
    if (lane == 0) cnt[row * CNT_STRIDE + (h - 1)] = n;
    nb_h[h - 1] = n;
    pos += n;
  }
  if constexpr (!DESC) return;
  // the list passes between lanes of this one wavefront: LDS serves its accesses in order, the fences keep the
  // compiler from moving the reads above the writes
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int i = (int)(row % a.nq);
  const int q = lane & (a.words - 1), w = q >> a.lg_ri, k = q & (a.ri - 1);     // words, ri: powers of two
  const int sub = lane >> a.lg_words, per_pass = 64 >> a.lg_words;               // tiles per pass
  const uint64_t group_mask = ((1ull << a.words) - 1ull) << ((lane >> a.lg_words) << a.lg_words);
  uint32_t* dmine = desc + row * (int64_t)a.pitch * a.words + (int64_t)w * a.pitch * a.ri + k;
  int first = 0, start = 0;
#pragma unroll
  for (int h = 0; h < PSA_MAX_LEVELS; ++h) {           // h = level - 1
    const int nb = nb_h[h];
    if (nb == 0) continue;
    const int lg_th = a.lg_bk - h;
    const int ntl = ((nb << lg_th) + 63) >> 6;
    int lim = a.N >> h;                                // rows below cover 2^h valid tokens
    if (a.causal) {
      const int vis = (i * a.bq + 1) >> h;             // rows below end at or before the block's first query row
      lim = vis < lim ? vis : lim;
    }
    for (int t0 = 0; t0 < ntl; t0 += per_pass) {
      const int tl = t0 + sub;
      const int g = (tl << 6) + q * a.rpi, e = g >> lg_th;
      const int jl = (int)lst[start + (e < nb ? e : nb - 1)];
      const int prow = (jl << lg_th) | (g & ((1 << lg_th) - 1));
      const bool mine = tl < ntl && ((e >= nb) | (prow + a.rpi - 1 >= lim));
      const bool irregular = (__ballot(mine) & group_mask) != 0ull;
      if (tl < ntl)
        dmine[(int64_t)(first + tl) * a.ri] =
            ((uint32_t)prow * (uint32_t)a.rowb + a.bias - 1024u * (uint32_t)k) | (k == 0 ? (uint32_t)h | (irregular ? 16u : 0u) : 0u);
    }
    first += ntl;
    start += nb;
  }
  for (int t = sub; t < 4; t += per_pass) dmine[(int64_t)(first + t) * a.ri] = k == 0 ? 15u : 0u;   // null tiles
}

template <int NCH>
static hipError_t launch_lists_t(const uint8_t* M, uint16_t* idx, int32_t* cnt, uint32_t* desc, const ListArgs& a, hipStream_t s) {
  constexpr int WAVES = NCH ? 4 : 1;
  const unsigned grid = (unsigned)((a.rows + WAVES - 1) / WAVES);
  if (a.pitch == 0) {
    lists_kernel<NCH, false><<<grid, 64 * WAVES, 0, s>>>(M, idx, cnt, desc, a);
    return hipGetLastError();
  }
  const size_t smem = (size_t)WAVES * ((a.nk + 7) & ~7) * sizeof(uint16_t);
  static LdsOptIn optin;
  const hipError_t e = allow_max_lds(reinterpret_cast<const void*>(lists_kernel<NCH, true>), &optin);
  if (e != hipSuccess) return e;
  lists_kernel<NCH, true><<<grid, 64 * WAVES, smem, s>>>(M, idx, cnt, desc, a);
  return hipGetLastError();
}

hipError_t launch_lists(const Plan& pl, const uint8_t* M, uint16_t* idx, int32_t* cnt, uint32_t* desc, hipStream_t s) {
  ListArgs a;
  a.rows = (int64_t)pl.B * pl.Hq * pl.nq;
  a.N = pl.N; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.H = pl.H; a.causal = pl.causal;
  a.lg_bk = 0;
  while ((1 << a.lg_bk) < pl.bk) ++a.lg_bk;
  a.rowb = pl.d * 2;
  a.words = pl.desc_words;
  a.rpi = 64 / a.words;
  a.lg_words = a.words == 16 ? 4 : 3;
  a.ri = a.words / 4;                                  // four wavefronts
  a.lg_ri = a.ri == 4 ? 2 : 1;
  a.bias = 1024u * (uint32_t)(a.ri - 1);
  a.pitch = desc ? pl.desc_pitch : 0;
  int nch = 1;
  while (64 * nch < pl.nk) nch <<= 1;
  switch (nch) {
    case 1:  return launch_lists_t<1>(M, idx, cnt, desc, a, s);
    case 2:  return launch_lists_t<2>(M, idx, cnt, desc, a, s);
    case 4:  return launch_lists_t<4>(M, idx, cnt, desc, a, s);
    case 8:  return launch_lists_t<8>(M, idx, cnt, desc, a, s);
    case 16: return launch_lists_t<16>(M, idx, cnt, desc, a, s);
    case 32: return launch_lists_t<32>(M, idx, cnt, desc, a, s);
    case 64: return launch_lists_t<64>(M, idx, cnt, desc, a, s);
    default: return launch_lists_t<0>(M, idx, cnt, desc, a, s);
  }
}

}  // namespace psa
