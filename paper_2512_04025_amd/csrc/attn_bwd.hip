// Backward pass of the adaptive pyramid attention (Sec. 3.4, Alg. 1 / Eq. 8; the paper states that its
// kernel supports backpropagation, Sec. 1, and prints no formulas: these follow by the chain rule).
//
// For a query row with kept pooled keys g, logits s_g = scale q.kbar_g + ln c_g, P_g = exp(s_g - lse):
//   dP_g = dO . vbar_g,  D = dO . O,  dS_g = P_g (dP_g - D),
//   dq = scale sum_g dS_g kbar_g,  dkbar_g = scale sum_rows dS_g q,  dvbar_g = sum_rows P_g dO,
// and the gradient of a pooled token is shared equally by the c_g tokens under it (Eq. 2-3).
// The level map is a constant.  Everything is in fp32 arithmetic, deterministic, without atomics; it serves
// float32 and the bfloat16 shapes that attn_bwd_mfma.hip does not take:
//   bwd_dq_kernel   one workgroup per 32, 64 or 128 query rows, walking the row's level-sorted block list; also
//                   leaves D = dO . O per query row for the next kernel
//   bwd_dkv_kernel  one workgroup (short launches: several, see bwd_parts) per (key head, up to 32 pooled keys of a block, level), walking
//                   the column of the level map; writes the gradient of every pooled token of every level (fp32)
//   unpool_kernel   dK, dV = sum over the levels of the pooled gradients / c_g
// The products run on v_mfma_f32_32x32x2_f32 and are bound by its rate (64 FLOP per cycle and SIMD); the
// operands of a 32 x 32 tile are read from LDS in an eighth of that time, so tiles are staged through registers
// during the products and one wavefront per SIMD (up to 512 registers at d = 128) keeps the pipe busy.  At d = 64, with two
// wavefronts per SIMD, bwd_dkv_kernel<float> spills 11 registers.
// Measured against four lanes per row on the vector unit, which this replaces (2 heads x 1000 tokens, d = 64,
// four levels): dK, dV 641 -> 45 us (four launches -> one), dQ 78 -> 16 us, the whole call 735 -> 62 us.
#include "psa_dev.h"
#include "psa_internal.h"

namespace psa {

struct BwdArgs {
  int N, Hq, Hkv, nq, nk, bq, bk, lg_bk, H, causal;
  int parts;                             // workgroups that share a column of the level map (bwd_dkv_kernel)
  float scale;
  int64_t lvl_off[PSA_MAX_LEVELS + 2];   // level h >= 2 inside one pyramid buffer (elements)
  int64_t glvl_off[PSA_MAX_LEVELS + 2];  // level h >= 1 inside one pooled-gradient buffer (elements)
};

// Rows of an LDS tile (one per lane, read 16 bytes at a time) times the operand x in registers, contracted over the D channels
// in CHAINS interleaved sums that are added pairwise: one chain of D roundings would leave dS = P (dP - D) less exact than the
// D / 4 of four lanes that share a row.  Error against fp64, 2 and 12 heads x 150 to 2000 tokens, four masks, relative to those
// four lanes (mean and worst), one chain -> as below: dQ 1.006, 1.22 -> 0.928, 1.005 (S in one chain, dP in four; S in two or
// four changes nothing); dK 0.943, 1.148 -> 0.859, 1.002; dV 0.822, 1.034 -> 0.793, 0.924 (two chains each; one and two: dK 1.09).
// One fragment ahead of the products, no more; and the sum is made before the next product starts, not where it is used
// first: with the chains of both products open at once bwd_dkv_kernel spills 24 to 71 registers.
template <int D, int CHAINS>
__device__ __forceinline__ f32x16 tile_product(const float* frag, const float* x) {
  f32x16 acc[CHAINS];
#pragma unroll
  for (int c = 0; c < CHAINS; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
  f32x4 next = *reinterpret_cast<const f32x4*>(frag);
#pragma unroll
  for (int k8 = 0; k8 < D / 8; ++k8) {
    const f32x4 now = next;
    if (k8 + 1 < D / 8) next = *reinterpret_cast<const f32x4*>(frag + (k8 + 1) * 8);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc[e % CHAINS] = __builtin_amdgcn_mfma_f32_32x32x2f32(now[e], x[k8 * 4 + e], acc[e % CHAINS], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int w = 1; w < CHAINS; w *= 2)
#pragma unroll
    for (int c = 0; c < CHAINS; c += 2 * w) acc[c] += acc[c + w];
  asm volatile("" : "+v"(acc[0]));
  return acc[0];
}

// LDS rows carry four floats of padding: the 16-byte reads of 16 rows then cover every bank once.
template <int D, int TEAM>
struct BwdDqShape {
  static constexpr int KS = 4 / TEAM, ROWS = 32 * TEAM, PITCH = D + 4;
  static constexpr int TILEF = 2 * 32 * PITCH + 64;                    // K | V | bias [32] | last token [32]
  static constexpr int MERGEF = KS * ROWS * PITCH;
  static constexpr int OFF_LIST = 4 * KS * TILEF;                      // blocks per level | list (rows whose list the kernel makes)
  static constexpr int END = OFF_LIST + 4 * PSA_MAX_LEVELS + 2 * ROW_LISTS_NK;
  static constexpr size_t BYTES = END > 4 * MERGEF ? END : 4 * MERGEF;
};

// dQ.  Operand roles, tiles and teams as in attn_f32_kernel: S^T = K Q^T and dP^T = V dO^T put one query row in
// each lane, register v of dS^T is the B operand of dQ^T += K^T dS^T for the two keys of the lane's halves.
template <typename T, int D, int TEAM>
__global__ __launch_bounds__(256, (D == 64 && TEAM > 1 ? 2 : 1))
void bwd_dq_kernel(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ Kp,
                   const T* __restrict__ Vp, const uint8_t* __restrict__ M, const uint16_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                   const T* __restrict__ O, const float* __restrict__ lse, float* __restrict__ Dr, const T* __restrict__ dO,
                   T* __restrict__ dQ, BwdArgs a) {
  using S = BwdDqShape<D, TEAM>;
  constexpr int KS = S::KS, ROWS = S::ROWS, PITCH = S::PITCH, CPR = D / 4, MD = D / 32, TT = 64 * TEAM, NCH = 32 * CPR / TT;
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = wave / TEAM, wr = wave % TEAM, tt = tid & (TT - 1);
  float* Ks = fsm + team * S::TILEF;
  float* Vs = Ks + 32 * PITCH;
  float* bias_s = Vs + 32 * PITCH;
  int* last_s = reinterpret_cast<int*>(bias_s + 32);
  const int slices = (a.bq + ROWS - 1) / ROWS;
  const int slice = blockIdx.x % slices;
  int i = blockIdx.x / slices;
  if (a.causal) i = a.nq - 1 - i;                        // longest rows first
  const int hq = blockIdx.y, b = blockIdx.z, hk = hq / (a.Hq / a.Hkv);
  const int64_t qhead = (int64_t)b * a.Hq + hq, khead = (int64_t)b * a.Hkv + hk;
  int row_end = (i + 1) * a.bq;
  row_end = row_end < a.N ? row_end : a.N;
  const int row0 = i * a.bq + slice * ROWS;
  if (row0 >= row_end) return;
  const int row = row0 + wr * 32 + l32;
  const bool active = row < row_end;

  float q[D / 2], go[D / 2], dots[D / 8];                // dots: dO . O, four channels at a time
#pragma unroll
  for (int k8 = 0; k8 < D / 8; ++k8) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x, z = x;
    if (active) {
      x = Four<T>::widen(Four<T>::load(Q + (qhead * a.N + row) * D + k8 * 8 + hf * 4));
      y = Four<T>::widen(Four<T>::load(dO + (qhead * a.N + row) * D + k8 * 8 + hf * 4));
      z = Four<T>::widen(Four<T>::load(O + (qhead * a.N + row) * D + k8 * 8 + hf * 4));
    }
    dots[k8] = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      q[k8 * 4 + e] = x[e];
      go[k8 * 4 + e] = y[e];
      dots[k8] = fmaf(y[e], z[e], dots[k8]);
    }
  }
#pragma unroll
  for (int w = 1; w < D / 8; w *= 2)
#pragma unroll
    for (int k8 = 0; k8 < D / 8; k8 += 2 * w) dots[k8] += dots[k8 + w];
  const float my_D = dots[0] + __shfl_xor(dots[0], 32, 64);            // D of the row, also for bwd_dkv_kernel
  if (active && team == 0 && hf == 0) Dr[qhead * a.N + row] = my_D;
  const float my_lse = active ? lse[qhead * a.N + row] : INFINITY;     // a row that does not exist: all weights 0
  f32x16 dq[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[md][v] = 0.f;

  const int64_t srow = qhead * a.nq + i;
  const uint16_t* my_idx = idx + srow * a.nk;
  const int32_t* my_cnt = cnt + srow * CNT_STRIDE;
  int* cnt_s = reinterpret_cast<int*>(reinterpret_cast<unsigned char*>(fsm) + S::OFF_LIST);
  uint16_t* list_s = reinterpret_cast<uint16_t*>(cnt_s + PSA_MAX_LEVELS);
  if (M) {                                               // (short rows, see lists_in_kernel)
    row_lists<4>(M + srow * a.nk, a.nk, a.H, list_s, cnt_s, wave, lane);
    __syncthreads();
  }
  struct Tile { int h, tl, ntl, nblk, start; bool ok; };
  auto enter = [&](Tile& t) __attribute__((always_inline)) {
    t.nblk = M ? __builtin_amdgcn_readfirstlane(cnt_s[t.h - 1]) : my_cnt[t.h - 1];
    t.ntl = ((t.nblk << (a.lg_bk - (t.h - 1))) + 31) >> 5;
  };
  auto settle = [&](Tile& t) __attribute__((always_inline)) {          // carry tl over to the level that holds it
    for (;;) {
      if (t.tl < t.ntl) { t.ok = true; return; }
      t.tl -= t.ntl;
      t.start += t.nblk;
      if (++t.h > a.H) { t.h = a.H; t.ok = false; t.ntl = 0; t.nblk = 0; return; }
      enter(t);
    }
  };
  auto locate = [&](const Tile& t) __attribute__((always_inline)) -> int {   // pooled row of tile row l32; -1: none
    if (!t.ok) return -1;
    const int lg_th = a.lg_bk - (t.h - 1), g = (t.tl << 5) + l32, e = g >> lg_th;
    return e < t.nblk ? ((M ? (int)list_s[t.start + e] : (int)my_idx[t.start + e]) << lg_th) | (g & ((1 << lg_th) - 1)) : -1;
  };
  typename Four<T>::raw kreg[NCH], vreg[NCH];
  auto fetch = [&](const Tile& t, int prow) __attribute__((always_inline)) {
    const int lg_th = a.lg_bk - (t.h - 1), hm1 = t.h - 1;
    const int64_t off = a.lvl_off[t.h] + khead * ((int64_t)a.nk << lg_th) * D;
    const T* kbase = hm1 == 0 ? K + khead * (int64_t)a.N * D : Kp + off;
    const T* vbase = hm1 == 0 ? V + khead * (int64_t)a.N * D : Vp + off;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = tt + TT * c, pr = __shfl(prow, x / CPR, 64), ch = (x % CPR) * 4;
      kreg[c] = typename Four<T>::raw{0, 0, 0, 0};
      vreg[c] = typename Four<T>::raw{0, 0, 0, 0};
      if (pr >= 0 && ((int64_t)pr << hm1) < a.N) {
        kreg[c] = Four<T>::load(kbase + (int64_t)pr * D + ch);
        vreg[c] = Four<T>::load(vbase + (int64_t)pr * D + ch);
      }
    }
  };
  auto deposit = [&](const Tile& t, int prow) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = tt + TT * c, at = (x / CPR) * PITCH + (x % CPR) * 4;
      *reinterpret_cast<f32x4*>(Ks + at) = Four<T>::widen(kreg[c]);
      *reinterpret_cast<f32x4*>(Vs + at) = Four<T>::widen(vreg[c]);
    }
    if (tt < 32) {
      const int span = 1 << (t.h - 1);
      const int64_t first = (int64_t)prow * span;
      int64_t c = a.N - first;
      c = prow < 0 || c < 0 ? 0 : (c > span ? span : c);
      bias_s[tt] = c > 0 ? logf((float)c) : -INFINITY;
      last_s[tt] = (int)(first + (c > 0 ? c : 1) - 1);
    }
  };
  // a team of one wavefront owns its buffer: its LDS operations complete in order, nothing to wait for
  auto barrier = [&]() __attribute__((always_inline)) {
    if constexpr (TEAM == 1) asm volatile("" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };
  int total = 0;
  for (int h = 1; h <= a.H; ++h) {
    Tile t;
    t.h = h;
    enter(t);
    total += t.ntl;
  }
  Tile cur = {1, team, 0, 0, 0, false};
  enter(cur);
  settle(cur);
  int pc = locate(cur);
  fetch(cur, pc);
  deposit(cur, pc);
  Tile nxt = cur;
  nxt.tl += KS;
  if (nxt.ok) settle(nxt);
  int pn = locate(nxt);
  for (int step = 0; step < total; step += KS) {
    barrier();                                           // the tile's rows are in LDS
    Tile nn = nxt;
    int pnn = -1;
    if (nxt.ok) {
      fetch(nxt, pn);
      nn.tl += KS;
      settle(nn);
      pnn = locate(nn);
    }
    if (cur.ok) {
      f32x16 sc = tile_product<D, 1>(Ks + l32 * PITCH + hf * 4, q);
      const f32x16 dp = tile_product<D, 4>(Vs + l32 * PITCH + hf * 4, go);
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 bs = *reinterpret_cast<const f32x4*>(bias_s + g4 * 8 + hf * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x = bs[e] == -INFINITY ? -INFINITY : fmaf(sc[g4 * 4 + e], a.scale, bs[e]);
          if (a.causal && last_s[g4 * 8 + hf * 4 + e] > row) x = -INFINITY;
          sc[g4 * 4 + e] = expf(x - my_lse) * (dp[g4 * 4 + e] - my_D);
        }
      }
      float ka[MD], kn[MD];
#pragma unroll
      for (int md = 0; md < MD; ++md) ka[md] = Ks[hf * 4 * PITCH + md * 32 + l32];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        if (v + 1 < 16) {
#pragma unroll
          for (int md = 0; md < MD; ++md) kn[md] = Ks[(((v + 1) >> 2) * 8 + hf * 4 + ((v + 1) & 3)) * PITCH + md * 32 + l32];
        }
#pragma unroll
        for (int md = 0; md < MD; ++md) {
          dq[md] = __builtin_amdgcn_mfma_f32_32x32x2f32(ka[md], sc[v], dq[md], 0, 0, 0);
          ka[md] = kn[md];
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    barrier();                                           // everyone has read it
    if (nxt.ok) deposit(nxt, pn);
    cur = nxt;
    nxt = nn;
    pn = pnn;
  }
  // the teams' sums through LDS, added in a fixed order
  __syncthreads();
  const int slot = team * ROWS + wr * 32 + l32;
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(fsm + slot * PITCH + md * 32 + g * 8 + hf * 4) =
          f32x4{dq[md][4 * g], dq[md][4 * g + 1], dq[md][4 * g + 2], dq[md][4 * g + 3]};
  __syncthreads();
  for (int x = tid; x < ROWS * CPR; x += 256) {
    const int r = x / CPR, c = (x % CPR) * 4;
    if (row0 + r >= row_end) continue;
    f32x4 sum = *reinterpret_cast<const f32x4*>(fsm + r * PITCH + c);
#pragma unroll
    for (int k = 1; k < KS; ++k) sum += *reinterpret_cast<const f32x4*>(fsm + (k * ROWS + r) * PITCH + c);
    Four<T>::store(dQ + (qhead * a.N + row0 + r) * D + c, sum * a.scale);
  }
}

template <int D>
struct BwdDkvShape {
  static constexpr int PITCH = D + 4;
  static constexpr int WAVEF = 2 * 32 * PITCH + 64;                    // Q | dO | lse [32] | D [32] of one wavefront
  static constexpr int LIST = 256;                                     // column entries tested at a time
  static constexpr size_t BYTES = sizeof(float) * (4 * WAVEF + LIST + 4);
};

// Pooled dK, dV of up to 32 pooled keys of a key block at one level (all levels in one launch, the coarsest first: their
// columns are the longest).  Larger blocks are split over several workgroups; smaller ones leave lanes idle and are
// not packed together, because a query row that is not finite would reach the blocks that do not use it as 0 * inf.
// Queries and keys exchanged: the keys and values sit in registers as B operands (one key per lane), the four
// wavefronts take the 32-row chunks of the query blocks that use the block at this level in turn, each
// through an LDS buffer of its own (no barrier in between), and their sums meet at the end in a fixed order.
// The column of the level map is tested 256 entries at a time, so its length is not limited.
template <typename T, int D>
__global__ __launch_bounds__(256, (D == 64 ? 2 : 1))
void bwd_dkv_kernel(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ Kp,
                    const T* __restrict__ Vp, const uint8_t* __restrict__ M, const float* __restrict__ lse,
                    const float* __restrict__ Dr, const T* __restrict__ dO, float* __restrict__ dKp, float* __restrict__ dVp,
                    BwdArgs a) {
  using S = BwdDkvShape<D>;
  constexpr int PITCH = S::PITCH, CPR = D / 4, MD = D / 32, NCH = 32 * CPR / 64;
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  float* Qs = fsm + wave * S::WAVEF;
  float* Gs = Qs + 32 * PITCH;
  float* lse_s = Gs + 32 * PITCH;
  float* D_s = lse_s + 32;
  int* kept = reinterpret_cast<int*>(fsm + 4 * S::WAVEF);
  int* wcount = kept + S::LIST;
  const int hk = blockIdx.y / a.parts, part = blockIdx.y % a.parts, b = blockIdx.z, group = a.Hq / a.Hkv;
  int h = a.H, pieces = 1, bx = blockIdx.x;
  for (;; --h) {
    const int th = a.bk >> (h - 1);
    pieces = th > 32 ? th / 32 : 1;
    if (bx < pieces * a.nk || h == 1) break;
    bx -= pieces * a.nk;
  }
  const int lg_th = a.lg_bk - (h - 1), span = 1 << (h - 1);
  const int j = bx / pieces, koff = (bx % pieces) * 32;                // key block; first key inside it
  const int64_t khead = (int64_t)b * a.Hkv + hk;
  const int prow = (j << lg_th) + koff + l32;
  const int64_t first = (int64_t)prow * span;
  int64_t c64 = a.N - first;
  c64 = c64 < 0 ? 0 : (c64 > span ? span : c64);
  const bool valid = koff + l32 < (1 << lg_th) && c64 > 0;
  const float bias = valid ? logf((float)c64) : -INFINITY;
  const int last = (int)(first + (c64 > 0 ? c64 : 1) - 1);
  const int64_t off = a.lvl_off[h] + khead * ((int64_t)a.nk << lg_th) * D;
  const T* kbase = h == 1 ? K + khead * (int64_t)a.N * D : Kp + off;
  const T* vbase = h == 1 ? V + khead * (int64_t)a.N * D : Vp + off;

  float k[D / 2], v[D / 2];
#pragma unroll
  for (int k8 = 0; k8 < D / 8; ++k8) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f}, y = x;
    if (valid) {
      x = Four<T>::widen(Four<T>::load(kbase + (int64_t)prow * D + k8 * 8 + hf * 4));
      y = Four<T>::widen(Four<T>::load(vbase + (int64_t)prow * D + k8 * 8 + hf * 4));
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      k[k8 * 4 + e] = x[e];
      v[k8 * 4 + e] = y[e];
    }
  }
  f32x16 dk[MD], dv[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int u = 0; u < 16; ++u) { dk[md][u] = 0.f; dv[md][u] = 0.f; }

  // this workgroup's share of the column: entries (query head of the group, query block)
  const int E_all = group * a.nq, share = (E_all + a.parts - 1) / a.parts, nchunk = (a.bq + 31) / 32;
  const int E_lo = part * share, E = E_lo + share < E_all ? E_lo + share : E_all;
  struct Chunk { int64_t row0; int r0, seg; };
  typename Four<T>::raw reg[NCH];                                      // the Q or dO rows on their way into LDS
  float lreg = INFINITY, dreg = 0.f;
  const uint32_t lane_off = (uint32_t)(((lane / CPR) * D + (lane % CPR) * 4) * (int)sizeof(T));   // bytes
  auto place = [&](int f) __attribute__((always_inline)) -> Chunk {    // chunk f of the batch's list
    Chunk c;
    const int e = __builtin_amdgcn_readfirstlane(kept[f / nchunk]);
    const int i = e % a.nq;
    c.r0 = i * a.bq + (f % nchunk) * 32;
    int row_end = (i + 1) * a.bq;
    row_end = row_end < a.N ? row_end : a.N;
    c.seg = row_end - c.r0 < 32 ? row_end - c.r0 : 32;                 // <= 0: past the end of a short last block
    c.row0 = ((int64_t)b * a.Hq + hk * group + e / a.nq) * a.N + c.r0;
    return c;
  };
  auto fetch = [&](const T* src, const Chunk& c) __attribute__((always_inline)) {
    // a scalar base and one 32-bit offset per lane: an address per chunk costs 14 to 40 registers more
    const char* base = reinterpret_cast<const char*>(src + c.row0 * D);
#pragma unroll
    for (int n = 0; n < NCH; ++n) {
      const int down = n * (64 / CPR);
      reg[n] = typename Four<T>::raw{0, 0, 0, 0};
      if (lane / CPR + down < c.seg) reg[n] = Four<T>::load(reinterpret_cast<const T*>(base + (lane_off + (uint32_t)(down * D * (int)sizeof(T)))));
    }
  };
  auto deposit = [&](float* dst) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < NCH; ++n) {
      const int x = lane + 64 * n;
      *reinterpret_cast<f32x4*>(dst + (x / CPR) * PITCH + (x % CPR) * 4) = Four<T>::widen(reg[n]);
    }
  };
  auto fetch_stats = [&](const Chunk& c) __attribute__((always_inline)) {
    lreg = l32 < c.seg ? lse[c.row0 + l32] : INFINITY;
    dreg = l32 < c.seg ? Dr[c.row0 + l32] : 0.f;
  };
  // acc += tile^T w: 32 rows of the tile, w[u] = weight of row (u/4)*8 + hf*4 + u%4 for this lane's key
  auto accumulate = [&](f32x16 (&acc)[MD], const float* tile, const f32x16& w) __attribute__((always_inline)) {
    float now[MD], nxt[MD];
#pragma unroll
    for (int md = 0; md < MD; ++md) now[md] = tile[hf * 4 * PITCH + md * 32 + l32];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      if (u + 1 < 16) {
#pragma unroll
        for (int md = 0; md < MD; ++md) nxt[md] = tile[(((u + 1) >> 2) * 8 + hf * 4 + ((u + 1) & 3)) * PITCH + md * 32 + l32];
      }
#pragma unroll
      for (int md = 0; md < MD; ++md) {
        acc[md] = __builtin_amdgcn_mfma_f32_32x32x2f32(now[md], w[u], acc[md], 0, 0, 0);
        now[md] = nxt[md];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int e0 = E_lo; e0 < E; e0 += S::LIST) {
    // which of the next column entries (query head of the group, query block) use this block at this level
    const int e = e0 + tid;
    const bool hit = e < E && (int)M[(((int64_t)b * a.Hq + hk * group) * a.nq + e) * a.nk + j] == h;
    const uint64_t mask = __ballot(hit);
    __syncthreads();                                                   // the list of the batch before is done with
    if (lane == 0) wcount[wave] = __popcll(mask);
    __syncthreads();
    int base = 0, nkept = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      base += w < wave ? wcount[w] : 0;
      nkept += wcount[w];
    }
    if (hit) kept[base + __popcll(mask & ((1ull << lane) - 1ull))] = e;
    __syncthreads();
    const int nf = nkept * nchunk;
    // dO is done with before Q is, so its next rows travel during the product with dO^T and those of Q during the one
    // with Q^T, through the same registers.
    Chunk c = {};
    if (wave < nf) {
      c = place(wave);
      fetch(dO, c);
      fetch_stats(c);
      deposit(Gs);
      fetch(Q, c);
    }
    for (int f = wave; f < nf; f += 4) {
      deposit(Qs);
      if (hf == 0) {
        lse_s[l32] = lreg;
        D_s[l32] = dreg;
      }
      asm volatile("" ::: "memory");                                   // this wavefront's LDS operations complete in order
      f32x16 sc = tile_product<D, 2>(Qs + l32 * PITCH + hf * 4, k);
      f32x16 dp = tile_product<D, 2>(Gs + l32 * PITCH + hf * 4, v);
      // this lane: its key, rows (u/4)*8 + hf*4 + u%4; sc becomes dS, dp becomes P
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int r = g4 * 8 + hf * 4;
        const f32x4 ls = *reinterpret_cast<const f32x4*>(lse_s + r), dd = *reinterpret_cast<const f32x4*>(D_s + r);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          float x = valid ? fmaf(sc[g4 * 4 + u], a.scale, bias) : -INFINITY;
          if (a.causal && last > c.r0 + r + u) x = -INFINITY;
          const float p = expf(x - ls[u]);
          sc[g4 * 4 + u] = p * (dp[g4 * 4 + u] - dd[u]);
          dp[g4 * 4 + u] = p;
        }
      }
      const bool more = f + 4 < nf;
      if (more) {
        c = place(f + 4);
        fetch(dO, c);
        fetch_stats(c);
      }
      accumulate(dv, Gs, dp);
      asm volatile("" ::: "memory");
      if (more) {
        deposit(Gs);
        fetch(Q, c);
      }
      accumulate(dk, Qs, sc);
      asm volatile("" ::: "memory");
    }
  }
  // the wavefronts' sums through LDS, first dK, then dV; every pooled key of the group is written
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        f32x4 x;
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = which ? dv[md][4 * g + u] : dk[md][4 * g + u];
        *reinterpret_cast<f32x4*>(fsm + (wave * 32 + l32) * PITCH + md * 32 + g * 8 + hf * 4) = x;
      }
    __syncthreads();
    float* dst = (which ? dVp : dKp) + a.glvl_off[h] + ((khead * a.parts + part) * ((int64_t)a.nk << lg_th) + ((int64_t)j << lg_th) + koff) * D;
    const float mul = which ? 1.f : a.scale;
    for (int x = tid; x < 32 * CPR; x += 256) {
      const int kk = x / CPR, c = (x % CPR) * 4;
      if (koff + kk >= (1 << lg_th)) break;
      f32x4 sum = *reinterpret_cast<const f32x4*>(fsm + kk * PITCH + c);
#pragma unroll
      for (int w = 1; w < 4; ++w) sum += *reinterpret_cast<const f32x4*>(fsm + (w * 32 + kk) * PITCH + c);
      *reinterpret_cast<f32x4*>(dst + (int64_t)kk * D + c) = sum * mul;
    }
  }
}

// dK[t] = sum_h dKbar^h[t >> (h-1)] / c  (Eq. 2-3 backwards); same for V.  One thread per 4 channels of TOK consecutive
// tokens: a pooled gradient is read once for all of them, and the rows of a level are independent loads.
// The pooled gradients of a key head come in `parts` consecutive partial tensors (one per query head of
// its group when the matrix-core kernel wrote them), added here in a fixed order.
template <typename T, int TOK>
__global__ __launch_bounds__(256) void unpool_kernel(const float* __restrict__ dKp, const float* __restrict__ dVp,
                                                     T* __restrict__ dK, T* __restrict__ dV, int heads, int parts, int d,
                                                     BwdArgs a) {
  // (32-bit arithmetic: a grid has fewer than 2^32 threads)
  const uint32_t gid = blockIdx.x * 256u + threadIdx.x, q4 = (uint32_t)d / 4u, groups = ((uint32_t)a.N + TOK - 1) / TOK, rest = gid / q4;
  const int c4 = (int)(gid - rest * q4);
  const int64_t bh = rest / groups;
  if (bh >= heads) return;
  const int t0 = (int)(rest - (uint32_t)bh * groups) * TOK;
  const float* src = blockIdx.y ? dVp : dKp;
  T* dst = blockIdx.y ? dV : dK;
  f32x4 acc[TOK];
#pragma unroll
  for (int u = 0; u < TOK; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int h = 1; h <= PSA_MAX_LEVELS; ++h) {
    if (h > a.H) break;
    const int span = 1 << (h - 1), n = TOK >> (h - 1) > 1 ? TOK >> (h - 1) : 1;     // tokens under a row, rows
    const int row0 = t0 >> (h - 1), rows = a.nk * (a.bk >> (h - 1));                // (TOK divides the tokens of a block)
    const float* at = src + a.glvl_off[h] + (bh * parts * (int64_t)rows + row0) * d + c4 * 4;
    f32x4 g[TOK];
#pragma unroll
    for (int x = 0; x < n; ++x) g[x] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int part = 0; part < parts; ++part, at += (int64_t)rows * d) {
#pragma unroll
      for (int x = 0; x < n; ++x) g[x] += *reinterpret_cast<const f32x4*>(at + x * d);
    }
#pragma unroll
    for (int x = 0; x < n; ++x) {
      int c = a.N - (row0 + x) * span;
      c = c > span ? span : c;                     // < 1: no token of this thread is under this row
      const float inv = 1.f / (float)c;
      g[x] *= inv;
    }
#pragma unroll
    for (int u = 0; u < TOK; ++u) acc[u] += g[u >> (h - 1)];
  }
#pragma unroll
  for (int u = 0; u < TOK; ++u) {
    if (t0 + u >= a.N) break;
    T* o = dst + (bh * a.N + t0 + u) * d + c4 * 4;
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = Elem<T>::from_f32(acc[u][v]);
  }
}

bool bwd_uses_mfma(const Plan& pl);
int dkv_split(const Plan& pl);
hipError_t launch_attn_bwd_mfma(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                                const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const void* O, const float* lse,
                                const void* dO, float* Dr, float* dKp, float* dVp, void* dQ, hipStream_t s);

// workgroups of bwd_dkv_kernel for one key head and part, as the kernel counts them
static int dkv_groups(const Plan& pl) {
  int n = 0;
  for (int h = 1; h <= pl.H; ++h) {
    const int th = pl.bk >> (h - 1);
    n += (th > 32 ? th / 32 : 1) * pl.nk;
  }
  return n;
}

// Partial pooled-gradient tensors per key head.  The matrix-core kernel writes one per query head of the group and share of a walk.
int bwd_parts(const Plan& pl) {
  if (bwd_uses_mfma(pl)) return pl.group * dkv_split(pl);
  // The other one splits the columns of short launches over up to eight workgroups, whose sums unpool_kernel adds: while there are fewer than 500 workgroups (d = 64:
  // 1000; the chip holds 256 and 512) and the column is worth it.  A part more saves less the more there are, and costs each time what the workgroups write (a
  // block of fewer than 32 pooled keys takes as long as a full one) and what is added again: the column's length, squared where it is long, against both sums, times
  // the parts squared.  Length: chunks of 32 rows, of which a causal column sees about a third; which blocks are kept is not known here.  950 shapes at a tenth to
  // three tenths of the keys: 4 more than 3 % slower than with one workgroup, the worst 8 %, the mean of all 9.6 % faster (the best choice for each: 15 %).  Whole call,
  // us, one / two / four / eight, one level: 8 heads in groups of four x 1258 tokens, d = 64 176 / 115 / 82 / 76; 28 in groups of seven x 902 112 / 85 / 84 / 87, x 900
  // causal at d = 128 141 / 114 / 123 / 142; 2 x 697 54 / 43 / 38 / 40; four levels 8 in groups of four x 1185, d = 128 409 / 270 / 209 / 193; not two levels
  // 2 x 1721 causal 35 / 42 / 47 / 55, one level 16 x 928 at d = 128 130 / 159 / 177 / 226, blocks of 8 keys 4 x 1047 in pairs causal 43 / 50.
  const int64_t wgs = (int64_t)pl.B * pl.Hkv * dkv_groups(pl), walk = pl.group * column_chunks(pl) * (pl.causal ? 1 : 3);   // (in thirds of a chunk)
  int64_t cost = wgs * 32 * pl.d;
  for (int h = 1; h <= pl.H; ++h) cost += ((int64_t)pl.B * pl.Hkv * pl.N * pl.d) >> (h - 1);
  const double gain = 40.0 * walk * std::max<int64_t>(walk, 200);
  int parts = 1;
  while (parts < 8 && wgs * parts < (pl.d == 64 ? 1000 : 500) && walk >= 12 * parts && gain >= (double)cost * parts * parts) parts *= 2;
  return parts;
}

size_t bwd_pooled_grad_elems(const Plan& pl) {      // one tensor: levels 1..H, every part
  size_t n = 0;
  for (int h = 1; h <= pl.H; ++h) n += (size_t)pl.B * pl.Hkv * bwd_parts(pl) * pl.nk * (pl.bk >> (h - 1)) * pl.d;
  return n;
}

template <typename T, int D, int TEAM>
static hipError_t launch_dq_t(const Plan& pl, const BwdArgs& a, const T* q, const T* k, const T* v, const T* kp, const T* vp,
                              const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const T* o, const float* lse, float* Dr, const T* go,
                              T* dq, hipStream_t s) {
  using S = BwdDqShape<D, TEAM>;
  auto kern = bwd_dq_kernel<T, D, TEAM>;
  static LdsOptIn optin;
  const hipError_t e = allow_max_lds(reinterpret_cast<const void*>(kern), &optin);
  if (e != hipSuccess) return e;
  kern<<<dim3(pl.nq * ((pl.bq + S::ROWS - 1) / S::ROWS), pl.Hq, pl.B), 256, S::BYTES, s>>>(q, k, v, kp, vp, M, idx, cnt, o, lse, Dr, go, dq, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_bwd_t(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                               const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const void* O, const float* lse,
                               const void* dO, float* Dr, float* dKp, float* dVp, void* dQ, void* dK, void* dV, bool use_mfma,
                               hipStream_t s) {
  BwdArgs a;
  a.N = pl.N; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.bk = pl.bk;
  a.H = pl.H; a.causal = pl.causal; a.scale = pl.scale;
  a.lg_bk = 0;
  while ((1 << a.lg_bk) < pl.bk) ++a.lg_bk;
  const int parts = bwd_parts(pl);
  a.parts = parts;
  int64_t off = 0;
  for (int h = 0; h < PSA_MAX_LEVELS + 2; ++h) { a.lvl_off[h] = pl.lvl_off[h]; a.glvl_off[h] = 0; }
  for (int h = 1; h <= pl.H; ++h) {
    a.glvl_off[h] = off;
    off += (int64_t)pl.B * pl.Hkv * parts * pl.nk * (pl.bk >> (h - 1)) * pl.d;
  }
  const T* q = static_cast<const T*>(Q);
  const T* k = static_cast<const T*>(K);
  const T* v = static_cast<const T*>(V);
  const T* kp = static_cast<const T*>(Kp);
  const T* vp = static_cast<const T*>(Vp);
  const T* go = static_cast<const T*>(dO);
  const T* o = static_cast<const T*>(O);
  hipError_t e = hipSuccess;
  if (use_mfma) {     // bfloat16: dQ and the pooled gradients on the matrix cores
    e = launch_attn_bwd_mfma(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, s);
    if (e != hipSuccess) return e;
  } else {
    // Rows per workgroup: the forward's rule (launch_f32_d), within 8 % of the best of the three at every size measured.
    // Whole call, 12 heads (128-row blocks of the problem: us for team 1 / 2 / 4), d = 64: 48: 55 / 59 / 63, 96: 110 / 99 / 108,
    // 192: 248 / 239 / 244, 252: 378 / 345 / 352, 288: 504 / 481 / 495, 432: 912 / 845 / 837, 564: 1478 / 1349 / 1413 (the rule
    // takes 4); d = 128: 48: 73 / 80 / 88, 96: 157 / 137 / 151, 144: 316 / 307 / 285, 192: 391 / 393 / 378, 252: 623 / 586 / 568,
    // 288: 816 / 808 / 845, 432: 1601 / 1574 / 1525.
    const int64_t blocks = (int64_t)pl.B * pl.Hq * pl.nq;
    auto groups = [&](int rows_wg) { return blocks * ((pl.bq + rows_wg - 1) / rows_wg); };
    const int team = pl.bq > 64 && groups(128) >= 256 ? 4 : (pl.bq > 32 && groups(64) >= 192 ? 2 : 1);
    T* dq = static_cast<T*>(dQ);
    const uint8_t* own = lists_in_kernel(pl, false) ? M : nullptr;
    e = team == 4 ? launch_dq_t<T, D, 4>(pl, a, q, k, v, kp, vp, own, idx, cnt, o, lse, Dr, go, dq, s)
      : team == 2 ? launch_dq_t<T, D, 2>(pl, a, q, k, v, kp, vp, own, idx, cnt, o, lse, Dr, go, dq, s)
                  : launch_dq_t<T, D, 1>(pl, a, q, k, v, kp, vp, own, idx, cnt, o, lse, Dr, go, dq, s);
    if (e != hipSuccess) return e;
    static LdsOptIn optin;
    e = allow_max_lds(reinterpret_cast<const void*>(bwd_dkv_kernel<T, D>), &optin);
    if (e != hipSuccess) return e;
    const int wgs = dkv_groups(pl);
    bwd_dkv_kernel<T, D><<<dim3(wgs, pl.Hkv * parts, pl.B), 256, BwdDkvShape<D>::BYTES, s>>>(q, k, v, kp, vp, M, lse, Dr, go, dKp, dVp, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  const int heads = pl.B * pl.Hkv;
  auto unpool = [&](auto kernel, int tokens) {
    const int64_t n = (int64_t)heads * ((pl.N + tokens - 1) / tokens) * (pl.d / 4);
    kernel<<<dim3((unsigned)((n + 255) / 256), 2), 256, 0, s>>>(dKp, dVp, static_cast<T*>(dK), static_cast<T*>(dV), heads, parts, pl.d, a);
  };
  // Four tokens a thread where that still fills the chip.  Whole call, us for one / four, d = 128, four levels: 12 heads x 32760 tokens
  // 6268 / 6225, x 8000 509 / 493, x 2000 91.7 / 91.3, x 1000 56.2 / 55.4, 40 x 4000 512 / 494, 28 in groups of seven x 8000 768 / 764,
  // x 3000 202 / 200, but x 1000 69.1 / 73.1 and 2 heads x 1000 at d = 64 36.5 / 37.5 (eight tokens: 6220, 494, 91.1, 56.1, 492, 765, 207, 85.1, 38.7).
  if ((int64_t)heads * pl.N * (pl.d / 4) >= 300000 && pl.bk >= 4) unpool(unpool_kernel<T, 4>, 4);
  else unpool(unpool_kernel<T, 1>, 1);
  return hipGetLastError();
}

hipError_t launch_attn_bwd(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                           const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const void* O, const float* lse,
                           const void* dO, float* Dr, float* dKp, float* dVp, void* dQ, void* dK, void* dV, hipStream_t s) {
  if (pl.dtype == PSA_F32)
    return pl.d == 64 ? launch_bwd_t<float, 64>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, dK, dV, false, s)
                      : launch_bwd_t<float, 128>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, dK, dV, false, s);
  const bool mfma = bwd_uses_mfma(pl);
  return pl.d == 64 ? launch_bwd_t<bf16_t, 64>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, dK, dV, mfma, s)
                    : launch_bwd_t<bf16_t, 128>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, dK, dV, mfma, s);
}

}  // namespace psa
