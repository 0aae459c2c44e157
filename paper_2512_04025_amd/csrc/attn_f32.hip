// Attention in fp32 arithmetic on the gfx950 matrix cores: psa_attention_fwd in float32 (Alg. 1 with accurate
// exp, the 1e-5 mode), psa_dense_ref (Eq. 1) for both element types, and the bfloat16 block sizes that
// attn_mfma_kernel does not take.  Products and sums are fp32 throughout (v_mfma_f32_32x32x2_f32).
//
// Bound: the fp32 matrix rate (64 FLOP per cycle and SIMD, 151 TFLOP/s measured on a large product).  A
// 32 x 32 x D tile keeps a wavefront's matrix pipe busy for 64 D cycles and needs 1 / 8 of that in LDS reads,
// so little has to be scheduled by hand (some registers spill all the same at d = 128 with two wavefronts per SIMD:
// teams of two 55 in float32 and 21 in bfloat16, teams of four 18 in float32): the V rows of a tile travel through registers into LDS during its
// first product, the K rows of the next one during its second, and each product is followed by one barrier.
//
// Operand roles as in the bfloat16 kernel: S^T = K Q^T puts one query row in each lane (lane l and l + 32 share
// row l: keys (v/4)*8 + (l/32)*4 + v%4 in register v), and register v of P^T is then directly the B operand of
// O^T += V^T P^T for the pair of keys that the two halves hold.  The contraction over channels runs in the
// order in which a 16-byte read delivers them, for both operands alike.
//
// What decides the speed of small problems is how many wavefronts there are, so the four wavefronts of a
// workgroup are dealt out in two ways: TEAM of them own 32 query rows each and share the tiles of one
// stream of keys, and there are 4 / TEAM such teams over the SAME 32 * TEAM rows, each taking every
// (4 / TEAM)-th tile of the row's list; their (maximum, sum, output) are merged through LDS at the end.
//
// Measured (pyramid and block lists included) against one thread per query row on the vector unit, which this
// replaces: 12 heads x 4680 tokens, d = 128, a fifth of the keys: 2250 -> 350 us (27 GFLOP: 77 TFLOP/s, half of
// the rate of a large product); 2 heads x 1024 tokens, d = 64, the attention alone: 217 -> 20 us.
#include "psa_dev.h"
#include "psa_internal.h"

namespace psa {

struct F32Args {
  int N, Hq, Hkv, nq, nk, bq, bk, lg_bk, H, causal;
  int slices;              // workgroups per query block
  float scale;
  int64_t lvl_off[PSA_MAX_LEVELS + 2];
};

// LDS rows: K + 4 floats (a 16-byte read of 16 rows covers every bank once), V + 8 (the two halves of a
// 4-byte read sit four rows, half the banks, apart).
template <int D, int TEAM>
struct F32Shape {
  static constexpr int KS = 4 / TEAM, ROWS = 32 * TEAM, KPITCH = D + 4, VPITCH = D + 8;
  static constexpr int TILEF = 32 * KPITCH + 32 * VPITCH + 128 + 4;    // K | V | (bias [32] | last token [32]) x 2 | flags
  static constexpr int MERGEF = 2 * KS * ROWS + KS * ROWS * KPITCH;     // m, l | O of every team
  static constexpr size_t BYTES = sizeof(float) * (KS * TILEF > MERGEF ? KS * TILEF : MERGEF);
};

template <typename T, int D, int TEAM>
__global__ __launch_bounds__(256, (F32Shape<D, TEAM>::BYTES <= 80 * 1024 ? 2 : 1))
void attn_f32_kernel(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ Kp,
                     const T* __restrict__ Vp, const uint16_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                     T* __restrict__ O, float* __restrict__ lse, F32Args a) {
  using S = F32Shape<D, TEAM>;
  constexpr int KS = S::KS, ROWS = S::ROWS, KPITCH = S::KPITCH, VPITCH = S::VPITCH, CPR = D / 4, MD = D / 32;
  constexpr int TT = 64 * TEAM, NCH = 32 * CPR / TT;     // threads of a team; 4-element chunks per thread, tile and tensor
  extern __shared__ __attribute__((aligned(16))) float fsm[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = wave / TEAM, wr = wave % TEAM, tt = tid & (TT - 1);
  float* Ks = fsm + team * S::TILEF;
  float* Vs = Ks + 32 * KPITCH;
  float* table_s = Vs + 32 * VPITCH;                     // of tile t in half t & 1: additive term and last covered token per key
  int* flag_s = reinterpret_cast<int*>(table_s + 128);   // per wavefront of the team: did it stage a value of V that is not finite

  const bool dense = idx == nullptr;
  const int slice = blockIdx.x % a.slices;
  int i = blockIdx.x / a.slices;
  if (a.causal) i = a.nq - 1 - i;                        // longest rows first
  const int hq = blockIdx.y, b = blockIdx.z, hk = hq / (a.Hq / a.Hkv);
  const int64_t qhead = (int64_t)b * a.Hq + hq, khead = (int64_t)b * a.Hkv + hk;
  int row_end = (i + 1) * a.bq;
  row_end = row_end < a.N ? row_end : a.N;
  const int row0 = i * a.bq + slice * ROWS;
  if (row0 >= row_end) return;                           // a slice past the end of a short last block
  const int row = row0 + wr * 32 + l32;
  const bool active = row < row_end;

  float q[D / 2];                                        // channels k8*8 + hf*4 + e of this lane's row
#pragma unroll
  for (int k8 = 0; k8 < D / 8; ++k8) {
    f32x4 x = {0.f, 0.f, 0.f, 0.f};
    if (active) x = Four<T>::widen(Four<T>::load(Q + (qhead * a.N + row) * D + k8 * 8 + hf * 4));
#pragma unroll
    for (int e = 0; e < 4; ++e) q[k8 * 4 + e] = x[e];
  }
  f32x16 o[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[md][v] = 0.f;
  float m = -INFINITY, l = 0.f;

  const int64_t srow = qhead * a.nq + i;
  const uint16_t* my_idx = dense ? nullptr : idx + srow * a.nk;
  const int32_t* my_cnt = dense ? nullptr : cnt + srow * CNT_STRIDE;
  const int H = dense ? 1 : a.H;
  int dense_blocks = a.nk;                               // dense and causal: blocks that start at or before the last row
  if (a.causal) dense_blocks = (row_end - 1) / a.bk + 1;

  // The pooled tokens of a level's kept blocks, in list order, are one stream that is cut into tiles of 32.
  struct Tile { int h, tl, ntl, nblk, start; bool ok; };
  auto enter = [&](Tile& t) __attribute__((always_inline)) {
    t.nblk = dense ? dense_blocks : my_cnt[t.h - 1];
    t.ntl = (int)((((int64_t)t.nblk << (a.lg_bk - (t.h - 1))) + 31) >> 5);
  };
  auto settle = [&](Tile& t) __attribute__((always_inline)) {   // carry tl over to the level that holds it
    for (;;) {
      if (t.tl < t.ntl) { t.ok = true; return; }
      t.tl -= t.ntl;
      t.start += t.nblk;
      if (++t.h > H) { t.h = H; t.ok = false; t.ntl = 0; t.nblk = 0; return; }
      enter(t);
    }
  };
  auto locate = [&](const Tile& t) __attribute__((always_inline)) -> int {   // pooled row of tile row l32; -1: none
    if (!t.ok) return -1;
    const int lg_th = a.lg_bk - (t.h - 1), g = (t.tl << 5) + l32, e = g >> lg_th;
    if (e >= t.nblk) return -1;
    return ((dense ? e : (int)my_idx[t.start + e]) << lg_th) | (g & ((1 << lg_th) - 1));
  };
  typename Four<T>::raw reg[NCH];                        // this thread's part of the K or V rows on their way into LDS
  auto fetch = [&](const T* level1, const T* pooled, const Tile& t, int prow) __attribute__((always_inline)) {
    const int lg_th = a.lg_bk - (t.h - 1), hm1 = t.h - 1;
    const T* base = hm1 == 0 ? level1 + khead * (int64_t)a.N * D : pooled + a.lvl_off[t.h] + khead * ((int64_t)a.nk << lg_th) * D;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = tt + TT * c, pr = __shfl(prow, x / CPR, 64);
      reg[c] = typename Four<T>::raw{0, 0, 0, 0};
      if (pr >= 0 && ((int64_t)pr << hm1) < a.N) reg[c] = Four<T>::load(base + (int64_t)pr * D + (x % CPR) * 4);
    }
  };
  auto deposit_k = [&](const Tile& t, int prow, int half) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = tt + TT * c;
      *reinterpret_cast<f32x4*>(Ks + (x / CPR) * KPITCH + (x % CPR) * 4) = Four<T>::widen(reg[c]);
    }
    if (tt < 32) {
      const int span = 1 << (t.h - 1);
      const int64_t first = (int64_t)prow * span;
      int64_t c = a.N - first;
      c = prow < 0 || c < 0 ? 0 : (c > span ? span : c);
      table_s[half * 64 + tt] = c > 0 ? logf((float)c) : -INFINITY;   // (h-1) ln 2 for a full pooled key
      reinterpret_cast<int*>(table_s)[half * 64 + 32 + tt] = (int)(first + (c > 0 ? c : 1) - 1);
    }
  };
  auto deposit_v = [&]() __attribute__((always_inline)) {
    bool bad = false;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = tt + TT * c;
      const f32x4 vv = Four<T>::widen(reg[c]);
      *reinterpret_cast<f32x4*>(Vs + (x / CPR) * VPITCH + (x % CPR) * 4) = vv;
      if (a.causal) bad |= not_finite(vv);
    }
    const bool any_bad = a.causal && __any(bad);
    if (lane == 0) flag_s[wr] = any_bad ? 1 : 0;
  };
  // a team of one wavefront owns its buffer: its LDS operations complete in order, nothing to wait for
  auto barrier = [&]() __attribute__((always_inline)) {
    if constexpr (TEAM == 1) asm volatile("" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  int total = 0;                                         // tiles of the row: the same for every team
  for (int h = 1; h <= H; ++h) {
    Tile t;
    t.h = h;
    enter(t);
    total += t.ntl;
  }
  Tile cur = {1, team, 0, 0, 0, false};
  enter(cur);
  settle(cur);
  int pc = locate(cur);
  fetch(K, Kp, cur, pc);
  deposit_k(cur, pc, 0);
  Tile nxt = cur;
  nxt.tl += KS;
  if (nxt.ok) settle(nxt);
  int pn = locate(nxt);
  barrier();
  for (int step = 0, half = 0; step < total; step += KS, half ^= 1) {
    const float* bias_s = table_s + half * 64;
    const int* last_s = reinterpret_cast<const int*>(bias_s + 32);
    Tile nn = nxt;
    int pnn = -1;
    if (cur.ok) fetch(V, Vp, cur, pc);
    if (nxt.ok) {
      nn.tl += KS;
      settle(nn);
      pnn = locate(nn);
    }
    f32x16 sc;
    float ref = 0.f;
    if (cur.ok) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = 0.f;
      // one fragment ahead of the products (256 cycles of matrix work each), no more: left alone the compiler
      // requests all of them first and spills
      f32x4 kk = *reinterpret_cast<const f32x4*>(Ks + l32 * KPITCH + hf * 4);
#pragma unroll
      for (int k8 = 0; k8 < D / 8; ++k8) {
        f32x4 kn = kk;
        if (k8 + 1 < D / 8) kn = *reinterpret_cast<const f32x4*>(Ks + l32 * KPITCH + (k8 + 1) * 8 + hf * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[e], q[k8 * 4 + e], sc, 0, 0, 0);
        kk = kn;
        __builtin_amdgcn_sched_barrier(0);
      }
      float tmax = -INFINITY;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 bs = *reinterpret_cast<const f32x4*>(bias_s + g4 * 8 + hf * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float s = bs[e] == -INFINITY ? -INFINITY : fmaf(sc[g4 * 4 + e], a.scale, bs[e]);
          if (a.causal && last_s[g4 * 8 + hf * 4 + e] > row) s = -INFINITY;
          sc[g4 * 4 + e] = s;
          tmax = fmaxf(tmax, s);
        }
      }
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
      const float mn = fmaxf(m, tmax);
      ref = mn == -INFINITY ? 0.f : mn;
      if (__any(mn > m)) {
        const float alpha = expf(m - ref);               // m = -inf: 0
        l *= alpha;
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[md][v] *= alpha;
        m = mn;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        sc[v] = expf(sc[v] - ref);
        l += sc[v];
      }
      deposit_v();
    }
    barrier();                                           // V rows in LDS; everyone is done with the K rows
    if (nxt.ok) fetch(K, Kp, nxt, pn);
    if (cur.ok) {
      int bad = 0;
      if (a.causal) {
#pragma unroll
        for (int w = 0; w < TEAM; ++w) bad |= flag_s[w];
      }
      if (__builtin_amdgcn_readfirstlane(bad) == 0) {
        float va[MD], vn[MD];
#pragma unroll
        for (int md = 0; md < MD; ++md) va[md] = Vs[hf * 4 * VPITCH + md * 32 + l32];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if (v + 1 < 16) {
#pragma unroll
            for (int md = 0; md < MD; ++md) vn[md] = Vs[(((v + 1) >> 2) * 8 + hf * 4 + ((v + 1) & 3)) * VPITCH + md * 32 + l32];
          }
#pragma unroll
          for (int md = 0; md < MD; ++md) {
            o[md] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[md], sc[v], o[md], 0, 0, 0);
            va[md] = vn[md];
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      } else {
        // Causal, and the tile holds a value that is not finite: a row must not see 0 * inf of a key that is
        // hidden from it, so hidden keys are left out one by one (rare: on the vector unit).
        for (int kk = 0; kk < 32; ++kk) {
          const int vi = (kk >> 3) * 4 + (kk & 3), from = l32 + ((kk >> 2) & 1) * 32;
          float pv = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) pv = v == vi ? sc[v] : pv;
          pv = __shfl(pv, from, 64);
          if (bias_s[kk] == -INFINITY || last_s[kk] > row) continue;
#pragma unroll
          for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int v = 0; v < 16; ++v)
              o[md][v] = fmaf(pv, Vs[kk * VPITCH + md * 32 + (v >> 2) * 8 + hf * 4 + (v & 3)], o[md][v]);
        }
      }
    }
    if (nxt.ok) deposit_k(nxt, pn, half ^ 1);
    barrier();                                           // the next K rows in LDS; everyone is done with the V rows
    cur = nxt;
    pc = pn;
    nxt = nn;
    pn = pnn;
  }

  // merge the teams through LDS (fixed order) and write whole rows
  float* ms = fsm;                                       // [KS][ROWS] maxima | [KS][ROWS] sums | [KS][ROWS][KPITCH] outputs
  float* os = fsm + 2 * KS * ROWS;
  l += __shfl_xor(l, 32, 64);
  __syncthreads();
  const int slot = team * ROWS + wr * 32 + l32;
  if (hf == 0) {
    ms[slot] = m;
    ms[KS * ROWS + slot] = l;
  }
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(os + slot * KPITCH + md * 32 + g * 8 + hf * 4) =
          f32x4{o[md][4 * g], o[md][4 * g + 1], o[md][4 * g + 2], o[md][4 * g + 3]};
  __syncthreads();
  for (int x = tid; x < ROWS * CPR; x += 256) {
    const int r = x / CPR, c = (x % CPR) * 4;
    if (row0 + r >= row_end) continue;
    float mm = -INFINITY;
#pragma unroll
    for (int k = 0; k < KS; ++k) mm = fmaxf(mm, ms[k * ROWS + r]);
    float ll = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      // A team that saw no key of the row adds 0 * 0.  None is left out for a maximum of -inf alone: fmaxf drops NaN, so
      // a team all of whose scores are NaN has that maximum too, with a sum and outputs that are NaN and have to stay.
      const float w = KS == 1 ? 1.f : expf(ms[k * ROWS + r] - (mm == -INFINITY ? 0.f : mm));
      ll += w * ms[KS * ROWS + k * ROWS + r];
      acc += w * *reinterpret_cast<const f32x4*>(os + (k * ROWS + r) * KPITCH + c);
    }
    const float inv = 1.f / ll;                          // no visible key at all: NaN
    Four<T>::store(O + (qhead * a.N + row0 + r) * D + c, acc * inv);
    if (lse && c == 0) lse[qhead * a.N + row0 + r] = mm + logf(ll);
  }
}

template <typename T, int D, int TEAM>
static hipError_t launch_f32_t(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                               const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  using S = F32Shape<D, TEAM>;
  F32Args a;
  a.N = pl.N; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.bk = pl.bk;
  a.H = pl.H; a.causal = pl.causal; a.scale = pl.scale;
  a.lg_bk = 0;
  while ((1 << a.lg_bk) < pl.bk) ++a.lg_bk;
  a.slices = (pl.bq + S::ROWS - 1) / S::ROWS;
  for (int h = 0; h < PSA_MAX_LEVELS + 2; ++h) a.lvl_off[h] = pl.lvl_off[h];
  auto kern = attn_f32_kernel<T, D, TEAM>;
  static LdsOptIn optin;                                 // one per kernel instantiation
  const hipError_t e = allow_max_lds(reinterpret_cast<const void*>(kern), &optin);
  if (e != hipSuccess) return e;
  kern<<<dim3(pl.nq * a.slices, pl.Hq, pl.B), 256, S::BYTES, s>>>(
      static_cast<const T*>(Q), static_cast<const T*>(K), static_cast<const T*>(V), static_cast<const T*>(Kp),
      static_cast<const T*>(Vp), idx, cnt, static_cast<T*>(O), lse, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_f32_d(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                               const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  // The largest team that still fills the chip: fewer rows per team cost more reads of the same keys, fewer
  // workgroups leave compute units idle.  Measured with 12 heads at d = 128 (128-row blocks of the problem: us for
  // team 1 / 2 / 4, pyramid included): 48: 26 / 33 / 37, 96: 62 / 47 / 55, 192: 121 / 105 / 106, 252: 194 / 137 / 136,
  // 288: 285 / 247 / 236, 432: 535 / 409 / 343, 564: 931 / 699 / 679; d = 64: 48: 20 / 23 / 27, 96: 30 / 30 / 37, 192: 65 / 62 / 72,
  // 252: 87 / 77 / 92, 288: 126 / 135 / 147, 348: 164 / 166 / 167, 432: 226 / 220 / 210, 564: 372 / 369 / 418.  One line for both
  // head dimensions: it is drawn for d = 128; at d = 64 a team of four is the slowest just behind the line (288) and again
  // where the last round of workgroups is nearly empty (564), by 16 and 13 %.
  const int64_t blocks = (int64_t)pl.B * pl.Hq * pl.nq;
  auto groups = [&](int rows) { return blocks * ((pl.bq + rows - 1) / rows); };
  const int team = pl.bq > 64 && groups(128) >= 256 ? 4 : (pl.bq > 32 && groups(64) >= 192 ? 2 : 1);
  if (team == 4) return launch_f32_t<T, D, 4>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s);
  if (team == 2) return launch_f32_t<T, D, 2>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s);
  return launch_f32_t<T, D, 1>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s);
}

hipError_t launch_attn_f32(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                           const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  if (pl.dtype == PSA_F32)
    return pl.d == 64 ? launch_f32_d<float, 64>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s)
                      : launch_f32_d<float, 128>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s);
  return pl.d == 64 ? launch_f32_d<bf16_t, 64>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s)
                    : launch_f32_d<bf16_t, 128>(pl, Q, K, V, Kp, Vp, idx, cnt, O, lse, s);
}

}  // namespace psa
