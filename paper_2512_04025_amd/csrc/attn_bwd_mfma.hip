// Backward pass of the adaptive pyramid attention on the gfx950 matrix cores, bfloat16 (the chain rule
// through Eq. 8 and the mean pooling of Eq. 2-3; see attn_bwd.hip for the formulas and for the fp32
// version that serves float32 and the shapes this one does not take).
//
// Two kernels with fp32 accumulation, P and dS rounded to bfloat16 for the
// products that consume them, no atomics on results, two wavefronts per SIMD (at most 256 registers per lane),
// double-buffered tiles that are loaded straight into LDS:
//   bwd_dq_mfma_kernel   one workgroup per 128 query rows (a wavefront per 32), walking the row's
//        level-sorted block list in tiles of 64 pooled keys gathered into LDS.  Same operand roles as the
//        forward kernel: S^T = Kbar Q^T and dP^T = Vbar dO^T put one query row in each lane (lse and
//        D = dO.O are per-lane scalars), dS^T is packed in registers as the B operand of
//        dQ^T += Kbar^T dS^T, whose A operand is read from the row-major Kbar tile with the transposing
//        LDS load.
//   bwd_dkv_mfma_kernel  the same with queries and keys exchanged, on 16x16x32 MFMAs: one workgroup per (64 adjacent pooled
//        keys of a level, query head); the pooled keys and values sit in registers as B operands (one key per lane), the
//        query blocks that use one of the workgroup's key blocks at this level (a walk down the level map's columns) are
//        staged through LDS 32 or 64 rows at a time; S = Q Kbar^T and dP = dO Vbar^T, then dVbar^T += dO^T P and
//        dKbar^T += Q^T dS with the transposing load on the staged dO and Q.
#include "bwd_walk.h"
#include "psa_dev.h"
#include "psa_internal.h"

namespace psa {

struct BwdMfmaArgs {
  int B, N, Hq, Hkv, group, nq, nk, bq, bk, lg_bk, H, causal;
  int split;                             // dK, dV: workgroups that share a walk (the query blocks of a column), each with a partial gradient
  int one_head;                          // dK, dV: all XCDs work on one head's neighbouring keys
  int dq_runs;                           // dQ: each XCD takes a contiguous run of all heads' query blocks
  int small_keys;                        // dK, dV: keys of a workgroup where blocks have fewer than 64
  int lg_cpe;                            // dK, dV: log2 of the 32-row chunks of a query block, or -1
  float scale, scale_log2;
  int64_t lvl_off[PSA_MAX_LEVELS + 2];   // level h >= 2 inside one pyramid buffer (elements)
  int64_t glvl_off[PSA_MAX_LEVELS + 2];  // level h >= 1 inside one pooled-gradient buffer (elements)
};

typedef __attribute__((ext_vector_type(4))) short bs16x4;
typedef __attribute__((ext_vector_type(8))) short bs16x8;
typedef __attribute__((ext_vector_type(4))) int i32x4;

constexpr float LOG2E = 1.44269504088896340736f;

// LDS reads with hand-counted waits: lds_wait<N> declares its operands arrived once at most N later LDS operations are outstanding
template <int OFF, typename T> __device__ __forceinline__ void lds_read(T& dst, uint32_t at) {
  static_assert(sizeof(T) == 16, "");
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(at), "n"(OFF));
}
template <int OFF> __device__ __forceinline__ void lds_read_t(bs16x4& dst, uint32_t at) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(dst) : "v"(at), "n"(OFF));
}
template <int N> __device__ __forceinline__ void lds_wait(bf16x8& x) { asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(N)); }
template <int N, typename T> __device__ __forceinline__ void lds_wait(T& x, f32x4& y, f32x4& z) {
  asm volatile("s_waitcnt lgkmcnt(%3)" : "+v"(x), "+v"(y), "+v"(z) : "n"(N));
}
template <int N, typename T, typename U> __device__ __forceinline__ void lds_wait(T& x, U& y) {
  asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x), "+v"(y) : "n"(N));
}

typedef __attribute__((ext_vector_type(4))) uint32_t rsrc_words;
// Loads straight into LDS, at `to` + lane * (16 or 4): source = buffer + v + s.  In assembly, so that the compiler does not track them:
// next to LDS reads it would make each of those wait for every load in flight, also for those into the other buffer.  They
// are waited for by hand (vmcnt) before the barrier behind which their bytes are read.
// (m0 is a reserved register: the compiler keeps nothing in it and warns that it would not restore it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_lds16(const rsrc_words& rsrc, uint32_t to, int v, int s) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(to), "v"(v), "s"(rsrc), "s"(s) : "memory", "m0");
}
__device__ __forceinline__ void load_lds4(const rsrc_words& rsrc, uint32_t to, int v, int s) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(to), "v"(v), "s"(rsrc), "s"(s) : "memory", "m0");
}
#pragma clang diagnostic pop
// buffer descriptor: base, bytes, 32-bit data format
__device__ __forceinline__ rsrc_words make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t at = (uint64_t)base;
  rsrc_words r = {(uint32_t)at, (uint32_t)(at >> 32) & 0xffffu, bytes, 0x00020000u};
#pragma unroll
  for (int i = 0; i < 4; ++i) r[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)r[i]);
  return r;
}

// Place of a row's 16-byte chunks in LDS: chunk ^ row_swizzle32(row) (psa_dev.h) for operands of 32 rows; row_swizzle serves
// operands of 16 rows (four lanes a row, 16 rows x 32 bytes transposed): no two of the rows that the LDS serves together meet either way.
template <int D> __host__ __device__ constexpr int row_swizzle(int row) {
  const int r = D == 128 ? row : row >> 1;                   // rows per 256 bytes of LDS: 1, 2
  const int fold = ((row >> 2) ^ (row >> 3)) & 1;
  return D == 128 ? (((r & 3) | (fold << 2)) << 1) | ((row >> 3) & 1) : (((r & 1) | (fold << 1)) << 1) | ((row >> 3) & 1);
}

// dQ, and D = dO.O for the kernel after it.  One workgroup per 128 query rows, a wavefront per 32 with its Q and dO fragments and
// the accumulators of dQ^T in registers.  The row's level-sorted block list is walked in tiles of 64 pooled keys; the
// rows of a tile go straight into LDS, one tile ahead, with one barrier per tile, and the block ids that say where the
// rows of the tile after that lie are on their way at the same time.
//
// As in the forward kernel the order of a tile is fixed by hand: every operand fragment is requested two fragments ahead of its MFMA, a
// slice of the vector work stands behind each MFMA (S and dP of the second 32 keys take turns while the weights of the first are made),
// tiles whose keys all count the same take one constant, and the rare others have their scores rewritten first.  Workgroups are dealt
// to the XCDs as in the forward kernel.
template <int D>
__global__ __launch_bounds__(256, D == 64 ? 3 : 2) void bwd_dq_mfma_kernel(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
                                                             const bf16_t* __restrict__ V, const bf16_t* __restrict__ Kp,
                                                             const bf16_t* __restrict__ Vp, const uint8_t* __restrict__ M,
                                                             const uint16_t* __restrict__ idx,
                                                             const int32_t* __restrict__ cnt, const bf16_t* __restrict__ O,
                                                             const float* __restrict__ lse, float* __restrict__ Dr,
                                                             const bf16_t* __restrict__ dO, bf16_t* __restrict__ dQ, BwdMfmaArgs a) {
  constexpr int ROWB = D * 2, TILEB = 64 * ROWB, BUFB = 2 * TILEB, CPR = D / 8, RPI = 64 / CPR, NI = 16 / RPI, KS = D / 16, MD = D / 32;
  // two buffers (Kbar rows [64][ROWB] | Vbar rows [64][ROWB]), a table per wavefront for irregular tiles (term [64] | last token [64])
  constexpr int OFF_FIX = 2 * BUFB, OFF_CNT = OFF_FIX + 4 * 512, OFF_LIST = OFF_CNT + 4 * PSA_MAX_LEVELS;   // and the row's blocks per level, a short row's list
  // The kernel's only LDS object: the addresses in the assembly are offsets into it, so it has to start at LDS address 0.
  __shared__ __attribute__((aligned(1024))) unsigned char smem[OFF_LIST + 2 * ROW_LISTS_NK];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slices = (a.bq + 127) / 128, per_head = a.nq * slices;
  // not causal: all XCDs on one head at a time, a contiguous run of query blocks each, or a contiguous run of all heads' blocks to each XCD
  // (dq_runs, see launch_bwd_mfma_t); causal: whole heads to each XCD and an even share of the others, the longest rows first (with
  // the same rule for dK, dV, whole backward calls, us: 12 heads x 8000 tokens 375 -> 349, x 20000 at d = 64 840 -> 778, 2 x 30000 822 -> 654,
  // 28 x 8000 775 -> 768)
  const int xcd = (int)(blockIdx.x & 7), slot = (int)(blockIdx.x >> 3);
  int head, item;
  if (a.causal) {
    if (!xcd_item(a.Hq * a.B, per_head, xcd, slot, head, item)) return;
  } else if (!dq_item(a.Hq * a.B, per_head, a.dq_runs, xcd, slot, head, item)) {
    return;
  }
  const int slice = item % slices, i = a.causal ? a.nq - 1 - item / slices : item / slices;
  const int hq = head % a.Hq, b = head / a.Hq;
  const int hk = hq / a.group;
  const int64_t qhead = (int64_t)b * a.Hq + hq, khead = (int64_t)b * a.Hkv + hk;
  int row_end = (i + 1) * a.bq;
  row_end = row_end < a.N ? row_end : a.N;
  const int row0 = i * a.bq + slice * 128, qrow = row0 + wave * 32 + l32;
  const bool active = qrow < row_end;

  bf16x8 qf[KS], gf[KS];
  // D = dO . O of the row: eight channels at a time, the sums of eight added pairwise.  The dKbar, dVbar kernel, which
  // runs after this one, reads -D from memory.  (A kernel of its own read dO once more and cost
  // a launch: 1 % of a call on 2 heads x 1000 tokens, 0.4 % on 28 x 8000.)
  float dots[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    u32x4 x = {0u, 0u, 0u, 0u}, y = x, z = x;
    if (active) {
      x = *reinterpret_cast<const u32x4*>(Q + (qhead * a.N + qrow) * D + ks * 16 + hf * 8);
      y = *reinterpret_cast<const u32x4*>(dO + (qhead * a.N + qrow) * D + ks * 16 + hf * 8);
      z = *reinterpret_cast<const u32x4*>(O + (qhead * a.N + qrow) * D + ks * 16 + hf * 8);
    }
    qf[ks] = __builtin_bit_cast(bf16x8, x);
    gf[ks] = __builtin_bit_cast(bf16x8, y);
    const bf16x8 of = __builtin_bit_cast(bf16x8, z);
    dots[ks] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) dots[ks] = fmaf((float)gf[ks][e], (float)of[e], dots[ks]);
  }
#pragma unroll
  for (int w = 1; w < KS; w *= 2)
#pragma unroll
    for (int ks = 0; ks < KS; ks += 2 * w) dots[ks] += dots[ks + w];
  float my_D = dots[0] + __shfl_xor(dots[0], 32, 64);
  if (active && hf == 0) Dr[qhead * a.N + qrow] = -my_D;
  float lse2 = active ? lse[qhead * a.N + qrow] * LOG2E : INFINITY;   // inactive rows: every weight 0
  // The wait for these loads stands here and not at their first use inside the tile loop, where it would
  // also wait for the rows fetched ahead.
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(qf[ks]), "v"(gf[ks]));
  asm volatile("" : "+v"(lse2), "+v"(my_D));
  f32x16 dq[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[md][v] = 0.f;

  const int64_t srow = qhead * a.nq + i;
  const uint16_t* my_idx = idx + srow * a.nk;
  // (in LDS: read from memory at a change of level it would wait for the rows that are under way)
  int* my_cnt = reinterpret_cast<int*>(smem + OFF_CNT);
  uint16_t* list_s = reinterpret_cast<uint16_t*>(smem + OFF_LIST);
  if (M) row_lists<4>(M + srow * a.nk, a.nk, a.H, list_s, my_cnt, wave, lane);   // (short rows, see lists_in_kernel)
  else if (tid < a.H) my_cnt[tid] = cnt[srow * CNT_STRIDE + tid];
  __syncthreads();

  // ---- the tiles of 64 pooled keys, level after level down the row's list
  struct Tile { int h, tl, ntl, nblk, start, ok; };   // (no padding: its bytes were copied through LDS)
  auto settle = [&](Tile t) __attribute__((always_inline)) -> Tile {   // first existing tile at or after (h, tl)
    for (; t.h <= a.H; ++t.h, t.tl = 0, t.start += t.nblk, t.ntl = -1) {
      if (t.ntl < 0) {
        t.nblk = __builtin_amdgcn_readfirstlane(my_cnt[t.h - 1]);
        t.ntl = ((t.nblk << (a.lg_bk - (t.h - 1))) + 63) >> 6;
      }
      if (t.tl < t.ntl) {
        t.ok = true;
        return t;
      }
    }
    t.ok = false;
    return t;
  };
  auto next = [&](Tile t) __attribute__((always_inline)) -> Tile {
    t.tl += 1;
    return settle(t);
  };
  // the block that tile row `lane` is of (rows past the level's last block: that block)
  auto block_of = [&](const Tile& t) __attribute__((always_inline)) -> int {
    const int e = ((t.tl << 6) + lane) >> (a.lg_bk - (t.h - 1));
    const int at = t.start + (e < t.nblk ? e : t.nblk - 1);
    return M ? (int)list_s[at] : (int)my_idx[at];
  };
  // its row in the level's array, from the block's id
  auto row_of = [&](const Tile& t, int block) __attribute__((always_inline)) -> int {
    const int lg_th = a.lg_bk - (t.h - 1);
    return (block << lg_th) | (((t.tl << 6) + lane) & ((1 << lg_th) - 1));
  };
  // whether some row of the tile is past the kept blocks, covers fewer tokens than others of its level or is not visible to every row
  auto irregular = [&](const Tile& t, int prow) __attribute__((always_inline)) -> bool {
    const int lg_th = a.lg_bk - (t.h - 1);
    int lim = a.N >> (t.h - 1);
    if (a.causal) {
      const int vis = (row0 + 1) >> (t.h - 1);
      lim = vis < lim ? vis : lim;
    }
    return ((t.tl + 1) << 6) > (t.nblk << lg_th) || __any(prow >= lim);
  };
  // this wavefront's 16 rows of a tile, RPI to an instruction -> buffer `to`
  auto fire = [&](const Tile& t, int prow, int to) __attribute__((always_inline)) {
    const int lg_th = a.lg_bk - (t.h - 1);
    const int64_t rows = (int64_t)a.nk << lg_th;
    const int n = t.h == 1 ? a.N : (int)rows;       // rows of this head's level array: level 1 is not padded to whole blocks
    const bf16_t* kbase = t.h == 1 ? K + khead * (int64_t)a.N * D : Kp + a.lvl_off[t.h] + khead * rows * D;
    const bf16_t* vbase = t.h == 1 ? V + khead * (int64_t)a.N * D : Vp + a.lvl_off[t.h] + khead * rows * D;
    const rsrc_words krsrc = make_rsrc(kbase, (uint32_t)n * (uint32_t)ROWB), vrsrc = make_rsrc(vbase, (uint32_t)n * (uint32_t)ROWB);
    // (a row past the end: the last one, whose weight is 0 there and which takes part elsewhere)
    const int off = (prow < n ? prow : n - 1) * ROWB;
    const int ln = lane_again(), lrow = ln / CPR;
    const uint32_t dst = to * BUFB + wave * NI * 1024;
    each<NI>([&](auto tag) __attribute__((always_inline)) {
      constexpr int k = decltype(tag)::value;
      const int r = wave * 16 + k * RPI + lrow;
      const int v = __shfl(off, r, 64) + (((ln % CPR) ^ row_swizzle32<D>(r)) << 4);
      load_lds16(krsrc, dst + k * 1024, v, 0);
      load_lds16(vrsrc, dst + k * 1024 + TILEB, v, 0);
    });
  };

  uint32_t rowaddr = l32 * ROWB + ((hf ^ row_swizzle32<D>(l32)) << 4);                                       // k-step ks: ^ ks * 32
  const int trow = hf * 4 + ((lane & 15) >> 2);
  uint32_t traddr = trow * ROWB + (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ row_swizzle32<D>(trow)) << 4) + (lane & 1) * 8;   // channels md * 32: ^ md * 64

  Tile cur = settle(Tile{1, 0, -1, 0, 0, 0}), nxt = cur;
  int prow = 0, id = 0;                            // rows of the current tile; block ids of the next one
  bool irr = false;
  if (cur.ok) {
    prow = row_of(cur, block_of(cur));
    irr = irregular(cur, prow);
    fire(cur, prow, 0);
    nxt = next(cur);
    if (nxt.ok) id = block_of(nxt);
  }
  for (int buf = 0; cur.ok; buf ^= 1) {
    // this wavefront's rows of the tile and the ids of the next have landed; behind the barrier everyone's rows have, and the
    // other buffer is no longer being read
    asm volatile("s_waitcnt vmcnt(0)" : "+v"(id)::"memory");
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    int prow_next = 0;
    bool irr_next = false;
    Tile nn = nxt;
    if (nxt.ok) {
      prow_next = row_of(nxt, id);
      irr_next = irregular(nxt, prow_next);
      fire(nxt, prow_next, buf ^ 1);
      nn = next(nxt);
      if (nn.ok) id = block_of(nn);
    }
    // S and dP of the tile's first 32 keys in turn, of its second 32, then dQ for the first and the second: 6 KS fragments
    constexpr int PF = 2, RING = 3, NR = 4 * KS, NF = 6 * KS;
    bf16x8 fr[RING], ds[2][2];
    bs16x4 lo[RING], hi[RING];
    f32x16 sc[2], dp[2];
    const float shift = (float)(cur.h - 1) - lse2;
    constexpr auto later = [](int j) {              // LDS reads issued behind those of fragment j when it is waited for
      int n = 0;
      for (int x = j + 1; x <= j + PF && x < NF; ++x) n += x < NR ? 1 : 2;
      return n;
    };
    auto request = [&](auto tag) __attribute__((always_inline)) {
      constexpr int j = decltype(tag)::value;
      if constexpr (j < NR) {
        constexpr int mb = j / (2 * KS), ks = (j % (2 * KS)) >> 1;
        lds_read<(j & 1) * TILEB + mb * 32 * ROWB>(fr[j % RING], flip<ks * 32>(rowaddr));
      } else if constexpr (j < NF) {
        constexpr int x = j - NR, md = x % MD, r0 = x / MD * 16;                  // 16 keys, 32 channels; eight rows further down the swizzle differs in one bit
        lds_read_t<r0 * ROWB>(lo[j % RING], flip<md * 64>(traddr));
        lds_read_t<(r0 + 8) * ROWB>(hi[j % RING], flip<(md * 64) ^ 32>(traddr));
      }
    };
    auto weight = [&](auto mb_tag, auto e_tag) __attribute__((always_inline)) {
      constexpr int mb = decltype(mb_tag)::value, e = decltype(e_tag)::value;
      sc[mb][e] = __builtin_amdgcn_exp2f(fmaf(sc[mb][e], a.scale_log2, shift));
      sc[mb][e] *= dp[mb][e] - my_D;
      if constexpr (e & 1) {
        ds[mb][e >> 3][(e & 7) - 1] = (__bf16)sc[mb][e - 1];
        ds[mb][e >> 3][e & 7] = (__bf16)sc[mb][e];
      }
    };
    // Scores of an irregular tile: rewritten so that the constant of the regular path gives log2 of the tokens under the key, -inf for
    // a key that must not be seen.  Each lane works out one key of the tile.
    auto fixup = [&](auto mb_tag) __attribute__((always_inline)) {
      constexpr int mb = decltype(mb_tag)::value;
      float* term = reinterpret_cast<float*>(smem + OFF_FIX + wave * 512);
      int* last = reinterpret_cast<int*>(smem + OFF_FIX + wave * 512 + 256);
      {
        const int ln = lane_again(), span = 1 << (cur.h - 1), first = prow * span;
        int c = a.N - first;
        c = c < 0 ? 0 : (c > span ? span : c);
        if (((cur.tl << 6) + ln) >> (a.lg_bk - (cur.h - 1)) >= cur.nblk) c = 0;
        term[ln] = c == 0 ? -INFINITY : (__log2f((float)c) - (float)(cur.h - 1)) / a.scale_log2;
        last[ln] = first + c - 1;
      }
      const int qlim = a.causal ? qrow : 0x7fffffff;
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const int col = mb * 32 + g4 * 8 + hf * 4;
        const f32x4 tm = *reinterpret_cast<const f32x4*>(term + col);
        const i32x4 la = *reinterpret_cast<const i32x4*>(last + col);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const float x = sc[mb][g4 * 4 + e4] + tm[e4];
          sc[mb][g4 * 4 + e4] = la[e4] > qlim ? -INFINITY : x;
        }
      }
    };
    using std::integral_constant;
    const integral_constant<int, 0> c0;
    const integral_constant<int, 1> c1;
    __builtin_amdgcn_sched_barrier(0);
    each<PF>([&](auto tag) __attribute__((always_inline)) { request(tag); });
    each<NF>([&](auto tag) __attribute__((always_inline)) {
      constexpr int j = decltype(tag)::value;
      request(integral_constant<int, j + PF>{});
      if constexpr (j < NR) {
        constexpr int mb = j / (2 * KS), ks = (j % (2 * KS)) >> 1;
        lds_wait<later(j)>(fr[j % RING]);
        const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if constexpr ((j & 1) == 0) sc[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j % RING], qf[ks], ks == 0 ? z : sc[mb], 0, 0, 0);
        else dp[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j % RING], gf[ks], ks == 0 ? z : dp[mb], 0, 0, 0);
      } else {
        constexpr int x = j - NR, md = x % MD, kq = x / MD;
        lds_wait<later(j)>(lo[j % RING], hi[j % RING]);
        const bf16x8 f = __builtin_bit_cast(bf16x8, (bs16x8)__builtin_shufflevector(lo[j % RING], hi[j % RING], 0, 1, 2, 3, 4, 5, 6, 7));
        dq[md] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, ds[kq >> 1][kq & 1], dq[md], 0, 0, 0);
      }
      // weights of the first 32 keys beside S and dP of the second, of the second beside dQ of the first
      if constexpr (j == 2 * KS) {
        if (irr) fixup(c0);
      }
      if constexpr (j == NR) {
        if (irr) fixup(c1);
      }
      if constexpr (j > 2 * KS && j < NR)
        each<16>([&](auto e) __attribute__((always_inline)) {
          constexpr int at = decltype(e)::value * (2 * KS - 1) / 16;
          if constexpr (at == j - 2 * KS - 1) weight(c0, e);
        });
      if constexpr (j >= NR && j < NR + KS)
        each<16>([&](auto e) __attribute__((always_inline)) {
          constexpr int at = decltype(e)::value * KS / 16;
          if constexpr (at == j - NR) weight(c1, e);
        });
      __builtin_amdgcn_sched_barrier(0);
    });
    rowaddr ^= BUFB;
    traddr ^= BUFB;
    cur = nxt;
    nxt = nn;
    prow = prow_next;
    irr = irr_next;
  }
  if (active) {
    bf16_t* op = dQ + (qhead * a.N + qrow) * D;
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (__bf16)(dq[md][4 * g + e] * a.scale);
        *reinterpret_cast<bf16x4*>(op + md * 32 + g * 8 + hf * 4) = w;
      }
  }
}

// One workgroup (short launches: a few, see dkv_split) per (64 adjacent pooled keys, QUERY head, level): the query heads that share a key
// head each write a partial gradient of their own (added up when the levels are folded back into dK, dV),
// so that a key block which every query block uses is not one workgroup's walk over the whole group.
// A block of 128 pooled keys is shared by two workgroups; smaller blocks are packed to a workgroup (at most 32).
//
// A wavefront owns two tiles of 16 keys with both of their gradients (128 accumulator registers at d = 128) and every second
// chunk of 32 query rows: S and dP are computed once, P and dS stay in registers, and where blocks are smaller than the
// workgroup's keys a chunk costs only the 16-key tiles that it uses.  (Two halves of wavefronts, one a gradient each, computed S
// twice, on tiles of 32 keys: of four 8-key blocks that were packed to such a tile a query block uses one and a third on average.)
// The row fragments, transposed fragments and MFMAs of a chunk follow one another in a fixed order (see `chunk`).
//
// What bounds it, 12 heads x 32760 tokens, d = 128, four levels, a fifth of the keys: the launch takes 4.1-4.4 ms (before the 16-key tiles 6.4 in two),
// the matrix pipe busy in 0.34 of the cycles, LDS in 0.30 without conflicts, the wavefronts waiting in 0.42 of theirs.  40 GB of
// rows are requested from the L2, 65 % of them miss it.  By parts, measured when four wavefronts were a workgroup and the launch took
// 4.7-4.8 ms, levels 2-4 / level 1: staging without products 1.93 / 1.29, products without staging 2.04 / 1.50, all 2.8 / 1.9.  128 keys to a
// workgroup of eight wavefronts stage a quarter less and were slower (3.85 for levels 2-4: one lock-step group on a compute unit).
constexpr int DKV_LIST = 1024;     // query blocks tested before their rows are walked
// RH: 32-row chunks of a stage, one for every two wavefronts.  With one the workgroups are of two wavefronts: four of them on a compute
// unit (d = 64: six) wait for each other less at their barriers than two of four wavefronts (12 heads x 32760 tokens 6.57 -> 6.32 ms for
// the call, causal 28 x 8000 0.849 -> 0.780), but a walk takes twice as long (the rule stands at the launch).
template <int D, int RH>
struct DkvShape {
  static constexpr int NW = 2 * RH, NT = NW * 64, KEYS = 64, ROWS = 32 * RH, CHUNKS = RH;
  static constexpr int ROWB = D * 2, TILEB = ROWS * ROWB, WPS = D == 64 ? 3 : 2;
  static constexpr int LDSB = 4 * TILEB + 16 * ROWS + 6 * DKV_LIST + 4 * NW;
};
struct DkvPtrs {
  const bf16_t *Q, *K, *V, *Kp, *Vp, *dO;
  const uint8_t* M;
  const float *lse, *Dr;
  float *dKp, *dVp;
};
// What a workgroup does: level, (batch, query head, share of its query blocks), number among the head's workgroups of this level
struct DkvItem { int h, head, bx; };

template <int D, int RH, bool FULL, bool CAUSAL>
__device__ __forceinline__ void dkv_body(unsigned char* smem, const DkvPtrs& ptr, const BwdMfmaArgs& a, const DkvItem it) {
  using S = DkvShape<D, RH>;
  constexpr int NW = S::NW, NT = S::NT, KEYS = S::KEYS, ROWS = S::ROWS, ROWB = S::ROWB, TILEB = S::TILEB, CHUNKS = S::CHUNKS;
  constexpr int CPR = D / 8, KS = D / 32, MD = D / 16, RPI = 64 / CPR, WROWS = ROWS / NW, NI = WROWS / RPI;   // rows and load instructions per wavefront, stage and tensor
  static_assert(WROWS == DKV_PART && WROWS == 16, "a wavefront's rows are of one chunk and start where the swizzle does");
  // two stage buffers (Q rows [ROWS][ROWB] | dO rows [ROWS][ROWB]), two of statistics (lse [ROWS] | -D [ROWS]), the list of query
  // blocks (the group's blocks that each uses, its number), counts per wavefront
  constexpr int BUFB = 2 * TILEB, STATB = 8 * ROWS, OFF_STAT = 2 * BUFB, OFF_BITS = OFF_STAT + 2 * STATB, OFF_ROW = OFF_BITS + 4 * DKV_LIST,
                OFF_COUNT = OFF_ROW + 2 * DKV_LIST;
  static_assert((BUFB & (BUFB - 1)) == 0 && OFF_STAT % (2 * STATB) == 0, "the buffers alternate by one address bit");
  static_assert(OFF_COUNT + 4 * NW <= S::LDSB, "LDS");
  uint32_t* kept_bits = reinterpret_cast<uint32_t*>(smem + OFF_BITS);
  uint16_t* kept_row = reinterpret_cast<uint16_t*>(smem + OFF_ROW);
  int* wcount = reinterpret_cast<int*>(smem + OFF_COUNT);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int lane = lane_again(), l16 = lane & 15, g = lane >> 4;
  const int rh = wave >> 1, pair = wave & 1;         // which 32 rows of a stage; which 16-key tiles: pair, pair + 2
  const bf16_t *Q = ptr.Q, *K = ptr.K, *V = ptr.V, *Kp = ptr.Kp, *Vp = ptr.Vp, *dO = ptr.dO;
  const uint8_t* M = ptr.M;
  const float *lse = ptr.lse, *Dr = ptr.Dr;
  const int h = it.h, head = it.head / a.split, share = it.head % a.split, bx = it.bx;
  const DkvGroup grp = dkv_group(a.lg_bk - (h - 1), a.nk, a.small_keys);
  const int G = 1 << grp.lg_G, keys = FULL ? KEYS : grp.keys;
  const int hq = head % a.Hq, b = head / a.Hq;
  const int hk = hq / a.group;
  const int lg_th = a.lg_bk - (h - 1), span = 1 << (h - 1);
  const int j0 = (bx >> grp.lg_pieces) << grp.lg_G, koff = (bx & ((1 << grp.lg_pieces) - 1)) * keys;       // first block; first key inside it
  const int64_t qhead = (int64_t)b * a.Hq + hq, khead = (int64_t)b * a.Hkv + hk;
  const bf16_t* kbase = h == 1 ? K + khead * (int64_t)a.N * D : Kp + a.lvl_off[h] + khead * ((int64_t)a.nk << lg_th) * D;
  const bf16_t* vbase = h == 1 ? V + khead * (int64_t)a.N * D : Vp + a.lvl_off[h] + khead * ((int64_t)a.nk << lg_th) * D;

  // This lane's two pooled keys (B operands of the first products, 16 keys each): key l16 of tile `pair` + u * 2
  bf16x8 kf[2][KS], vf[2][KS];
  [[maybe_unused]] int seen_from[2], kblk[2];      // causal: the key's last token - 4 g (rows from there on see it)
  uint32_t tile_bits[2];                           // the blocks that the tile's keys belong to
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int t0 = koff + (pair + u * 2) * 16, key = t0 + l16;
    kblk[u] = key >> lg_th;                        // the key's block within the group
    const int prow = (j0 << lg_th) + key, first = prow * span;
    int ctok = a.N - first;
    ctok = ctok < 0 ? 0 : (ctok > span ? span : ctok);
    const bool valid = kblk[u] < G && j0 + kblk[u] < a.nk && ctok > 0 && (FULL || (pair + u * 2) * 16 < keys);
    seen_from[u] = first + (ctok > 0 ? ctok : 1) - 1 - g * 4;
    const int wb0 = t0 >> lg_th, wb1 = (t0 + 15) >> lg_th;
    tile_bits[u] = wb0 < G && (FULL || (pair + u * 2) * 16 < keys) ? ((2u << (wb1 < G ? wb1 : G - 1)) - 1u) & ~((1u << wb0) - 1u) : 0u;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      u32x4 x = {0u, 0u, 0u, 0u}, y = {0u, 0u, 0u, 0u};
      if (valid) {
        x = *reinterpret_cast<const u32x4*>(kbase + (int64_t)prow * D + ks * 32 + g * 8);
        y = *reinterpret_cast<const u32x4*>(vbase + (int64_t)prow * D + ks * 32 + g * 8);
      }
      kf[u][ks] = __builtin_bit_cast(bf16x8, x);
      vf[u][ks] = __builtin_bit_cast(bf16x8, y);
    }
  }
  f32x4 dk[2][MD], dv[2][MD];                      // dKbar^T, dVbar^T: channels md * 16 + g * 4 .. +3 of this lane's keys
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int md = 0; md < MD; ++md) dk[u][md] = dv[u][md] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- loads: a wavefront fetches rows wave * WROWS .. of a stage, RPI rows per instruction
  const rsrc_words qrsrc = make_rsrc(Q + qhead * a.N * D, (uint32_t)a.N * (uint32_t)ROWB), grsrc = make_rsrc(dO + qhead * a.N * D, (uint32_t)a.N * (uint32_t)ROWB);
  // chunk number c of the walk: 32 rows of the query block kept[c / cpe]
  const int cpe = (a.bq + 31) >> 5;
  auto entry_of = [&](int c) __attribute__((always_inline)) { return a.lg_cpe >= 0 ? c >> a.lg_cpe : c / cpe; };
  const rsrc_words lrsrc = make_rsrc(lse + qhead * a.N, (uint32_t)a.N * 4u), drsrc = make_rsrc(Dr + qhead * a.N, (uint32_t)a.N * 4u);
  auto part_of = [&](int c) __attribute__((always_inline)) -> DkvPart {     // this wavefront's rows of the chunk
    const int e = entry_of(c);
    const int blk = __builtin_amdgcn_readfirstlane((int)kept_row[e]);
    return dkv_part(a.N, a.bq, blk, (c - e * cpe) * 32 + wave * WROWS % 32);
  };
  auto fire = [&](int c0, int total, int to) __attribute__((always_inline)) {
    const int c = c0 + wave * WROWS / 32;
    if (c >= total) return;
    const DkvPart p = part_of(c);
    const int ln = lane_again(), lrow = ln / CPR;
    // byte offset that this lane reads with load 0; with load k, RPI rows further down: ^ row_swizzle(k * RPI) << 4
    const uint32_t lane_off = lrow * ROWB + (((ln % CPR) ^ row_swizzle<D>(lrow)) << 4);
    const uint32_t dst = to * BUFB + wave * NI * 1024, st = OFF_STAT + to * STATB + wave * WROWS * 4;
    if (p.valid >= WROWS) {
      each<NI>([&](auto tag) __attribute__((always_inline)) {
        constexpr int k = decltype(tag)::value;
        const int v = (int)flip<(row_swizzle<D>(k * RPI) << 4)>(lane_off), at = (p.row + k * RPI) * ROWB;
        load_lds16(qrsrc, dst + k * 1024, v, at);
        load_lds16(grsrc, dst + k * 1024 + TILEB, v, at);
      });
    } else {
      // past its end a block repeats its last row: the weights of the rows past it are 0, and what they multiply has to be a
      // row that takes part anyway
      each<NI>([&](auto tag) __attribute__((always_inline)) {
        constexpr int k = decltype(tag)::value;
        const int v = (int)flip<(row_swizzle<D>(k * RPI) << 4)>(lane_off);
        const int r = k * RPI + lrow, at = (dkv_source_row(p, r) - lrow) * ROWB + v;
        load_lds16(qrsrc, dst + k * 1024, at, 0);
        load_lds16(grsrc, dst + k * 1024 + TILEB, at, 0);
      });
    }
    if (dkv_reads_stat(p, ln)) {                   // lse and -D of the rows that there are (step() makes up the others')
      load_lds4(lrsrc, st, ln * 4, p.row * 4);
      load_lds4(drsrc, st + 4 * ROWS, ln * 4, p.row * 4);
    }
  };
  // ---- LDS addresses in buffer 0 of this wavefront's 32-row chunk: row fragments (k-step ks: ^ ks * 64), transposed ones
  // (channels md * 16: ^ md * 32), statistics
  int total = 0, at = 0;                           // chunks of the walk; buffer of the next stage
  uint32_t rowaddr = (rh * 32 + l16) * ROWB + ((g ^ row_swizzle<D>(l16)) << 4);
  uint32_t traddr = (rh * 32 + g * 4 + (l16 >> 2)) * ROWB + ((((l16 & 3) >> 1) ^ row_swizzle<D>(g * 4 + (l16 >> 2))) << 4) + (l16 & 1) * 8;

  // One chunk of 32 rows (two row tiles of 16) against the tiles LO .. HI of this wavefront: 4 KS + 2 MD operand fragments,
  // each requested PF fragments ahead of the MFMAs that read it, in the order
  //   both tiles: S of row tile 0, dP of row tile 0, S of row tile 1, dP of row tile 1, dV, dK (two MFMAs a fragment)
  //   one tile:   S of the row tiles in turn, dP of the row tiles in turn, dV, dK (one MFMA a fragment)
  // Behind every fragment's MFMAs stands a slice of the vector work.  The reads are assembly with counted waits: left to the
  // compiler every fragment was waited for right after its read (LDS latency: two thirds of the time).
  auto chunk = [&](auto lo_tag, auto hi_tag, uint32_t bits, int row0) __attribute__((always_inline)) {
    constexpr int LO = decltype(lo_tag)::value, HI = decltype(hi_tag)::value;
    constexpr bool BOTH = LO != HI;
    constexpr int NR = 4 * KS, NF = NR + 2 * MD, PF = 2, RING = PF + 1;
    bf16x8 fr[RING], pf[2], df[2];
    bs16x4 lo[RING], hi[RING];
    f32x4 sc[2][2], dp[2][2], ls[2];                // [row tile][tile]
    // a key counts only if its block is used.  (A pooled key's token count multiplies its gradients at the end; keys that do not exist
    // get gradients that are dropped there.)
    float off[2];
#pragma unroll
    for (int u = LO; u <= HI; ++u) off[u] = FULL || ((bits >> kblk[u]) & 1u) != 0u ? 0.f : -INFINITY;
    // row fragment j: product (0: S, 1: dP), row tile, k-step
    constexpr auto prod = [](int j) { return BOTH ? (j / KS) & 1 : j / (2 * KS); };
    constexpr auto rtile = [](int j) { return BOTH ? j / (2 * KS) : j & 1; };
    constexpr auto kstep = [](int j) { return BOTH ? j % KS : (j % (2 * KS)) >> 1; };
    // slot in which the statistics of row tile 1 are requested, ahead of that slot's fragment
    constexpr int SR = BOTH ? 3 * KS - PF : -1;
    constexpr auto later = [](int j) {               // LDS reads issued behind those of fragment j when it is waited for
      int n = 0;
      for (int i = j + 1; i <= j + PF && i < NF; ++i) n += i < NR ? 1 : 2;
      if (BOTH && SR + PF - 1 >= j && SR <= j) n += 3;   // (they stand between the fragments SR + PF - 1 and SR + PF)
      return n;
    };
    auto request = [&](auto tag) __attribute__((always_inline)) {
      constexpr int j = decltype(tag)::value;
      if constexpr (j < NR) {
        lds_read<prod(j) * TILEB + rtile(j) * 16 * ROWB>(fr[j % RING], flip<kstep(j) * 64>(rowaddr));
      } else if constexpr (j < NF) {
        constexpr int md = (j - NR) % MD, off = j - NR < MD ? TILEB : 0;
        const uint32_t x = flip<md * 32>(traddr);
        lds_read_t<off>(lo[j % RING], x);
        lds_read_t<off + 16 * ROWB>(hi[j % RING], x);
      }
    };
    // lse of a row tile's rows, and -D straight into the accumulators of dP
    auto request_stat = [&](auto rt_tag) __attribute__((always_inline)) {
      constexpr int rt = decltype(rt_tag)::value;
      const uint32_t staddr = OFF_STAT + at * STATB + rh * 128 + (lane_again() & 0x30);
      lds_read<rt * 64>(ls[rt], staddr);
      lds_read<4 * ROWS + rt * 64>(dp[rt][LO], staddr);
      if constexpr (BOTH) lds_read<4 * ROWS + rt * 64>(dp[rt][HI], staddr);
    };
    // weight number e of a row tile: tile LO + e / 4, row g * 4 + e % 4
    auto weight = [&](auto rt_tag, auto e_tag) __attribute__((always_inline)) {
      constexpr int rt = decltype(rt_tag)::value, e = decltype(e_tag)::value, u = LO + e / 4, v = e % 4;
      if constexpr (u == LO) ls[rt][v] *= -LOG2E;
      float x = fmaf(sc[rt][u][v], a.scale_log2, FULL ? ls[rt][v] : ls[rt][v] + off[u]);
      if (CAUSAL) x = seen_from[u] > row0 + (rt * 16 + v) ? -INFINITY : x;
      sc[rt][u][v] = __builtin_amdgcn_exp2f(x);
      if constexpr (v & 1) {
        pf[u][rt * 4 + v - 1] = (__bf16)sc[rt][u][v - 1];
        pf[u][rt * 4 + v] = (__bf16)sc[rt][u][v];
      }
    };
    auto dscore = [&](auto rt_tag, auto e_tag) __attribute__((always_inline)) {
      constexpr int rt = decltype(rt_tag)::value, e = decltype(e_tag)::value, u = LO + e / 4, v = e % 4;
      sc[rt][u][v] *= dp[rt][u][v];
      if constexpr (v & 1) {
        df[u][rt * 4 + v - 1] = (__bf16)sc[rt][u][v - 1];
        df[u][rt * 4 + v] = (__bf16)sc[rt][u][v];
      }
    };
    // f(0) .. f(7) spread over the slots FROM .. TO - 1
    auto spread = [&](auto slot_tag, auto from_tag, auto to_tag, auto&& f) __attribute__((always_inline)) {
      constexpr int J = decltype(slot_tag)::value, FROM = decltype(from_tag)::value, TO = decltype(to_tag)::value;
      if constexpr (J >= FROM && J < TO)
        each<8>([&](auto e_tag) __attribute__((always_inline)) {
          constexpr int e = decltype(e_tag)::value;
          if constexpr (e >= 8 * (J - FROM) / (TO - FROM) && e < 8 * (J + 1 - FROM) / (TO - FROM)) f(e_tag);
        });
    };
    const std::integral_constant<int, 0> c0;
    const std::integral_constant<int, 1> c1;
    __builtin_amdgcn_sched_barrier(0);
    request_stat(c0);
    if constexpr (!BOTH) request_stat(c1);
    each<PF>([&](auto tag) __attribute__((always_inline)) { request(tag); });
    each<NF>([&](auto tag) __attribute__((always_inline)) {
      constexpr int j = decltype(tag)::value;
      if constexpr (j == SR) request_stat(c1);
      request(std::integral_constant<int, j + PF>{});
      if constexpr (j < NR) {
        constexpr int rt = rtile(j), ks = kstep(j);
        // (the statistics read before this fragment have arrived with it)
        if constexpr (prod(j) == 0) lds_wait<later(j)>(fr[j % RING], ls[rt]);
        else lds_wait<later(j)>(fr[j % RING], dp[rt][LO], dp[rt][HI]);
#pragma unroll
        for (int u = LO; u <= HI; ++u) {
          if (prod(j) == 0) sc[rt][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[j % RING], kf[u][ks], ks == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sc[rt][u], 0, 0, 0);
          else dp[rt][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[j % RING], vf[u][ks], dp[rt][u], 0, 0, 0);
        }
      } else {
        constexpr int md = (j - NR) % MD;
        lds_wait<later(j)>(lo[j % RING], hi[j % RING]);
        const bf16x8 f = __builtin_bit_cast(bf16x8, (bs16x8)__builtin_shufflevector(lo[j % RING], hi[j % RING], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
        for (int u = LO; u <= HI; ++u) {
          if (j - NR < MD) dv[u][md] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, pf[u], dv[u][md], 0, 0, 0);
          else dk[u][md] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, df[u], dk[u][md], 0, 0, 0);
        }
      }
      auto range = [&](auto from, auto to, auto&& f) __attribute__((always_inline)) { spread(tag, from, to, f); };
      using std::integral_constant;
      if constexpr (BOTH) {
        range(integral_constant<int, KS + 1>{}, integral_constant<int, 2 * KS>{}, [&](auto e) __attribute__((always_inline)) { weight(c0, e); });
        range(integral_constant<int, 2 * KS>{}, integral_constant<int, 3 * KS - KS / 2>{}, [&](auto e) __attribute__((always_inline)) { dscore(c0, e); });
        range(integral_constant<int, 3 * KS + 1>{}, integral_constant<int, 4 * KS>{}, [&](auto e) __attribute__((always_inline)) { weight(c1, e); });
        range(integral_constant<int, 4 * KS + 1>{}, integral_constant<int, 4 * KS + MD>{}, [&](auto e) __attribute__((always_inline)) { dscore(c1, e); });
      } else {                                       // (four weights a row tile)
        range(integral_constant<int, 2 * KS + 1>{}, integral_constant<int, 4 * KS>{}, [&](auto e) __attribute__((always_inline)) {
          weight(integral_constant<int, decltype(e)::value / 4>{}, integral_constant<int, decltype(e)::value % 4>{});
        });
        range(integral_constant<int, 4 * KS + 1>{}, integral_constant<int, 4 * KS + MD>{}, [&](auto e) __attribute__((always_inline)) {
          dscore(integral_constant<int, decltype(e)::value / 4>{}, integral_constant<int, decltype(e)::value % 4>{});
        });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // one stage: its chunks have been requested into buffer `at`, those of the stage after it go into the other one
  auto step = [&](int c0) __attribute__((always_inline)) {
    // this wavefront's part of the stage has landed; behind the barrier everyone's has, and the other buffer is
    // no longer being read
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (c0 + wave * WROWS / 32 < total) {
      const DkvPart p = part_of(c0 + wave * WROWS / 32);
      if (p.valid < WROWS) {                       // rows past the end of the query block: weight 0
        const int ln = lane_again();
        float* stat = reinterpret_cast<float*>(smem + OFF_STAT + at * STATB);
        if (ln < WROWS && ln >= p.valid) {
          stat[wave * WROWS + ln] = INFINITY;
          stat[ROWS + wave * WROWS + ln] = 0.f;
        }
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    fire(c0 + CHUNKS, total, at ^ 1);
    const int c = c0 + rh;
    if (c < total) {
      const int e = entry_of(c);
      const uint32_t bits = (uint32_t)__builtin_amdgcn_readfirstlane((int)kept_bits[e]);
      int row0 = 0;
      if (CAUSAL) row0 = __builtin_amdgcn_readfirstlane((int)kept_row[e]) * a.bq + (c - e * cpe) * 32;
      const std::integral_constant<int, 0> t0;
      const std::integral_constant<int, 1> t1;
      if constexpr (FULL) {
        chunk(t0, t1, bits, row0);
      } else {
        if ((bits & tile_bits[0]) != 0u) chunk(t0, t0, bits, row0);
        if ((bits & tile_bits[1]) != 0u) chunk(t1, t1, bits, row0);
      }
    }
    rowaddr ^= BUFB;
    traddr ^= BUFB;
    at ^= 1;
  };

  const int per_share = (a.nq + a.split - 1) / a.split, e_end = (share + 1) * per_share < a.nq ? (share + 1) * per_share : a.nq;
  for (int e_lo = share * per_share; e_lo < e_end; e_lo += DKV_LIST) {
    const int tid = wave * 64 + lane_again(), lane = tid & 63;
    // The columns of the level map: which of the next query blocks of this query head use any of the group's key blocks
    // at this level, as an ordered list in LDS with the blocks used as a bit mask (one round of independent
    // loads per NT entries; a walk that tests one entry after the other spends a memory latency on each of them).
    int nkept = 0;
    const int e_hi = e_lo + DKV_LIST < e_end ? e_lo + DKV_LIST : e_end;
    for (int e0 = e_lo; e0 < e_hi; e0 += NT) {
      const int e = e0 + tid;
      uint32_t bits = 0u;
      if (e < e_hi) {
        const uint8_t* mrow = M + (qhead * a.nq + e) * a.nk + j0;
        const int n = j0 + G < a.nk ? G : a.nk - j0;
        if constexpr (FULL) {
          bits = (int)mrow[0] == h ? 1u : 0u;
        } else {
          for (int x0 = 0; x0 < n; x0 += 8) {      // eight loads in flight
            int m[8];
#pragma unroll
            for (int x = 0; x < 8; ++x) m[x] = mrow[x0 + x < n ? x0 + x : n - 1];
#pragma unroll
            for (int x = 0; x < 8; ++x) bits |= (x0 + x < n && m[x] == h ? 1u : 0u) << (x0 + x);
          }
        }
      }
      const uint64_t mask = __ballot(bits != 0u);
      if (lane == 0) wcount[wave] = __popcll(mask);
      __syncthreads();                             // (and the list before is done with)
      int base = nkept, found = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        base += w < wave ? wcount[w] : 0;
        found += wcount[w];
      }
      if (bits) {
        const int at = base + __popcll(mask & ((1ull << lane) - 1ull));
        kept_bits[at] = bits;
        kept_row[at] = (uint16_t)e;
      }
      nkept += found;
      __syncthreads();
    }
    total = __builtin_amdgcn_readfirstlane(nkept);
    total = dkv_chunks(a.N, a.bq, a.nq, total, total > 0 ? __builtin_amdgcn_readfirstlane((int)kept_row[total - 1]) : 0);
    // The operands are declared used here, so that the wait for their loads stands here, where those of the level map have been waited for
    // too, and not at their first use inside the stage loop, where it would also wait for the rows fetched ahead.
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) asm volatile("" ::"v"(kf[u][ks]), "v"(vf[u][ks]));
    fire(0, total, at);
    for (int c0 = 0; c0 < total; c0 += CHUNKS) step(c0);
    __syncthreads();                               // everyone has read the last stage: the buffers may be filled again
  }
  // The two row halves' partial sums -> LDS [half][pair][tile][key][channel], added in a fixed order, first dKbar, then
  // dVbar.  Every pooled key of the group is written (zeros where no query block used it).
  const int tid = wave * 64 + lane_again(), l16e = tid & 15, ge = (tid & 63) >> 4;
  auto red = [&](int half, int p, int u) __attribute__((always_inline)) {   // 16 x D floats
    return reinterpret_cast<float*>(smem + ((half * 2 + p) * 2 + u) * 16 * D * 4);
  };
  static_assert(RH * 2 * 2 * 16 * D * 4 <= OFF_STAT, "the partial sums fit the buffers");
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int md = 0; md < MD; ++md)              // (rows spread over the banks)
        *reinterpret_cast<f32x4*>(red(rh, pair, u) + (l16e * D + ((md * 16 + ge * 4) ^ (l16e << 2)))) = which ? dv[u][md] : dk[u][md];
    __syncthreads();
    float* dst = (which ? ptr.dVp : ptr.dKp) + a.glvl_off[h] + ((qhead * a.split + share) * ((int64_t)a.nk << lg_th) + ((int64_t)j0 << lg_th)) * D;
    for (int x = tid; x < keys * (D / 4); x += NT) {
      const int kk = x / (D / 4), c4 = x % (D / 4);     // key of the workgroup, group of four channels
      const int blk = (koff + kk) >> lg_th;
      if (blk >= G || j0 + blk >= a.nk) continue;
      const int t = kk >> 4, k16 = kk & 15, at = k16 * D + ((c4 * 4) ^ (k16 << 2));
      f32x4 sum = *reinterpret_cast<const f32x4*>(red(0, t & 1, t >> 1) + at);
      if constexpr (RH == 2) sum += *reinterpret_cast<const f32x4*>(red(1, t & 1, t >> 1) + at);
      int ctok = a.N - ((j0 << lg_th) + koff + kk) * span;      // tokens under the key
      ctok = ctok < 0 ? 0 : (ctok > span ? span : ctok);
      const f32x4 none = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4*>(dst + (int64_t)(koff + kk) * D + c4 * 4) = ctok > 0 ? sum * ((float)ctok * (which ? 1.f : a.scale)) : none;
    }
  }
}

// One launch covers all levels.  Workgroup ids are dealt round-robin to the 8 XCDs.  Each XCD takes one contiguous run of a
// level's (head, key block) items (causal, where a head's columns differ in length: whole heads and an even share of the others), so that what runs on it at one time are columns of one head and level, of
// like length, whose query rows meet in its L2; or all XCDs take the same head, a block each in turn (one_head, see
// launch_bwd_mfma_t).  An XCD's items, level after level from the coarsest down, are its slots.
__device__ __forceinline__ bool dkv_item(const BwdMfmaArgs& a, int xcd, int slot, DkvItem& it) {
  for (int h = a.H; h >= 1; --h) {
    const int heads = a.B * a.Hq * a.split, ng = dkv_group(a.lg_bk - (h - 1), a.nk, a.small_keys).ng, items = heads * ng, run = a.causal ? xcd_slots(heads, ng) : (items + 7) >> 3;
    if (slot >= run) {
      slot -= run;
      continue;
    }
    if (a.causal) {
      it.h = h;
      return xcd_item(heads, ng, xcd, slot, it.head, it.bx);
    }
    const int item = a.one_head ? slot * 8 + xcd : xcd * run + slot;
    it = {h, item / ng, item % ng};
    return item < items;
  }
  return false;
}

template <int D, int RH, bool CAUSAL>
__global__ __launch_bounds__((DkvShape<D, RH>::NT), (DkvShape<D, RH>::WPS)) void bwd_dkv_mfma_kernel(DkvPtrs ptr, const uint32_t* __restrict__ order, BwdMfmaArgs a) {
  // The kernel's only LDS object: the addresses in the assembly are offsets into it, so it has to start at LDS address 0.
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DkvShape<D, RH>::LDSB];
  const int xcd = (int)(blockIdx.x & 7);
  int slot = (int)(blockIdx.x >> 3);
  if (order) slot = (int)order[xcd * (int)(gridDim.x >> 3) + slot];
  DkvItem it;
  if (!dkv_item(a, xcd, slot, it)) return;
  if (a.lg_bk - (it.h - 1) >= 6) dkv_body<D, RH, true, CAUSAL>(smem, ptr, a, it);
  else dkv_body<D, RH, false, CAUSAL>(smem, ptr, a, it);
}

// The walks of an XCD differ in length (12 heads x 32760 tokens: 7 to 171 query blocks on level 1, 205 to 242 on level 4), so the long ones are
// started first: in the order of the slots the last walks ended 1.2 to 1.4 times the mean later, 1.8 to 2.3 times in causal problems.
// bwd_dkv_length_kernel counts the query blocks of every item (64 columns of the level map a workgroup, the rows dealt to its
// wavefronts), bwd_dkv_order_kernel sorts each XCD's slots into classes of length, an eighth of an octave each (within a class as they
// come: neighbours in the key sequence stay close; in half octaves the calls took up to 1.5 % longer).  Both are latency: with the rocprofv3 trace's idle GPU
// before each, 9.6 and 9.2 us there, 9.8 and 17 at 28 x 32768.
constexpr int LEN_WAVES = 8;
__global__ __launch_bounds__(LEN_WAVES * 64) void bwd_dkv_length_kernel(const uint8_t* __restrict__ M, uint32_t* __restrict__ len, int pitch, BwdMfmaArgs a) {
  __shared__ int part[LEN_WAVES][PSA_MAX_LEVELS][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, head = blockIdx.z * a.Hq + blockIdx.y, j = blockIdx.x * 64 + lane;
  const uint8_t* col = M + (int64_t)head * a.nq * a.nk + (j < a.nk ? j : a.nk - 1);
  int n[PSA_MAX_LEVELS];
  uint64_t mates[PSA_MAX_LEVELS];                  // the lanes whose blocks share a workgroup with this lane's
#pragma unroll
  for (int h = 1; h <= PSA_MAX_LEVELS; ++h) {
    const int lg_G = h <= a.H ? dkv_group(a.lg_bk - (h - 1), a.nk, a.small_keys).lg_G : 0, G = 1 << lg_G;
    n[h - 1] = 0;
    mates[h - 1] = ((1ull << G) - 1ull) << (lane >> lg_G << lg_G);     // (G is at most 32)
  }
  for (int e0 = wave; e0 < a.nq; e0 += LEN_WAVES * 8) {
    int m[8];
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int e = e0 + x * LEN_WAVES;
      m[x] = e < a.nq && j < a.nk ? (int)col[(int64_t)e * a.nk] : 0;
    }
#pragma unroll
    for (int h = 1; h <= PSA_MAX_LEVELS; ++h) {
      if (h > a.H) break;
#pragma unroll
      for (int x = 0; x < 8; ++x) n[h - 1] += (__ballot(m[x] == h) & mates[h - 1]) != 0ull;
    }
  }
#pragma unroll
  for (int h = 1; h <= PSA_MAX_LEVELS; ++h) part[wave][h - 1][lane] = n[h - 1];
  __syncthreads();
  int base = 0;                                    // slots of the coarser levels
  for (int h = a.H; h >= 1; --h) {
    const DkvGroup g = dkv_group(a.lg_bk - (h - 1), a.nk, a.small_keys);
    const int items = a.B * a.Hq * g.ng, run = a.causal ? xcd_slots(a.B * a.Hq, g.ng) : (items + 7) >> 3;
    if (wave == h % LEN_WAVES && j < a.nk && (lane & ((1 << g.lg_G) - 1)) == 0) {
      int sum = 0;
      for (int w = 0; w < LEN_WAVES; ++w) sum += part[w][h - 1][lane];
      // in fifths of a query block of a small block's walk; what a workgroup costs besides its walk is worth about three
      const uint32_t cost = (uint32_t)(sum * (a.lg_bk - (h - 1) >= 6 ? 7 : 5) + 15);
      for (int p = 0; p < 1 << g.lg_pieces; ++p) {
        const int item = head * g.ng + (j >> g.lg_G << g.lg_pieces) + p;
        int xcd = a.one_head ? item & 7 : item / run, slot = a.one_head ? item >> 3 : item % run;
        if (a.causal) xcd_of_item(a.B * a.Hq, g.ng, head, item - head * g.ng, xcd, slot);
        len[xcd * pitch + base + slot] = cost;
      }
    }
    base += run;
  }
}

constexpr int ORDER_CLASSES = 160;
__global__ __launch_bounds__(1024) void bwd_dkv_order_kernel(const uint32_t* __restrict__ len, uint32_t* __restrict__ order, int pitch, BwdMfmaArgs a) {
  __shared__ int count[ORDER_CLASSES];
  const int xcd = blockIdx.x, tid = threadIdx.x;
  auto class_of = [&](int slot) __attribute__((always_inline)) -> int {      // the longest walks: class 0
    DkvItem it;
    if (!dkv_item(a, xcd, slot, it)) return ORDER_CLASSES - 1;               // a slot without an item
    const uint32_t c = len[xcd * pitch + slot];                              // 15 .. 7 * 8192 + 15
    const int top = 31 - __clz((int)c), eighth = 8 * top + (int)((c >> (top - 3)) & 7u);
    return ORDER_CLASSES - 2 - eighth;
  };
  if (tid < ORDER_CLASSES) count[tid] = 0;
  __syncthreads();
  for (int s = tid; s < pitch; s += 1024) atomicAdd(&count[class_of(s)], 1);
  __syncthreads();
  if (tid == 0) {
    int at = 0;
    for (int c = 0; c < ORDER_CLASSES; ++c) {
      const int n = count[c];
      count[c] = at;
      at += n;
    }
  }
  __syncthreads();
  for (int s0 = 0; s0 < pitch; s0 += 1024) {
    const int s = s0 + tid;
    if (s < pitch) order[xcd * pitch + atomicAdd(&count[class_of(s)], 1)] = (uint32_t)s;
    __syncthreads();
  }
}

// (32-bit byte offsets reach every row of a head: at most 65535 key blocks of 128 keys of 256 bytes are less than 2^31.
// Addresses need no more than element alignment, in the direct-to-LDS loads as in all others.)
// Workgroups that share a walk of dK, dV, each with a share of the query blocks and a partial gradient (added up with those of the query heads): while
// workgroups (of 32 keys) are fewer than the chip holds (four levels or more, whose deepest walks are the longest: twice that), and the walk is worth
// it: its chunks of 32 rows (causal: half of them; more than two levels, whose blocks are used by more rows: twice) at least 16 a share, and one for every 10000 gradient elements that the shares write, times the shares (a share more
// costs the same traffic, and saves less the more there are).  Which blocks are kept is not known here.  1150 shapes at a tenth to three tenths of the
// keys: 5 more than 3 % slower than with one workgroup, the worst 4 %, the mean of all 2.3 % faster (the best choice for each: 4.1 %).  Whole call, us, one / two / four:
// d = 128 1 head x 3825 tokens 130 / 101 / 89, 2 x 6109 186 / 149 / 176, 1 x 14018 423 / 335 / 330; d = 64 4 x 2869 69.5 / 60.5 / 65.2, 1 x 5413 112 / 80 / 67,
// causal 2 x 11280 227 / 165 / 171, one level 2 x 10891 177 / 148 / 152; not in one level causal 4 x 2396 at d = 128 46 / 50 / 57, 28 x 1295 39 / 46 / 60, nor in two
// causal 8 x 1549 at d = 128 41 / 50 / 63.
int dkv_split(const Plan& pl) {
  int64_t groups = 0, elems = 0;
  for (int h = 1; h <= pl.H; ++h) {
    int lg_th = 0;
    while ((1 << (lg_th + 1)) <= (pl.bk >> (h - 1))) ++lg_th;
    groups += (int64_t)pl.B * pl.Hq * dkv_group(lg_th, pl.nk, 32).ng;
    elems += ((int64_t)pl.B * pl.Hq * pl.N * pl.d) >> (h - 1);
  }
  const int64_t resident = 256 * (pl.d == 64 ? 3 : 2);
  int64_t walk = 2 * column_chunks(pl);            // in half chunks
  if (pl.causal) walk /= 2;
  if (pl.H > 2) walk *= 2;
  int split = 1;
  while (groups * split < (pl.H > 3 ? 2 : 1) * resident && walk >= 2 * 16 * split && 5000 * walk >= elems * split * split) split *= 2;
  return split;
}

bool bwd_uses_mfma(const Plan& pl) {
  return pl.dtype == PSA_BF16 && pl.bk >= 8 && pl.bk <= 128 && (pl.d == 64 || pl.d == 128) &&
         pl.nq <= 8192;                            // (the bound that the header states)
}

template <int D>
static hipError_t launch_bwd_mfma_t(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp,
                                    const void* Vp, const uint8_t* M, const uint16_t* idx, const int32_t* cnt,
                                    const void* O, const float* lse, const void* dO, float* Dr, float* dKp, float* dVp, void* dQ,
                                    hipStream_t s) {
  BwdMfmaArgs a;
  a.B = pl.B; a.N = pl.N; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.group = pl.group; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.bk = pl.bk;
  a.H = pl.H; a.causal = pl.causal; a.scale = pl.scale; a.scale_log2 = pl.scale * LOG2E;
  a.lg_bk = 0;
  while ((1 << a.lg_bk) < pl.bk) ++a.lg_bk;
  const int cpe = (pl.bq + 31) / 32;
  a.lg_cpe = 0;
  while ((1 << a.lg_cpe) < cpe) ++a.lg_cpe;
  if ((1 << a.lg_cpe) != cpe) a.lg_cpe = -1;
  // With a run of items to each XCD the Q and dO of eight heads are in flight, next to which the memory-side cache (256 MB) has little room from 5 million
  // elements a head on (4 million with grouped heads); with all XCDs on one head it has room at any length.  Runs are better all the same, but for few
  // heads, of which they leave an XCD less than a whole one.  Whole call, ms for runs / one head, not causal, d = 128: 5 heads x 60000 tokens 8.92 / 10.0, 12 x 40000 9.52 / 10.6,
  // 40 x 75600 116 / 125, single level 8 x 42000 5.22 / 5.46; 64-row blocks 16 x 40000 7.90 / 9.05; d = 64 6 x 100000 15.0 / 16.7, 32 x 131072 127 / 135; grouped 28 x 32000
  // 7.48 / 8.45, 8 x 40000 6.20 / 7.17.  One head: 1 x 40000 0.929 / 0.924, 2 x 100000 in a single level 8.04 / 7.55, d = 64 4 x 120000 11.4 / 11.0 (2 x 40000 1.61 / 1.63).
  a.one_head = !pl.causal && pl.B * pl.Hq <= 4 && (int64_t)pl.N * pl.d >= (pl.group > 1 ? 4000000 : 5000000);
  a.split = dkv_split(pl);
  int64_t off = 0;
  for (int h = 0; h < PSA_MAX_LEVELS + 2; ++h) { a.lvl_off[h] = pl.lvl_off[h]; a.glvl_off[h] = 0; }
  for (int h = 1; h <= pl.H; ++h) {
    a.glvl_off[h] = off;
    off += (int64_t)pl.B * pl.Hq * a.split * pl.nk * (pl.bk >> (h - 1)) * pl.d;   // partial tensors of every QUERY head
  }
  const bf16_t* q = static_cast<const bf16_t*>(Q);
  const bf16_t* k = static_cast<const bf16_t*>(K);
  const bf16_t* v = static_cast<const bf16_t*>(V);
  const bf16_t* kp = static_cast<const bf16_t*>(Kp);
  const bf16_t* vp = static_cast<const bf16_t*>(Vp);
  const bf16_t* go = static_cast<const bf16_t*>(dO);
  const int slices = (pl.bq + 127) / 128;
  // A head of few query blocks does not reach all XCDs (2 blocks: two of the eight; 9: five, two blocks each but the last): there each XCD
  // takes an eighth of all heads' blocks.  Whole call, us for a head's runs / this, 40 heads, one level: x 130 tokens 37.0 / 31.1, x 350
  // 44.0 / 38.4, x 1100 92.7 / 80.5, d = 64 x 161 24.9 / 22.4, x 1100 55.3 / 50.4; four levels 12 x 2000 92.0 / 91.6.  From 32 blocks on the two are
  // within 1 % of each other (12 x 4000 197.0 / 198.3, x 32760 6199 / 6254, 40 x 20000 8399 / 8391, 24 x 60000 46488 / 46609).
  const int dq_items = pl.nq * slices, heads = pl.B * pl.Hq;
  a.dq_runs = dq_runs(dq_items);
  const int dq_slot_count = pl.causal ? xcd_slots(heads, dq_items) : dq_slots(heads, dq_items);
  const unsigned dq_grid = 8u * (unsigned)dq_slot_count;
  bwd_dq_mfma_kernel<D><<<dq_grid, 256, 0, s>>>(q, k, v, kp, vp, lists_in_kernel(pl, false) ? M : nullptr, idx, cnt, static_cast<const bf16_t*>(O), lse, Dr, go, static_cast<bf16_t*>(dQ), a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  auto groups = [&](int small_keys) {            // workgroups of an XCD, as the kernel counts them
    int64_t n = 0;
    for (int h = 1; h <= pl.H; ++h) {
      const int ng = dkv_group(a.lg_bk - (h - 1), pl.nk, small_keys).ng;
      n += pl.causal ? (int64_t)xcd_slots(heads * a.split, ng) : ((int64_t)heads * a.split * ng + 7) / 8;
    }
    return n;
  };
  // Where blocks have fewer than 64 pooled keys a workgroup takes 64 keys, or 32 (half of its tiles) while the longest walk (half of
  // the query blocks, say) would end after the work that there is for every resident workgroup (walks of a fifth of the query blocks,
  // a tenth if causal; what a workgroup costs besides is worth four).  Whole call, us for 64 / 32, d = 128, four levels: 2 heads x 3000 tokens 112 / 90,
  // x 8000 241 / 193, x 20000 644 / 505; 12 x 3000 148 / 147, x 8000 489 / 512, 28 grouped causal x 8000 674 / 709; d = 64 2 x 8000 164 / 129, 12 x 8000 256 / 266.
  const int64_t nq = (pl.nq + a.split - 1) / a.split, walk = nq / (pl.causal ? 10 : 5) + 4;   // of a workgroup's share
  // Workgroups of two wavefronts (twice as many resident, each walk twice as long) where the work for every resident one is at least the
  // longest walk that there can be.  Whole call, time in four wavefronts over time in two, 70 shapes, by that work over that walk: up to
  // 0.2 0.60-0.91, 0.2-0.5 0.63-0.97 (32-row blocks up to 1.07), 0.5-0.95 0.71-1.08, from 1.0 on 1.01-1.06.
  const bool pairs = groups(64) * 8 * walk >= 256 * DkvShape<D, 1>::WPS * 2 * nq;
  const int64_t resident = 256 * DkvShape<D, 2>::WPS * (pairs ? 2 : 1);
  a.small_keys = groups(64) * 8 * walk < resident * (nq / 2 + 4) ? 32 : 64;
  const DkvPtrs ptr = {q, k, v, kp, vp, go, M, lse, Dr, dKp, dVp};
  const int pitch = (int)groups(a.small_keys);
  // Started in the order of their lengths once they are more than fit at a time and the launch is long enough to gain more than the two
  // small kernels take (about 36 query blocks for every resident workgroup).  Whole call, us in the order of the keys / of their lengths: 12 heads x
  // 3000 tokens 148 / 159, x 4000 198 / 193, x 5000 255 / 235, x 32760 6659 / 6170, 2 x 8000 193 / 205, x 20000 555 / 502, causal 28 x 3000 192 / 197, x 4000
  // 281 / 274, x 8000 690 / 674; 40 x 3000 392 / 342, which the line leaves in the order of the keys.  The dQ kernel was the last to read the block
  // lists: their place takes the lengths and the order.
  uint32_t* order = nullptr;
  if (a.split == 1 && 8 * pitch > resident && 8 * pitch * walk > 36 * resident && (size_t)pitch * 8 * 2 * sizeof(uint32_t) <= (size_t)pl.B * pl.Hq * pl.nq * pl.nk * sizeof(uint16_t)) {
    uint32_t* len = const_cast<uint32_t*>(reinterpret_cast<const uint32_t*>(idx));
    order = len + 8 * pitch;
    bwd_dkv_length_kernel<<<dim3((pl.nk + 63) / 64, pl.Hq, pl.B), LEN_WAVES * 64, 0, s>>>(M, len, pitch, a);
    bwd_dkv_order_kernel<<<8, 1024, 0, s>>>(len, order, pitch, a);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  auto launch = [&](auto kernel, int threads) { kernel<<<8 * pitch, threads, 0, s>>>(ptr, order, a); };
  if (pairs) launch(pl.causal ? bwd_dkv_mfma_kernel<D, 1, true> : bwd_dkv_mfma_kernel<D, 1, false>, DkvShape<D, 1>::NT);
  else launch(pl.causal ? bwd_dkv_mfma_kernel<D, 2, true> : bwd_dkv_mfma_kernel<D, 2, false>, DkvShape<D, 2>::NT);
  return hipGetLastError();
}

// dQ, D = dO.O per row and the pooled gradients dKp, dVp of every level (bfloat16 inputs)
hipError_t launch_attn_bwd_mfma(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                                const uint8_t* M, const uint16_t* idx, const int32_t* cnt, const void* O, const float* lse,
                                const void* dO, float* Dr, float* dKp, float* dVp, void* dQ, hipStream_t s) {
  return pl.d == 64 ? launch_bwd_mfma_t<64>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, s)
                    : launch_bwd_mfma_t<128>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, dO, Dr, dKp, dVp, dQ, s);
}

}  // namespace psa
