// Attention with float32 operands and sums on the gfx950 matrix cores: psa_attention_fwd in float32 (Alg. 1, the 1e-5 mode),
// psa_dense_ref (Eq. 1) for both element types, and the bfloat16 block sizes that
// attn_mfma_kernel does not take.  Sums are fp32 throughout; a float32 operand is the sum of three bfloat16 planes (psa_dev.h: exact but for
// small values, see far_q and small_v below), and a product of two is six of the nine products of planes on v_mfma_f32_32x32x16_bf16 (what is left out is below
// 2^-24 of it): 192 cycles of the matrix pipe for 16 channels where v_mfma_f32_32x32x2_f32 needs 512.  A bfloat16 operand is one plane, the weights, by
// v_exp_f32 (1 ulp), are three either way.  Scores or values that are not finite, values of 2^80 and more and rows of small operands take float32 instructions.
// In S the products of the leading planes and all others are two sums that are added at the end; error against 64 bits
// of 12 heads x 4680 tokens 4.1e-7 (float32 instructions) -> 1.0e-7, of 2 x 1024 at d = 64 1.4e-7 -> 0.9e-7, of lse 4.8e-8 -> 2.4e-8.
//
// What bounds it: 12 heads x 4680 tokens, d = 128, a fifth of the keys: a wavefront issues about 1040 vector instructions a
// tile (72 conversions and what belongs to them, addresses, softmax) next to 96 MFMAs, two wavefronts on a SIMD: the vector port is
// busy as long as the matrix pipe, and 444 workgroups take one and a half rounds of the chip.  The V rows of a tile travel through registers into LDS during its
// first product, the K rows of the next one during its second, and each product is followed by one barrier; the block ids that say
// where rows lie are requested a step ahead.
//
// Operand roles as in the bfloat16 kernel: S^T = K Q^T puts one query row in each lane (lane l and l + 32 share
// row l: keys (v/4)*8 + (l/32)*4 + v%4 in register v), and the planes of P^T are directly the B operands of
// O^T += V^T P^T, whose A operands the transposing LDS load makes from the row-major V planes.
//
// What decides the speed of small problems is how many wavefronts there are, so the four wavefronts of a
// workgroup are dealt out in two ways: TEAM of them own 32 query rows each and share the tiles of one
// stream of keys, and there are 4 / TEAM such teams over the SAME 32 * TEAM rows, each taking every
// (4 / TEAM)-th tile of the row's list; their (maximum, sum, output) are merged through LDS at the end.
//
// Registers: float32 at d = 128 in teams of four spills 16 (68 bytes), some of them stored and reloaded inside the tile loop; no other instantiation spills vector registers.
//
// Measured (pyramid and block lists included, a fifth of the keys), products on v_mfma_f32_32x32x2_f32 -> here, us: 12 heads x 4680 tokens, d = 128,
// 342 -> 236, x 1000 46.8 -> 35.2, x 6000 at d = 64 417 -> 228; causal 12 x 2634 133 -> 107, 2 x 2435 58.5 -> 43.0; 4 x 3433 at d = 64 70.8 -> 50.9.
#include <limits.h>
#include <math.h>

#include "psa_dev.h"
#include "psa_internal.h"

namespace psa {

struct F32Args {
  int N, Hq, Hkv, nq, nk, bq, bk, lg_bk, H, causal;
  int slices;              // workgroups per query block
  float scale_hi, scale_lo;  // scale * log2(e) as a sum of two
  int64_t lvl_off[PSA_MAX_LEVELS + 2];
};

// bfloat16 planes of an element type: what a value is the exact sum of
template <typename T> struct Planes { static constexpr int N = 1; };
template <> struct Planes<float> { static constexpr int N = 3; };

// A tile: its planes one after the other, rows of D bfloat16, 16-byte chunks at chunk ^ row_swizzle32(row).  A team of one wavefront puts V
// where K was (it has nobody to wait for), so that four such teams fit the LDS at d = 128.
constexpr int LATER_TILES = 2048;
template <typename T, int D, int TEAM>
struct F32Shape {
  static constexpr int KS = 4 / TEAM, ROWS = 32 * TEAM, PITCH = D + 4, NPL = Planes<T>::N;
  static constexpr int ROWB = 2 * D, PLANEB = 32 * ROWB, TENSORB = NPL * PLANEB;
  static constexpr int OFF_V = TEAM == 1 ? 0 : TENSORB, OFF_TAB = OFF_V + TENSORB;
  static constexpr int TILEB = OFF_TAB + TEAM * 256;                   // K | V | (term [32] | last token [32]) per wavefront
  static constexpr int MERGEB = 4 * (2 * KS * ROWS + KS * ROWS * PITCH);   // m, l | O of every team
  static constexpr int OFF_FLAG = KS * TILEB;                          // behind the teams' tiles: one flag per wavefront
  static constexpr int OFF_LATER = OFF_FLAG + 16;                      // a bit per tile and wavefront: left for the end
  static constexpr int OFF_LIST = OFF_LATER + 4 * LATER_TILES / 8;                        // blocks per level | list (rows whose list the kernel makes)
  static constexpr int END = OFF_LIST + 4 * PSA_MAX_LEVELS + 2 * ROW_LISTS_NK;
  static constexpr size_t BYTES = END > MERGEB ? END : MERGEB;
};

// Four consecutive elements as their planes: put(plane, its four bfloat16); their leading planes' range is added to `range`.
template <typename F> __device__ __forceinline__ void to_planes(f32x4 x, PairRange& range, F&& put) {
  const Split2 a = split2(x[0], x[1]), b = split2(x[2], x[3]);
  range.add(a.h);
  range.add(b.h);
  put(0, u32x2{a.h, b.h});
  put(1, u32x2{a.m, b.m});
  put(2, u32x2{a.l, b.l});
}
template <typename F> __device__ __forceinline__ void to_planes(Four<bf16_t>::raw x, PairRange& range, F&& put) {
  const u32x2 w = __builtin_bit_cast(u32x2, x);
  range.add(w[0]);
  range.add(w[1]);
  put(0, w);
}

typedef short f32_s16x4 __attribute__((ext_vector_type(4)));
typedef short f32_s16x8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) f32_s16x4 f32_lds_s16x4;

template <typename T, int D, int TEAM>
__global__ __launch_bounds__(256, (F32Shape<T, D, TEAM>::BYTES <= 80 * 1024 ? 2 : 1))
void attn_f32_kernel(const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ Kp,
                     const T* __restrict__ Vp, const uint8_t* __restrict__ M, const uint16_t* __restrict__ idx, const int32_t* __restrict__ cnt,
                     T* __restrict__ O, float* __restrict__ lse, F32Args a) {
  using S = F32Shape<T, D, TEAM>;
  constexpr int KS = S::KS, ROWS = S::ROWS, PITCH = S::PITCH, NPL = S::NPL, ROWB = S::ROWB, PLANEB = S::PLANEB, CPR = D / 4, MD = D / 32, KSTEPS = D / 16;
  constexpr int TT = 64 * TEAM, NCH = 32 * CPR / TT;     // threads of a team; 4-element chunks per thread, tile and tensor
  extern __shared__ __attribute__((aligned(16))) unsigned char fsm[];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int team = wave / TEAM, wr = wave % TEAM;
  unsigned char* Ks = fsm + team * S::TILEB;
  unsigned char* Vs = Ks + S::OFF_V;
  float* term_s = reinterpret_cast<float*>(Ks + S::OFF_TAB + wr * 256);   // irregular tiles: additive term per key, its last token
  int* last_s = reinterpret_cast<int*>(term_s + 32);
  int* flag_s = reinterpret_cast<int*>(fsm + S::OFF_FLAG);               // what the wavefront staged of V: FAR, SMALL
  uint32_t* later_s = reinterpret_cast<uint32_t*>(fsm + S::OFF_LATER) + wave * (LATER_TILES / 32);

  const bool own_list = M != nullptr, dense = !own_list && idx == nullptr;
  int* cnt_s = reinterpret_cast<int*>(fsm + S::OFF_LIST);
  uint16_t* list_s = reinterpret_cast<uint16_t*>(cnt_s + PSA_MAX_LEVELS);
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

  PairRange q_range;
  bf16x8 q[NPL][KSTEPS];                                 // planes of channels ks * 16 + hf * 8 .. +7 of this lane's row
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    u32x4 w[NPL];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      typename Four<T>::raw x = {0, 0, 0, 0};
      if (active) x = Four<T>::load(Q + (qhead * a.N + row) * D + ks * 16 + hf * 8 + u * 4);
      to_planes(x, q_range, [&](int plane, u32x2 v) __attribute__((always_inline)) {
        w[plane][2 * u] = v[0];
        w[plane][2 * u + 1] = v[1];
      });
    }
#pragma unroll
    for (int pl = 0; pl < NPL; ++pl) q[pl][ks] = __builtin_bit_cast(bf16x8, w[pl]);
  }
  f32x16 o[MD];
#pragma unroll
  for (int md = 0; md < MD; ++md)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[md][v] = 0.f;
  float m = -INFINITY, l = 0.f;                          // reference of the weights (log2, a whole number), sum of the weights

  const int64_t srow = qhead * a.nq + i;
  const uint16_t* my_idx = idx + srow * a.nk;
  const int32_t* my_cnt = cnt + srow * CNT_STRIDE;
  if (own_list) {
    row_lists<4>(M + srow * a.nk, a.nk, a.H, list_s, cnt_s, wave, lane);
    __syncthreads();
  }
  const int H = dense ? 1 : a.H;
  int dense_blocks = a.nk;                               // dense and causal: blocks that start at or before the last row
  if (a.causal) dense_blocks = (row_end - 1) / a.bk + 1;

  // The pooled tokens of a level's kept blocks, in list order, are one stream that is cut into tiles of 32.
  struct Tile { int h, tl, ntl, nblk, start, ok; };      // (no padding: its bytes were copied through memory)
  auto enter = [&](Tile& t) __attribute__((always_inline)) {
    t.nblk = dense ? dense_blocks : own_list ? __builtin_amdgcn_readfirstlane(cnt_s[t.h - 1]) : my_cnt[t.h - 1];
    t.ntl = (int)((((int64_t)t.nblk << (a.lg_bk - (t.h - 1))) + 31) >> 5);
  };
  auto settle = [&](Tile& t) __attribute__((always_inline)) {   // carry tl over to the level that holds it
    for (;;) {
      if (t.tl < t.ntl) { t.ok = 1; return; }
      t.tl -= t.ntl;
      t.start += t.nblk;
      if (++t.h > H) { t.h = H; t.ok = 0; t.ntl = 0; t.nblk = 0; return; }
      enter(t);
    }
  };
  // The block of tile row l32 (past the level's last block: that block) is requested a step before its row is worked out.
  auto block_of = [&](const Tile& t) __attribute__((always_inline)) -> int {
    const int e = ((t.tl << 5) + l32) >> (a.lg_bk - (t.h - 1)), f = e < t.nblk ? e : t.nblk - 1;
    return dense ? f : own_list ? (int)list_s[t.start + f] : (int)my_idx[t.start + f];
  };
  auto row_of = [&](const Tile& t, int block) __attribute__((always_inline)) -> int {   // pooled row of tile row l32; -1: none
    const int lg_th = a.lg_bk - (t.h - 1), g = (t.tl << 5) + l32, pr = (block << lg_th) | (g & ((1 << lg_th) - 1));
    return t.ok && g >> lg_th < t.nblk && ((int64_t)pr << (t.h - 1)) < a.N ? pr : -1;
  };
  auto base_of = [&](const T* level1, const T* pooled, const Tile& t) __attribute__((always_inline)) -> const T* {
    return t.h == 1 ? level1 + khead * (int64_t)a.N * D : pooled + a.lvl_off[t.h] + khead * ((int64_t)a.nk << (a.lg_bk - (t.h - 1))) * D;
  };
  // this thread's number in its team; where registers are short what depends on it is worked out again at every use
  auto place = [&]() __attribute__((always_inline)) -> int { return wr * 64 + (D == 128 && TEAM == 4 && NPL == 3 ? lane_again() : lane); };
  typename Four<T>::raw reg[NCH];                        // this thread's part of the K or V rows on their way into LDS
  // (a row that does not exist: row 0, which is replaced by zeros on its way into LDS)
  auto fetch = [&](const T* level1, const T* pooled, const Tile& t, int prow) __attribute__((always_inline)) {
    const T* base = base_of(level1, pooled, t);
    const int at = prow < 0 ? 0 : prow, x0 = place();
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = x0 + TT * c;
      reg[c] = Four<T>::load(base + (int64_t)__shfl(at, x / CPR, 64) * D + (x % CPR) * 4);
    }
  };
  auto deposit = [&](unsigned char* tensor, int prow) __attribute__((always_inline)) -> PairRange {
    const int x0 = place();
    if (__any(prow < 0)) {
#pragma unroll
      for (int c = 0; c < NCH; ++c)
        if (__shfl(prow, (x0 + TT * c) / CPR, 64) < 0) reg[c] = typename Four<T>::raw{0, 0, 0, 0};
    }
    PairRange range;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      const int x = x0 + TT * c, r = x / CPR, ch = x % CPR;
      unsigned char* at = tensor + r * ROWB + (((ch >> 1) ^ row_swizzle32<D>(r)) << 4) + (ch & 1) * 8;
      to_planes(reg[c], range, [&](int plane, u32x2 v) __attribute__((always_inline)) { *reinterpret_cast<u32x2*>(at + plane * PLANEB) = v; });
    }
    return range;
  };
  // scores of tile t -> weights of its keys for this lane's row and their sum; reference, sum and output so far follow.  Weights below 2^-109, whose planes would
  // not hold them (and those below 2^-126, which v_exp_f32 makes 0): the tile's weights and their sum are 2^24 times what they are, `unscale` takes that back (dense
  // 16 heads x 3000 tokens, scores of deviation 1 / 16: 619 / 624 us, error 2.9e-7 / 1.0e-6; float32 instructions 1011 / 1013 us, 1.2e-6 / 2.6e-6).  EXACT: never,
  // by exp2f.  With `discard` the scores may be anything: reference, sum and output stay.
  constexpr float LAG = 8.f;
  float unscale = 1.f;
  auto weights = [&](const Tile& t, int prow, f32x16& sc, auto exact, bool discard) __attribute__((always_inline)) -> float {
    constexpr bool EXACT = decltype(exact)::value;
    constexpr float TINY = -109.f;
    // log2 of the tokens under a key: one constant, unless the tile holds keys that do not exist, cover fewer tokens than others of the level
    // or (causal) are hidden from a row of this wavefront
    const int hm1 = t.h - 1;
    int lim = a.N >> hm1;
    if (a.causal) {
      const int vis = (row0 + wr * 32 + 1) >> hm1;
      lim = vis < lim ? vis : lim;
    }
    const bool irregular = __any(prow < 0 || prow >= lim);
    float tmax = -INFINITY, tmin = INFINITY;
    if (irregular) {
      const int span = 1 << hm1;
      const int64_t first = (int64_t)prow << hm1;
      int64_t c = a.N - first;
      c = prow < 0 ? 0 : (c > span ? span : c);
      if (hf == 0) {
        term_s[l32] = c > 0 ? (c == span ? (float)hm1 : log2f((float)c)) : -INFINITY;
        last_s[l32] = (int)(first + (c > 0 ? c : 1) - 1);
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");          // (LDS serves one wavefront in order)
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x4 ts = *reinterpret_cast<const f32x4*>(term_s + g4 * 8 + hf * 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float s = ts[e] == -INFINITY ? -INFINITY : fmaf(sc[g4 * 4 + e], a.scale_lo, fmaf(sc[g4 * 4 + e], a.scale_hi, ts[e]));
          if (a.causal && last_s[g4 * 8 + hf * 4 + e] > row) s = -INFINITY;
          sc[g4 * 4 + e] = s;
          tmax = fmaxf(tmax, s);
          if (!EXACT) tmin = fminf(tmin, s == -INFINITY ? INFINITY : s);
        }
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        tmax = fmaxf(tmax, sc[v]);
        tmin = fminf(tmin, sc[v]);
      }
      tmax = fmaf(tmax, a.scale_hi, (float)hm1);
      tmin = fmaf(tmin, a.scale_hi, (float)hm1);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    // The reference is a whole number, so that changing it rounds nothing, and is raised when a weight would pass 2^LAG (with every
    // larger score 12 heads x 4680 tokens take 244 us instead of 240): no sum overflows as long as values are below 2^80, and tiles with others are EXACT.
    // (One test for all that is rare, and `discard` only behind it: what a step waits for before its weights counts.)
    bool tiny = false;
    if (__any(EXACT ? tmax > m : tmax - m > LAG || tmin - m < TINY) && !discard) {
      const float mn = tmax - m > LAG || EXACT ? fmaxf(m, ceilf(tmax)) : m;
      const float alpha = mn == -INFINITY ? 1.f : exp2f(m - mn);      // m = -inf: 0
      l *= alpha;
#pragma unroll
      for (int md = 0; md < MD; ++md)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[md][v] *= alpha;
      m = mn;
      tiny = !EXACT && __any(tmin - (m == -INFINITY ? 0.f : m) < TINY);
    }
    unscale = tiny ? 0x1p-24f : 1.f;
    const float ref = m == -INFINITY ? 0.f : m;
    const float shift = irregular ? -ref : (float)hm1 - ref;
    auto power = [&](int v) __attribute__((always_inline)) { return irregular ? sc[v] + shift : fmaf(sc[v], a.scale_lo, fmaf(sc[v], a.scale_hi, shift)); };
    if (EXACT) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = exp2f(power(v));
    } else if (tiny) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float x = power(v);
        const bool down = x < -64.f;
        sc[v] = __builtin_amdgcn_exp2f(down ? x + 24.f : x) * (down ? 1.f : 0x1p24f);
      }
    } else if (irregular) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = __builtin_amdgcn_exp2f(sc[v] + shift);
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = __builtin_amdgcn_exp2f(fmaf(sc[v], a.scale_lo, fmaf(sc[v], a.scale_hi, shift)));
    }
    float sum[8];                                        // pairwise: l is rounded once a tile, the parts at their own size
#pragma unroll
    for (int v = 0; v < 8; ++v) sum[v] = sc[2 * v] + sc[2 * v + 1];
#pragma unroll
    for (int w = 1; w < 8; w *= 2)
#pragma unroll
      for (int v = 0; v < 8; v += 2 * w) sum[v] += sum[v + w];
    return sum[0];
  };
  // a team of one wavefront owns its buffer: its LDS operations complete in order, nothing to wait for
  auto barrier = [&]() __attribute__((always_inline)) {
    if constexpr (TEAM == 1) asm volatile("" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  };

  // Of float32 operands below 2^-109 the planes may hold all but 2^-134.  Of keys this counts next to large queries only, of queries it is not asked whether
  // there are large keys: such rows leave every tile for the end.  Of values it counts where the output is as small: SMALL is noted, and looked into at the end.
  const bool far_q = NPL == 3 && __any(q_range.small() || q_range.large());
  constexpr int FAR = 1, SMALL = 2;                      // of the rows of V: one is large or not finite, one is small
  bool small_v = false;
  int total = 0;                                         // tiles of the row: the same for every team
  for (int h = 1; h <= H; ++h) {
    Tile t;
    t.h = h;
    enter(t);
    total += t.ntl;
  }
  Tile cur = {1, team, 0, 0, 0, 0};
  enter(cur);
  settle(cur);
  Tile nxt = cur;
  int pc = -1, id = 0;                                   // rows of this tile; blocks of the next one
  if (cur.ok) {
    pc = row_of(cur, block_of(cur));
    fetch(K, Kp, cur, pc);
    nxt.tl += KS;
    settle(nxt);
    if (nxt.ok) id = block_of(nxt);
    deposit(Ks, pc);
  }
#pragma unroll
  for (int x = 0; x < LATER_TILES / 32; x += 64) if (x + lane < LATER_TILES / 32) later_s[x + lane] = 0u;
  barrier();
  int n = 0, later_from = INT_MAX;                       // tiles of the team so far; the first of those that are all left for the end
  bool later = false, again = false;                     // there are such tiles; all are
  for (int step = 0; step < total; step += KS, ++n) {
    const int pn = row_of(nxt, id);
    Tile nn = nxt;
    if (nxt.ok) {
      nn.tl += KS;
      settle(nn);
      if (nn.ok) id = block_of(nn);
    }
    if (cur.ok) fetch(V, Vp, cur, pc);
    f32x16 sc;
    float sum = 0.f;
    int v_state = 0;
    bool bad = far_q;
    if (cur.ok) {
      // S: the large terms in one sum, the others in another that is added at the end (fewer roundings than one chain of D products).  One k-step's
      // fragments ahead of the products, no more.
      f32x16 low;
      const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      const uint32_t kaddr = (uint32_t)(l32 * ROWB + ((hf ^ row_swizzle32<D>(l32)) << 4));
      bf16x8 fr[2][NPL];
      auto read_k = [&](bf16x8 (&dst)[NPL], auto tag) __attribute__((always_inline)) {
        const unsigned char* at = Ks + flip<decltype(tag)::value * 32>(kaddr);
#pragma unroll
        for (int pl = 0; pl < NPL; ++pl) dst[pl] = *reinterpret_cast<const bf16x8*>(at + pl * PLANEB);
      };
      read_k(fr[0], std::integral_constant<int, 0>{});
      each<KSTEPS>([&](auto tag) __attribute__((always_inline)) {
        constexpr int ks = decltype(tag)::value;
        if constexpr (ks + 1 < KSTEPS) read_k(fr[(ks + 1) & 1], std::integral_constant<int, ks + 1>{});
        const bf16x8(&kk)[NPL] = fr[ks & 1];
        if constexpr (NPL == 3) {
          low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[2], q[0][ks], ks == 0 ? zero : low, 0, 0, 0);
          low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[0], q[2][ks], low, 0, 0, 0);
          low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[1], q[1][ks], low, 0, 0, 0);
          low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[1], q[0][ks], low, 0, 0, 0);
          low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[0], q[1][ks], low, 0, 0, 0);
        }
        sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[0], q[0][ks], ks == 0 ? zero : sc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (NPL == 3) {
        float any[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) any[v] = sc[v] += low[v];
#pragma unroll
        for (int w = 1; w < 16; w *= 2)
#pragma unroll
          for (int v = 0; v < 16; v += 2 * w) any[v] += any[v + w];
        bad |= (bool)__any(!(fabsf(any[0]) < INFINITY));       // a row or key that is not finite, or a product that overflows
      }
      sum = weights(cur, pc, sc, std::false_type{}, bad);
      const PairRange range = deposit(Vs, pc);
      v_state = (__any(range.large()) ? FAR : 0) | (NPL == 3 && __any(range.small()) ? SMALL : 0);
      if (TEAM > 1 && lane == 0) flag_s[wave] = v_state;
    }
    barrier();                                           // V rows in LDS; everyone is done with the K rows
    if constexpr (TEAM > 1) {
      v_state = 0;
#pragma unroll
      for (int w = 0; w < TEAM; ++w) v_state |= flag_s[team * TEAM + w];
      v_state = __builtin_amdgcn_readfirstlane(v_state);
    }
    bad |= v_state & FAR;
    if (nxt.ok) fetch(K, Kp, nxt, pn);
    if (cur.ok && (bad || n >= later_from)) {
      later = true;
      if (n >= LATER_TILES) later_from = n < later_from ? n : later_from;
      else if (lane == 0) later_s[n >> 5] |= 1u << (n & 31);
    } else if (cur.ok) {
      l = fmaf(sum, unscale, l);
      small_v |= v_state & SMALL;
      bf16x8 p[3][2];                                    // planes of the weights: keys f * 16 .. as they stand in the registers
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        u32x4 w[3];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const Split2 t = split2(sc[8 * f + 2 * x], sc[8 * f + 2 * x + 1]);
          w[0][x] = t.h;
          w[1][x] = t.m;
          w[2][x] = t.l;
        }
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) p[pl][f] = __builtin_bit_cast(bf16x8, w[pl]);
      }
      const int trow = hf * 4 + ((lane & 15) >> 2);
      const uint32_t taddr = (uint32_t)(trow * ROWB + (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ row_swizzle32<D>(trow)) << 4) + (lane & 1) * 8);
      auto read_v = [&](bf16x8 (&dst)[NPL], auto tag) __attribute__((always_inline)) {   // 16 keys j % 2, channels (j / 2) * 32 ..
        constexpr int j = decltype(tag)::value, down = (j % 2) * 16 * ROWB, md = j / 2;
        unsigned char *at = Vs + flip<md * 64>(taddr), *at8 = Vs + flip<(md * 64) ^ 32>(taddr);   // (eight rows further down the swizzle differs in one bit)
#pragma unroll
        for (int pl = 0; pl < NPL; ++pl) {
          const f32_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((f32_lds_s16x4*)(at + pl * PLANEB + down));
          const f32_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((f32_lds_s16x4*)(at8 + pl * PLANEB + down + 8 * ROWB));
          dst[pl] = __builtin_bit_cast(bf16x8, (f32_s16x8)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        }
      };
      // The tile's twelve products for 32 channels are summed from zero and join o in one addition: twelve roundings a tile at the size of o made
      // the error against 64 bits of causal 12 heads x 2634 tokens 3.5e-7, where one makes it 1.1e-7 (float32 instructions 2.5e-7).  It costs 223 -> 236 us at
      // 12 heads x 4680 tokens: `part` takes the registers of a second set of V fragments, the other wavefront of the SIMD covers their loads.
      bf16x8 va[NPL];
      f32x16 part;
      each<2 * MD>([&](auto tag) __attribute__((always_inline)) {
        constexpr int j = decltype(tag)::value, f = j % 2, md = j / 2;
        read_v(va, tag);
        if constexpr (f == 0)
#pragma unroll
          for (int v = 0; v < 16; ++v) part[v] = 0.f;
        if constexpr (NPL == 3) part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[2], p[0][f], part, 0, 0, 0);
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[0], p[2][f], part, 0, 0, 0);
        if constexpr (NPL == 3) {
          part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[1], p[1][f], part, 0, 0, 0);
          part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[1], p[0][f], part, 0, 0, 0);
        }
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[0], p[1][f], part, 0, 0, 0);
        part = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[0], p[0][f], part, 0, 0, 0);
        if constexpr (f == 1)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[md][v] = fmaf(part[v], unscale, o[md][v]);
        __builtin_amdgcn_sched_barrier(0x7);             // (arithmetic may pass: the next weights' planes, addresses; causal 12 heads x 2634 tokens 110 -> 107 us)
      });
    }
    if (nxt.ok) deposit(Ks, pn);
    barrier();                                           // the next K rows in LDS; everyone is done with the V rows
    cur = nxt;
    pc = pn;
    nxt = nn;
  }
  if (small_v) {                                         // an output so small that 2^-134 of a value is more than 2^-25 of it: the whole row again, in float32
    const float bar = (l + __shfl_xor(l, 32, 64)) * 0x1p-109f;
    bool below = false;
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int v = 0; v < 16; ++v) below |= fabsf(o[md][v]) < bar;
    if (__any(below)) {
      later = again = true;
      m = -INFINITY;
      l = 0.f;
#pragma unroll
      for (int md = 0; md < MD; ++md)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[md][v] = 0.f;
    }
  }
  if (later) {
    // Tiles with scores or values that are not finite (the planes of an infinity give NaN where the product has a sign) or values that are large, and rows of small
    // operands: taken from memory in float32, at the end (a wavefront's sums do not ask for an order), since next to the planes in the loop above this would take
    // registers from it (12 heads x 4680 tokens 229 -> 255 us with no such tile).  No weight is more than one here, so that values up to the largest float32 can be summed.
    m += LAG;
    l *= exp2f(-LAG);
#pragma unroll
    for (int md = 0; md < MD; ++md)
#pragma unroll
      for (int v = 0; v < 16; ++v) o[md][v] *= exp2f(-LAG);
    const int tiles = (total + KS - 1 - team) / KS;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll 1
    for (int x = 0; x < tiles; ++x) {
      if (!again && (x < LATER_TILES ? !((__builtin_amdgcn_readfirstlane(later_s[x >> 5]) >> (x & 31)) & 1u) : x < later_from)) continue;
      Tile t = {1, team + x * KS, 0, 0, 0, 0};
      enter(t);
      settle(t);
      const int prow = row_of(t, block_of(t));
      f32x16 sc;
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[v] = 0.f;
      const T* krow = base_of(K, Kp, t) + (int64_t)(prow < 0 ? 0 : prow) * D + hf * 4;
      const T* qrow = Q + (qhead * a.N + (active ? row : row0)) * D + hf * 4;
#pragma unroll
      for (int c = 0; c < D; c += 8) {
        f32x4 kk = Four<T>::widen(Four<T>::load(krow + c)), qq = Four<T>::widen(Four<T>::load(qrow + c));
        if (prow < 0) kk = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!active) qq = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 4; ++e) sc = __builtin_amdgcn_mfma_f32_32x32x2f32(kk[e], qq[e], sc, 0, 0, 0);
      }
      l += weights(t, prow, sc, std::true_type{}, false);
      const T* vbase = base_of(V, Vp, t);
      if (a.causal && __any(prow >= (row0 + wr * 32 + 1) >> (t.h - 1))) {
        // A row must not see 0 * inf of a key that is hidden from it: hidden keys are left out one by one, on the vector unit.
#pragma unroll 1
        for (int kk = 0; kk < 32; ++kk) {
          const int vi = (kk >> 3) * 4 + (kk & 3), from = l32 + ((kk >> 2) & 1) * 32, pr = __shfl(prow, kk, 64);
          if (pr < 0) continue;                          // no such key
          float pv = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) pv = v == vi ? sc[v] : pv;
          pv = __shfl(pv, from, 64);
          const int64_t end = ((int64_t)pr + 1) << (t.h - 1);
          const bool hidden = (end < a.N ? end : a.N) - 1 > row;
#pragma unroll
          for (int md = 0; md < MD; ++md)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
              const f32x4 y = Four<T>::widen(Four<T>::load(vbase + (int64_t)pr * D + md * 32 + g * 8 + hf * 4));
#pragma unroll
              for (int e = 0; e < 4; ++e) o[md][g * 4 + e] = hidden ? o[md][g * 4 + e] : fmaf(pv, y[e], o[md][g * 4 + e]);
            }
        }
      } else {
        f32x16 part[MD];                                 // (from zero for every tile, as above)
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
          for (int v = 0; v < 16; ++v) part[md][v] = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {                   // the key of register v, and the one four rows further down
          const int pr = __shfl(prow, (v >> 2) * 8 + hf * 4 + (v & 3), 64);
          const T* vrow = vbase + (int64_t)(pr < 0 ? 0 : pr) * D + l32;
#pragma unroll
          for (int md = 0; md < MD; ++md)
            part[md] = __builtin_amdgcn_mfma_f32_32x32x2f32(pr < 0 ? 0.f : Elem<T>::to_f32(vrow[md * 32]), sc[v], part[md], 0, 0, 0);
        }
#pragma unroll
        for (int md = 0; md < MD; ++md)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[md][v] += part[md][v];
      }
    }
  }

  // merge the teams through LDS (fixed order) and write whole rows
  float* ms = reinterpret_cast<float*>(fsm);             // [KS][ROWS] maxima | [KS][ROWS] sums | [KS][ROWS][PITCH] outputs
  float* os = ms + 2 * KS * ROWS;
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
      *reinterpret_cast<f32x4*>(os + slot * PITCH + md * 32 + g * 8 + hf * 4) =
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
      const float w = KS == 1 ? 1.f : exp2f(ms[k * ROWS + r] - (mm == -INFINITY ? 0.f : mm));
      ll += w * ms[KS * ROWS + k * ROWS + r];
      acc += w * *reinterpret_cast<const f32x4*>(os + (k * ROWS + r) * PITCH + c);
    }
    const float inv = 1.f / ll;                          // no visible key at all: NaN
    Four<T>::store(O + (qhead * a.N + row0 + r) * D + c, acc * inv);
    if (lse && c == 0) {
      int e;                                             // the sum's power of two joins the reference: ln 2 in two parts, one rounding at the size of lse
      const float f = frexpf(ll, &e), w = mm + (float)e;
      lse[qhead * a.N + row0 + r] = fmaf(w, 0.693145751953125f, fmaf(w, 1.42860677e-6f, logf(f)));
    }
  }
}

template <typename T, int D, int TEAM>
static hipError_t launch_f32_t(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                               const uint8_t* M, const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  using S = F32Shape<T, D, TEAM>;
  F32Args a;
  a.N = pl.N; a.Hq = pl.Hq; a.Hkv = pl.Hkv; a.nq = pl.nq; a.nk = pl.nk; a.bq = pl.bq; a.bk = pl.bk;
  a.H = pl.H; a.causal = pl.causal;
  const double scale2 = (double)pl.scale * 1.4426950408889634074;
  a.scale_hi = (float)scale2;
  if ((double)a.scale_hi >= scale2) a.scale_hi = nextafterf(a.scale_hi, 0.f);   // both parts positive: times -inf they must not meet as NaN
  a.scale_lo = (float)(scale2 - (double)a.scale_hi);
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
      static_cast<const T*>(Vp), M, idx, cnt, static_cast<T*>(O), lse, a);
  return hipGetLastError();
}

template <typename T, int D>
static hipError_t launch_f32_d(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                               const uint8_t* M, const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  // The largest team that still fills the chip: fewer rows per team cost more reads (and conversions) of the same keys, fewer
  // workgroups leave compute units idle.  Measured with 12 heads at d = 128 (128-row blocks of the problem: us for team 1 / 2 / 4, pyramid and
  // block lists included): 48: 25 / 31 / 33, 96: 55 / 38 / 45, 192: 106 / 93 / 80, 252: 183 / 127 / 107, 288: 225 / 190 / 151, 432: 415 / 328 / 240,
  // 564: 673 / 515 / 417; d = 64: 48: 20 / 28 / 29, 96: 28 / 31 / 32, 192: 52 / 47 / 53, 252: 77 / 61 / 66, 288: 97 / 94 / 87, 432: 177 / 151 / 129,
  // 564: 284 / 242 / 232.  So teams of four from 150 such blocks on at d = 128 and from 256 on at d = 64, where a row of keys is converted in half the time.
  // Counted in parts of 64 rows, so that a part of 128 rows that is half empty counts as half: blocks of 192 rows, dense, teams of four / two: 16 heads x 926 tokens
  // 156 / 88, 8 x 2000 298 / 162, 28 x 926 at d = 64 113 / 69 (but 16 x 1024 153 / 163).
  const int64_t parts = (int64_t)pl.B * pl.Hq * pl.nq * ((pl.bq + 63) / 64);
  const int team = pl.bq > 64 && parts >= (D == 128 ? 300 : 512) ? 4 : (pl.bq > 32 && parts >= 192 ? 2 : 1);
  if (team == 4) return launch_f32_t<T, D, 4>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s);
  if (team == 2) return launch_f32_t<T, D, 2>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s);
  return launch_f32_t<T, D, 1>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s);
}

hipError_t launch_attn_f32(const Plan& pl, const void* Q, const void* K, const void* V, const void* Kp, const void* Vp,
                           const uint8_t* M, const uint16_t* idx, const int32_t* cnt, void* O, float* lse, hipStream_t s) {
  if (pl.dtype == PSA_F32)
    return pl.d == 64 ? launch_f32_d<float, 64>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s)
                      : launch_f32_d<float, 128>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s);
  return pl.d == 64 ? launch_f32_d<bf16_t, 64>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s)
                    : launch_f32_d<bf16_t, 128>(pl, Q, K, V, Kp, Vp, M, idx, cnt, O, lse, s);
}

}  // namespace psa
