// Which work a workgroup of the backward kernels takes and which rows the dK, dV walk over the query blocks touches (attn_bwd_mfma.hip), and what fits one launch.  Plain arithmetic, the same on host and device, so
// that its bounds can be checked without a GPU (tests/test_bwd_walk_host.py).
#ifndef PSA_BWD_WALK_H
#define PSA_BWD_WALK_H

namespace psa {

constexpr int DKV_PART = 16;       // rows of a stage that one wavefront fetches

// Rows row .. row + DKV_PART - 1 of the sequence, of which the first `valid` are of the query block (none if <= 0: a 32-row chunk
// is two parts).
struct DkvPart { int row, valid; };
constexpr DkvPart dkv_part(int N, int bq, int blk, int sub) {
  const int left = N - blk * bq, rows = left < bq ? left : bq;
  return DkvPart{blk * bq + sub, rows - sub};
}
// The row whose Q and dO stand for row r of the part: past the block's end its last row
constexpr int dkv_source_row(DkvPart p, int r) { return p.row + (r < p.valid ? r : p.valid - 1); }
// Whether lse and D are read for row r of the part.  They are arrays of exactly N entries a head, so nothing past the end may be.
constexpr bool dkv_reads_stat(DkvPart p, int r) { return r < DKV_PART && r < p.valid; }

// 32-row chunks in the walk over `kept` query blocks, given in order, of which the last one is `last`: the short block at the sequence's end has
// no more of them than it has rows for.
constexpr int dkv_chunks(int N, int bq, int nq, int kept, int last) {
  const int cpe = (bq + 31) / 32, rows = N - (nq - 1) * bq;
  return kept * cpe - (kept > 0 && last == nq - 1 ? cpe - (rows + 31) / 32 : 0);
}

// Work order of dQ (and of the forward, which takes runs for other problems too), not causal: workgroup `slot` of XCD `xcd` takes query block `item` of head `head`, or nothing.  All XCDs are on one head at a time, a
// contiguous run of its blocks each; with `runs` each XCD takes a contiguous run of all heads' blocks (see launch_bwd_mfma_t).
constexpr bool dq_runs(int per_head) { return per_head < 32; }
constexpr int dq_slots(int heads, int per_head) { return dq_runs(per_head) ? (heads * per_head + 7) / 8 : heads * ((per_head + 7) / 8); }
constexpr bool dq_item(int heads, int per_head, bool runs, int xcd, int slot, int& head, int& item) {
  if (runs) {
    const int at = xcd * ((heads * per_head + 7) >> 3) + slot;
    head = at / per_head;
    item = at % per_head;
    return at < heads * per_head;
  }
  const int run = (per_head + 7) >> 3;
  head = slot / run;
  item = xcd * run + slot % run;
  return item < per_head;
}

// Whether the work of two launches, in workgroups of 256 threads each, may go out as one: a launch has fewer than 2^32 threads
constexpr bool one_launch(long long first, long long second) { return (first + second) * 256 < (1ll << 32); }

// log2 of the most key blocks of a workgroup: one bit each
constexpr int DKV_LG_MAXG = 5;
// pooled keys of a workgroup, log2 of the key blocks they belong to and of the workgroups that share a block, workgroups per head.
// (All but the last are powers of two, and shifts: 19 integer divisions stood before a workgroup's first load, which short calls wait for.
// Whole call, us, one level: 2 heads x 161 tokens 25.7 -> 25.1, in 32-token key blocks 24.8 -> 24.2, 12 x 300 30.8 -> 30.3, 40 x 161 31.5 -> 30.8.)
struct DkvGroup { int keys, lg_G, lg_pieces, ng; };
constexpr DkvGroup dkv_group(int lg_th, int nk, int small_keys) {
  const int lg_keys = lg_th >= 6 || small_keys == 64 ? 6 : 5, packed = lg_keys - lg_th;
  DkvGroup r{};
  r.keys = 1 << lg_keys;
  r.lg_G = packed < 0 ? 0 : (packed > DKV_LG_MAXG ? DKV_LG_MAXG : packed);
  r.lg_pieces = packed < 0 ? -packed : 0;
  r.ng = ((nk + (1 << r.lg_G) - 1) >> r.lg_G) << r.lg_pieces;
  return r;
}

}  // namespace psa
#endif
