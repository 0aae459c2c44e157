// Which rows the dK, dV walk over the query blocks touches (attn_bwd_mfma.hip).  Plain arithmetic, the same on host and device, so
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

}  // namespace psa
#endif
