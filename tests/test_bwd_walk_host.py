"""The work that the backward kernels' workgroups take, worked out by the kernel's own arithmetic (csrc/bwd_walk.h) compiled for the host:
every row of a query block once, nothing outside it and no chunk without a row, also where the last block is short."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_04025_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "bwd_walk.h"
using namespace psa;
int main(int argc, char** argv) {
  if (argc == 4) {
    const DkvGroup g = dkv_group(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]));
    printf("group %d %d\ngroup %d %d\n", g.keys, g.lg_G, g.lg_pieces, g.ng);
    return 0;
  }
  if (argc == 5) {
    printf("first 0 %d\n", one_launch(atoll(argv[1]) * atoll(argv[2]), atoll(argv[3]) * atoll(argv[4])));
    return 0;
  }
  if (argc == 3 && atoi(argv[1]) < 0) {
    const int heads = -atoi(argv[1]), per_head = atoi(argv[2]);
    for (int xcd = 0; xcd < 8; ++xcd)
      for (int slot = 0; slot < dq_slots(heads, per_head); ++slot) {
        int head = 0, item = 0;
        if (dq_item(heads, per_head, dq_runs(per_head), xcd, slot, head, item)) printf("x%d %d %d\n", xcd, head, item);
      }
    return 0;
  }
  const int N = atoi(argv[1]), bq = atoi(argv[2]), nq = (N + bq - 1) / bq, cpe = (bq + 31) / 32;
  const int total = dkv_chunks(N, bq, nq, nq, nq - 1), first = dkv_chunks(N, bq, nq, nq / 2, nq / 2 - 1);
  printf("first 0 %d\n", first);
  for (int blk = 0; blk < nq; ++blk)
    for (int sub = 0; sub < cpe * 32; sub += DKV_PART) {
      if (blk * cpe + sub / 32 >= total) continue;
      if (sub % 32 == 0) printf("chunk %d %d\n", blk, sub);
      const DkvPart p = dkv_part(N, bq, blk, sub);
      for (int r = 0; r < 64; ++r)
        if (dkv_reads_stat(p, r)) printf("stat %d %d\n", blk, p.row + r);
      for (int r = 0; r < DKV_PART; ++r) printf("row %d %d\n", blk, dkv_source_row(p, r));
    }
}
"""


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    folder = tmp_path_factory.mktemp("walk")
    (folder / "walk.cpp").write_text(PROGRAM)
    exe = str(folder / "walk")
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(folder / "walk.cpp"), "-o", exe], check=True)

    def run(*args):
        lines = subprocess.run([exe, *map(str, args)], check=True, capture_output=True, text=True).stdout.split("\n")
        out = {f"x{x}": [] for x in range(8)} | {"stat": [], "row": [], "chunk": [], "first": [], "group": []}
        for line in filter(None, lines):
            kind, blk, row = line.split()
            out[kind].append((int(blk), int(row)))
        return out
    return run


@pytest.mark.parametrize("N,bq", [(1, 128), (8, 8), (200, 128), (256, 128), (257, 128), (283, 24), (300, 32), (461, 96), (523, 40), (1000, 128)])
def test_walk_stays_inside_the_query_blocks(walk, N, bq):
    got = walk(N, bq)
    assert got["stat"] == [(row // bq, row) for row in range(N)]       # lse and D: every row once, none past the end
    assert all(0 <= row < N and row // bq == blk for blk, row in got["row"])
    assert set(got["row"]) == set(got["stat"])
    assert all(blk * bq + sub < N for blk, sub in got["chunk"])        # every chunk has a row
    assert got["first"] == [(0, -(-N // bq) // 2 * -(-bq // 32))]      # (blocks before the last one have all of theirs)


@pytest.mark.parametrize("small_keys", [32, 64])
@pytest.mark.parametrize("nk", [1, 2, 31, 32, 33, 500])
@pytest.mark.parametrize("lg_th", range(8))
def test_groups_take_every_key_once(walk, lg_th, nk, small_keys):
    (keys, lg_G), (lg_pieces, ng) = walk(lg_th, nk, small_keys)["group"]
    th, taken = 1 << lg_th, []
    assert keys == (64 if th >= 64 else small_keys) and 1 << lg_G <= 32
    for bx in range(ng):                                              # as the kernel reads it
        j0, koff = (bx >> lg_pieces) << lg_G, (bx & ((1 << lg_pieces) - 1)) * keys
        taken += [j0 * th + koff + k for k in range(min(keys, (th << lg_G) - koff)) if j0 + (koff + k) // th < nk]
    assert taken == list(range(nk * th))


@pytest.mark.parametrize("heads,per_head", [(1, 1), (40, 2), (12, 9), (3, 4), (16, 31), (2, 32), (5, 33), (12, 256), (7, 257)])
def test_query_blocks_are_dealt_once_and_evenly(walk, heads, per_head):
    got = walk(-heads, per_head)
    shares = [got[f"x{x}"] for x in range(8)]
    assert sorted(sum(shares, [])) == [(h, i) for h in range(heads) for i in range(per_head)]
    most = -(-heads * per_head // 8) if per_head < 32 else heads * -(-per_head // 8)
    assert max(map(len, shares)) <= most                              # from 32 blocks on: at most a quarter more than an even share


@pytest.mark.parametrize("first,second,fits", [((1, 1), (0, 0), 1), ((4096, 4095), (1, 4095), 1), ((4096, 4095), (1, 4096), 0), ((1024, 12000), (1024, 6000), 0),
                                               ((65536, 65536), (0, 0), 0)])
def test_two_launches_go_out_as_one_below_the_limit_of_a_launch(walk, first, second, fits):
    """Workgroups of 256 threads: 2^24 of them are 2^32 threads, which no launch has."""
    assert walk(*first, *second)["first"] == [(0, fits)]
