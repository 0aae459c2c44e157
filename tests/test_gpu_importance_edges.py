"""Block importance (bfloat16, 8 x 8 representatives) where its tiles and slices end: representatives without a token past a ragged
query or key block, the causal diagonal, one tile and many, both pooling rules and both kinds of representatives.

Tolerance: the bar of the other importance tests (fast exp2 of bfloat16 dots, 1e-3 relative)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import psa_oracle as orc
from tests.psa_testlib import Buffers, gpu_params, to_dev

pytestmark = pytest.mark.gpu

psa = pytest.importorskip("paper_2512_04025_amd")


@pytest.mark.parametrize("Hq,Hkv,N,d,bq,bk,causal,rep,est", [
    (1, 1, 50, 128, 32, 32, False, "pooled", "max"),      # one tile; representatives without a token on both sides
    (2, 2, 1003, 128, 32, 32, False, "pooled", "max"),    # the last row group holds rows without a token: four tiles
    (2, 2, 1003, 64, 32, 32, False, "pooled", "mean"),
    (2, 1, 4700, 128, 128, 64, True, "pooled", "max"),    # ten tiles, diagonal tiles in every row group, slices that end early
    (2, 1, 4700, 64, 64, 64, True, "pooled", "max"),
    (2, 1, 2900, 128, 64, 64, True, "pooled", "mean"),
    (1, 1, 1500, 128, 64, 32, True, "strided", "max"),
    (1, 1, 777, 64, 64, 32, False, "strided", "mean"),
    (24, 24, 1540, 64, 32, 32, False, "pooled", "max"),   # slices of two tiles
])
def test_importance_edges(Hq, Hkv, N, d, bq, bk, causal, rep, est):
    import torch
    op = orc.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, d=d, bq=bq, bk=bk, levels=2, dtype="bf16", causal=causal, sq=8, sk=8,
                    rep_mode=rep, est_pool=est, alloc_mode="budget", budget=0.3)
    gp = gpu_params(op)
    host = si.random_qkv(11, 1, Hq, Hkv, N, d, "bf16")
    Qd, Kd, Vd = (to_dev(x, "bf16") for x in host)
    buf = Buffers(gp)
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    psa.psa_allocate_levels(gp, Qd, Kd, buf.Kpyr, buf.M, buf.scratch, scores_out=buf.S)
    torch.cuda.synchronize()
    Q64, K64 = (si.to_f64(x, "bf16") for x in host[:2])
    np.testing.assert_allclose(buf.S.cpu().numpy().astype(np.float64), orc.importance(Q64, K64, op), rtol=1e-3, atol=1e-9)


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("est", ["max", "mean"])
def test_logits_below_the_range_of_float32(est, causal):
    """Every second tile of 64 representative keys gives some rows logits that overflow to -inf, next to rows of the same wavefront
    for which they are finite: such a key has weight 0, and what the row sees later (or has seen) counts as ever.  Two tiles a slice."""
    import torch
    N, d, bq, bk = 8192, 64, 128, 64
    op = orc.Params(B=1, Hq=1, Hkv=1, N=N, d=d, bq=bq, bk=bk, levels=2, dtype="bf16", causal=causal, sq=8, sk=8, est_pool=est,
                    rep_mode="pooled", alloc_mode="budget", budget=0.3)
    gp = gpu_params(op)
    rng = np.random.default_rng(3)
    token = np.arange(N)
    q = rng.uniform(0.5, 1.5, (N, d)) * np.where(token // bq % 4 == 0, 1e30, 1e-10)[:, None]
    k = np.where((token // (8 * bk) % 2 == 0)[:, None], -1e10, 1e-30 * rng.standard_normal((N, d)))
    if causal:
        k[:bk] = 1e-30                             # (every row sees a key with a finite logit)
    def bits(x):
        return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)[None, None]
    host = bits(q), bits(k)
    Qd, Kd = (to_dev(x, "bf16") for x in host)
    buf = Buffers(gp)
    psa.psa_build_pyramid(gp, Kd, Kd, buf.Kpyr, buf.Vpyr)
    psa.psa_allocate_levels(gp, Qd, Kd, buf.Kpyr, buf.M, buf.scratch, scores_out=buf.S)
    torch.cuda.synchronize()
    Q64, K64 = (si.to_f64(x, "bf16") for x in host)
    np.testing.assert_allclose(buf.S.cpu().numpy().astype(np.float64), orc.importance(Q64, K64, op), rtol=1e-3, atol=1e-9)


def test_other_numbers_of_representatives_in_bfloat16_and_float32():
    """Four representatives a key block: the general kernel for both types, whose multiply-adds are the same (float32 reads twice the
    bytes).  Timed in turn, the shortest of ten each; widening the query rows' channels for every multiply-add takes bfloat16 1.65
    times as long as float32, widening them once 1.23."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(1)
    problems = []
    for dtype in ("bf16", "f32"):
        op = orc.Params(B=2, Hq=8, Hkv=8, N=11049, d=128, bq=32, bk=32, levels=1, dtype=dtype, causal=True, sq=8, sk=4)
        Q, K = (torch.randn((2, 8, op.N, 128), generator=gen, device="cuda").to(torch.bfloat16 if dtype == "bf16" else torch.float32) for _ in range(2))
        gp = gpu_params(op)
        problems.append((gp, Q, K, Buffers(gp)))
    best = [float("inf")] * 2
    for _ in range(10):
        for x, (gp, Q, K, buf) in enumerate(problems):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            psa.psa_allocate_levels(gp, Q, K, buf.Kpyr, buf.M, buf.scratch)
            end.record()
            torch.cuda.synchronize()
            best[x] = min(best[x], start.elapsed_time(end))
    assert best[0] <= 1.45 * best[1]
