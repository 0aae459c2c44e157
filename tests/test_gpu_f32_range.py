"""float32 attention and dense attention over the range of float32: values near its largest, operands and weights near its
smallest, and what one value that is not finite costs the rest of a call.

Tolerance: the fp32 bar of the parity tests, relative to the largest entry of the result (which is of the order of the scaled
operand), unless a test derives its own."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import psa_oracle as orc
from tests.psa_testlib import Buffers, from_dev, gpu_params, to_dev

pytestmark = pytest.mark.gpu

psa = pytest.importorskip("paper_2512_04025_amd")

TEAMS = [(289, 2, 64), (993, 12, 64), (993, 32, 128)]       # (tokens, heads, block): teams of one, two and four wavefronts


def _run(op, Q, K, V):
    """Every block kept at level 1: the sparse call and the dense one, which are the same attention."""
    import torch
    gp = gpu_params(op)
    buf = Buffers(gp)
    buf.M.fill_(1)
    dev = [to_dev(x, "f32") for x in (Q, K, V)]
    out = []
    for call in ("sparse", "dense"):
        buf.O.fill_(float("nan"))
        if call == "sparse":
            psa.psa_attention_fwd(gp, *dev, None, None, buf.M, buf.O, buf.scratch, lse=buf.lse)
        else:
            psa.psa_dense_ref(gp, *dev, buf.O, lse=buf.lse)
        torch.cuda.synchronize()
        out.append((from_dev(buf.O, "f32"), buf.lse.cpu().numpy()))
    return out


def _single_level(N, Hq, d, bq):
    return orc.Params(B=1, Hq=Hq, Hkv=1, N=N, d=d, bq=bq, bk=32, levels=1, dtype="f32", sq=8, sk=1)


def _scored(op, scores, seed):
    """Q and K whose scores are `scores` (natural, one per key) for every row, all in the first channel."""
    Q = np.zeros((1, op.Hq, op.N, op.d), np.float32)
    K = np.zeros((1, 1, op.N, op.d), np.float32)
    Q[..., 0] = 1
    K[0, 0, :, 0] = scores * np.sqrt(op.d)
    V = np.random.default_rng(seed).uniform(0.5, 1.0, K.shape)
    return Q, K, V


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Hq,bq", TEAMS)
def test_values_whose_weighted_sum_just_fits(N, Hq, bq, d):
    """128 keys of value 0, then keys of almost 2^8 times their weight and values whose plain sum is a little below 2^127:
    finite as long as no weight on the way is more than one."""
    op = _single_level(N, Hq, d, bq)
    Q, K, V = _scored(op, np.where(np.arange(N) < 128, 0.0, 7.9 * np.log(2)), 1)
    V = (V * 2.0 ** (127 - np.ceil(np.log2(N)))).astype(np.float32)
    V[:, :, :128] = 0
    want, lse = orc.dense_attention(*(x.astype(np.float64) for x in (Q, K, V)), op)
    for got, l in _run(op, Q, K, V):
        assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()
        assert np.abs(l - lse).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Hq,bq", TEAMS)
@pytest.mark.parametrize("which", ["V", "K", "Q"])
@pytest.mark.parametrize("power", [104, 112, 116, 120])
def test_small_operands(N, Hq, bq, d, which, power):
    """One operand scaled by 2^-power (keys and queries: the other one by 2^power, so that the scores stay)."""
    op = _single_level(N, Hq, d, bq)
    host = dict(zip("QKV", si.random_qkv(power, 1, Hq, 1, N, d, "f32")))
    host[which] = np.ldexp(host[which], -power)
    if which != "V":
        other = "K" if which == "Q" else "Q"
        host[other] = np.ldexp(host[other], power)
    want, lse = orc.dense_attention(*(host[x].astype(np.float64) for x in "QKV"), op)
    for got, l in _run(op, *(host[x] for x in "QKV")):
        assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()
        assert np.abs(l - lse).max() <= 1e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Hq,bq", TEAMS)
@pytest.mark.parametrize("log2_weight", [-112, -118, -130])
@pytest.mark.parametrize("log2_value", [80, 120])
def test_small_weights(N, Hq, bq, d, log2_weight, log2_value):
    """128 keys of weight 1 and value 0, all others of weight 2^-112 and less and values of 2^80 or 2^120.  A score of 130 is rounded
    to 2^-17 (twice: the product, the maximum taken off), which moves its weight by 1.1e-5; a weight of 2^-130 is a
    subnormal number of 20 bits (1e-6): 2e-5."""
    op = _single_level(N, Hq, d, bq)
    Q, K, V = _scored(op, np.where(np.arange(N) < 128, 0.0, log2_weight * np.log(2)), 2)
    V = (V * 2.0 ** log2_value).astype(np.float32)
    V[:, :, :128] = 0
    want, _ = orc.dense_attention(*(x.astype(np.float64) for x in (Q, K, V)), op)
    for got, _ in _run(op, Q, K, V):
        assert np.abs(got - want).max() <= 2e-5 * np.abs(want).max()


@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("what", ["key", "value", "small values"])
def test_single_values_do_not_slow_the_call(what, causal):
    """The first token's key or value is infinite in one channel and every row keeps its block: one tile of a row's list.  Or
    every seventh token has a value of 1e-36 among ordinary ones.  The two calls are timed in turn, the shortest of 20 each, so that
    what else the machine does drops out."""
    import torch
    op = orc.Params(B=1, Hq=12, Hkv=12, N=4680, d=128, bq=128, bk=64, levels=4, dtype="f32", causal=causal, sq=8, sk=8)
    gp = gpu_params(op)
    Q, K, V = (to_dev(x, "f32") for x in si.random_qkv(6, 1, 12, 12, op.N, 128, "f32"))
    rng = np.random.default_rng(7)
    vis = orc.block_visibility(op)
    M = rng.integers(1, 5, size=(1, 12, op.nq, op.nk)) * (rng.random((1, 12, op.nq, op.nk)) < 0.4)
    M[..., 0] = 1
    M = torch.from_numpy(np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)).cuda()
    problems = []
    for bad in (False, True):
        k, v = K.clone(), V.clone()
        if bad and what == "small values":
            v[:, :, ::7, 3] = 1e-36
        elif bad:
            (k if what == "key" else v)[:, :, 0, 0] = float("inf")
        buf = Buffers(gp)
        psa.psa_build_pyramid(gp, k, v, buf.Kpyr, buf.Vpyr)
        problems.append((k, v, buf))
    best = [float("inf")] * 2
    for _ in range(20):
        for x, (k, v, buf) in enumerate(problems):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            psa.psa_attention_fwd(gp, Q, k, v, buf.Kpyr, buf.Vpyr, M, buf.O, buf.scratch)
            end.record()
            torch.cuda.synchronize()
            best[x] = min(best[x], start.elapsed_time(end))
    assert best[1] <= 1.5 * best[0]


def test_infinities_far_down_a_row():
    """A row of 2195 tiles of 32 keys: infinite values in the first tile, in the 2063rd and in the last.  The channels without one stay
    what they are, here of three rows in torch at 64 bits."""
    import torch
    op = orc.Params(B=1, Hq=1, Hkv=1, N=70219, d=128, bq=128, bk=64, levels=1, dtype="f32", sq=8, sk=8)
    Q, K, V = (to_dev(x, "f32") for x in si.random_qkv(8, 1, 1, 1, op.N, 128, "f32"))
    for token, channel in ((3, 5), (66007, 6), (70218, 7)):
        V[:, :, token, channel] = float("inf")
    O = torch.full_like(Q, float("nan"))
    psa.psa_dense_ref(gpu_params(op), Q, K, V, O)
    torch.cuda.synchronize()
    assert bool((O[..., 5:8] == float("inf")).all()) and bool(torch.isfinite(O[..., 8:]).all())
    rows = torch.tensor([0, 35000, 70218], device="cuda")
    P = torch.softmax(Q[0, 0, rows].double() @ K[0, 0].double().T.contiguous() / np.sqrt(128), 1)
    want = P @ V[0, 0, :, 8:].double()
    assert float((O[0, 0, rows, 8:].double() - want).abs().max()) <= 1e-5
