"""The fp32 matrix-core kernels at the sizes where their tiles and teams end, against the oracle.

Tolerance: fp32 products and sums of at most a few thousand terms with accurate exp: the fp32 bar of the
parity tests (1e-5); bfloat16 inputs through the same arithmetic are rounded once on the way out (2^-9 of
values below 4)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import psa_oracle as orc
from tests.psa_testlib import Buffers, from_dev, gpu_params, rel_l2, to_dev

pytestmark = pytest.mark.gpu

psa = pytest.importorskip("paper_2512_04025_amd")


def _problem(dtype, B, Hq, Hkv, N, d, bq, bk, levels, causal, seed=3):
    op = orc.Params(B=B, Hq=Hq, Hkv=Hkv, N=N, d=d, bq=bq, bk=bk, levels=levels, dtype=dtype, causal=causal, sq=8, sk=1)
    host = si.random_qkv(seed, B, Hq, Hkv, N, d, dtype)
    rng = np.random.default_rng(seed + 1)
    vis = orc.block_visibility(op)
    M = rng.integers(0, levels + 1, size=(B, Hq, op.nq, op.nk)).astype(np.uint8)
    M[..., 0] = 1
    M = np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)
    return op, gpu_params(op), host, M


# (dtype, B, Hq, Hkv, N, d, bq, bk, levels, causal): teams of 1, 2 and 4; ragged tails; blocks of one pooled key, of more
# keys than a tile; query blocks that are no multiple of a team's rows
SHAPES = [
    ("f32", 1, 2, 1, 333, 64, 64, 64, 4, False),
    ("f32", 1, 2, 2, 40, 128, 32, 8, 4, False),
    ("f32", 2, 2, 1, 515, 128, 24, 16, 5, True),
    ("f32", 1, 12, 12, 1000, 64, 128, 64, 3, False),
    ("f32", 1, 12, 4, 1021, 128, 64, 32, 3, True),
    ("f32", 2, 16, 4, 1001, 64, 128, 256, 4, True),
    ("f32", 1, 32, 8, 1023, 128, 128, 64, 4, False),
    ("bf16", 1, 2, 2, 700, 128, 96, 64, 3, True),
    ("bf16", 1, 32, 8, 1530, 64, 192, 32, 2, False),
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_attention_and_dense_at_the_edges(shape):
    import torch
    op, gp, host, M = _problem(*shape)
    Q64, K64, V64 = (si.to_f64(x, op.dtype) for x in host)
    Qd, Kd, Vd = (to_dev(x, op.dtype) for x in host)
    buf = Buffers(gp)
    tol = 1e-5 if op.dtype == "f32" else 1e-2
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    buf.O.fill_(float("nan"))
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, torch.from_numpy(M).cuda(), buf.O, buf.scratch, lse=buf.lse)
    torch.cuda.synchronize()
    O, lse = orc.psa_attention(Q64, orc.build_pyramid(K64, op), orc.build_pyramid(V64, op), M, op)
    assert np.abs(from_dev(buf.O, op.dtype) - O).max() <= tol
    assert np.abs(buf.lse.cpu().numpy() - lse).max() <= 1e-4
    buf.O.fill_(float("nan"))
    psa.psa_dense_ref(gp, Qd, Kd, Vd, buf.O, lse=buf.lse)
    torch.cuda.synchronize()
    O, lse = orc.dense_attention(Q64, K64, V64, op)
    assert np.abs(from_dev(buf.O, op.dtype) - O).max() <= tol
    assert np.abs(buf.lse.cpu().numpy() - lse).max() <= 1e-4


BWD_SHAPES = [s for s in SHAPES if s[0] == "f32" and s[7] <= 128] + [
    ("f32", 1, 4, 2, 2070, 64, 8, 8, 4, True),            # more column entries than are tested at a time; blocks of one pooled key
    ("bf16", 1, 2, 2, 300, 128, 64, 4, 3, False),         # key blocks smaller than the bfloat16 kernels take
    ("f32", 1, 32, 8, 1023, 64, 128, 64, 4, False),       # the remaining teams of the dQ kernel: d = 64 in teams of four,
    ("bf16", 1, 12, 6, 1000, 64, 64, 4, 3, True),         # bfloat16 in teams of two ...
    ("bf16", 1, 12, 6, 1000, 128, 64, 4, 2, False),
    ("bf16", 1, 32, 4, 1000, 64, 128, 4, 2, False),       # ... and of four
    ("bf16", 1, 32, 4, 1000, 128, 128, 4, 3, True),
]


@pytest.mark.parametrize("shape", BWD_SHAPES, ids=lambda s: "-".join(map(str, s)))
def test_backward_at_the_edges(shape):
    """Gradients against the oracle: 1e-5 of the largest entry for float32, one bfloat16 rounding otherwise (O, which
    enters through dO . O, is rounded too: the bar of the backward tests)."""
    import torch
    op, gp, host, M = _problem(*shape)
    dO = si.random_qkv(9, op.B, op.Hq, op.Hq, op.N, op.d, op.dtype)[0]
    Q64, K64, V64, dO64 = (si.to_f64(x, op.dtype) for x in (*host, dO))
    Qd, Kd, Vd, dOd = (to_dev(x, op.dtype) for x in (*host, dO))
    buf = Buffers(gp)
    Md = torch.from_numpy(M).cuda()
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.scratch, lse=buf.lse)
    grads = [torch.full_like(x, float("nan")) for x in (Qd, Kd, Vd)]
    scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
    psa.psa_attention_bwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.lse, dOd, *grads, scratch)
    torch.cuda.synchronize()
    ref = orc.psa_attention_backward(Q64, orc.build_pyramid(K64, op), orc.build_pyramid(V64, op), M, dO64, op)
    for name, got, want in zip(("dQ", "dK", "dV"), grads, ref):
        bar = (1e-5 if op.dtype == "f32" else 2e-2) * max(1.0, float(np.abs(want).max()))
        assert np.abs(from_dev(got, op.dtype) - want).max() <= bar, name


@pytest.mark.parametrize("N,Hq,bq", [(333, 2, 64), (1000, 12, 64), (1000, 32, 128)])
def test_values_hidden_by_the_causal_mask_may_be_infinite(N, Hq, bq):
    """The last token's value is infinite: no row before it sees that token, so no row before it changes."""
    import torch
    op, gp, host, M = _problem("f32", 1, Hq, 1, N, 64, bq, 64, 3, True)
    Qd, Kd, Vd = (to_dev(x, "f32") for x in host)
    outs = []
    for bad in (None, float("inf")):
        V = Vd.clone()
        if bad is not None:
            V[:, :, -1] = bad
        buf = Buffers(gp)
        psa.psa_build_pyramid(gp, Kd, V, buf.Kpyr, buf.Vpyr)
        psa.psa_attention_fwd(gp, Qd, Kd, V, buf.Kpyr, buf.Vpyr, torch.from_numpy(M).cuda(), buf.O, buf.scratch)
        torch.cuda.synchronize()
        outs.append(from_dev(buf.O, "f32"))
    assert np.abs(outs[1][:, :, :-1] - outs[0][:, :, :-1]).max() <= 1e-5
    assert np.all(np.isinf(outs[1][:, :, -1]) | np.isnan(outs[1][:, :, -1]))


@pytest.mark.parametrize("N,Hq,bq", [(97, 2, 64), (993, 12, 64), (993, 32, 128)])
def test_a_key_that_is_not_a_number_reaches_every_row_that_keeps_it(N, Hq, bq):
    """The last token's key is NaN, alone in the last key block and in the last tile of a row's list, at sizes that
    deal out the wavefronts in teams of one, two and four: rows that keep the block are NaN, the others untouched."""
    import torch
    op = orc.Params(B=1, Hq=Hq, Hkv=1, N=N, d=64, bq=bq, bk=32, levels=1, dtype="f32", sq=8, sk=1)
    gp = gpu_params(op)
    Qd, Kd, Vd = (to_dev(x, "f32") for x in si.random_qkv(4, 1, Hq, 1, N, 64, "f32"))
    M = np.zeros((1, Hq, op.nq, op.nk), np.uint8)
    M[..., 0] = 1
    M[:, :, ::2, -1] = 1
    keeps = np.repeat(np.arange(op.nq) % 2 == 0, bq)[:N]
    outs = []
    for key in (None, float("nan")):
        K = Kd.clone()
        if key is not None:
            K[:, :, -1] = key
        buf = Buffers(gp)
        psa.psa_attention_fwd(gp, Qd, K, Vd, None, None, torch.from_numpy(M).cuda(), buf.O, buf.scratch, lse=buf.lse)
        torch.cuda.synchronize()
        outs.append((from_dev(buf.O, "f32"), buf.lse.cpu().numpy()))
    for clean, bad in zip(*outs):
        assert np.all(np.isnan(bad[:, :, keeps]))
        assert np.array_equal(bad[:, :, ~keeps], clean[:, :, ~keeps])
    psa.psa_dense_ref(gp, Qd, K, Vd, buf.O, lse=buf.lse)
    torch.cuda.synchronize()
    assert bool(torch.isnan(buf.O).all()) and bool(torch.isnan(buf.lse).all())


@pytest.mark.parametrize("d", [64, 128])
def test_gradients_where_the_channels_cancel(d):
    """Values of +16 and -16 in the two halves of the channels under a constant output gradient: dP is what is left of sums
    that reach 16 d / 2.  One chain of d roundings has an rms error of about 0.45 * 2^-24 * 8 d * sqrt(d / 3), relative to
    dP - dO . O of about 1.4 sqrt(d): 1.1e-5 at d = 128, proportional to d; in c interleaved chains 1 / c of it, next to
    the 3e-6 that the rounding of O leaves in dO . O.  The bar lies between two chains and one."""
    import torch
    op = orc.Params(B=1, Hq=2, Hkv=2, N=160, d=d, bq=64, bk=64, levels=1, dtype="f32", sq=8, sk=8)
    gp = gpu_params(op)
    Q, K, V = si.random_qkv(3, 1, 2, 2, op.N, d, "f32")
    V = (V + np.where(np.arange(d) < d // 2, 16, -16)).astype(np.float32)
    dO = si.random_qkv(4, 1, 2, 2, op.N, d, "f32")[0] + np.float32(1)
    M = np.ones((1, 2, op.nq, op.nk), np.uint8)
    Qd, Kd, Vd, dOd = (to_dev(x, "f32") for x in (Q, K, V, dO))
    buf = Buffers(gp)
    Md = torch.from_numpy(M).cuda()
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, None, None, Md, buf.O, buf.scratch, lse=buf.lse)
    grads = [torch.empty_like(x) for x in (Qd, Kd, Vd)]
    scratch = torch.empty(psa.psa_query_bwd_sizes(gp), dtype=torch.uint8, device="cuda")
    psa.psa_attention_bwd(gp, Qd, Kd, Vd, None, None, Md, buf.O, buf.lse, dOd, *grads, scratch)
    torch.cuda.synchronize()
    Q64, K64, V64, dO64 = (si.to_f64(x, "f32") for x in (Q, K, V, dO))
    ref = orc.psa_attention_backward(Q64, orc.build_pyramid(K64, op), orc.build_pyramid(V64, op), M, dO64, op)
    for name, got, want in zip(("dQ", "dK"), grads, ref):
        assert rel_l2(from_dev(got, "f32"), want) <= 9e-6 * d / 128, name


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,Hq,bq", [(97, 2, 64), (993, 12, 64), (993, 32, 128)])
def test_infinite_keys_and_values_act_as_in_float32(N, Hq, bq, d):
    """Products of the bfloat16 planes of an infinity would be NaN; teams of one, two and four.  The last key has an infinite
    channel: rows whose query is negative there do not see it, the others are NaN.  One value is infinite, one is finite but
    rounds to infinity in bfloat16.  Bars: the fp32 bar of the parity tests, relative where values are of the order of 1e36."""
    import torch
    op = orc.Params(B=1, Hq=Hq, Hkv=1, N=N, d=d, bq=bq, bk=32, levels=1, dtype="f32", sq=8, sk=1)
    gp = gpu_params(op)
    Q, K, V = si.random_qkv(6, 1, Hq, 1, N, d, "f32")
    K[:, :, -1, 0] = np.inf
    V[:, :, 3, 5] = -np.inf
    V[:, :, 4, 6] = 3.4e38
    buf = Buffers(gp)
    buf.M.fill_(1)
    psa.psa_attention_fwd(gp, *(to_dev(x, "f32") for x in (Q, K, V)), None, None, buf.M, buf.O, buf.scratch, lse=buf.lse)
    torch.cuda.synchronize()
    got, lse = from_dev(buf.O, "f32"), buf.lse.cpu().numpy()
    sees = Q[..., 0] < 0
    assert np.all(np.isnan(got[~sees]))
    x = Q.astype(np.float64) @ K[:, :, :-1].astype(np.float64).swapaxes(2, 3) / np.sqrt(d)
    top = x.max(-1, keepdims=True)
    P = np.exp(x - top)
    total = P.sum(-1, keepdims=True)
    with np.errstate(invalid="ignore"):
        want = (P / total) @ V[:, :, :-1].astype(np.float64)
    assert np.all(got[sees][:, 5] == -np.inf)
    assert np.allclose(got[sees][:, 6], want[sees][:, 6], rtol=1e-5, atol=0)
    rest = [c for c in range(d) if c not in (5, 6)]
    assert np.abs(got[sees][:, rest] - want[sees][:, rest]).max() <= 1e-5
    assert np.abs(lse[sees] - (top + np.log(total))[..., 0][sees]).max() <= 1e-4


@pytest.mark.parametrize("shape", [("f32", 1, 8, 2, 611, 128, 128, 64, 3, True), ("f32", 1, 8, 2, 611, 64, 128, 64, 3, False), ("f32", 1, 8, 1, 1201, 64, 128, 64, 4, False), ("f32", 1, 2, 2, 1000, 64, 64, 64, 4, False)],
                         ids=lambda s: "-".join(map(str, s)))
def test_gradients_of_split_columns(shape):
    """Short launches whose columns of the level map are shared by two, four, eight and two workgroups (same bars)."""
    test_backward_at_the_edges(shape)


@pytest.mark.parametrize("Hq,N,d", [(16, 926, 128), (28, 926, 64)])
def test_half_empty_parts_of_a_query_block_do_not_count_as_work(Hq, N, d):
    """Blocks of 192 rows: with teams of four wavefronts every second part of 128 rows is half empty, and these calls, too short to fill
    the chip with them, took 1.7 times as long as in blocks of 128 rows; with teams of two as long."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V, O = (torch.randn((1, Hq, N, d), generator=gen, device="cuda") for _ in range(4))

    def best(bq):
        gp = psa.make_params(1, Hq, Hq, N, d, bq, 64, 1, dtype=psa.PSA_F32, sq=8, sk=8)
        times = []
        for _ in range(8):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(10):
                psa.psa_dense_ref(gp, Q, K, V, O)
            end.record()
            torch.cuda.synchronize()
            times.append(start.elapsed_time(end))
        return min(times)

    assert best(192) <= 1.3 * best(128)
