"""Rows of up to 128 key blocks, whose lists the kernels make themselves, and the first length beyond them, whose lists (and,
with 128-row query blocks, tile descriptors) are made by a launch of their own: forward and gradients against the oracle.

Tolerances: the bars of the parity and backward tests (bfloat16: P rounded to 8 bits, results once more; float32: 1e-5)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import psa_oracle as orc
from tests.psa_testlib import Buffers, from_dev, gpu_params, rel_l2, to_dev

pytestmark = pytest.mark.gpu

psa = pytest.importorskip("paper_2512_04025_amd")


@pytest.mark.parametrize("N", [1021, 1030])
@pytest.mark.parametrize("dtype,d,bq,levels,causal", [("bf16", 128, 128, 2, False), ("bf16", 64, 128, 1, True), ("bf16", 128, 32, 2, False), ("bf16", 128, 64, 2, True),
                                                      ("bf16", 64, 32, 3, True), ("f32", 64, 64, 3, True), ("f32", 128, 128, 2, False), ("bf16", 64, 96, 2, False),
                                                      ("bf16", 128, 256, 2, False), ("bf16", 128, 256, 2, True), ("bf16", 64, 256, 1, True)])   # two workgroups to a row's list and descriptors
def test_short_rows(N, dtype, d, bq, levels, causal):
    import torch
    op = orc.Params(B=1, Hq=2, Hkv=1, N=N, d=d, bq=bq, bk=8, levels=levels, dtype=dtype, causal=causal, sq=8, sk=1)
    assert op.nk == (128 if N == 1021 else 129)
    gp = gpu_params(op)
    host = si.random_qkv(N + d, 1, 2, 1, N, d, dtype)
    dO = si.random_qkv(9, 1, 2, 2, N, d, dtype)[0]
    rng = np.random.default_rng(N + bq)
    vis = orc.block_visibility(op)
    M = rng.integers(0, levels + 1, size=(1, 2, op.nq, op.nk))
    M[:, 0, 0] = 1                                       # a full row
    M[:, 1, -1] = 0                                      # a row of its first and last block
    M[:, 1, -1, [0, -1]] = levels
    M[..., 0] = np.maximum(M[..., 0], 1)
    M = np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)
    Qd, Kd, Vd, dOd = (to_dev(x, dtype) for x in (*host, dO))
    Q64, K64, V64, dO64 = (si.to_f64(x, dtype) for x in (*host, dO))
    buf, Md = Buffers(gp), torch.from_numpy(M).cuda()
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    buf.O.fill_(float("nan"))
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.scratch, lse=buf.lse)
    torch.cuda.synchronize()
    pyramids = orc.build_pyramid(K64, op), orc.build_pyramid(V64, op)
    O, lse = orc.psa_attention(Q64, *pyramids, M, op)
    bf16 = dtype == "bf16"
    got = from_dev(buf.O, dtype)
    assert np.abs(got - O).max() <= (2e-2 if bf16 else 1e-5) and rel_l2(got, O) <= (1e-2 if bf16 else 1e-5)
    assert np.abs(buf.lse.cpu().numpy() - lse).max() <= (2e-2 if bf16 else 1e-4)
    grads = [torch.full_like(x, float("nan")) for x in (Qd, Kd, Vd)]
    scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
    psa.psa_attention_bwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.lse, dOd, *grads, scratch)
    torch.cuda.synchronize()
    for name, x, want in zip(("dQ", "dK", "dV"), grads, orc.psa_attention_backward(Q64, *pyramids, M, dO64, op)):
        bar = (2e-2 if bf16 else 1e-5) * max(1.0, float(np.abs(want).max()))
        assert np.abs(from_dev(x, dtype) - want).max() <= bar, name


@pytest.mark.parametrize("N,d,bq,levels,causal", [(2601, 128, 128, 3, False), (2601, 64, 64, 2, True), (4301, 64, 128, 1, False), (2601, 64, 16, 3, False)])
def test_gradients_of_shared_walks(N, d, bq, levels, causal):
    """Few key blocks under long columns: one, two and four workgroups share a walk of the bfloat16 dK, dV kernel."""
    import torch
    op = orc.Params(B=1, Hq=2, Hkv=1, N=N, d=d, bq=bq, bk=64, levels=levels, dtype="bf16", causal=causal, sq=8, sk=1)
    gp = gpu_params(op)
    host = si.random_qkv(N + d, 1, 2, 1, N, d, "bf16")
    dO = si.random_qkv(9, 1, 2, 2, N, d, "bf16")[0]
    rng = np.random.default_rng(N)
    vis = orc.block_visibility(op)
    M = rng.integers(1, levels + 1, size=(1, 2, op.nq, op.nk)) * (rng.random((1, 2, op.nq, op.nk)) < 0.2)
    M[..., 0] = 1
    M[:, :, -1, -1] = 1
    M = np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)
    Qd, Kd, Vd, dOd = (to_dev(x, "bf16") for x in (*host, dO))
    Q64, K64, V64, dO64 = (si.to_f64(x, "bf16") for x in (*host, dO))
    buf, Md = Buffers(gp), torch.from_numpy(M).cuda()
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.scratch, lse=buf.lse)
    grads = [torch.full_like(x, float("nan")) for x in (Qd, Kd, Vd)]
    scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
    psa.psa_attention_bwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.lse, dOd, *grads, scratch)
    torch.cuda.synchronize()
    want = orc.psa_attention_backward(Q64, orc.build_pyramid(K64, op), orc.build_pyramid(V64, op), M, dO64, op)
    for name, x, w in zip(("dQ", "dK", "dV"), grads, want):
        assert np.abs(from_dev(x, "bf16") - w).max() <= 2e-2 * max(1.0, float(np.abs(w).max())), name


@pytest.mark.parametrize("Hq,N,bk,bq,own", [(12, 1000, 64, 128, True), (1, 5100, 64, 128, True), (1, 14634, 128, 128, False), (40, 3033, 128, 128, False),
                                            (1, 14634, 128, 64, True), (1, 8200, 64, 64, False)])
def test_which_calls_make_their_lists_themselves(Hq, N, bk, bq, own):
    """Rows of up to 128 blocks; 128-row query blocks, which lose their tile descriptors with it, only where tokens times rounds of the
    chip are few.  Calls that make them write nothing into the workspace."""
    import torch
    gp = psa.make_params(1, Hq, 1, N, 128, bq, bk, 1, causal=True, sq=8, sk=8)
    gen = torch.Generator(device="cuda").manual_seed(N)
    Q, K, V = (torch.randn((1, h, N, 128), generator=gen, device="cuda").to(torch.bfloat16) for h in (Hq, 1, 1))
    buf = Buffers(gp)
    buf.M.zero_()
    buf.M[..., 0] = 1
    buf.scratch.fill_(255)
    psa.psa_attention_fwd(gp, Q, K, V, None, None, buf.M, buf.O, buf.scratch)
    torch.cuda.synchronize()
    assert bool((buf.scratch == 255).all()) == own
