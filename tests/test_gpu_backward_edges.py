"""bfloat16 gradients where the staging of the matrix-core kernels ends: columns longer than one list, ragged last
stages, every tile width, and tensors that start between two 16-byte chunks.

Tolerance: the bfloat16 bar of the backward tests (P, dS, O and the gradients are rounded to 8 bits)."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import psa_oracle as orc
from tests.psa_testlib import Buffers, from_dev, gpu_params, rel_l2, to_dev

pytestmark = pytest.mark.gpu

psa = pytest.importorskip("paper_2512_04025_amd")


def _off_by_one(x):
    """The same tensor at an address that is 2 bytes past a 16-byte boundary."""
    import torch
    flat = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
    y = flat[1:1 + x.numel()].view(x.shape)
    y.copy_(x)
    return y


@pytest.mark.parametrize("Hq,Hkv,N,d,bq,bk,levels,causal,keep,shifted", [
    (1, 1, 8300, 128, 8, 64, 3, False, 0.04, False),      # 1038 query blocks: two lists; stages of 8 rows
    (2, 1, 1050, 128, 128, 128, 4, True, 0.6, False),     # 128-key blocks: two workgroups each
    (2, 2, 530, 64, 64, 128, 5, False, 0.6, False),       # d = 64: a 128-key block split over two workgroups
    (3, 1, 333, 64, 96, 32, 3, True, 0.8, False),         # 9 (head, block) runs on 8 XCDs; 96-row blocks: stages of 64 and 32
    (2, 1, 300, 128, 128, 64, 4, False, 0.7, True),
    (1, 1, 39100, 128, 128, 64, 3, False, 0.02, False),   # long: all XCDs on one head
])
def test_backward_edges(Hq, Hkv, N, d, bq, bk, levels, causal, keep, shifted):
    import torch
    op = orc.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, d=d, bq=bq, bk=bk, levels=levels, dtype="bf16", causal=causal, sq=8, sk=8)
    gp = gpu_params(op)
    host = si.random_qkv(5, 1, Hq, Hkv, N, d, "bf16")
    dO = si.random_qkv(6, 1, Hq, Hq, N, d, "bf16")[0]
    rng = np.random.default_rng(7)
    vis = orc.block_visibility(op)
    M = rng.integers(1, levels + 1, size=(1, Hq, op.nq, op.nk)) * (rng.random((1, Hq, op.nq, op.nk)) < keep)
    M[..., 0] = 1
    M = np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)
    Qd, Kd, Vd, dOd = (to_dev(x, "bf16") for x in (*host, dO))
    if shifted:
        Qd, dOd = _off_by_one(Qd), _off_by_one(dOd)
    buf = Buffers(gp)
    Md = torch.from_numpy(M).cuda()
    psa.psa_build_pyramid(gp, Kd, Vd, buf.Kpyr, buf.Vpyr)
    psa.psa_attention_fwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.scratch, lse=buf.lse)
    grads = [torch.full_like(x, float("nan")) for x in (Qd, Kd, Vd)]
    scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
    psa.psa_attention_bwd(gp, Qd, Kd, Vd, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.lse, dOd, *grads, scratch)
    torch.cuda.synchronize()
    Q64, K64, V64, dO64 = (si.to_f64(x, "bf16") for x in (*host, dO))
    ref = orc.psa_attention_backward(Q64, orc.build_pyramid(K64, op), orc.build_pyramid(V64, op), M, dO64, op)
    for name, got, want in zip(("dQ", "dK", "dV"), grads, ref):
        g = from_dev(got, "bf16")
        assert np.abs(g - want).max() <= 2e-2 * max(1.0, float(np.abs(want).max())), name
        assert rel_l2(g, want) <= 1e-2, name


@pytest.mark.parametrize("dtype,d,bq,bk,levels,causal", [
    ("bf16", 128, 128, 64, 4, False), ("bf16", 64, 128, 128, 4, True), ("bf16", 128, 32, 32, 3, False), ("bf16", 64, 64, 64, 3, True),
    ("f32", 128, 128, 64, 4, False), ("f32", 64, 64, 32, 3, True)])
def test_tensors_between_two_chunks_give_the_same_bits(dtype, d, bq, bk, levels, causal):
    """Every tensor one element past a 16-byte boundary: the same kernels, so the same bits as on aligned tensors."""
    import torch
    N, Hq, Hkv = 333, 4, 2
    op = orc.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, d=d, bq=bq, bk=bk, levels=levels, dtype=dtype, causal=causal, sq=8, sk=8)
    gp = gpu_params(op)
    host = si.random_qkv(5, 1, Hq, Hkv, N, d, dtype)
    dO = si.random_qkv(6, 1, Hq, Hq, N, d, dtype)[0]
    rng = np.random.default_rng(7)
    vis = orc.block_visibility(op)
    M = rng.integers(1, levels + 1, size=(1, Hq, op.nq, op.nk)) * (rng.random((1, Hq, op.nq, op.nk)) < 0.7)
    M[..., 0] = 1
    Md = torch.from_numpy(np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)).cuda()
    results = []
    for place in (lambda x: x, _off_by_one):
        Q, K, V, go = (place(to_dev(x, dtype)) for x in (*host, dO))
        buf = Buffers(gp)
        Kp, Vp, O = place(buf.Kpyr), place(buf.Vpyr), place(buf.O)
        psa.psa_build_pyramid(gp, K, V, Kp, Vp)
        psa.psa_allocate_levels(gp, Q, K, Kp, buf.M, buf.scratch, scores_out=buf.S)
        psa.psa_attention_fwd(gp, Q, K, V, Kp, Vp, Md, O, buf.scratch, lse=buf.lse)
        grads = [place(torch.full_like(x, float("nan"))) for x in (Q, K, V)]
        scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
        psa.psa_attention_bwd(gp, Q, K, V, Kp, Vp, Md, O, buf.lse, go, *grads, scratch)
        torch.cuda.synchronize()
        results.append([x.clone() for x in (buf.M, buf.S, O, buf.lse, *grads)])
    for name, a, b in zip(("M", "S", "O", "lse", "dQ", "dK", "dV"), *results):
        assert torch.equal(a, b), name


def _before_nan(x):
    """The same tensor with 64 KB of NaN right behind it."""
    import torch
    flat = torch.full((x.numel() + 65536 // x.element_size(),), float("nan"), dtype=x.dtype, device=x.device)
    y = flat[:x.numel()].view(x.shape)
    y.copy_(x)
    return y


@pytest.mark.parametrize("N,d,bq,bk,levels,causal", [
    (321, 128, 128, 64, 4, False), (450, 64, 128, 128, 4, True), (449, 128, 128, 128, 1, False), (290, 128, 32, 32, 3, True), (1000, 64, 128, 64, 2, False),
    # more than 128 key blocks: the forward's 128-row workgroups read lists and tile descriptors made by a launch of their own, as all long calls do;
    # with 256-row blocks two of them share a set
    (2099, 128, 128, 16, 2, False), (2099, 128, 128, 16, 2, True), (2099, 64, 128, 16, 2, False), (2099, 64, 128, 16, 2, True), (2081, 128, 256, 16, 2, False),
    (2081, 64, 256, 16, 2, True)])
def test_what_lies_behind_the_tensors_does_not_count(N, d, bq, bk, levels, causal):
    """Ragged lengths whose last tiles, stages and chunks reach far past the last row: the same bits with NaN behind every input."""
    import torch
    Hq, Hkv = 2, 1
    op = orc.Params(B=1, Hq=Hq, Hkv=Hkv, N=N, d=d, bq=bq, bk=bk, levels=levels, dtype="bf16", causal=causal, sq=8, sk=8)
    gp = gpu_params(op)
    host = si.random_qkv(5, 1, Hq, Hkv, N, d, "bf16")
    dO = si.random_qkv(6, 1, Hq, Hq, N, d, "bf16")[0]
    vis = orc.block_visibility(op)
    M = np.broadcast_to(np.arange(op.nk) % levels + 1, (1, Hq, op.nq, op.nk))
    Md = torch.from_numpy(np.where(vis[None, None] == 0, 0, np.where(vis[None, None] == 2, 1, M)).astype(np.uint8)).cuda()
    results = []
    for place in (lambda x: x, _before_nan):
        Q, K, V, go = (place(to_dev(x, "bf16")) for x in (*host, dO))
        buf = Buffers(gp)
        psa.psa_build_pyramid(gp, K, V, buf.Kpyr, buf.Vpyr)
        psa.psa_attention_fwd(gp, Q, K, V, buf.Kpyr, buf.Vpyr, Md, buf.O, buf.scratch, lse=buf.lse)
        O, lse = place(buf.O), place(buf.lse)
        grads = [torch.full_like(x, float("nan")) for x in (Q, K, V)]
        scratch = torch.full((psa.psa_query_bwd_sizes(gp),), 255, dtype=torch.uint8, device="cuda")
        psa.psa_attention_bwd(gp, Q, K, V, buf.Kpyr, buf.Vpyr, Md, O, lse, go, *grads, scratch)
        torch.cuda.synchronize()
        results.append([x.clone() for x in (buf.O, buf.lse, *grads)])
    for name, a, b in zip(("O", "lse", "dQ", "dK", "dV"), *results):
        assert torch.equal(a, b), name
        assert not torch.isnan(a).any(), name
