"""GPU parity of the single kernels against the CPU oracle, element by element.
Tolerance: max|gpu - oracle| / max|oracle| <= 1e-5 in fp32 mode, 2e-2 in bf16 mode."""
import math

import numpy as np
import pytest
import torch

import bf_inputs
import paper_2211_05953_amd as bf
from oracle import layer as L
from oracle import stack as K
from util import TOL, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

MODES = [("fp32", bf.BF_FP32), ("bf16", bf.BF_BF16)]


def _dt(bf16):
    return torch.bfloat16 if bf16 else torch.float32


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("kernels", [bf.BF_KERNELS_PLAIN, bf.BF_KERNELS_AUTO])
@pytest.mark.parametrize("M,N,K", [(128, 768, 256), (200, 136, 72), (256, 512, 384), (2048, 256, 512), (64, 64, 2048), (1, 1, 1)])
def test_gemm_all_layouts_and_epilogues(mode, dtype, kernels, M, N, K):
    b16 = dtype == bf.BF_BF16
    A = bf_inputs.normal(1, 0, (M, K), bf16=b16)
    B = bf_inputs.normal(1, 1, (K, N), 0.05, bf16=b16)
    bias = bf_inputs.normal(1, 2, (N,), 0.5)
    R = bf_inputs.normal(1, 3, (M, N), bf16=b16)
    A64, B64, R64 = A.astype(np.float64), B.astype(np.float64), R.astype(np.float64)
    acc = A64 @ B64
    dA, dB, dR, dbias = to_dev(A, b16), to_dev(B, b16), to_dev(R, b16), to_dev(bias, False)
    out = torch.empty(M, N, dtype=_dt(b16), device="cuda")
    out2 = torch.empty_like(out)
    # forward layouts
    bf.bf_op_gemm(dtype, kernels, bf.BF_NN, bf.BF_EPI_NONE, M, N, K, dA, dB, out)
    assert rel_err(to_host(out), acc) <= TOL[mode]
    bf.bf_op_gemm(dtype, kernels, bf.BF_NN, bf.BF_EPI_BIAS, M, N, K, dA, dB, out, bias=dbias)
    assert rel_err(to_host(out), acc + bias) <= TOL[mode]
    bf.bf_op_gemm(dtype, kernels, bf.BF_NN, bf.BF_EPI_BIAS_RES, M, N, K, dA, dB, out, bias=dbias, R=dR)
    assert rel_err(to_host(out), acc + bias + R64) <= TOL[mode]
    bf.bf_op_gemm(dtype, kernels, bf.BF_NN, bf.BF_EPI_BIAS_GELU, M, N, K, dA, dB, out, bias=dbias, C2=out2)
    assert rel_err(to_host(out), acc + bias) <= TOL[mode]
    assert rel_err(to_host(out2), L.gelu(acc + bias)) <= TOL[mode]
    # dgrad layout: B passed as [N, K]
    dBt = to_dev(np.ascontiguousarray(B.T), b16)
    bf.bf_op_gemm(dtype, kernels, bf.BF_NT, bf.BF_EPI_NONE, M, N, K, dA, dBt, out)
    assert rel_err(to_host(out), acc) <= TOL[mode]
    bf.bf_op_gemm(dtype, kernels, bf.BF_NT, bf.BF_EPI_GELU_BWD, M, N, K, dA, dBt, out, R=dR)
    assert rel_err(to_host(out), acc * L.gelu_grad(R64)) <= TOL[mode]
    # wgrad layout: A passed as [K, M], fp32 output, overwrite then accumulate
    dAt = to_dev(np.ascontiguousarray(A.T), b16)
    G = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    bf.bf_op_gemm(dtype, kernels, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, dAt, dB, G, accumulate=0)
    assert rel_err(to_host(G), acc) <= TOL["fp32"] * (1 if not b16 else 1)
    bf.bf_op_gemm(dtype, kernels, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, dAt, dB, G, accumulate=1)
    assert rel_err(to_host(G), 2 * acc) <= TOL["fp32"]


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("kernels", [bf.BF_KERNELS_PLAIN, bf.BF_KERNELS_AUTO])
@pytest.mark.parametrize("M,N,K", [(128, 768, 256), (200, 136, 72), (512, 512, 128), (1280, 384, 192), (2048, 256, 512)])
def test_gelu_backward_product_with_the_bias_gradient_on_the_way(mode, dtype, kernels, M, N, K):
    """dU = (dY W^T) gelu'(U) and db = column sums of dU: in the MFMA kernel's epilogue (per-tile partial sums in a
    scratch buffer, then a fixed-order reduction), or as a second pass when there is no scratch or the plain kernel
    runs; overwriting and accumulating.  In bf16 all of these are products of few tiles, which take the second pass with
    the scratch or without (test_gemm_on_whole_tiles has those whose epilogue leaves partial sums)."""
    b16 = dtype == bf.BF_BF16
    A = bf_inputs.normal(4, 0, (M, K), bf16=b16)
    Bt = bf_inputs.normal(4, 1, (N, K), 0.05, bf16=b16)
    R = bf_inputs.normal(4, 3, (M, N), bf16=b16)
    ref = (A.astype(np.float64) @ Bt.astype(np.float64).T) * L.gelu_grad(R.astype(np.float64))
    dA, dBt, dR = to_dev(A, b16), to_dev(Bt, b16), to_dev(R, b16)
    for with_part in (True, False):
        out = torch.empty(M, N, dtype=_dt(b16), device="cuda")
        db = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
        part = torch.full(((M + 127) // 128, N), float("nan"), dtype=torch.float32, device="cuda") if with_part else None
        bf.bf_op_gemm_gelu_bwd_colsum(dtype, kernels, M, N, K, dA, dBt, out, dR, db, part, accumulate=0)
        assert rel_err(to_host(out), ref) <= TOL[mode]
        assert rel_err(to_host(db), ref.sum(axis=0)) <= TOL[mode]
        # the sums are those of the stored output, up to fp32 summation order
        assert rel_err(to_host(db), to_host(out).astype(np.float64).sum(axis=0)) <= 1e-5
        first = to_host(db).copy()
        bf.bf_op_gemm_gelu_bwd_colsum(dtype, kernels, M, N, K, dA, dBt, out, dR, db, part, accumulate=1)
        assert rel_err(to_host(db), 2.0 * first.astype(np.float64)) <= 1e-6
        # same launch, same bits
        db2 = torch.empty_like(db)
        bf.bf_op_gemm_gelu_bwd_colsum(dtype, kernels, M, N, K, dA, dBt, out, dR, db2, part, accumulate=0)
        assert np.array_equal(to_host(db2), first)


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("T,h", [(128, 256), (77, 100), (300, 2048), (1024, 6144), (2048, 8192), (520, 1000), (3, 8200), (64, 16384)])
def test_layernorm_backward_in_one_pass(mode, dtype, T, h):
    """bf_op_layernorm_bwd_fused: dx, the gain / bias gradients and the column sums of dx from one pass over dy and x
    (workgroups of consecutive rows with partial sums in a scratch buffer, then a fixed-order reduction), or in separate
    passes when there is no scratch or the row does not fit; overwriting and accumulating; row counts that do not
    divide into equal runs; widths with idle lanes (256), of 3 and 4 vectors per thread, and beyond the one-pass form."""
    b16 = dtype == bf.BF_BF16
    x = bf_inputs.normal(6, 0, (T, h), 2.0, bf16=b16) + np.float32(0.5)
    if b16:
        x = bf_inputs.round_bf16(x)
    g = 1 + bf_inputs.normal(6, 1, (h,), 0.2)
    dy = bf_inputs.normal(6, 3, (T, h), bf16=b16)
    dres = bf_inputs.normal(6, 4, (T, h), bf16=b16)
    eps = 1e-5
    g64 = g.astype(np.float64)
    _, saved = L.layernorm_fwd(x.astype(np.float64), g64, np.zeros(h), eps)
    dx_ref, dg_ref, db_ref = L.layernorm_bwd(dy.astype(np.float64), g64, saved)
    dx_ref = dx_ref + dres.astype(np.float64)
    dX, dG, dDY, dRES = to_dev(x, b16), to_dev(g, False), to_dev(dy, b16), to_dev(dres, b16)
    stats = torch.empty(T, 2, dtype=torch.float32, device="cuda")
    bf.bf_op_layernorm_fwd(dtype, T, h, dX, dG, torch.zeros(h, device="cuda"), eps, torch.empty_like(dX), stats)
    n_part = bf.bf_op_layernorm_bwd_part_elems(T, h)
    assert n_part == 3 * h * -(-T // -(-T // 256)) and n_part <= 3 * h * 256
    results = []
    for with_part in (True, False):
        part = torch.full((n_part,), float("nan"), dtype=torch.float32, device="cuda") if with_part else None
        dx = torch.empty_like(dX)
        dg, db, dcs = (torch.full((h,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(3))
        bf.bf_op_layernorm_bwd_fused(dtype, T, h, dDY, dX, dG, stats, dRES, dx, dg, db, dcs, part, accumulate=0)
        assert rel_err(to_host(dx), dx_ref) <= TOL[mode]
        assert rel_err(to_host(dg), dg_ref) <= TOL[mode] and rel_err(to_host(db), db_ref) <= TOL[mode]
        assert rel_err(to_host(dcs), dx_ref.sum(axis=0)) <= TOL[mode]
        assert rel_err(to_host(dcs), to_host(dx).astype(np.float64).sum(axis=0)) <= 1e-5   # sums of the stored dx
        first = [to_host(t).copy() for t in (dg, db, dcs)]
        bf.bf_op_layernorm_bwd_fused(dtype, T, h, dDY, dX, dG, stats, dRES, dx, dg, db, dcs, part, accumulate=1)
        for t, f0 in zip((dg, db, dcs), first):
            assert rel_err(to_host(t), 2.0 * f0.astype(np.float64)) <= 1e-6
        # without the residual gradient and without the column sums of dx
        dx2 = torch.empty_like(dX)
        bf.bf_op_layernorm_bwd_fused(dtype, T, h, dDY, dX, dG, stats, None, dx2, dg, db, None, part, accumulate=0)
        assert rel_err(to_host(dx2), dx_ref - dres.astype(np.float64)) <= TOL[mode]
        assert np.array_equal(to_host(dg), first[0]) and np.array_equal(to_host(db), first[1])
        results.append((to_host(dx), first))
    # the two forms agree to the rounding of the output (their fused multiply-adds may associate differently)
    assert rel_err(results[0][0], results[1][0].astype(np.float64)) <= (2.0 ** -8 if b16 else 1e-6)


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("T,h", [(128, 256), (77, 100), (512, 2048), (3, 8200)])
def test_layernorm_fwd_bwd_and_colsum(mode, dtype, T, h):
    b16 = dtype == bf.BF_BF16
    x = bf_inputs.normal(2, 0, (T, h), 2.0, bf16=b16) + np.float32(0.5)
    if b16:
        x = bf_inputs.round_bf16(x)
    g = 1 + bf_inputs.normal(2, 1, (h,), 0.2)
    b = bf_inputs.normal(2, 2, (h,), 0.2)
    dy = bf_inputs.normal(2, 3, (T, h), bf16=b16)
    dres = bf_inputs.normal(2, 4, (T, h), bf16=b16)
    eps = 1e-5
    y_ref, saved = L.layernorm_fwd(x.astype(np.float64), g.astype(np.float64), b.astype(np.float64), eps)
    dx_ref, dg_ref, db_ref = L.layernorm_bwd(dy.astype(np.float64), g.astype(np.float64), saved)
    dX, dG, dB, dDY, dRES = to_dev(x, b16), to_dev(g, False), to_dev(b, False), to_dev(dy, b16), to_dev(dres, b16)
    y = torch.empty(T, h, dtype=_dt(b16), device="cuda")
    stats = torch.empty(T, 2, dtype=torch.float32, device="cuda")
    bf.bf_op_layernorm_fwd(dtype, T, h, dX, dG, dB, eps, y, stats)
    assert rel_err(to_host(y), y_ref) <= TOL[mode]
    st = to_host(stats).astype(np.float64)
    assert rel_err(st[:, 0], x.astype(np.float64).mean(-1)) <= 1e-5
    assert rel_err(st[:, 1], saved[1][:, 0]) <= 1e-5
    dx = torch.empty_like(y)
    dg = torch.full((h,), float("nan"), dtype=torch.float32, device="cuda")
    db = torch.full((h,), float("nan"), dtype=torch.float32, device="cuda")
    bf.bf_op_layernorm_bwd(dtype, T, h, dDY, dX, dG, stats, dRES, dx, dg, db, 0)
    assert rel_err(to_host(dx), dx_ref + dres) <= TOL[mode]
    assert rel_err(to_host(dg), dg_ref) <= 1e-5 and rel_err(to_host(db), db_ref) <= 1e-5
    bf.bf_op_layernorm_bwd(dtype, T, h, dDY, dX, dG, stats, None, dx, dg, db, 1)
    assert rel_err(to_host(dx), dx_ref) <= TOL[mode]
    assert rel_err(to_host(dg), 2 * dg_ref) <= 1e-5 and rel_err(to_host(db), 2 * db_ref) <= 1e-5
    out = torch.full((h,), float("nan"), dtype=torch.float32, device="cuda")
    bf.bf_op_colsum(dtype, T, h, dDY, out, 0)
    assert rel_err(to_host(out), dy.astype(np.float64).sum(0)) <= 1e-5
    bf.bf_op_colsum(dtype, T, h, dDY, out, 1)
    assert rel_err(to_host(out), 2 * dy.astype(np.float64).sum(0)) <= 1e-5


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("kernels", [bf.BF_KERNELS_PLAIN, bf.BF_KERNELS_AUTO])
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(1, 128, 4, 64), (2, 256, 2, 128), (2, 100, 3, 40), (1, 1, 1, 8), (1, 384, 2, 128)])
def test_attention_fwd_bwd(mode, dtype, kernels, causal, S_mb, S_seq, a, d):
    b16 = dtype == bf.BF_BF16
    h = a * d
    qkv = bf_inputs.normal(3, 0, (S_mb, S_seq, 3 * h), bf16=b16)
    dctx = bf_inputs.normal(3, 1, (S_mb, S_seq, h), bf16=b16)
    ctx_ref, saved = L.attention_fwd(qkv.astype(np.float64), a, bool(causal))
    dqkv_ref = L.attention_bwd(dctx.astype(np.float64), saved, a)
    dQKV, dDC = to_dev(qkv, b16), to_dev(dctx, b16)
    ctx = torch.empty(S_mb, S_seq, h, dtype=_dt(b16), device="cuda")
    lse = torch.empty(S_mb, a, S_seq, dtype=torch.float32, device="cuda")
    bf.bf_op_attention_fwd(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
    assert rel_err(to_host(ctx), ctx_ref) <= TOL[mode]
    # log-sum-exp of the scaled masked scores, from the definition
    q, k, v, p = saved
    s = np.matmul(q, k.transpose(0, 1, 3, 2)) / math.sqrt(d)
    if causal:
        s = np.where(np.tril(np.ones((S_seq, S_seq), dtype=bool)), s, -np.inf)
    lse_ref = np.log(np.exp(s - s.max(-1, keepdims=True)).sum(-1)) + s.max(-1)
    assert np.abs(to_host(lse) - lse_ref).max() <= (1e-4 if not b16 else 2e-2)
    dqkv = torch.empty(S_mb, S_seq, 3 * h, dtype=_dt(b16), device="cuda")
    delta = torch.empty(S_mb * a * S_seq, dtype=torch.float32, device="cuda")
    bf.bf_op_attention_bwd(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta)
    got = to_host(dqkv)
    for i, name in enumerate(("dq", "dk", "dv")):
        assert rel_err(got[..., i * h:(i + 1) * h], dqkv_ref[..., i * h:(i + 1) * h]) <= TOL[mode], name
    # the same with the QKV bias gradient (column sums of dqkv) on the way: with the scratch for the kernels' partial
    # sums (where the matrix-core kernels serve the shape) and without it (dqkv read a second time); overwrite, then add
    n_part = bf.bf_op_attention_bwd_part_elems(S_mb, S_seq, a, d)
    mfma = bf.bf_op_attention_uses_mfma(S_seq, d)
    q_rows = S_mb * (S_seq // (256 if S_seq % 256 == 0 else 128)) if mfma else 0
    assert n_part == (q_rows * h + S_mb * (S_seq // 128) * 2 * h if mfma else 0)
    db_ref = dqkv_ref.reshape(-1, 3 * h).sum(axis=0)
    for with_part in (True, False):
        part = torch.full((max(n_part, 1),), float("nan"), dtype=torch.float32, device="cuda") if with_part and n_part else None
        dqkv2 = torch.full_like(dqkv, float("nan"))
        db = torch.full((3 * h,), float("nan"), dtype=torch.float32, device="cuda")
        bf.bf_op_attention_bwd_bias(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv2, delta, db, part, 0)
        assert torch.equal(dqkv2, dqkv)
        first = to_host(db).copy()
        # (the K third is zero in exact arithmetic: a softmax row does not move when every score of it is shifted by the
        # same amount, which is all a key bias does; so the thirds are judged together, on the scale of the whole vector)
        assert rel_err(first, db_ref) <= TOL[mode]
        for i, name in ((0, "dq"), (2, "dv")):
            assert rel_err(first[i * h:(i + 1) * h], db_ref[i * h:(i + 1) * h]) <= TOL[mode], name
        # against the sums of what was stored: the fused form adds the values before they are rounded to bf16
        stored = got.astype(np.float64).reshape(-1, 3 * h).sum(axis=0)
        assert rel_err(first, stored) <= (2.0 ** -8 if b16 else 1e-5)
        bf.bf_op_attention_bwd_bias(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv2, delta, db, part, 1)
        assert rel_err(to_host(db), 2.0 * first.astype(np.float64)) <= 1e-6


@pytest.mark.parametrize("M,N,K", [(2048, 2048, 8192), (2048, 2048, 2048), (1024, 1024, 4608), (256, 128, 4608)])
def test_gemm_with_a_split_contraction(M, N, K):
    """bf_op_gemm_splitk: few tiles and a long contraction run K in two slices into fp32 planes that a second kernel adds
    in order, with each of the epilogues it serves, in both layouts; the result agrees with the unsplit product to the
    rounding of the output (the fp32 sum associates differently) and with the fp64 product to the bf16 bar."""
    assert bf.bf_op_gemm_splitk_slices(bf.BF_NN, bf.BF_EPI_BIAS_RES, M, N, K) == 2
    assert bf.bf_op_gemm_splitk_slices(bf.BF_NT, bf.BF_EPI_NONE, M, N, K) == 2
    A = bf_inputs.normal(15, 0, (M, K), bf16=True)
    B = bf_inputs.normal(15, 1, (K, N), 0.05, bf16=True)
    bias = bf_inputs.normal(15, 2, (N,), 0.5)
    R = bf_inputs.normal(15, 3, (M, N), bf16=True)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    dA, dB, dBt, dR, dbias = to_dev(A, True), to_dev(B, True), to_dev(np.ascontiguousarray(B.T), True), to_dev(R, True), to_dev(bias, False)
    planes = torch.full((2 * M * N,), float("nan"), dtype=torch.float32, device="cuda")
    for layout, Bd in ((bf.BF_NN, dB), (bf.BF_NT, dBt)):
        for epi, want in ((bf.BF_EPI_NONE, acc), (bf.BF_EPI_BIAS, acc + bias), (bf.BF_EPI_BIAS_RES, acc + bias + R)):
            out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            ref = torch.empty_like(out)
            bf.bf_op_gemm_splitk(bf.BF_BF16, 0, layout, epi, M, N, K, dA, Bd, out, bias=dbias, R=dR, planes=planes)
            bf.bf_op_gemm(bf.BF_BF16, 0, layout, epi, M, N, K, dA, Bd, ref, bias=dbias, R=dR)
            assert bool(torch.isfinite(planes).all())   # both slices were run
            planes.fill_(float("nan"))
            assert rel_err(to_host(out), want) <= TOL["bf16"], (layout, epi)
            assert rel_err(to_host(out), to_host(ref).astype(np.float64)) <= 2.0 ** -7, (layout, epi)
            # deterministic: a second call gives the same bits
            again = torch.empty_like(out)
            bf.bf_op_gemm_splitk(bf.BF_BF16, 0, layout, epi, M, N, K, dA, Bd, again, bias=dbias, R=dR, planes=planes)
            assert torch.equal(out, again)
    # without the scratch, or with too little of it, the call is the plain product
    out, ref = torch.empty((M, N), dtype=torch.bfloat16, device="cuda"), torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_NN, bf.BF_EPI_BIAS, M, N, K, dA, dB, ref, bias=dbias)
    bf.bf_op_gemm_splitk(bf.BF_BF16, 0, bf.BF_NN, bf.BF_EPI_BIAS, M, N, K, dA, dB, out, bias=dbias, planes=None)
    assert torch.equal(out, ref)
    bf.bf_op_gemm_splitk(bf.BF_BF16, 0, bf.BF_NN, bf.BF_EPI_BIAS, M, N, K, dA, dB, out, bias=dbias, planes=planes[:M * N])
    assert torch.equal(out, ref)


def test_split_contraction_is_chosen_only_where_it_pays():
    s = bf.bf_op_gemm_splitk_slices
    assert s(bf.BF_NN, bf.BF_EPI_BIAS_RES, 2048, 2048, 2048) == 2
    assert s(bf.BF_NN, bf.BF_EPI_BIAS_RES, 2048, 2048, 1024) == 1      # contraction too short
    assert s(bf.BF_NN, bf.BF_EPI_BIAS, 1024, 1024, 4608) == 2          # few tiles: only a longer one pays
    assert s(bf.BF_NN, bf.BF_EPI_BIAS, 1024, 1024, 4096) == 1 and s(bf.BF_NT, bf.BF_EPI_NONE, 256, 512, 2048) == 1
    assert s(bf.BF_NN, bf.BF_EPI_BIAS, 2048, 8192, 8192) == 1          # a full round of tiles already
    assert s(bf.BF_NT, bf.BF_EPI_NONE, 2048, 6144, 18432) == 1
    assert s(bf.BF_NN, bf.BF_EPI_BIAS_GELU, 2048, 2048, 8192) == 1     # epilogues with a second output are not split
    assert s(bf.BF_NT, bf.BF_EPI_GELU_BWD, 2048, 2048, 8192) == 1
    assert s(bf.BF_TN, bf.BF_EPI_ACCUM, 2048, 2048, 8192) == 1
    assert s(bf.BF_NN, bf.BF_EPI_NONE, 2000, 2048, 8192) == 1          # not a shape of the matrix-core kernel
    assert s(bf.BF_NN, bf.BF_EPI_NONE, 2048, 2048, 8192 + 64) == 1     # slices must be whole k-tiles


@pytest.mark.parametrize("M,N,K", [(2048, 4096, 512), (4096, 2048, 192), (512, 16384, 128)])
def test_gemm_mfma_large_tile(M, N, K):
    """Products of many tiles of the MFMA kernel (256 x 128 ones), all layouts."""
    assert bf.bf_op_gemm_uses_mfma(bf.BF_NN, bf.BF_EPI_NONE, M, N, K)
    A = bf_inputs.normal(5, 0, (M, K), bf16=True)
    B = bf_inputs.normal(5, 1, (K, N), 0.05, bf16=True)
    bias = bf_inputs.normal(5, 2, (N,), 0.5)
    R = bf_inputs.normal(5, 3, (M, N), bf16=True)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    dA, dB, dR, dbias = to_dev(A, True), to_dev(B, True), to_dev(R, True), to_dev(bias, False)
    out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    out2 = torch.empty_like(out)
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_NN, bf.BF_EPI_BIAS_RES, M, N, K, dA, dB, out, bias=dbias, R=dR)
    assert rel_err(to_host(out), acc + bias + R) <= TOL["bf16"]
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_NN, bf.BF_EPI_BIAS_GELU, M, N, K, dA, dB, out, bias=dbias, C2=out2)
    assert rel_err(to_host(out2), L.gelu(acc + bias)) <= TOL["bf16"]
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_NT, bf.BF_EPI_GELU_BWD, M, N, K, dA, to_dev(np.ascontiguousarray(B.T), True), out, R=dR)
    assert rel_err(to_host(out), acc * L.gelu_grad(R.astype(np.float64))) <= TOL["bf16"]
    G = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    dAt = to_dev(np.ascontiguousarray(A.T), True)
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, dAt, dB, G, accumulate=0)
    bf.bf_op_gemm(bf.BF_BF16, 0, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, dAt, dB, G, accumulate=1)
    assert rel_err(to_host(G), 2 * acc) <= 1e-5   # bf16 products are exact in fp32; only the summation order differs


@pytest.mark.parametrize("M,N,K", [(4096, 3072, 192), (2048, 6144, 64), (256, 49152, 128), (2048, 6144, 320)])
def test_gemm_mfma_tile_of_192_columns(M, N, K):
    """Forward and dgrad products with a one-output epilogue whose column count is a multiple of 192 take a 256 x 192
    tile where that fills the rounds better (6144 columns: 32 tiles where 256-column tiles give 24); the epilogues
    with a second output or with column sums, and the weight-gradient layout, keep their tiles."""
    for layout, epi in ((bf.BF_NT, bf.BF_EPI_NONE), (bf.BF_NN, bf.BF_EPI_NONE), (bf.BF_NN, bf.BF_EPI_BIAS), (bf.BF_NN, bf.BF_EPI_BIAS_RES)):
        assert bf.bf_op_gemm_tile(layout, epi, M, N, K) == (256, 192), (layout, epi)
    for layout, epi in ((bf.BF_NT, bf.BF_EPI_GELU_BWD), (bf.BF_NN, bf.BF_EPI_BIAS_GELU), (bf.BF_TN, bf.BF_EPI_ACCUM)):
        assert bf.bf_op_gemm_tile(layout, epi, M, N, K)[1] != 192, (layout, epi)
    assert bf.bf_op_gemm_tile(bf.BF_NT, bf.BF_EPI_NONE, 2048, 8192, 8192) == (256, 256)   # 8192 is no multiple of 192
    assert bf.bf_op_gemm_tile(bf.BF_NN, bf.BF_EPI_BIAS, 2048, 24576, 8192) == (256, 256)  # three whole rounds already
    assert bf.bf_op_gemm_tile(bf.BF_NT, bf.BF_EPI_NONE, 100, 72, 64) is None
    A = bf_inputs.normal(6, 0, (M, K), bf16=True)
    B = bf_inputs.normal(6, 1, (K, N), 0.05, bf16=True)
    bias = bf_inputs.normal(6, 2, (N,), 0.5)
    R = bf_inputs.normal(6, 3, (M, N), bf16=True)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    dA, dB, dBt = to_dev(A, True), to_dev(B, True), to_dev(np.ascontiguousarray(B.T), True)
    dR, dbias = to_dev(R, True), to_dev(bias, False)
    cases = (("dgrad", bf.BF_NT, bf.BF_EPI_NONE, dBt, acc), ("fwd", bf.BF_NN, bf.BF_EPI_NONE, dB, acc),
             ("fwd+bias", bf.BF_NN, bf.BF_EPI_BIAS, dB, acc + bias), ("fwd+bias+res", bf.BF_NN, bf.BF_EPI_BIAS_RES, dB, acc + bias + R))
    for name, layout, epi, dOp, ref in cases:
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        bf.bf_op_gemm(bf.BF_BF16, 0, layout, epi, M, N, K, dA, dOp, out, bias=dbias, R=dR)
        got = to_host(out)
        assert np.isfinite(got).all() and rel_err(got, ref) <= TOL["bf16"], name
        # one rounding of the fp32 result: the plain kernel (fp32 FMA over the same bf16 products) agrees to that rounding
        plain = torch.empty_like(out)
        bf.bf_op_gemm(bf.BF_BF16, bf.BF_KERNELS_PLAIN, layout, epi, M, N, K, dA, dOp, plain, bias=dbias, R=dR)
        assert rel_err(got, to_host(plain)) <= 2.0 ** -7, name


@pytest.mark.parametrize("mode,dtype,kernels", [("fp32", bf.BF_FP32, bf.BF_KERNELS_AUTO), ("bf16", bf.BF_BF16, bf.BF_KERNELS_PLAIN),
                                                ("bf16", bf.BF_BF16, bf.BF_KERNELS_AUTO)])
@pytest.mark.parametrize("M,N,K,n_seg,gap", [(256, 512, 128, 3, 0), (1024, 768, 128, 2, 64), (128, 384, 64, 2, 8), (512, 256, 192, 4, 0),
                                             (768, 128, 64, 1, 0), (200, 136, 72, 3, 16), (256, 256, 64, 2, 4)])
def test_wgrad_over_the_micro_batches_of_a_stage(mode, dtype, kernels, M, N, K, n_seg, gap):
    """G = sum_i X_i^T dY_i and db = sum_i colsum(dY_i) in one call (Sec. 4.2: the gradient of a stage
    is needed only after all its micro-batches); segments lie `gap` elements apart beyond their size.  (bf16 products of few
    tiles, and ragged ones; test_gemm_on_whole_tiles has segments on the larger tiles.)"""
    b16 = dtype == bf.BF_BF16
    sx, sy = K * M + gap, K * N + gap
    X = bf_inputs.normal(9, 0, (n_seg * sx,), bf16=b16)
    dY = bf_inputs.normal(9, 1, (n_seg * sy,), 0.3, bf16=b16)
    G_ref, db_ref = np.zeros((M, N)), np.zeros(N)
    for i in range(n_seg):
        Xi = X[i * sx:i * sx + K * M].reshape(K, M).astype(np.float64)
        dYi = dY[i * sy:i * sy + K * N].reshape(K, N).astype(np.float64)
        G_ref += Xi.T @ dYi
        db_ref += dYi.sum(0)
    dX, ddY = to_dev(X, b16), to_dev(dY, b16)
    G = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    db = torch.full((N,), float("nan"), dtype=torch.float32, device="cuda")
    bf.bf_op_wgrad(dtype, kernels, M, N, K, n_seg, dX, sx, ddY, sy, G, db, accumulate=0)
    assert rel_err(to_host(G), G_ref) <= 1e-5 and rel_err(to_host(db), db_ref) <= 1e-5
    bf.bf_op_wgrad(dtype, kernels, M, N, K, n_seg, dX, sx, ddY, sy, G, db, accumulate=1)
    assert rel_err(to_host(G), 2 * G_ref) <= 1e-5 and rel_err(to_host(db), 2 * db_ref) <= 1e-5
    # without the bias gradient: db is left alone
    keep = to_host(db).copy()
    bf.bf_op_wgrad(dtype, kernels, M, N, K, n_seg, dX, sx, ddY, sy, G, None, accumulate=0)
    assert rel_err(to_host(G), G_ref) <= 1e-5 and np.array_equal(to_host(db), keep)


@pytest.mark.parametrize("n", [1, 1000, 4096 * 33 + 4])
def test_adam_kernel(n):
    rng = np.random.default_rng(4)
    w = rng.standard_normal(n).astype(np.float32)
    g = (rng.standard_normal(n) * 10.0 ** rng.integers(-4, 2, n)).astype(np.float32)
    m0 = (rng.standard_normal(n) * 0.1).astype(np.float32)
    v0 = (rng.random(n) * 0.1).astype(np.float32)
    dW, dM, dV, dGr = (torch.from_numpy(t).cuda() for t in (w, m0, v0, g))
    wlp = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    args = dict(lr=1e-2, beta1=0.9, beta2=0.999, adam_eps=1e-8, weight_decay=0.01)
    bf.bf_op_adam(n, dW, dM, dV, dGr, wlp, 3, **args)
    # the C ABI carries the constants as fp32: the oracle gets those exact values
    f32 = {k: float(np.float32(v)) for k, v in args.items()}
    w1, m1, v1 = K.adam_update(w.astype(np.float64), g.astype(np.float64), m0.astype(np.float64), v0.astype(np.float64),
                               3, f32["lr"], f32["beta1"], f32["beta2"], f32["adam_eps"], f32["weight_decay"])
    assert rel_err(to_host(dM), m1) <= 1e-6 and rel_err(to_host(dV), v1) <= 1e-6
    assert rel_err(to_host(dW) - w, w1 - w) <= 1e-4          # the update itself
    assert np.array_equal(to_host(wlp), bf_inputs.round_bf16(to_host(dW)))  # recast = RNE of the new master


def test_op_argument_errors():
    t = torch.zeros(16, device="cuda")
    with pytest.raises(bf.BfError) as e:
        bf.bf_op_gemm(bf.BF_FP32, 0, bf.BF_NN, bf.BF_EPI_BIAS, 4, 4, 4, t, t, t)   # bias missing
    assert e.value.status == bf.BF_EINVAL
    with pytest.raises(bf.BfError):
        bf.bf_op_gemm(bf.BF_FP32, 0, bf.BF_TN, bf.BF_EPI_NONE, 4, 4, 4, t, t, t)
    with pytest.raises(bf.BfError):
        bf.bf_op_gemm(9, 0, bf.BF_NN, bf.BF_EPI_NONE, 4, 4, 4, t, t, t)
    with pytest.raises(bf.BfError):
        bf.bf_op_layernorm_fwd(bf.BF_FP32, 0, 4, t, t, t, 1e-5, t, t)
    with pytest.raises(bf.BfError):
        bf.bf_op_attention_fwd(bf.BF_FP32, 0, 1, 5000, 1, 4, 1, t, t, t)


def _guarded(a, b16):
    """A device copy of `a` with NaN on both sides: a read outside the operand that reaches a result shows."""
    flat = torch.full((a.size + 128,), float("nan"), dtype=_dt(b16), device="cuda")
    flat[64:64 + a.size] = to_dev(a, b16).reshape(-1)
    return flat[64:64 + a.size]


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (100, 72, 64), (127, 136, 200), (129, 264, 72), (1000, 8200, 72), (300, 1000, 24), (520, 264, 1000),
                                   (33, 35, 37), (1, 1, 1), (130, 66, 101), (2048, 392, 40)])
def test_gemm_on_partly_empty_tiles(mode, dtype, M, N, K):
    """Sizes around the tiles' edges, down to one element and with rows that are not 16-byte chunks: every layout and
    epilogue, operands between NaNs, outputs that must not be written outside.  fp32: a chain of K products, error
    under 2^-24 sqrt(K) of the sum's scale, far below the bar of 1e-5, and the same chain as the plain kernel's: the same
    bits; bf16: one rounding of such a sum, 2^-8, below 2e-2."""
    b16 = dtype == bf.BF_BF16
    A = bf_inputs.normal(21, 0, (M, K), bf16=b16)
    B = bf_inputs.normal(21, 1, (K, N), 0.05, bf16=b16)
    bias = bf_inputs.normal(21, 2, (N,), 0.5)
    R = bf_inputs.normal(21, 3, (M, N), bf16=b16)
    R64 = R.astype(np.float64)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    gA, gB, gBt, gR, gbias = _guarded(A, b16), _guarded(B, b16), _guarded(np.ascontiguousarray(B.T), b16), _guarded(R, b16), to_dev(bias, False)
    gAt = _guarded(np.ascontiguousarray(A.T), b16)

    def outbuf(td):
        return torch.full((M * N + 128,), 7.0, dtype=td, device="cuda")

    def taken(buf):
        assert bool((buf[:64] == 7.0).all()) and bool((buf[64 + M * N:] == 7.0).all())
        return to_host(buf[64:64 + M * N].reshape(M, N))
    for layout, op in ((bf.BF_NN, gB), (bf.BF_NT, gBt)):
        for epi, ref in ((bf.BF_EPI_NONE, acc), (bf.BF_EPI_BIAS, acc + bias), (bf.BF_EPI_BIAS_RES, acc + bias + R64),
                         (bf.BF_EPI_BIAS_GELU, acc + bias), (bf.BF_EPI_GELU_BWD, acc * L.gelu_grad(R64))):
            out, out2 = outbuf(_dt(b16)), outbuf(_dt(b16))
            bf.bf_op_gemm(dtype, 0, layout, epi, M, N, K, gA, op, out[64:], bias=gbias, R=gR, C2=out2[64:])
            assert rel_err(taken(out), ref) <= TOL[mode], (layout, epi)
            if epi == bf.BF_EPI_BIAS_GELU:
                assert rel_err(taken(out2), L.gelu(acc + bias)) <= TOL[mode]
            if not b16:
                plain, plain2 = outbuf(_dt(b16)), outbuf(_dt(b16))
                bf.bf_op_gemm(dtype, bf.BF_KERNELS_PLAIN, layout, epi, M, N, K, gA, op, plain[64:], bias=gbias, R=gR, C2=plain2[64:])
                assert torch.equal(out, plain) and torch.equal(out2, plain2), (layout, epi)
    G = outbuf(torch.float32)
    for accumulate in (0, 1):
        bf.bf_op_gemm(dtype, 0, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, gAt, gB, G[64:], accumulate=accumulate)
        assert rel_err(taken(G), (1 + accumulate) * acc) <= 1e-5
    # the column sums that go with the GeLU backward, through the scratch rows and without
    if M >= 100:
        ref = (acc * L.gelu_grad(R64)).sum(axis=0)
        for part in (torch.full(((M + 127) // 128, N), float("nan"), device="cuda"), None):
            out, db = outbuf(_dt(b16)), torch.full((N,), float("nan"), device="cuda")
            bf.bf_op_gemm_gelu_bwd_colsum(dtype, 0, M, N, K, gA, gBt, out[64:], gR, db, part)
            taken(out)
            assert rel_err(to_host(db), ref) <= TOL[mode]


@pytest.mark.parametrize("K", [31, 64, 97, 200])
@pytest.mark.parametrize("M,N", [(1021, 4092), (509, 4092), (500, 1990), (61, 260)])
def test_fp32_products_of_odd_and_even_numbers_of_k_tiles(M, N, K):
    """Each of the four fp32 tiles, one to seven k-tiles with remainders, ragged rows and columns: the chain of the plain
    kernel, so the same bits, with the epilogues that read (all of their reads are requested in front of the first
    product or behind the last) and with what an accumulated weight gradient starts from, over two segments as well."""
    A, B = bf_inputs.normal(23, 0, (M, K)), bf_inputs.normal(23, 1, (K, N), 0.05)
    bias, R = to_dev(bf_inputs.normal(23, 2, (N,), 0.5), False), _guarded(bf_inputs.normal(23, 3, (M, N)), False)
    gA, gB, gBt, gAt = (_guarded(np.ascontiguousarray(x), False) for x in (A, B, B.T, A.T))

    def both(call):
        outs = []
        for kernels in (bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN):
            out = torch.full((2, M * N + 128), 7.0, device="cuda")
            call(kernels, out[0][64:], out[1][64:])
            outs.append(out)
        assert bool((outs[0][:, :64] == 7.0).all()) and bool((outs[0][:, 64 + M * N:] == 7.0).all())
        assert torch.equal(outs[0], outs[1])
    for layout, op in ((bf.BF_NN, gB), (bf.BF_NT, gBt)):
        for epi in (bf.BF_EPI_BIAS_RES, bf.BF_EPI_BIAS_GELU, bf.BF_EPI_GELU_BWD):
            both(lambda kern, o, o2: bf.bf_op_gemm(bf.BF_FP32, kern, layout, epi, M, N, K, gA, op, o, bias=bias, R=R, C2=o2))
    both(lambda kern, o, o2: bf.bf_op_gemm(bf.BF_FP32, kern, bf.BF_TN, bf.BF_EPI_ACCUM, M, N, K, gAt, gB, o, accumulate=1))
    if K % 2 == 0:
        both(lambda kern, o, o2: bf.bf_op_wgrad(bf.BF_FP32, kern, M, N, K // 2, 2, gAt, K // 2 * M, gB, K // 2 * N, o))


@pytest.mark.parametrize("mode,dtype", MODES)
@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("poison", [False, True])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(1, 1, 1, 8), (1, 128, 4, 60), (2, 65, 2, 33), (2, 100, 3, 40), (1, 200, 20, 128), (3, 129, 30, 64), (1, 1900, 1, 16),
                                            (3, 65, 24, 33), (2, 100, 24, 40), (1, 200, 48, 16), (1, 500, 4, 60), (2, 48, 3, 20), (2, 32, 2, 100)])
def test_attention_on_the_fp32_matrix_instructions(mode, dtype, causal, poison, S_mb, S_seq, a, d):
    """The same bits as the plain kernels (ascending chains, the same order of every sum): tiles of 64 with remainders,
    16 and 32 rows per workgroup, odd head sizes, and infinities and NaN that the mask keeps from earlier rows.  (Few
    or short rows and small heads run forward on the plain kernels by themselves.)"""
    b16 = dtype == bf.BF_BF16
    if b16 and d in (64, 128):
        pytest.skip("bf16 heads of 64 and 128 run on the bf16 matrix instructions")
    h = a * d
    qkv, dctx = (bf_inputs.normal(31, i, (S_mb, S_seq, n * h), bf16=b16) for i, n in ((0, 3), (1, 1)))
    if poison and S_seq > 2:
        qkv[:, 2 * S_seq // 3, 2 * h + 3], qkv[:, 2 * S_seq // 3 + 1, h + 1] = np.inf, np.nan
        qkv[:, S_seq // 3, 5], dctx[:, S_seq // 2, 2] = -np.inf, np.nan
    dQKV, dDC = to_dev(qkv, b16), to_dev(dctx, b16)
    got = []
    for kernels in (bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN):
        ctx, dqkv = (torch.full((S_mb, S_seq, n * h), 7.0, dtype=_dt(b16), device="cuda") for n in (1, 3))
        lse, delta = (torch.full((S_mb, a, S_seq), 7.0, device="cuda") for _ in range(2))
        bf.bf_op_attention_fwd(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
        bf.bf_op_attention_bwd(dtype, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta)
        got.append((ctx, lse, dqkv))
    for x, y in zip(*got):
        assert torch.equal(torch.nan_to_num(x.float(), 123.0), torch.nan_to_num(y.float(), 123.0))


@pytest.mark.parametrize("M,N,K", [(256, 128, 4608), (1024, 1024, 4608), (1024, 2048, 8192)])
def test_split_contraction_of_few_tiles(M, N, K):
    """Long contractions of at most 512 tiles of 64 x 64: two slices on 64 x 64 tiles (up to 256 of them) or 256 x 128 ones,
    with the epilogue in the second pass.  The sums associate differently from the unsplit product's: fp32 rounding of
    the sum, then one bf16 rounding on either side, 2^-7."""
    A, B = bf_inputs.normal(16, 0, (M, K), bf16=True), bf_inputs.normal(16, 1, (K, N), 0.05, bf16=True)
    bias, R = bf_inputs.normal(16, 2, (N,), 0.5), bf_inputs.normal(16, 3, (M, N), bf16=True)
    dA, dB, dBt, dR, dbias = to_dev(A, True), to_dev(B, True), to_dev(np.ascontiguousarray(B.T), True), to_dev(R, True), to_dev(bias, False)
    planes = torch.full((2 * M * N,), float("nan"), dtype=torch.float32, device="cuda")
    want = A.astype(np.float64) @ B.astype(np.float64) + bias + R
    for layout, op in ((bf.BF_NN, dB), (bf.BF_NT, dBt)):
        out, ref = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        bf.bf_op_gemm_splitk(bf.BF_BF16, 0, layout, bf.BF_EPI_BIAS_RES, M, N, K, dA, op, out, bias=dbias, R=dR, planes=planes)
        bf.bf_op_gemm(bf.BF_BF16, 0, layout, bf.BF_EPI_BIAS_RES, M, N, K, dA, op, ref, bias=dbias, R=dR)
        assert bool(torch.isfinite(planes).all())   # both slices were run
        assert rel_err(to_host(out), want) <= TOL["bf16"] and rel_err(to_host(out), to_host(ref).astype(np.float64)) <= 2.0 ** -7


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(1, 2, 2, 64), (2, 63, 2, 64), (1, 65, 2, 128), (1, 129, 2, 128), (2, 300, 2, 64), (1, 255, 3, 128),
                                           (1, 451, 2, 128), (1, 257, 70, 64)])
def test_attention_of_any_length_in_bf16(causal, S_mb, S_seq, a, d):
    """Sequences that are not whole blocks of 128 on the bf16 matrix instructions, probabilities in three parts: no further
    from the oracle than the fp32 kernels that served them (2 % of the rounding of the outputs, which both share, for
    the chance of single roundings), nothing written outside, and finite wherever those are finite when infinities
    and NaN lie behind the mask."""
    h = a * d
    for poison in (False, True):
        qkv, dctx = (bf_inputs.normal(33, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
        if poison:
            qkv[:, S_seq - 1, 2 * h + 3], qkv[:, 2 * S_seq // 3, h + 1] = np.inf, np.nan
            qkv[:, S_seq // 3, 5], dctx[:, S_seq // 2, 2] = -np.inf, np.nan
        dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
        got = []
        for kernels in (bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN):
            ctx, dqkv = (torch.full((S_mb * S_seq * n * h + 64,), 7.0, dtype=torch.bfloat16, device="cuda") for n in (1, 3))
            lse, delta = (torch.full((S_mb * a * S_seq + 64,), 7.0, device="cuda") for _ in range(2))
            bf.bf_op_attention_fwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
            bf.bf_op_attention_bwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta)
            for t in (ctx, dqkv, lse, delta):
                assert bool((t[-64:] == 7.0).all())
            got.append([to_host(ctx[:-64].reshape(S_mb, S_seq, h)), to_host(dqkv[:-64].reshape(S_mb, S_seq, 3 * h)), to_host(lse[:-64])])
        if poison:
            for x, y in zip(*got):
                assert np.array_equal(np.isfinite(x), np.isfinite(y))
            continue
        ctx_ref, saved = L.attention_fwd(qkv.astype(np.float64), a, bool(causal))
        dqkv_ref = L.attention_bwd(dctx.astype(np.float64), saved, a)
        for x, y, ref in ((got[0][0], got[1][0], ctx_ref), (got[0][1], got[1][1], dqkv_ref)):
            off = [np.linalg.norm(t - ref) / np.linalg.norm(ref) for t in (x, y)]
            assert off[0] <= 1.02 * off[1] + 1e-6, off
        assert np.abs(got[0][2] - got[1][2]).max() <= 4e-6


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(1, 256, 2, 64), (1, 384, 1, 128), (2, 640, 1, 64), (1, 1024, 1, 128), (2, 1152, 1, 64)])
def test_attention_with_two_key_groups(causal, S_mb, S_seq, a, d):
    """Launches of few rows: two groups of waves share a row's key tiles and merge; odd and even numbers of tiles per block,
    rows that only one group sees a key of, and the folded partial column sums of dQ (4 and 2 rows into one)."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(35, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    qkv[..., :h] *= 3.0  # peaked rows: the two groups' maxima differ
    qkv = bf_inputs.round_bf16(qkv)
    ctx_ref, saved = L.attention_fwd(qkv.astype(np.float64), a, bool(causal))
    dqkv_ref = L.attention_bwd(dctx.astype(np.float64), saved, a)
    dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
    ctx, dqkv = (torch.full((S_mb, S_seq, n * h), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (1, 3))
    lse, delta = (torch.full((S_mb, a, S_seq), float("nan"), device="cuda") for _ in range(2))
    part = torch.full((bf.bf_op_attention_bwd_part_elems(S_mb, S_seq, a, d) + 64,), float("nan"), device="cuda")
    db = torch.full((3 * h,), float("nan"), device="cuda")
    bf.bf_op_attention_fwd(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
    bf.bf_op_attention_bwd_bias(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta, db, part, 0)
    assert bool(torch.isnan(part[-64:]).all())
    assert rel_err(to_host(ctx), ctx_ref) <= TOL["bf16"]
    for i in range(3):
        assert rel_err(to_host(dqkv)[..., i * h:(i + 1) * h], dqkv_ref[..., i * h:(i + 1) * h]) <= TOL["bf16"]
    assert rel_err(to_host(db), dqkv_ref.reshape(-1, 3 * h).sum(0)) <= TOL["bf16"]
    assert rel_err(to_host(db), to_host(dqkv).astype(np.float64).reshape(-1, 3 * h).sum(0)) <= 2.0 ** -8


def _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx):
    """ctx, lse, dqkv of a bf16 call by the kernels the sizes choose, and by the plain ones."""
    h = a * d
    dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
    got = []
    for kernels in (bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN):
        ctx, dqkv = (torch.full((S_mb, S_seq, n * h), 7.0, dtype=torch.bfloat16, device="cuda") for n in (1, 3))
        lse, delta = (torch.full((S_mb, a, S_seq), 7.0, device="cuda") for _ in range(2))
        bf.bf_op_attention_fwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
        bf.bf_op_attention_bwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta)
        got.append([to_host(t) for t in (ctx, lse, dqkv)])
    return got


# one and two key groups, whole lengths (128 and 256 rows per workgroup) and others
ATTENTION_FORMS = [(1, 128, 2, 128), (1, 256, 2, 64), (1, 384, 50, 128), (1, 256, 256, 64), (1, 1024, 2, 128), (1, 200, 2, 128), (1, 300, 2, 128),
                   (1, 300, 2, 64), (1, 451, 70, 128), (1, 451, 200, 64)]


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("keys", [(64, 65), (64, 128), (0, 64)])
@pytest.mark.parametrize("value", [-np.inf, -3.3895313892515355e38])
@pytest.mark.parametrize("S_mb,S_seq,a,d", ATTENTION_FORMS)
def test_attention_keys_without_a_finite_score(causal, keys, value, S_mb, S_seq, a, d):
    """Keys that hold -inf, or bf16's lowest value against a query component above 1 (the product overflows), score -inf: one
    key, a whole tile of 64, the first tile.  Results are finite exactly where the plain kernels' are (rows with no other
    key have none), and there within the bf16 bar of them."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(37, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    qkv[..., 5:h:d] = bf_inputs.round_bf16(np.abs(qkv[..., 5:h:d]) + np.float32(1.5))
    qkv[:, keys[0]:keys[1], h + 5:2 * h:d] = value
    got = _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx)
    for name, x, y in zip(("ctx", "lse", "dqkv"), *got):
        if name == "dqkv" and S_seq % 128 == 0 and np.isinf(value):  # dQ: the whole-length kernels contract masked pairs too, 0 x inf
            x, y = x[..., h:], y[..., h:]
        there = np.isfinite(y)
        assert np.array_equal(np.isfinite(x), there), (name, int((~np.isfinite(x)).sum()), int((~there).sum()))
        assert there.any() and np.abs(np.where(there, x, 0) - np.where(there, y, 0)).max() <= TOL["bf16"] * np.abs(y[there]).max(), name


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("where", ["q", "k", "v", "dctx"])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [f for f in ATTENTION_FORMS if f[1] % 128])
def test_attention_of_any_length_keeps_infinities(causal, where, S_mb, S_seq, a, d):
    """One infinite component per head: every output is an infinity of the same sign, a NaN or finite where the plain
    kernels' is (the parts of a probability must not all meet it, nor a masked pair)."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(39, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    if where == "dctx":
        dctx[:, S_seq // 3, 3::d] = np.inf
    else:
        part = "qkv".index(where)
        qkv[:, S_seq // 3, part * h + 3:(part + 1) * h:d] = np.inf
    got = _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx)
    for name, x, y in zip(("ctx", "lse", "dqkv"), *got):
        kind = [np.where(np.isnan(t), 2, np.where(np.isinf(t), np.sign(t), 0)) for t in (x, y)]
        assert np.array_equal(*kind), (name, [[int((k == c).sum()) for c in (-1, 1, 2)] for k in kind])


@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(1, 1000, 2, 64), (1, 1000, 2, 128), (1, 451, 70, 128), (1, 451, 200, 64)])
def test_attention_of_any_length_keeps_the_bits_of_probabilities(causal, S_mb, S_seq, a, d):
    """Nearly uniform rows over values that cancel: the outputs are the differences of the probabilities, 1e-3 of them, so
    that 16 bits of a probability show above the outputs' rounding.  No further from the oracle than the plain fp32
    kernels, 2 % for the chance of single roundings; neither is the log-sum-exp of ordinary rows, which is fp32."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(41, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    ordinary = _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx)
    q, k = (qkv[..., i * h:(i + 1) * h].astype(np.float64).reshape(S_mb, S_seq, a, d).transpose(0, 2, 1, 3) for i in (0, 1))
    s = np.matmul(q[:, :8], k[:, :8].transpose(0, 1, 3, 2)) / math.sqrt(d)
    if causal:
        s = np.where(np.tril(np.ones((S_seq, S_seq), dtype=bool)), s, -np.inf)
    lse = np.log(np.exp(s - s.max(-1, keepdims=True)).sum(-1)) + s.max(-1)
    off = [np.linalg.norm(got[1][:, :8] - lse) for got in ordinary]
    assert off[0] <= 1.02 * off[1], ("lse", off)
    sign = np.where(np.arange(S_seq) % 2, -1, 1).astype(np.float32)[None, :, None]
    qkv[..., :h] = bf_inputs.round_bf16(qkv[..., :h] * np.float32(2e-3))
    qkv[..., 2 * h:] = sign
    dctx[...] = sign
    ctx, saved = L.attention_fwd(qkv.astype(np.float64), a, bool(causal))
    dqkv = L.attention_bwd(dctx.astype(np.float64), saved, a)
    got = _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx)
    even = slice(1, None, 2)   # rows of an even number of keys, where the values cancel
    thirds = [("ctx", got[0][0][:, even], got[1][0][:, even], ctx[:, even])]
    thirds += [(n, *(t[..., i * h:(i + 1) * h] for t in (got[0][2], got[1][2], dqkv))) for i, n in enumerate(("dq", "dk", "dv"))]
    for name, x, y, ref in thirds:
        off = [np.linalg.norm(t - ref) / np.linalg.norm(ref) for t in (x, y)]
        assert off[0] <= 1.02 * off[1] + 1e-6, (name, off)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("causal,S_mb,S_seq,a", [(1, 2, 31, 3), (1, 1, 97, 2), (0, 1, 161, 2), (1, 1, 607, 2), (0, 2, 200, 32), (0, 1, 200, 65), (0, 1, 300, 96),
                                                 (1, 1, 140, 144), (1, 1, 140, 150), (0, 1, 140, 256), (1, 1, 140, 130), (1, 1, 140, 136), (1, 1, 140, 163),
                                                 (1, 1, 140, 164), (1, 1, 65, 217), (1, 1, 65, 218), (1, 1, 607, 84), (1, 1, 607, 110)])
def test_attention_backward_with_one_and_two_query_groups(d, causal, S_mb, S_seq, a):
    """The dK / dV kernel for any length with 64 and with 128 keys a workgroup, on both sides of what decides (rounds of 256
    workgroups; causal, the tiles per compute unit against the longest block's, 0.68 at S_head 64 and 0.85 to 1.25 here at 128), last blocks of 31, 33 and 64 keys and last query tiles with an empty second half.
    Against the plain kernels: fp32 sums in another order and one bf16 rounding on either side, 2^-7."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(47, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    got = _attention_by_both(S_mb, S_seq, a, d, causal, qkv, dctx)
    for i in range(3):
        x, y = (t[2][..., i * h:(i + 1) * h].astype(np.float64) for t in got)
        assert np.isfinite(x).all() and rel_err(x, y) <= 2.0 ** -7, i


@pytest.mark.parametrize("d,causal,S_mb,S_seq,a", [(128, 1, 6, 1024, 16), (128, 1, 4, 2048, 12), (128, 0, 4, 256, 64), (128, 0, 3, 768, 22)])
def test_attention_backward_is_the_same_bits_in_batches(d, causal, S_mb, S_seq, a):
    """dK / dV of a batch run on 256 keys a workgroup, of its sequences one by one on 128: the same roundings and sums, so the same
    bits; and the column sums' partial rows, in the batch's order, too."""
    h = a * d
    assert S_seq % 256 == 0
    qkv, dctx = (to_dev(bf_inputs.normal(67, i, (S_mb, S_seq, n * h), bf16=True), True) for i, n in ((0, 3), (1, 1)))
    ctx, lse = torch.empty_like(dctx), torch.empty((S_mb, a, S_seq), device="cuda")
    bf.bf_op_attention_fwd(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, qkv, ctx, lse)

    def backward(m0, m1):
        n = m1 - m0
        dqkv, delta = torch.empty_like(qkv[m0:m1]), torch.empty((n, a, S_seq), device="cuda")
        part = torch.zeros(bf.bf_op_attention_bwd_part_elems(n, S_seq, a, d), device="cuda")
        db = torch.empty(3 * h, device="cuda")
        bf.bf_op_attention_bwd_bias(bf.BF_BF16, 0, n, S_seq, a, d, causal, qkv[m0:m1], ctx[m0:m1], lse[m0:m1], dctx[m0:m1], dqkv, delta, db, part, 0)
        return dqkv, part

    dqkv, part = backward(0, S_mb)
    rows = S_mb * S_seq // 128                      # of [dK | dV], at the end of the partial rows
    kv = part[part.numel() - rows * 2 * h:].reshape(S_mb, -1)
    for m in range(S_mb):
        one, p1 = backward(m, m + 1)
        assert torch.equal(one[0, :, h:], dqkv[m, :, h:]), m
        assert torch.equal(p1[p1.numel() - kv.shape[1]:], kv[m]), m


@pytest.mark.parametrize("causal,S_mb,S_seq,a", [(1, 1, 384, 90), (1, 1, 640, 60), (1, 2, 1024, 20), (0, 2, 384, 50), (0, 3, 1024, 12), (1, 4, 128, 64),
                                                 (1, 5, 128, 52), (0, 5, 128, 52), (0, 4, 128, 64)])
def test_attention_backward_of_heads_of_64_in_large_launches(causal, S_mb, S_seq, a):
    """256 to 340 blocks of 128 keys: the dK / dV kernel of 32 keys a wave, and, in short rows, the one of eight waves in pairs.  A
    handful of heads against the oracle, and the bias gradient's partial rows against the sums of what was stored."""
    d, h = 64, a * 64
    qkv, dctx = (bf_inputs.normal(43, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
    ctx, dqkv = (torch.full((S_mb, S_seq, n * h), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (1, 3))
    lse, delta = (torch.full((S_mb, a, S_seq), float("nan"), device="cuda") for _ in range(2))
    part = torch.full((bf.bf_op_attention_bwd_part_elems(S_mb, S_seq, a, d) + 64,), float("nan"), device="cuda")
    db = torch.full((3 * h,), float("nan"), device="cuda")
    bf.bf_op_attention_fwd(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
    bf.bf_op_attention_bwd_bias(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta, db, part, 0)
    assert bool(torch.isnan(part[-64:]).all())
    for head in (0, 1, a // 2, a - 1):
        cols = slice(head * d, (head + 1) * d)
        one = np.concatenate([qkv[..., i * h:][..., cols] for i in range(3)], axis=-1).astype(np.float64)
        ref, saved = L.attention_fwd(one, 1, bool(causal))
        ref_d = L.attention_bwd(dctx[..., cols].astype(np.float64), saved, 1)
        assert rel_err(to_host(ctx)[..., cols], ref) <= TOL["bf16"]
        for i in range(3):
            assert rel_err(to_host(dqkv)[..., i * h:][..., cols], ref_d[..., i * d:(i + 1) * d]) <= TOL["bf16"], (head, i)
    assert rel_err(to_host(db), to_host(dqkv).astype(np.float64).reshape(-1, 3 * h).sum(0)) <= 2.0 ** -8


@pytest.mark.parametrize("causal,S_mb,S_seq,a", [(0, 66, 256, 2), (0, 1, 512, 70), (0, 3, 768, 20), (1, 2, 1024, 48), (1, 3, 1280, 24), (1, 1, 2048, 44)])
def test_attention_backward_on_256_key_workgroups(causal, S_mb, S_seq, a):
    """Heads of 128 in launches that fill the chip, of one key block per head to eight: a handful of heads against the oracle,
    and the bias gradient's partial rows (two per workgroup) against the sums of what was stored."""
    d, h = 128, a * 128
    qkv, dctx = (bf_inputs.normal(47, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
    ctx, dqkv = (torch.full((S_mb, S_seq, n * h), float("nan"), dtype=torch.bfloat16, device="cuda") for n in (1, 3))
    lse, delta = (torch.full((S_mb, a, S_seq), float("nan"), device="cuda") for _ in range(2))
    part = torch.full((bf.bf_op_attention_bwd_part_elems(S_mb, S_seq, a, d) + 64,), float("nan"), device="cuda")
    db = torch.full((3 * h,), float("nan"), device="cuda")
    bf.bf_op_attention_fwd(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
    bf.bf_op_attention_bwd_bias(bf.BF_BF16, 0, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta, db, part, 0)
    assert bool(torch.isnan(part[-64:]).all())
    got = to_host(dqkv)
    for m, head in ((0, 0), (S_mb - 1, 1), (S_mb // 2, a // 2), (S_mb - 1, a - 1)):
        cols = slice(head * d, (head + 1) * d)
        one = np.concatenate([qkv[m:m + 1, :, i * h:][..., cols] for i in range(3)], axis=-1).astype(np.float64)
        ref, saved = L.attention_fwd(one, 1, bool(causal))
        ref_d = L.attention_bwd(dctx[m:m + 1, :, cols].astype(np.float64), saved, 1)
        for i in range(3):
            assert rel_err(got[m:m + 1, :, i * h:][..., cols], ref_d[..., i * d:(i + 1) * d]) <= TOL["bf16"], (m, head, i)
    assert rel_err(to_host(db), got.astype(np.float64).reshape(-1, 3 * h).sum(0)) <= 2.0 ** -8


@pytest.mark.parametrize("M,N,K", [(1, 8, 1024), (100, 72, 1032), (65, 64, 4104), (128, 256, 4224), (1000, 1000, 4096), (1100, 1000, 1032), (1030, 1024, 2048)])
def test_gemm_of_few_tiles_by_groups_of_waves(M, N, K):
    """Two and four groups of waves on the k-tiles of one output tile: contractions that leave a group with fewer of them than
    the others, output tiles that are mostly empty, both tiles, every epilogue of the forward and dgrad layouts."""
    A, B = bf_inputs.normal(61, 0, (M, K), bf16=True), bf_inputs.normal(61, 1, (K, N), 0.05, bf16=True)
    bias, R = bf_inputs.normal(61, 2, (N,), 0.5), bf_inputs.normal(61, 3, (M, N), bf16=True)
    dA, dB, dBt, dR, dbias = to_dev(A, True), to_dev(B, True), to_dev(np.ascontiguousarray(B.T), True), to_dev(R, True), to_dev(bias, False)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    r64 = R.astype(np.float64)
    u = to_host(to_dev(acc + bias, True)).astype(np.float64)
    for layout, op, epi, want in ((bf.BF_NN, dB, bf.BF_EPI_NONE, acc), (bf.BF_NN, dB, bf.BF_EPI_BIAS_RES, acc + bias + r64),
                                  (bf.BF_NN, dB, bf.BF_EPI_BIAS_GELU, acc + bias), (bf.BF_NT, dBt, bf.BF_EPI_NONE, acc),
                                  (bf.BF_NT, dBt, bf.BF_EPI_GELU_BWD, acc * L.gelu_grad(r64))):
        out, out2 = (torch.full((M + 1, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        bf.bf_op_gemm(bf.BF_BF16, 0, layout, epi, M, N, K, dA, op, out, bias=dbias, R=dR, C2=out2)
        assert rel_err(to_host(out[:M]), want) <= TOL["bf16"], (layout, epi)
        if epi == bf.BF_EPI_BIAS_GELU:
            assert rel_err(to_host(out2[:M]), L.gelu(u)) <= TOL["bf16"]
        assert bool(torch.isnan(out[M:]).all()) and bool(torch.isnan(out2[M:]).all())


@pytest.mark.parametrize("M,N,K,n_seg,gap", [(8, 8, 512, 1, 0), (72, 40, 584, 1, 0), (64, 128, 200, 3, 0), (64, 128, 200, 3, 64), (1000, 1024, 520, 1, 0)])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_weight_gradient_of_few_tiles_by_groups_of_waves(M, N, K, n_seg, gap, accumulate):
    """The same in the weight-gradient layout, added to or not, over segments that follow each other without a gap (one
    contraction, and long enough only as one) or with one."""
    X, dY = bf_inputs.normal(62, 0, (n_seg, K * M + gap), bf16=True), bf_inputs.normal(62, 1, (n_seg, K * N + gap), bf16=True)
    G = torch.full((M + 1, N), 2.0, device="cuda")
    bf.bf_op_wgrad(bf.BF_BF16, 0, M, N, K, n_seg, to_dev(X, True), K * M + gap, to_dev(dY, True), K * N + gap, G, accumulate=accumulate)
    x, d = (t[:, :K * w].astype(np.float64).reshape(n_seg * K, w) for t, w in ((X, M), (dY, N)))
    assert rel_err(to_host(G)[:M], x.T @ d + 2.0 * accumulate) <= 1e-5
    assert bool((G[M:] == 2.0).all())


@pytest.mark.parametrize("layout,epi,M,N,K", [(bf.BF_NT, bf.BF_EPI_NONE, 2048, 8320, 1536), (bf.BF_NN, bf.BF_EPI_BIAS_RES, 2048, 8320, 1536),
                                              (bf.BF_NN, bf.BF_EPI_BIAS_GELU, 1024, 16640, 1536), (bf.BF_NT, bf.BF_EPI_GELU_BWD, 2048, 8320, 1536),
                                              (bf.BF_TN, bf.BF_EPI_ACCUM, 8576, 2048, 1536), (bf.BF_TN, bf.BF_EPI_ACCUM, 16768, 1024, 2048)])
def test_gemm_in_whole_rounds_and_a_rest(layout, epi, M, N, K):
    """A round of 256 x 256 tiles over the chip and one, two or three blocks of 128 rows or columns more, which run as a launch of
    their own: against fp32 products of the same operands on either side of the seam, and the first and last of both."""
    g = torch.Generator(device="cuda").manual_seed(63)
    mk = lambda *s, sc=1.0: (torch.randn(s, generator=g, device="cuda") * sc).bfloat16()
    A, B = mk(*((K, M) if layout == bf.BF_TN else (M, K))), mk(*((N, K) if layout == bf.BF_NT else (K, N)), sc=0.05)
    bias, R = torch.randn(N, generator=g, device="cuda"), mk(M, N)
    out = torch.full((M, N), 1.0 if epi == bf.BF_EPI_ACCUM else float("nan"), dtype=torch.float32 if epi == bf.BF_EPI_ACCUM else torch.bfloat16, device="cuda")
    out2 = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    bf.bf_op_gemm(bf.BF_BF16, 0, layout, epi, M, N, K, A, B, out, bias=bias, R=R, C2=out2, accumulate=1)
    a32, b32 = (A.t() if layout == bf.BF_TN else A).float(), (B.t() if layout == bf.BF_NT else B).float()
    assert bool(torch.isfinite(out).all())
    for rows, cols in ((slice(0, 300), slice(0, 300)), (slice(M - 700, M), slice(N - 700, N)), (slice(M - 700, M), slice(0, 200)), (slice(0, 200), slice(N - 700, N))):
        want = a32[rows] @ b32[:, cols]
        if epi == bf.BF_EPI_ACCUM:
            want = want + 1.0
        if epi in (bf.BF_EPI_BIAS_RES, bf.BF_EPI_BIAS_GELU):
            want = want + bias[cols]
        if epi == bf.BF_EPI_BIAS_RES:
            want = want + R[rows, cols].float()
        if epi == bf.BF_EPI_GELU_BWD:
            want = want * torch.from_numpy(L.gelu_grad(to_host(R[rows, cols]).astype(np.float64))).float().cuda()
        tol = 1e-5 if epi == bf.BF_EPI_ACCUM else TOL["bf16"]
        assert rel_err(to_host(out[rows, cols]), to_host(want)) <= tol, (rows, cols)
        if epi == bf.BF_EPI_BIAS_GELU:
            assert rel_err(to_host(out2[rows, cols]), L.gelu(to_host(out[rows, cols]).astype(np.float64))) <= TOL["bf16"]


@pytest.mark.parametrize("M,N,K", [(256, 256, 16384), (512, 256, 16512), (256, 512, 50304)])
def test_very_long_contraction_in_slices_on_large_tiles(M, N, K):
    """Contractions of a vocabulary's length in more than two slices, all of whose planes are used; with room for two planes only,
    and for one, in two and unsplit."""
    s = bf.bf_op_gemm_splitk_slices(bf.BF_NN, bf.BF_EPI_BIAS_RES, M, N, K)
    assert s > 2 and K % (64 * s) == 0
    g = torch.Generator(device="cuda").manual_seed(64)
    A, B = torch.randn((M, K), generator=g, device="cuda").bfloat16(), (torch.randn((K, N), generator=g, device="cuda") * 0.02).bfloat16()
    Bt, bias, R = B.t().contiguous(), torch.randn(N, generator=g, device="cuda"), torch.randn((M, N), generator=g, device="cuda").bfloat16()
    acc = to_host(A).astype(np.float64) @ to_host(B).astype(np.float64)
    for layout, op, epi, want in ((bf.BF_NN, B, bf.BF_EPI_BIAS_RES, acc + to_host(bias) + to_host(R)), (bf.BF_NT, Bt, bf.BF_EPI_NONE, acc)):
        for n in (s, 2, 1):
            planes = torch.full((n, M, N), float("nan"), device="cuda")
            out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
            bf.bf_op_gemm_splitk(bf.BF_BF16, 0, layout, epi, M, N, K, A, op, out, bias=bias, R=R, planes=planes.reshape(-1))
            assert bool(torch.isfinite(planes).all()) if n > 1 else bool(torch.isnan(planes).all())
            assert rel_err(to_host(out), want) <= TOL["bf16"], (layout, n)


@pytest.mark.parametrize("dtype,layout,M,N", [(bf.BF_BF16, bf.BF_TN, 128, 128), (bf.BF_BF16, bf.BF_TN, 72, 40), (bf.BF_BF16, bf.BF_NN, 128, 128),
                                              (bf.BF_BF16, bf.BF_NT, 128, 256), (bf.BF_FP32, bf.BF_TN, 40, 36)])
def test_gemm_of_few_tiles_over_more_than_two_million(dtype, layout, M, N):
    """Contractions longer than the 32-bit offsets of the small-tile kernel's rows reach, in layouts where K is a row's length
    and in the weight gradient's, where it is not: still on the matrix cores.  Ones in A and small whole numbers in B: every
    partial sum is exact, in any order.  That the vector kernel did not run shows in random bf16 values, whose sums round
    differently there (in fp32 the bits are the same, so only the sums are looked at)."""
    K = 2 ** 21 + 128
    td = torch.bfloat16 if dtype == bf.BF_BF16 else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    B = torch.randint(-2, 3, (K, N), generator=gen, device="cuda").to(td)
    A = torch.ones((K, M), device="cuda", dtype=td)
    def run(kernels, A, B):
        out = torch.full((M, N), float("nan"), dtype=torch.float32 if layout == bf.BF_TN else td, device="cuda")
        a, b = (A if layout == bf.BF_TN else A.t().contiguous()), (B.t().contiguous() if layout == bf.BF_NT else B)
        bf.bf_op_gemm(dtype, kernels, layout, bf.BF_EPI_ACCUM if layout == bf.BF_TN else bf.BF_EPI_NONE, M, N, K, a, b, out, accumulate=0)
        return out
    want = B.float().sum(0).to(torch.float32 if layout == bf.BF_TN else td).expand(M, N)
    assert torch.equal(run(bf.BF_KERNELS_AUTO, A, B), want)
    if dtype == bf.BF_BF16 and layout == bf.BF_TN:
        B = torch.randn((K, N), generator=gen, device="cuda").to(td)
        A = torch.randn((K, M), generator=gen, device="cuda").to(td)
        auto, plain = run(bf.BF_KERNELS_AUTO, A, B), run(bf.BF_KERNELS_PLAIN, A, B)
        assert rel_err(to_host(auto), to_host(plain).astype(np.float64)) <= 1e-4 and not torch.equal(auto, plain)


@pytest.mark.parametrize("K", [64, 128, 192])
@pytest.mark.parametrize("M,N,tile", [(384, 8192, (128, 128)), (512, 4224, (256, 128)), (2048, 8192, (256, 256))])
def test_gemm_on_whole_tiles(M, N, tile, K):
    """Each whole tile of the MFMA kernel on products of more tiles than the small-tile form takes: every layout and
    epilogue, the column sums from the epilogue's partial rows (one per row of tiles, which shows that it ran) and
    without them, and the weight gradient over three segments with a gap, 1 to 3 k-tiles each (a power of two or not)."""
    for layout, epi in ((bf.BF_NN, bf.BF_EPI_NONE), (bf.BF_NN, bf.BF_EPI_BIAS_GELU), (bf.BF_NT, bf.BF_EPI_GELU_BWD), (bf.BF_TN, bf.BF_EPI_ACCUM)):
        assert bf.bf_op_gemm_tile(layout, epi, M, N, K) == tile and (M // 64) * (N // 64) > 512
    A, B = bf_inputs.normal(51, 0, (M, K), bf16=True), bf_inputs.normal(51, 1, (K, N), 0.05, bf16=True)
    bias, R = bf_inputs.normal(51, 2, (N,), 0.5), bf_inputs.normal(51, 3, (M, N), bf16=True)
    acc, R64 = A.astype(np.float64) @ B.astype(np.float64), R.astype(np.float64)
    dA, dB, dBt, dR, dbias = to_dev(A, True), to_dev(B, True), to_dev(np.ascontiguousarray(B.T), True), to_dev(R, True), to_dev(bias, False)
    grad = acc * L.gelu_grad(R64)
    for layout, op in ((bf.BF_NN, dB), (bf.BF_NT, dBt)):
        for epi, ref in ((bf.BF_EPI_NONE, acc), (bf.BF_EPI_BIAS, acc + bias), (bf.BF_EPI_BIAS_RES, acc + bias + R64),
                         (bf.BF_EPI_BIAS_GELU, acc + bias), (bf.BF_EPI_GELU_BWD, grad)):
            out, out2 = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(2))
            bf.bf_op_gemm(bf.BF_BF16, 0, layout, epi, M, N, K, dA, op, out, bias=dbias, R=dR, C2=out2)
            assert rel_err(to_host(out), ref) <= TOL["bf16"], (layout, epi)
            if epi == bf.BF_EPI_BIAS_GELU:
                assert rel_err(to_host(out2), L.gelu(acc + bias)) <= TOL["bf16"]
    for with_part in (True, False):
        out, db = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda"), torch.full((N,), float("nan"), device="cuda")
        part = torch.full(((M + 127) // 128, N), float("nan"), device="cuda") if with_part else None
        bf.bf_op_gemm_gelu_bwd_colsum(bf.BF_BF16, 0, M, N, K, dA, dBt, out, dR, db, part)
        assert rel_err(to_host(out), grad) <= TOL["bf16"]
        assert rel_err(to_host(db), to_host(out).astype(np.float64).sum(0)) <= 1e-5
        if with_part:
            written = torch.isfinite(part).all(1).cpu().numpy()
            assert np.array_equal(written, np.arange(len(written)) < M // tile[0])
    n_seg, gap = 3, 64
    sx, sy = K * M + gap, K * N + gap
    X, dY = bf_inputs.normal(53, 0, (n_seg * sx,), bf16=True), bf_inputs.normal(53, 1, (n_seg * sy,), 0.3, bf16=True)
    G_ref, db_ref = np.zeros((M, N)), np.zeros(N)
    for i in range(n_seg):
        dYi = dY[i * sy:i * sy + K * N].reshape(K, N).astype(np.float64)
        G_ref += X[i * sx:i * sx + K * M].reshape(K, M).astype(np.float64).T @ dYi
        db_ref += dYi.sum(0)
    G, db = torch.full((M, N), float("nan"), device="cuda"), torch.full((N,), float("nan"), device="cuda")
    for accumulate in (0, 1):
        bf.bf_op_wgrad(bf.BF_BF16, 0, M, N, K, n_seg, to_dev(X, True), sx, to_dev(dY, True), sy, G, db, accumulate=accumulate)
        assert rel_err(to_host(G), (1 + accumulate) * G_ref) <= 1e-5 and rel_err(to_host(db), (1 + accumulate) * db_ref) <= 1e-5


def _check_heads(S_mb, S_seq, a, d, causal, poison=False):
    """Forward and backward of a launch of many heads, four of them against the oracle (or, with infinities and NaN behind the
    mask, against where the plain kernels are finite)."""
    h = a * d
    qkv, dctx = (bf_inputs.normal(57, i, (S_mb, S_seq, n * h), bf16=True) for i, n in ((0, 3), (1, 1)))
    if poison:
        qkv[:, S_seq - 1, 2 * h + 3::d], qkv[:, 2 * S_seq // 3, h + 1:2 * h:d] = np.inf, np.nan
        qkv[:, S_seq // 3, 5:h:d], dctx[:, S_seq // 2, 2::d] = -np.inf, np.nan
    dQKV, dDC = to_dev(qkv, True), to_dev(dctx, True)
    got = []
    for kernels in ((bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN) if poison else (bf.BF_KERNELS_AUTO,)):
        ctx, dqkv = (torch.full((S_mb, S_seq, n * h), 7.0, dtype=torch.bfloat16, device="cuda") for n in (1, 3))
        lse, delta = (torch.full((S_mb, a, S_seq), 7.0, device="cuda") for _ in range(2))
        bf.bf_op_attention_fwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse)
        bf.bf_op_attention_bwd(bf.BF_BF16, kernels, S_mb, S_seq, a, d, causal, dQKV, ctx, lse, dDC, dqkv, delta)
        got.append([to_host(t) for t in (ctx, dqkv, lse)])
    if poison:
        for x, y in zip(*got):
            assert np.array_equal(np.isfinite(x), np.isfinite(y))
        return
    for head in (0, 1, a // 2, a - 1):
        cols = slice(head * d, (head + 1) * d)
        one = np.concatenate([qkv[..., i * h:][..., cols] for i in range(3)], axis=-1).astype(np.float64)
        ref, saved = L.attention_fwd(one, 1, bool(causal))
        ref_d = L.attention_bwd(dctx[..., cols].astype(np.float64), saved, 1)
        assert rel_err(got[0][0][..., cols], ref) <= TOL["bf16"], head
        for i in range(3):
            assert rel_err(got[0][1][..., i * h:][..., cols], ref_d[..., i * d:(i + 1) * d]) <= TOL["bf16"], (head, i)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(2, 451, 33, 128), (2, 451, 70, 64), (1, 1000, 80, 64), (2, 1000, 16, 128), (1, 770, 70, 64), (1, 300, 64, 128),
                                            (1, 300, 65, 128)])
@pytest.mark.parametrize("poison", [False, True])
def test_attention_of_any_length_in_large_launches(causal, poison, S_mb, S_seq, a, d):
    """Both sides of the numbers of blocks up to which a row's keys go to two groups: 264 and 560 blocks of 128 rows
    (one group in both passes), 640, 256, 490, and 192 / 195 of short rows."""
    _check_heads(S_mb, S_seq, a, d, causal, poison)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_mb,S_seq,a,d", [(4, 1024, 16, 64), (1, 1024, 70, 64), (1, 384, 90, 128), (1, 384, 180, 64), (1, 1024, 40, 128), (1, 1024, 41, 128),
                                            (1, 256, 65, 128), (1, 384, 44, 128)])
def test_attention_of_whole_blocks_in_large_launches(causal, S_mb, S_seq, a, d):
    """The 256-row kernels with heads of 64 (512 and 560 blocks), the 128-row ones over several blocks of both head sizes, and
    both sides of the numbers of blocks that two key groups serve (320 / 328 forward, 130 at S_seq 256 and 132 at 384 for dQ)."""
    _check_heads(S_mb, S_seq, a, d, causal)


@pytest.mark.parametrize("causal", [1, 0])
@pytest.mark.parametrize("S_seq,a,d", [(2176, 1, 64), (2177, 1, 64), (1856, 2, 128), (1857, 2, 128), (4096, 1, 64), (4096, 1, 128)])
def test_fp32_attention_at_the_limits_of_the_scores_in_lds(causal, S_seq, a, d):
    """The longest rows whose scores fit the forward kernel's LDS, one past them (the plain kernel), and the longest rows
    there are: the same bits as the plain kernels, forward and backward."""
    h = a * d
    qkv, dctx = (to_dev(bf_inputs.normal(59, i, (1, S_seq, n * h)), False) for i, n in ((0, 3), (1, 1)))
    got = []
    for kernels in (bf.BF_KERNELS_AUTO, bf.BF_KERNELS_PLAIN):
        ctx, dqkv = (torch.full((1, S_seq, n * h), 7.0, device="cuda") for n in (1, 3))
        lse, delta = (torch.full((1, a, S_seq), 7.0, device="cuda") for _ in range(2))
        bf.bf_op_attention_fwd(bf.BF_FP32, kernels, 1, S_seq, a, d, causal, qkv, ctx, lse)
        bf.bf_op_attention_bwd(bf.BF_FP32, kernels, 1, S_seq, a, d, causal, qkv, ctx, lse, dctx, dqkv, delta)
        got.append((ctx, lse, dqkv))
    for x, y in zip(*got):
        assert torch.equal(x, y)
