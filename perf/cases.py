"""Workloads by which the speed of this framework is judged, through the entry points a program calls.

Two are whole training steps; the others are the layers and blocks that such steps consist of (attention, the
two-layer MLP, LayerNorm, the language-model head and the embedding), each forward and backward, in the data types
the framework has (bf16 with fp32 main-grads, and fp32), at sizes from launch-bound to chip-filling and at sequence
lengths that are not multiples of anything.

Sizes are those of the benchmark's configurations (256-, 2048- and 8192-wide stacks, S_seq 128, 1024 and 2048, a
50304-word vocabulary) or generic ones beside them.

listed() gives the cases, draw(rng) more of the same ranges; prepare / run / exact / work / tolerance are described
at each function."""
import math

import numpy as np
import torch

import paper_2211_05953_amd as bf

DEV = "cuda:0"
LR, BETA1, BETA2, ADAM_EPS, LN_EPS = 1e-5, 0.9, 0.999, 1e-8, 1e-5


def listed():
    return [
        # The smallest stack the framework is used with: 4 layers of 256 in fp32, breadth-first, optimizer included.
        # Every launch is a few microseconds of work: launch count and latency decide.
        {"name": "step_fp32_256", "kind": "step", "dtype": "fp32", "layers": 4, "loop": 2, "hidden": 256, "heads": 4, "mlp": 1024,
         "seq": 128, "mb": 4, "smb": 1, "order": "bf", "causal": 1},
        # One training step of the 1.3B-shaped rank share (6 layers in 3 stages, 8 micro-batches of 2048 tokens) in
        # breadth-first order with the stage-wide weight gradients and the optimizer: the whole path at once.
        {"name": "step_bf16_2048", "kind": "step", "dtype": "bf16", "layers": 6, "loop": 3, "hidden": 2048, "heads": 16, "mlp": 8192,
         "seq": 2048, "mb": 8, "smb": 1, "order": "bf", "causal": 1},
        # Attention of one layer of the 52B-shaped stack: causal, 64 heads of 128, forward and backward with the QKV bias
        # gradient.
        {"name": "attention_causal_2048", "kind": "attention", "dtype": "bf16", "smb": 1, "seq": 2048, "heads": 64, "head": 128, "causal": 1},
        # Attention as a bidirectional encoder has it: S_seq 1024, heads of 64, a micro-batch of 4 sequences.
        {"name": "attention_bidir_1024", "kind": "attention", "dtype": "bf16", "smb": 4, "seq": 1024, "heads": 16, "head": 64, "causal": 0},
        # Sequences of a length nobody rounded up.
        {"name": "attention_ragged_1000", "kind": "attention", "dtype": "bf16", "smb": 2, "seq": 1000, "heads": 16, "head": 128, "causal": 1},
        # The MLP of one 8192-wide layer on one micro-batch: both products forward, both input gradients, both weight
        # gradients, bias gradients.  The largest products there are.
        {"name": "mlp_8192", "kind": "mlp", "dtype": "bf16", "tokens": 2048, "hidden": 8192, "mlp": 32768},
        # The MLP of a 2048-wide layer on a ragged number of tokens.
        {"name": "mlp_ragged_1000", "kind": "mlp", "dtype": "bf16", "tokens": 1000, "hidden": 2048, "mlp": 8192},
        # The MLP in full fp32 precision.
        {"name": "mlp_fp32_1024", "kind": "mlp", "dtype": "fp32", "tokens": 512, "hidden": 1024, "mlp": 4096},
        # LayerNorm forward and backward (input gradient with the residual, gain / bias gradients, bias gradient of the
        # layer below) of an 8192-wide layer on one micro-batch.
        {"name": "norm_8192", "kind": "norm", "dtype": "bf16", "tokens": 2048, "hidden": 8192},
        # The same of the smallest stack: pure launch latency.
        {"name": "norm_fp32_256", "kind": "norm", "dtype": "fp32", "tokens": 128, "hidden": 256},
        # Language-model head of a 2048-wide model on one micro-batch: 50304 logits per token, cross-entropy, and the
        # gradients of its input and its weights.
        {"name": "head_50304", "kind": "head", "dtype": "bf16", "tokens": 2048, "hidden": 2048, "vocab": 50304},
        # Token and position embedding of that model, forward and backward, on Zipf-distributed token ids.
        {"name": "embedding_50304", "kind": "embedding", "dtype": "bf16", "smb": 1, "seq": 2048, "hidden": 2048, "vocab": 50304},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult(v, m):
    return max(m, v // m * m)


def draw(rng):
    kind = rng.choice(["step", "attention", "mlp", "norm", "head", "embedding"])
    dtype = rng.choice(["bf16", "bf16", "fp32"])
    if kind == "step":
        loop, per = rng.choice([1, 2, 3]), rng.choice([1, 2])
        head = rng.choice([64, 128])
        heads = _log(rng, 2, 16 if dtype == "bf16" else 8)
        hidden = min(heads * head, 2048 if dtype == "bf16" else 1024)
        seq = rng.choice([128, 256, 512, 1024, _log(rng, 96, 700)]) if dtype == "bf16" else rng.choice([128, 256, _log(rng, 64, 300)])
        return {"kind": kind, "dtype": dtype, "layers": loop * per, "loop": loop, "hidden": hidden, "heads": hidden // head,
                "mlp": 4 * hidden, "seq": seq, "mb": rng.choice([2, 3, 4]), "smb": rng.choice([1, 2]), "order": rng.choice(["bf", "bf", "df"]),
                "causal": rng.choice([1, 1, 0])}
    if kind == "attention":
        head = rng.choice([64, 128])
        heads = _log(rng, 4, 64 if dtype == "bf16" else 16)
        seq = rng.choice([128, 256, 512, 1024, 2048, _log(rng, 64, 2048), _log(rng, 64, 2048)])
        if dtype == "fp32":
            seq = min(seq, 512 + seq % 2)
        smb = max(1, min(rng.choice([1, 2, 4]), 2 ** 27 // (heads * seq * seq)))
        return {"kind": kind, "dtype": dtype, "smb": smb, "seq": seq, "heads": heads, "head": head, "causal": rng.choice([1, 1, 0])}
    if kind == "mlp":
        hidden = _mult(_log(rng, 256, 4096 if dtype == "bf16" else 1536), rng.choice([8, 64, 256]))
        tokens = rng.choice([_log(rng, 64, 4096), _mult(_log(rng, 128, 4096), 128)])
        tokens = max(64, min(tokens, int((5e11 if dtype == "bf16" else 8e10) / (48 * hidden * hidden))))
        return {"kind": kind, "dtype": dtype, "tokens": tokens, "hidden": hidden, "mlp": 4 * hidden}
    if kind == "norm":
        return {"kind": kind, "dtype": dtype, "tokens": _log(rng, 64, 4096), "hidden": _mult(_log(rng, 256, 8192), rng.choice([8, 64, 256]))}
    if kind == "head":
        hidden = _mult(_log(rng, 256, 1536 if dtype == "bf16" else 512), rng.choice([64, 128]))
        vocab = rng.choice([50304, 32000, _mult(_log(rng, 1000, 50000), 8)])
        tokens = rng.choice([_log(rng, 64, 2048), _mult(_log(rng, 128, 2048), 128)])
        tokens = max(64, min(tokens, int((3e11 if dtype == "bf16" else 4e10) / (6 * hidden * vocab))))
        return {"kind": kind, "dtype": dtype, "tokens": tokens, "hidden": hidden, "vocab": vocab}
    return {"kind": kind, "dtype": dtype, "smb": rng.choice([1, 1, 2, 4]), "seq": rng.choice([128, 512, 1024, 2048, _log(rng, 64, 2048)]),
            "hidden": _mult(_log(rng, 256, 2048), rng.choice([8, 64, 256])), "vocab": rng.choice([50304, 32000, _log(rng, 1000, 50000)])}


# ------------------------------------------------------------------------------------------------------ inputs
class _Draw:
    """Seeded normal draws on the GPU, rounded to the case's storage type."""

    def __init__(self, case, seed):
        self.gen = torch.Generator(device=DEV)
        self.gen.manual_seed(int(seed) * 1000003 + 12345)
        self.td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def act(self, *shape, std=1.0):
        return (torch.randn(shape, generator=self.gen, device=DEV) * std).to(self.td)

    def f32(self, *shape, std=1.0, mean=0.0):
        """fp32 values that the storage type holds exactly (a master weight and its low-precision copy agree)."""
        return (torch.randn(shape, generator=self.gen, device=DEV) * std + mean).to(self.td).float()

    def tokens(self, shape, vocab):
        """Zipf-distributed ids (exponent 1.1) over a shuffled vocabulary."""
        p = torch.arange(1, vocab + 1, device=DEV, dtype=torch.float64).pow(-1.1)
        n = int(np.prod(shape))
        rank = torch.searchsorted(torch.cumsum(p / p.sum(), 0), torch.rand(n, generator=self.gen, device=DEV, dtype=torch.float64)).clamp_(max=vocab - 1)
        return torch.randperm(vocab, generator=self.gen, device=DEV)[rank].to(torch.int32).reshape(shape)


TENSORS = ("ln1_g", "ln1_b", "w_qkv", "b_qkv", "w_o", "b_o", "ln2_g", "ln2_b", "w_fc1", "b_fc1", "w_fc2", "b_fc2")


def _shapes(case):
    h, f = case["hidden"], case["mlp"]
    return {"ln1_g": (h,), "ln1_b": (h,), "w_qkv": (h, 3 * h), "b_qkv": (3 * h,), "w_o": (h, h), "b_o": (h,), "ln2_g": (h,), "ln2_b": (h,),
            "w_fc1": (h, f), "b_fc1": (f,), "w_fc2": (f, h), "b_fc2": (h,)}


def _inputs(case, seed):
    """Every input of a case, from the seed alone: activations and incoming gradients ~ N(0, 1), weights ~ N(0, 0.02),
    biases and LayerNorm parameters as a trained model has them (not zero, not one)."""
    d, k = _Draw(case, seed), case["kind"]
    if k == "step":
        sh = _shapes(case)
        params = [{n: d.f32(*sh[n], std=0.02, mean=1.0 if n.endswith("_g") else 0.0) for n in TENSORS} for _ in range(case["layers"])]
        io = (case["mb"], case["smb"], case["seq"], case["hidden"])
        return {"params": params, "x": d.act(*io), "dy": d.act(*io)}
    if k == "attention":
        h = case["heads"] * case["head"]
        return {"qkv": d.act(case["smb"], case["seq"], 3 * h), "dctx": d.act(case["smb"], case["seq"], h)}
    if k == "mlp":
        t, h, f = case["tokens"], case["hidden"], case["mlp"]
        return {"c": d.act(t, h), "x1": d.act(t, h), "dy": d.act(t, h), "w1": d.act(h, f, std=0.02), "w2": d.act(f, h, std=0.02),
                "b1": d.f32(f, std=0.02), "b2": d.f32(h, std=0.02)}
    if k == "norm":
        t, h = case["tokens"], case["hidden"]
        return {"x": d.act(t, h), "dy": d.act(t, h), "dres": d.act(t, h), "g": d.f32(h, std=0.02, mean=1.0), "b": d.f32(h, std=0.02)}
    if k == "head":
        t, h, v = case["tokens"], case["hidden"], case["vocab"]
        return {"hn": d.act(t, h), "w": d.act(v, h, std=0.02), "labels": d.tokens((t,), v)}
    t, h, v = (case["smb"], case["seq"]), case["hidden"], case["vocab"]
    return {"tokens": d.tokens(t, v), "e_tok": torch.randn((v, h), generator=d.gen, device=DEV) * 0.02,
            "e_pos": torch.randn((case["seq"], h), generator=d.gen, device=DEV) * 0.02, "d": d.act(*t, h)}


# ----------------------------------------------------------------------------------------------------- prepare
def _planes(dt, layout, epi, m, n, k):
    """The scratch a program lends bf_op_gemm_splitk, as the library asks for it."""
    s = bf.bf_op_gemm_splitk_slices(layout, epi, m, n, k) if dt == bf.BF_BF16 else 1
    return torch.empty(s * m * n, device=DEV) if s > 1 else None


def prepare(case, seed):
    """What a program has in hand before the call: inputs, weights, the stack, output buffers and scratch."""
    i, k = _inputs(case, seed), case["kind"]
    s = {"case": case, "kind": k, "dt": bf.BF_BF16 if case["dtype"] == "bf16" else bf.BF_FP32}
    s.update({n: v for n, v in i.items() if n != "params"})
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def act(*shape):
        return torch.empty(shape, device=DEV, dtype=td)

    def f32(*shape):
        return torch.empty(shape, device=DEV)

    if k == "step":
        cfg = bf.make_config(case["hidden"], case["heads"], case["mlp"], case["seq"], case["layers"], case["mb"], case["smb"], dtype=s["dt"],
                             causal=case["causal"], lr=LR, fuse_wgrad=1, N_loop_min=case["loop"], seed=int(seed) + 1)
        s["stack"] = bf.Stack(cfg, device=DEV)
        for l, p in enumerate(i["params"]):
            for n in TENSORS:
                s["stack"].bf_set_params(l, bf.TENSOR_IDS[n], p[n].reshape(-1).cpu().numpy())
        s["y"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
        s["order"] = bf.BF_SCHED_BF if case["order"] == "bf" else bf.BF_SCHED_DF
        # where the workspace keeps master weights, moments and main-grads: [w32 | m | v | g32], each arena one block of
        # equally laid out layers whose tensors are padded to 128 elements, arenas padded to 256 bytes
        offs, off = {}, 0
        for n in TENSORS:
            offs[n] = off
            off += -(-int(np.prod(_shapes(case)[n])) // 128) * 128
        arena = -(-off * case["layers"] * 4 // 256) * 64
        ws = s["stack"].workspace[:16 * arena].view(torch.float32)
        out = {"y": s["y"], "dx": s["dx"]}
        for a, name in enumerate(("w", "m", "v", "g")):
            for n in TENSORS:
                out[name + "." + n] = torch.as_strided(ws, (case["layers"], int(np.prod(_shapes(case)[n]))), (off, 1), a * arena + offs[n])
        # The key third of b_qkv has no gradient (a softmax row does not move when all its scores shift), so what the
        # sums leave there is rounding, and the optimizer makes steps of +-lr of it: the updated bias without that third.
        out["w.b_qkv"] = torch.as_strided(ws, (case["layers"], 2, case["hidden"]), (off, 2 * case["hidden"], 1), offs["b_qkv"])
        s["out"] = out
    elif k == "attention":
        m, t, h = case["smb"], case["seq"], case["heads"] * case["head"]
        n_part = bf.bf_op_attention_bwd_part_elems(m, t, case["heads"], case["head"])
        s.update(ctx=act(m, t, h), lse=f32(m, case["heads"], t), dqkv=act(m, t, 3 * h), delta=f32(m * case["heads"] * t), db=f32(3 * h),
                 part=f32(n_part) if n_part and case["dtype"] == "bf16" else None)
    elif k == "mlp":
        t, h, f = case["tokens"], case["hidden"], case["mlp"]
        s.update(u=act(t, f), g=act(t, f), y=act(t, h), du=act(t, f), dc=act(t, h), dw1=f32(h, f), dw2=f32(f, h), db1=f32(f), db2=f32(h),
                 part=f32(-(-t // 128), f), planes_y=_planes(s["dt"], bf.BF_NN, bf.BF_EPI_BIAS_RES, t, h, f),
                 planes_dc=_planes(s["dt"], bf.BF_NT, bf.BF_EPI_NONE, t, h, f))
    elif k == "norm":
        t, h = case["tokens"], case["hidden"]
        s.update(y=act(t, h), stats=f32(t, 2), dx=act(t, h), dg=f32(h), db=f32(h), dcs=f32(h), part=f32(bf.bf_op_layernorm_bwd_part_elems(t, h)))
    elif k == "head":
        t, h, v = case["tokens"], case["hidden"], case["vocab"]
        s.update(z=act(t, v), row_loss=f32(t), loss=f32(1), dhn=act(t, h), dw=f32(v, h),
                 planes=_planes(s["dt"], bf.BF_NN, bf.BF_EPI_NONE, t, h, v))
    else:
        h, v = case["hidden"], case["vocab"]
        s.update(x=act(case["smb"], case["seq"], h), g_tok=torch.zeros((v, h), device=DEV), g_pos=f32(case["seq"], h))
    return s


# --------------------------------------------------------------------------------------------------------- run
def run(s):
    """One pass as a program makes it; the outputs whole."""
    c, k, dt = s["case"], s["kind"], s["dt"]
    if k == "step":
        s["stack"].bf_run_step(s["order"], c["loop"], c["mb"], c["smb"], s["x"], s["dy"], s["y"], s["dx"], apply_optimizer=1)
        return s["out"]
    if k == "attention":
        a = (dt, bf.BF_KERNELS_AUTO, c["smb"], c["seq"], c["heads"], c["head"], c["causal"])
        bf.bf_op_attention_fwd(*a, s["qkv"], s["ctx"], s["lse"])
        bf.bf_op_attention_bwd_bias(*a, s["qkv"], s["ctx"], s["lse"], s["dctx"], s["dqkv"], s["delta"], s["db"], s["part"], 0)
        return {n: s[n] for n in ("ctx", "lse", "dqkv", "db")}
    if k == "mlp":
        t, h, f = c["tokens"], c["hidden"], c["mlp"]
        auto = bf.BF_KERNELS_AUTO
        bf.bf_op_gemm(dt, auto, bf.BF_NN, bf.BF_EPI_BIAS_GELU, t, f, h, s["c"], s["w1"], s["u"], bias=s["b1"], C2=s["g"])
        bf.bf_op_gemm_splitk(dt, auto, bf.BF_NN, bf.BF_EPI_BIAS_RES, t, h, f, s["g"], s["w2"], s["y"], bias=s["b2"], R=s["x1"], planes=s["planes_y"])
        bf.bf_op_gemm_gelu_bwd_colsum(dt, auto, t, f, h, s["dy"], s["w2"], s["du"], s["u"], s["db1"], s["part"])
        bf.bf_op_gemm_splitk(dt, auto, bf.BF_NT, bf.BF_EPI_NONE, t, h, f, s["du"], s["w1"], s["dc"], planes=s["planes_dc"])
        bf.bf_op_wgrad(dt, auto, f, h, t, 1, s["g"], t * f, s["dy"], t * h, s["dw2"], s["db2"])
        bf.bf_op_wgrad(dt, auto, h, f, t, 1, s["c"], t * h, s["du"], t * f, s["dw1"])
        return {n: s[n] for n in ("u", "g", "y", "du", "db1", "dc", "dw1", "dw2", "db2")}
    if k == "norm":
        t, h = c["tokens"], c["hidden"]
        bf.bf_op_layernorm_fwd(dt, t, h, s["x"], s["g"], s["b"], LN_EPS, s["y"], s["stats"])
        bf.bf_op_layernorm_bwd_fused(dt, t, h, s["dy"], s["x"], s["g"], s["stats"], s["dres"], s["dx"], s["dg"], s["db"], s["dcs"], s["part"])
        return {n: s[n] for n in ("y", "stats", "dx", "dg", "db", "dcs")}
    if k == "head":
        t, h, v = c["tokens"], c["hidden"], c["vocab"]
        auto = bf.BF_KERNELS_AUTO
        bf.bf_op_gemm(dt, auto, bf.BF_NT, bf.BF_EPI_NONE, t, v, h, s["hn"], s["w"], s["z"])
        bf.bf_op_ce_loss(dt, t, v, s["z"], s["labels"], 1.0 / t, s["row_loss"], s["loss"])
        bf.bf_op_gemm_splitk(dt, auto, bf.BF_NN, bf.BF_EPI_NONE, t, h, v, s["z"], s["w"], s["dhn"], planes=s["planes"])
        bf.bf_op_gemm(dt, auto, bf.BF_TN, bf.BF_EPI_ACCUM, v, h, t, s["z"], s["hn"], s["dw"])
        return {n: s[n] for n in ("z", "row_loss", "loss", "dhn", "dw")}
    # the token rows' gradients are added to, as over the micro-batches of a step
    h, v, rows = c["hidden"], c["vocab"], c["smb"] * c["seq"]
    bf.bf_op_embedding_fwd(dt, rows, c["seq"], v, h, s["tokens"], s["e_tok"], s["e_pos"], s["x"])
    bf.bf_op_embedding_bwd(dt, c["smb"], c["seq"], v, h, s["tokens"], s["d"], s["g_tok"], s["g_pos"], 0)
    return {n: s[n] for n in ("x", "g_tok", "g_pos")}


# ------------------------------------------------------------------------------------------------- what it costs
def work(case):
    """Bytes (every input read once, every output written once) and flops (products, with the causal half of the
    attention scores; backward attention 2.5 times forward) of one pass."""
    es, k = (2 if case["dtype"] == "bf16" else 4), case["kind"]
    if k == "step":
        h, f, lay, t = case["hidden"], case["mlp"], case["layers"], case["mb"] * case["smb"] * case["seq"]
        mat = 4 * h * h + 2 * h * f
        att = 4.0 * case["seq"] * t * h * (0.5 if case["causal"] else 1.0)
        params = lay * (mat + 9 * h + f)
        return {"bytes": params * (16 + 16 + (2 if es == 2 else 0)) + 4.0 * es * t * h, "flops": lay * (6.0 * t * mat + 3.5 * att)}
    if k == "attention":
        m, t, h = case["smb"], case["seq"], case["heads"] * case["head"]
        att = 4.0 * m * t * t * h * (0.5 if case["causal"] else 1.0)
        return {"bytes": es * m * t * h * (3 + 1 + 1 + 3) + 4.0 * m * t * case["heads"] + 12.0 * h, "flops": 3.5 * att}
    if k == "mlp":
        t, h, f = case["tokens"], case["hidden"], case["mlp"]
        return {"bytes": es * (3.0 * t * h + 2.0 * h * f + 3.0 * t * f + 2.0 * t * h) + 8.0 * h * f + 8.0 * (h + f), "flops": 12.0 * t * h * f}
    if k == "norm":
        t, h = case["tokens"], case["hidden"]
        return {"bytes": es * t * h * 5.0 + 8.0 * t + 20.0 * h, "flops": 20.0 * t * h}
    if k == "head":
        t, h, v = case["tokens"], case["hidden"], case["vocab"]
        return {"bytes": es * (2.0 * t * h + float(v) * h + float(t) * v) + 4.0 * v * h + 8.0 * t, "flops": 6.0 * t * h * v}
    rows, h = case["smb"] * case["seq"], case["hidden"]
    # about 0.4 of the tokens of a Zipf stream are first uses: their gradient rows are read and written
    return {"bytes": rows * h * (0.4 * 4 + es) + 4.0 * case["seq"] * h + rows * h * (es + 0.4 * 8) + 4.0 * case["seq"] * h, "flops": 3.0 * rows * h}


def tolerance(case):
    """Measured against exact() and stated at about four times what was seen.  bf16: the roundings of the tensors that
    pass from kernel to kernel; fp32: the order of sums of up to 32768 terms.  The step's roundings add up over its
    layers."""
    if case["kind"] == "step":
        return {"rel": 0.03, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1e-3}
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 4e-4}
    return {"rel": 1e-2, "max": 0.4}


# ------------------------------------------------------------------------------------------- the answer in 64 bits
def _gelu(u):
    return 0.5 * u * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (u + 0.044715 * u ** 3)))


def _attention(qkv, heads, causal):
    m, t, h3 = qkv.shape
    h = h3 // 3
    d = h // heads
    q, k, v = (qkv[..., i * h:(i + 1) * h].reshape(m, t, heads, d).permute(0, 2, 1, 3).contiguous() for i in range(3))
    s = torch.matmul(q, k.transpose(-1, -2).contiguous()) / math.sqrt(d)
    if causal:
        s = s.masked_fill(torch.ones((t, t), dtype=torch.bool, device=qkv.device).triu(1), -math.inf)
    return torch.matmul(torch.softmax(s, -1), v).permute(0, 2, 1, 3).reshape(m, t, h), torch.logsumexp(s, -1)


def _norm(x, g, b):
    mean = x.mean(-1, keepdim=True)
    rstd = 1.0 / torch.sqrt(((x - mean) ** 2).mean(-1, keepdim=True) + float(np.float32(LN_EPS)))
    return (x - mean) * rstd * g + b, torch.cat([mean, rstd], -1)


def _layer(x, p, heads, causal):
    a, _ = _norm(x, p["ln1_g"], p["ln1_b"])
    ctx, _ = _attention(a @ p["w_qkv"] + p["b_qkv"], heads, causal)
    x1 = x + ctx @ p["w_o"] + p["b_o"]
    c, _ = _norm(x1, p["ln2_g"], p["ln2_b"])
    return x1 + _gelu(c @ p["w_fc1"] + p["b_fc1"]) @ p["w_fc2"] + p["b_fc2"]


def exact(case, seed):
    i, k = _inputs(case, seed), case["kind"]

    def d64(t):
        return t.double()

    if k == "step":
        params = [{n: d64(v).requires_grad_() for n, v in p.items()} for p in i["params"]]
        ys, dxs = [], []
        for m in range(case["mb"]):
            x0 = d64(i["x"][m]).requires_grad_()
            x = x0
            for p in params:
                x = _layer(x, p, case["heads"], case["causal"])
            x.backward(d64(i["dy"][m]))
            ys.append(x.detach())
            dxs.append(x0.grad)
        out = {"y": torch.stack(ys), "dx": torch.stack(dxs)}
        lr, b1, b2, eps = (float(np.float32(v)) for v in (LR, BETA1, BETA2, ADAM_EPS))
        for n in TENSORS:
            w = torch.stack([p[n].detach().reshape(-1) for p in params])
            g = torch.stack([p[n].grad.reshape(-1) for p in params])
            for p in params:
                p[n].grad = None
            mo, ve = (1.0 - b1) * g, (1.0 - b2) * g * g
            out["g." + n], out["m." + n], out["v." + n] = g, mo, ve
            out["w." + n] = w - lr * (mo / (1.0 - b1)) / (torch.sqrt(ve / (1.0 - b2)) + eps)
            if n == "b_qkv":
                out["w.b_qkv"] = out["w.b_qkv"].reshape(case["layers"], 3, case["hidden"])[:, ::2]
        return out
    if k == "attention":
        qkv = d64(i["qkv"]).requires_grad_()
        ctx, lse = _attention(qkv, case["heads"], case["causal"])
        ctx.backward(d64(i["dctx"]))
        return {"ctx": ctx.detach(), "lse": lse.detach(), "dqkv": qkv.grad, "db": qkv.grad.reshape(-1, qkv.shape[-1]).sum(0)}
    if k == "mlp":
        c, w1, w2, dy = d64(i["c"]), d64(i["w1"]), d64(i["w2"]), d64(i["dy"])
        u = (c @ w1 + i["b1"]).requires_grad_()
        g = _gelu(u)
        y = (g @ w2).detach() + i["b2"] + i["x1"]
        g.backward(dy @ w2.t())
        du = u.grad
        return {"u": u.detach(), "g": g.detach(), "y": y, "du": du, "db1": du.sum(0), "dc": du @ w1.t(), "dw1": c.t() @ du,
                "dw2": g.detach().t() @ dy, "db2": dy.sum(0)}
    if k == "norm":
        x, g, b = d64(i["x"]).requires_grad_(), d64(i["g"]).requires_grad_(), d64(i["b"]).requires_grad_()
        y, stats = _norm(x, g, b)
        y.backward(d64(i["dy"]))
        dx = x.grad + i["dres"]
        return {"y": y.detach(), "stats": stats.detach(), "dx": dx, "dg": g.grad, "db": b.grad, "dcs": dx.sum(0)}
    if k == "head":
        hn, w, t = d64(i["hn"]), d64(i["w"]), case["tokens"]
        z = hn @ w.t()
        lab = i["labels"].long()
        scale = float(np.float32(1.0 / t))
        row = (torch.logsumexp(z, -1) - z.gather(1, lab[:, None])[:, 0]) * scale
        dz = torch.softmax(z, -1)
        dz[torch.arange(t, device=DEV), lab] -= 1.0
        dz *= scale
        return {"z": dz, "row_loss": row, "loss": row.sum().reshape(1), "dhn": dz @ w, "dw": dz.t() @ hn}
    tok, d = i["tokens"].long(), d64(i["d"])
    g_tok = torch.zeros((case["vocab"], case["hidden"]), device=DEV, dtype=torch.float64)
    g_tok.index_add_(0, tok.reshape(-1), d.reshape(-1, case["hidden"]))
    return {"x": d64(i["e_tok"])[tok] + d64(i["e_pos"]), "g_tok": g_tok, "g_pos": d.sum(0)}
