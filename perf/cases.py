"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain sizes and options in the paper's notation (s, b, a, h, t; p = dropout probability).  Its `kind`:

  attn_fwd    attention core, forward only (evaluation, the forward of a microbatch)
  attn_train  attention core, forward and the backward that recomputes softmax and mask (`workspace`: "full" as
              attn_core_bwd_workspace asks for, or "min", the scratch of one float per query row)
  rows_train  the sequence-parallel region around one residual connection on a rank's rows: bias-dropout-add fused with the
              LayerNorm that reads it, then the backward of both
  mlp_train   bias + GeLU of the MLP block, forward and backward
  layer_train every one of the above in the order of one transformer layer's training step (all of the layer but its GEMMs)
"""
import torch

import paper_2205_05198_amd as sar

TORCH = {"bf16": torch.bfloat16, "f32": torch.float32}
BYTES = {"bf16": 2, "f32": 4}


def listed():
    return [
        # The smallest call: the tiny fp32 workload (b = 1, s = 128, 2 heads of 64), where launches and the host path count.
        dict(name="attn_tiny_f32", kind="attn_train", s=128, b=1, a=2, h=128, t=1, dtype="f32", p=0.1, causal=1, workspace="full"),
        # fp32 at an ordinary size: what a user runs to check a bf16 result, or trains a small model with.
        dict(name="attn_f32", kind="attn_train", s=1024, b=2, a=12, h=768, t=1, dtype="f32", p=0.1, causal=1, workspace="full"),
        # The tensor-parallel shards (t = 8, s = 2048) of the paper's 22B and 175B models: head dimensions 96 and 128.
        dict(name="attn_22B", kind="attn_train", s=2048, b=4, a=64, h=6144, t=8, dtype="bf16", p=0.1, causal=1, workspace="full"),
        dict(name="attn_175B", kind="attn_train", s=2048, b=1, a=96, h=12288, t=8, dtype="bf16", p=0.1, causal=1, workspace="full"),
        # A long sequence on the 530B model's heads (16 of 160): the largest case.
        dict(name="attn_530B_s8192", kind="attn_train", s=8192, b=1, a=128, h=20480, t=8, dtype="bf16", p=0.1, causal=1, workspace="full"),
        # A sequence that is not a multiple of the tile, in a memory-bound program: minimal scratch.
        dict(name="attn_ragged_min", kind="attn_train", s=1000, b=2, a=96, h=12288, t=8, dtype="bf16", p=0.1, causal=1, workspace="min"),
        # An encoder's forward in evaluation: no causal mask, no dropout, short sequences, many of them.
        dict(name="attn_fwd_eval", kind="attn_fwd", s=512, b=8, a=16, h=1024, t=1, dtype="bf16", p=0.0, causal=0),
        # One layer's training step of the 530B model's shard: the paper's headline shape.
        dict(name="layer_530B", kind="layer_train", s=2048, b=1, a=128, h=20480, t=8, dtype="bf16", p=0.1, causal=1, workspace="full"),
        # The residual connection on a rank's rows: the 22B model's shard, and a long sequence of the 530B model's.
        dict(name="rows_22B", kind="rows_train", rows=1024, h=6144, dtype="bf16", p=0.1),
        dict(name="rows_530B_s32768", kind="rows_train", rows=4096, h=20480, dtype="bf16", p=0.1),
        # A few rows of an odd width in fp32.
        dict(name="rows_small_f32", kind="rows_train", rows=37, h=1032, dtype="f32", p=0.25),
        # The MLP's non-linearity at the 22B model's shard: s b rows of 4 h / t.
        dict(name="mlp_22B", kind="mlp_train", rows=8192, h=3072, dtype="bf16", p=0.0),
    ]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _attn_size(rng, dtype, most):
    """Sizes of an attention call of at most `most` floating-point operations, forward and backward."""
    while True:
        d = rng.choice([64, 96, 128, 160]) if dtype == "bf16" else rng.choice([32, 64, 80, 96, 128])
        s = int(_log(rng, 64, 8192 if dtype == "bf16" else 1024))
        s = max(8, s // 64 * 64 if rng.random() < 0.6 else s // 8 * 8)
        b, t, heads = rng.choice([1, 1, 2, 3, 4, 8]), rng.choice([1, 2, 8]), rng.randint(1, 20)
        case = dict(s=s, b=b, a=heads * t, h=heads * t * d, t=t, dtype=dtype, p=rng.choice([0.1, 0.1, 0.1, 0.0, 0.25]), causal=rng.choice([1, 1, 1, 0]))
        if 2e7 < _attn_flops(case, 14) < most:
            return case


def draw(rng):
    kind = rng.choice(["attn_train"] * 9 + ["attn_fwd"] * 4 + ["rows_train"] * 4 + ["mlp_train"] * 2 + ["layer_train"])
    dtype = "f32" if rng.random() < 0.15 else "bf16"
    if kind in ("attn_train", "attn_fwd"):
        case = dict(_attn_size(rng, dtype, 1.2e12 if dtype == "bf16" else 1.1e10), kind=kind)
        if kind == "attn_train":
            case["workspace"] = rng.choice(["full", "full", "full", "min"])
        return case
    if kind == "layer_train":
        s, heads, d = rng.choice([1024, 2048, 3072, 4096]), rng.randint(4, 16), rng.choice([64, 96, 128, 160])
        return dict(kind=kind, s=s, b=1, a=8 * heads, h=8 * heads * d, t=8, dtype="bf16", p=0.1, causal=1, workspace="full")
    h = max(8, int(_log(rng, 256, 25600)) // 8 * 8)
    if rng.random() < 0.5:
        h = max(64, h // 64 * 64)
    rows = max(1, min(int(_log(rng, 16, 16384)), int(1.2e8 / h) // BYTES[dtype]))
    return dict(kind=kind, rows=rows, h=h, dtype=dtype, p=rng.choice([0.1, 0.1, 0.0, 0.25]) if kind == "rows_train" else 0.0)


# ---------------------------------------------------------------------------------------------------------------- states
class _Maker:
    """Seeded tensors on the GPU."""

    def __init__(self, dtype, seed):
        self.dtype = TORCH[dtype]
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape, std=1.0, mean=0.0):
        return (torch.randn(*shape, device="cuda", generator=self.g) * std + mean).to(self.dtype)

    def empty(self, *shape):
        return torch.empty(*shape, dtype=self.dtype, device="cuda")


def _floats(*shape):
    return torch.empty(*shape, dtype=torch.float32, device="cuda")


def _scratch(nbytes):
    return torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")


def _code(case):
    return sar.binding.SAR_BF16 if case["dtype"] == "bf16" else sar.binding.SAR_F32


def _attn_state(case, m, seed):
    s, b, A, d = case["s"], case["b"], case["a"] // case["t"], case["h"] // case["a"]
    desc = sar.AttnDesc.packed(s, b, case["a"], case["h"], t=case["t"], rank=0, dtype=_code(case), p=case["p"], seed=1234 + seed, offset=64 * seed,
                               causal=case["causal"])
    st = dict(desc=desc, o=m.empty(s, b, A, d), lse=_floats(b, A, s))
    for name in ("q", "k", "v", "do"):
        st[name] = m.normal(s, b, A, d)
    if case["kind"] != "attn_fwd":
        for name in ("dq", "dk", "dv"):
            st[name] = m.empty(s, b, A, d)
        st["ws"] = _scratch(sar.attn_core_bwd_workspace_min(desc) if case["workspace"] == "min" else sar.attn_core_bwd_workspace(desc))
    return st


def _rows_state(case, m, seed, rows, h, p):
    desc = sar.RowsDesc.make(rows, h, dtype=_code(case), p=p, seed=4321 + seed, offset=77 * seed)
    st = dict(desc=desc, bias=m.normal(h, std=0.02), gamma=m.normal(h, std=0.02, mean=1.0), beta=m.normal(h, std=0.02))
    for name in ("x", "resid", "dy"):
        st[name] = m.normal(rows, h)
    for name in ("out", "y", "dout", "dx"):
        st[name] = m.empty(rows, h)
    for name in ("dgamma", "dbeta", "dbias"):
        st[name] = _floats(h)
    st["mean"], st["rstd"] = _floats(rows), _floats(rows)
    st["ws_ln"], st["ws_bias"] = _scratch(sar.ln_bwd_workspace(desc)), _scratch(sar.bias_dropout_add_bwd_workspace(desc))
    return st


def _mlp_state(case, m, rows, h):
    desc = sar.RowsDesc.make(rows, h, dtype=_code(case))
    return dict(desc=desc, x=m.normal(rows, h), dy=m.normal(rows, h), bias=m.normal(h, std=0.02), y=m.empty(rows, h), dx=m.empty(rows, h), dbias=_floats(h),
                ws=_scratch(sar.bias_gelu_bwd_workspace(desc)))


def _layer_rows(case):
    return case["s"] * case["b"] // case["t"]


def prepare(case, seed):
    m, kind = _Maker(case["dtype"], seed), case["kind"]
    if kind in ("attn_fwd", "attn_train"):
        return kind, _attn_state(case, m, seed)
    if kind == "rows_train":
        return kind, _rows_state(case, m, seed, case["rows"], case["h"], case["p"])
    if kind == "mlp_train":
        return kind, _mlp_state(case, m, case["rows"], case["h"])
    rows = _layer_rows(case)
    return kind, dict(attn=_attn_state(case, m, seed), first=_rows_state(case, m, seed, rows, case["h"], case["p"]),
                      second=_rows_state(case, m, seed + 1, rows, case["h"], case["p"]), mlp=_mlp_state(case, m, case["s"] * case["b"], 4 * case["h"] // case["t"]))


# --------------------------------------------------------------------------------------------------------------- one pass
def _attn_fwd(a):
    sar.attn_core_fwd(a["desc"], a["q"], a["k"], a["v"], a["o"], a["lse"])


def _attn_bwd(a):
    sar.attn_core_bwd_recompute(a["desc"], a["q"], a["k"], a["v"], a["o"], a["lse"], a["do"], a["dq"], a["dk"], a["dv"], a["ws"])


def _bda_ln_fwd(r):
    sar.bias_dropout_add_ln_fwd(r["desc"], r["x"], r["bias"], r["resid"], r["gamma"], r["beta"], r["out"], r["y"], r["mean"], r["rstd"])


def _ln_bwd(r, x, dx):
    sar.ln_bwd(r["desc"], r["dy"], x, r["mean"], r["rstd"], r["gamma"], dx, r["dgamma"], r["dbeta"], r["ws_ln"])


def _bda_bwd(r, dout, dx):
    sar.bias_dropout_add_bwd(r["desc"], dout, dx, r["dbias"], r["ws_bias"])


def _gelu(g):
    sar.bias_gelu_fwd(g["desc"], g["x"], g["bias"], g["y"])


def _gelu_bwd(g):
    sar.bias_gelu_bwd(g["desc"], g["dy"], g["x"], g["bias"], g["dx"], g["dbias"], g["ws"])


def run(state):
    kind, st = state
    if kind == "attn_fwd":
        _attn_fwd(st)
        return st["o"], st["lse"]
    if kind == "attn_train":
        _attn_fwd(st)
        _attn_bwd(st)
        return st["o"], st["lse"], st["dq"], st["dk"], st["dv"]
    if kind == "rows_train":
        _bda_ln_fwd(st)
        _ln_bwd(st, st["out"], st["dout"])
        _bda_bwd(st, st["dout"], st["dx"])
        return [st[n] for n in ("out", "y", "mean", "rstd", "dout", "dx", "dgamma", "dbeta", "dbias")]
    if kind == "mlp_train":
        _gelu(st)
        _gelu_bwd(st)
        return st["y"], st["dx"], st["dbias"]
    a, f, s, g = st["attn"], st["first"], st["second"], st["mlp"]
    # forward: LayerNorm, attention core, dropout-add + LayerNorm, GeLU, dropout-add
    sar.ln_fwd(f["desc"], f["x"], f["gamma"], f["beta"], f["y"], f["mean"], f["rstd"])
    _attn_fwd(a)
    _bda_ln_fwd(s)
    _gelu(g)
    sar.bias_dropout_add(f["desc"], f["resid"], f["bias"], s["out"], f["out"])
    # backward, in the reverse order
    _bda_bwd(f, f["dy"], f["dx"])
    _gelu_bwd(g)
    _ln_bwd(s, s["out"], s["dout"])
    _bda_bwd(s, s["dout"], s["dx"])
    _attn_bwd(a)
    _ln_bwd(f, f["x"], f["dout"])
    got = [a[n] for n in ("o", "lse", "dq", "dk", "dv")] + [g[n] for n in ("y", "dx", "dbias")]
    return got + [r[n] for r in (f, s) for n in ("out", "y", "mean", "rstd", "dout", "dx", "dgamma", "dbeta", "dbias")]


# ------------------------------------------------------------------------------------------------------- work, tolerances
def _pairs(case):
    return case["s"] * (case["s"] + 1) // 2 if case["causal"] else case["s"] ** 2


def _attn_flops(case, contraction2):
    return contraction2 * (case["h"] // case["t"]) * _pairs(case) * case["b"]


def work(case):
    kind, esz = case["kind"], BYTES[case["dtype"]]
    if kind in ("attn_fwd", "attn_train"):
        n, stats = case["s"] * case["b"] * case["h"] // case["t"] * esz, 4 * case["s"] * case["b"] * case["a"] // case["t"]
        if kind == "attn_fwd":  # q, k, v in, o, lse out; two contractions over the allowed pairs
            return {"bytes": 4 * n + stats, "flops": _attn_flops(case, 4)}
        return {"bytes": 8 * n + stats, "flops": _attn_flops(case, 14)}  # q, k, v, do in; o, dq, dk, dv out; seven contractions
    if kind == "rows_train":  # x, resid, dy in; out, y, dout, dx out; per element some 60 operations
        n = case["rows"] * case["h"]
        return {"bytes": 7 * n * esz, "flops": 60 * n}
    if kind == "mlp_train":  # x, dy in; y, dx out
        n = case["rows"] * case["h"]
        return {"bytes": 4 * n * esz, "flops": 60 * n}
    attn, rows = work(dict(case, kind="attn_train")), _layer_rows(case) * case["h"]
    mlp = case["s"] * case["b"] * 4 * case["h"] // case["t"]
    return {"bytes": attn["bytes"] + 14 * rows * esz + 4 * mlp * esz, "flops": attn["flops"] + 120 * rows + 60 * mlp}


def tolerance(case):
    # About four times what the results of this path differ by from the same definitions evaluated in 64 bits: 2-norm 2.5e-3
    # (bf16: inputs of the second products and outputs rounded) and 8e-7 (f32; 1.4e-6 for a row's mean, which is small);
    # largest element 0.18 of the tensor's root mean square in bf16 (dQ, dK of the first rows, differences of large terms) and
    # 1.4e-5 in f32.
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.7}
