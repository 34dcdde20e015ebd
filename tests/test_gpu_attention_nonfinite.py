"""GPU: the attention core in fp32 (and bf16 of head dimensions that the bf16 kernels leave to the same kernels) on inputs that hold
an infinity, a NaN, or scores at the end of the type's range.  A pair (i, j) that the mask excludes takes no part in anything: a value that
is not finite reaches exactly the outputs that the definition, evaluated over the allowed pairs only, gives it, and as the same infinity.  Large finite scores keep their precision."""
import numpy as np
import pytest

import oracle
from paper_2205_05198_amd.workloads import attn_inputs

pytestmark = pytest.mark.gpu


def _definition(sh, q, k, v, do, heads):
    """O, LSE and the gradients of some (batch, head)s from the definition in fp64, one row of scores at a time over its allowed keys;
    beside each the sum of the magnitudes of its terms."""
    s, alpha, c = sh.s, sh.alpha(), 1.0 / (1.0 - float(np.float32(sh.p)))
    M = oracle.attn_mask(sh)
    out = {n: np.zeros(q.shape) for n in ("o", "dq", "dk", "dv")}
    mag = {n: np.zeros(q.shape) for n in ("o", "dq", "dk", "dv")}
    out["lse"] = np.zeros((sh.b, sh.A, s))
    with np.errstate(all="ignore"):
        for be, n in heads:
            Q, K, V, G = (np.asarray(t[:, be, n], dtype=np.float64) for t in (q, k, v, do))
            for i in range(s):
                e = i + 1 if sh.causal else s
                S = alpha * (K[:e] * Q[i]).sum(1)
                m = S[~np.isnan(S)].max(initial=-np.inf)
                P = np.exp(S - m)
                out["lse"][be, n, i] = m + np.log(P.sum())
                P = P / P.sum()
                keep = M[be, n, i, :e] != 0
                D = np.where(keep, P * c, 0.0)
                O = (D[:, None] * V[:e]).sum(0)
                dp = np.where(keep, (V[:e] * G[i]).sum(1) * c, 0.0)
                dS = alpha * P * (dp - (G[i] * O).sum())
                W = alpha * P * (np.abs(dp) + (np.abs(G[i]) * (D[:, None] * np.abs(V[:e])).sum(0)).sum())
                out["o"][i, be, n] = O
                out["dq"][i, be, n] = (dS[:, None] * K[:e]).sum(0)
                out["dk"][:e, be, n] += dS[:, None] * Q[i]
                out["dv"][:e, be, n] += D[:, None] * G[i]
                mag["o"][i, be, n] = (D[:, None] * np.abs(V[:e])).sum(0)
                mag["dq"][i, be, n] = (W[:, None] * np.abs(K[:e])).sum(0)
                mag["dk"][:e, be, n] += W[:, None] * np.abs(Q[i])
                mag["dv"][:e, be, n] += D[:, None] * np.abs(G[i])
    return out, mag


def _compare(tag, sh, dtype, q, k, v, do):
    from gpu_util import run_attn
    got = run_attn(sh, dtype, q, k, v, do)
    heads = [(0, 0), (sh.b - 1, 1)]
    ref, mag = _definition(sh, q, k, v, do, heads)
    at = tuple(np.transpose(heads))
    bar = 1e-4 if dtype == "f32" else 2e-2   # of the sum of the magnitudes of the terms: those of the other tests of either dtype
    for nm in ("o", "lse", "dq", "dk", "dv"):
        x, r, g = (t[nm][at] if nm == "lse" else t[nm][:, at[0], at[1]] for t in (got, ref, {**mag, "lse": ref["lse"]}))
        fin = np.isfinite(r)
        bad = int(np.count_nonzero(np.isfinite(x) != fin))
        assert bad == 0, (tag, nm, "finite in one, not in the other", bad, np.argwhere(np.isfinite(x) != fin)[:4].tolist())
        assert np.array_equal(x[~fin], r[~fin], equal_nan=True), (tag, nm, "another infinity, or NaN for one")
        if nm == "lse":
            assert np.max(np.abs(x[fin] - r[fin]) / (1.0 + np.abs(r[fin])), initial=0.0) < (1e-5 if dtype == "f32" else 2e-3), tag
        else:
            e = np.abs(x[fin] - r[fin]) / (g[fin] + 1e-30)
            assert np.all(e <= bar), (tag, nm, float(np.max(e)))


def _case(dtype, s, d, p, causal, heads, scale=None):
    b = 1 if heads == 2 else 512 // ((s + 31) // 32) // heads + 1    # 2 heads: blocks of 16 rows; 64: of 32
    return oracle.AttnShape(s=s, b=b, a=heads, h=heads * d, p=p, seed=5, offset=(1 << 32) - 9, causal=causal, **({} if scale is None else {"scale": scale}))


@pytest.mark.parametrize("heads", [2, 64])
@pytest.mark.parametrize("where", ["q", "k", "v", "do"])
@pytest.mark.parametrize("dtype,s,d,p,causal", [("f32", 72, 64, 0.1, 1), ("f32", 104, 96, 0.0, 1), ("f32", 40, 32, 0.1, 0), ("bf16", 72, 40, 0.1, 1), ("f32", 72, 128, 0.0, 0),
                                                 ("f32", 8, 64, 0.1, 1), ("bf16", 16, 72, 0.1, 1)])
def test_excluded_pairs_take_no_part(dtype, s, d, p, causal, where, heads):
    """One element of one tensor is not finite: inside a 32-wide tile that the diagonal crosses, and in the last row, which the
    clamped loads past the end repeat."""
    sh = _case(dtype, s, d, p, causal, heads)
    base = dict(zip(("q", "k", "v", "do"), attn_inputs(s, sh.b, sh.A, d, dtype, seed=11)))
    for row, value in ((5, np.nan), (min(37, s - 2), np.inf), (s - 1, -np.inf), (s - 1, np.nan)):
        t = dict(base)
        t[where] = base[where].copy()
        t[where][row, sh.b - 1, 1, d // 2] = value
        print(f"{where}[{row}] = {value} {dtype} s={s} d={d} p={p} causal={causal} heads={sh.b * heads}", flush=True)
        _compare(f"{where}[{row}]={value}", sh, dtype, t["q"], t["k"], t["v"], t["do"])


@pytest.mark.parametrize("heads", [2, 64])
@pytest.mark.parametrize("dtype,s,d", [("f32", 40, 36), ("f32", 72, 80), ("f32", 40, 100), ("bf16", 72, 40)])
def test_infinity_in_the_last_element_of_a_head(dtype, s, d, heads):
    """Head dimensions that are no multiple of 32: the operand pieces past the end of a row are loads of its last one.  K = -infinity in the
    last element, met by positive elements of Q, gives that key probability 0 and leaves all but its own row of scores finite."""
    sh = _case(dtype, s, d, 0.1, 1, heads)
    q, k, v, do = attn_inputs(s, sh.b, sh.A, d, dtype, seed=15)
    q[..., d - 1], k[..., d - 1] = np.abs(q[..., d - 1]), np.abs(k[..., d - 1])
    k[9, sh.b - 1, 1, d - 1] = -np.inf
    print(f"last element {dtype} s={s} d={d} heads={sh.b * heads}", flush=True)
    _compare("last element", sh, dtype, q, k, v, do)


def test_uninitialised_tail_of_a_causal_sequence():
    """A sequence padded with NaN to a multiple of 8: the rows before the padding keep their O and LSE."""
    from gpu_util import run_attn
    sh = _case("f32", 72, 64, 0.1, 1, 2)
    q, k, v, do = attn_inputs(72, sh.b, sh.A, 64, "f32", seed=12)
    for t in (q, k, v, do):
        t[67:] = np.nan
    got = run_attn(sh, "f32", q, k, v, do)
    ref, mag = _definition(sh, q, k, v, do, [(0, 0), (0, 1)])
    assert np.all(np.abs(got["o"] - ref["o"])[:67] <= 1e-4 * mag["o"][:67]) and np.all(np.isnan(got["o"][67:]))
    assert np.max(np.abs(got["lse"] - ref["lse"])[:, :, :67]) < 1e-4


@pytest.mark.parametrize("heads", [2, 64])
@pytest.mark.parametrize("d,scale,top,causal", [(64, None, 58, 1), (96, None, 58, 1), (64, 1.0, 62, 1), (64, None, 58, 0), (64, -0.125, 58, 1), (32, None, 50, 1)])
def test_scores_at_the_end_of_the_range(d, scale, top, causal, heads):
    """Finite scores of one sign in a row, far below -1e30 or far above 1e30: every row attends to one key (a sum of several exponentials
    would not show in a log-sum-exp of that size); a causal row 0 has no other."""
    s = 72
    sh = _case("f32", s, d, 0.1, causal, heads, scale)
    q, k, v, do = attn_inputs(s, sh.b, sh.A, d, "f32", seed=13)
    q[..., 0], q[..., 1:] = -2.0 ** top, 0.0
    q[40::3, ..., 0] = 2.0 ** top
    k[..., 0] = (2.0 ** top * (1.0 + (np.arange(s) * 29 % s) / 128.0))[:, None, None]
    print(f"scores of 2^{2 * top} d={d} scale={scale} causal={causal} heads={sh.b * heads}", flush=True)
    _compare("range", sh, "f32", q, k, v, do)


@pytest.mark.parametrize("d,heads", [(64, 2), (96, 2), (64, 64)])
def test_precision_of_large_scores(d, heads):
    """Scores up to some 300, a row's softmax spread over few keys.  A probability exp(score - LSE) carries one rounding of the score and
    one of the LSE, each uniform within 2^-17 where they lie between 128 and 256 as most row maxima do: sqrt 2 x 2^-17 / sqrt 3 = 6.2e-6
    of dV in the 2-norm, less what cancels in rows with a single key.  Measured 3.4e-6 to 3.8e-6."""
    s = 512
    sh = oracle.AttnShape(s=s, b=1, a=heads, h=heads * d, p=0.0, seed=5)
    q, k, v, do = attn_inputs(s, 1, heads, d, "f32", seed=14, qk_std=8.0)
    from gpu_util import run_attn
    got = run_attn(sh, "f32", q, k, v, do)
    ref = oracle.attn_bwd(sh, q, k, v, do)["dv"]
    e = float(np.linalg.norm(got["dv"] - ref) / np.linalg.norm(ref))
    print(f"large scores d={d} heads={heads}: dV error {e:.2e}", flush=True)
    assert e <= 2 ** 0.5 * 2.0 ** -17 / 3 ** 0.5
