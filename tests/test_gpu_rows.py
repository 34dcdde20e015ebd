"""GPU parity: LayerNorm forward/backward and bias-dropout-add against the fp64 oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import oracle
import paper_2205_05198_amd as sar
from paper_2205_05198_amd.workloads import WORKLOADS, rows_inputs

pytestmark = pytest.mark.gpu


def _run_ln(rows, h, dtype, inp, eps=1e-5):
    from gpu_util import DT, dev, host
    tdt, code = DT[dtype]
    desc = sar.RowsDesc.make(rows, h, dtype=code, eps=eps)
    x, dy, gamma, beta = (dev(inp[k], dtype) for k in ("x", "dy", "gamma", "beta"))
    y, dx = torch.empty_like(x), torch.empty_like(x)
    mean = torch.empty(rows, dtype=torch.float32, device="cuda")
    rstd = torch.empty_like(mean)
    dgamma = torch.empty(h, dtype=torch.float32, device="cuda")
    dbeta = torch.empty_like(dgamma)
    ws = torch.empty(sar.ln_bwd_workspace(desc), dtype=torch.uint8, device="cuda")
    sar.ln_fwd(desc, x, gamma, beta, y, mean, rstd)
    sar.ln_bwd(desc, dy, x, mean, rstd, gamma, dx, dgamma, dbeta, ws)
    torch.cuda.synchronize()
    return {k: host(v) for k, v in dict(y=y, mean=mean, rstd=rstd, dx=dx, dgamma=dgamma, dbeta=dbeta).items()}


@pytest.mark.parametrize("rows,h,dtype", [
    (128, 128, "f32"),            # tiny workload
    (37, 1032, "bf16"),           # ragged: h not a multiple of 64, rows not a multiple of 32
    (5, 8, "f32"),                # smallest row
    (3, 32768, "bf16"),           # widest supported row
    (1024, 6144, "bf16"), (256, 12288, "bf16"), (256, 20480, "bf16"), (256, 25600, "bf16"),  # 22B, 175B, 530B, 1T shards
])
def test_layernorm(rows, h, dtype):
    from gpu_util import BAR, err
    inp = rows_inputs(rows, h, dtype, seed=1234)
    print(f"ln rows={rows} h={h} {dtype}", flush=True)
    got = _run_ln(rows, h, dtype, inp)
    f = oracle.ln_fwd(inp["x"], inp["gamma"], inp["beta"], 1e-5)
    g = oracle.ln_bwd(inp["dy"], inp["x"], inp["gamma"], 1e-5)
    ref = {**f, **g}
    for nm in ("y", "dx"):
        e = err(got[nm], ref[nm], dtype)
        print(f"  {nm}: {e:.3e}", flush=True)
        assert e <= BAR[dtype], nm
    # statistics and parameter gradients are fp32 in both dtypes
    for nm in ("mean", "rstd", "dgamma", "dbeta"):
        e = err(got[nm], ref[nm], "f32")
        print(f"  {nm}: {e:.3e}", flush=True)
        assert e <= 1e-4, nm


def test_layernorm_large_mean():
    """Rows far from zero mean: the shifted single-pass variance must not cancel."""
    from gpu_util import err
    rows, h = 16, 4096
    inp = rows_inputs(rows, h, "f32", seed=5)
    inp["x"] = (inp["x"] * 0.5 + 300.0).astype(np.float32)
    got = _run_ln(rows, h, "f32", inp)
    f = oracle.ln_fwd(inp["x"], inp["gamma"], inp["beta"], 1e-5)
    e_y, e_r = err(got["y"], f["y"], "f32"), err(got["rstd"], f["rstd"], "f32")
    print(f"  large mean: y {e_y:.3e} rstd {e_r:.3e}", flush=True)
    assert e_y < 1e-4 and e_r < 1e-4


def _run_bda(rows, h, dtype, inp, p, seed, offset, row_offset=0, bias=True, mask=True, inplace=False):
    from gpu_util import DT, dev, host
    tdt, code = DT[dtype]
    desc = sar.RowsDesc.make(rows, h, dtype=code, p=p, seed=seed, offset=offset, row_offset=row_offset)
    x, resid = dev(inp["x"], dtype), dev(inp["resid"], dtype)
    b = dev(inp["bias"], dtype) if bias else None
    out = resid if inplace else torch.empty_like(x)
    m = torch.empty((rows, h), dtype=torch.uint8, device="cuda") if mask else None
    sar.bias_dropout_add(desc, x, b, resid, out, m)
    torch.cuda.synchronize()
    return host(out), (m.cpu().numpy() if mask else None)


@pytest.mark.parametrize("rows,h,dtype,p", [
    (128, 128, "f32", 0.1), (37, 1032, "bf16", 0.25), (9, 8, "bf16", 0.0),
    (1024, 6144, "bf16", 0.1), (256, 20480, "bf16", 0.1), (256, 25600, "bf16", 0.1),
])
def test_bias_dropout_add(rows, h, dtype, p):
    from gpu_util import BAR, err
    inp = rows_inputs(rows, h, dtype, seed=99)
    seed, offset, row_offset = 1234, (1 << 32) - 3, 7 * rows
    print(f"bda rows={rows} h={h} {dtype} p={p}", flush=True)
    ref = oracle.bias_dropout_add(inp["x"], inp["bias"], inp["resid"], p, seed, offset, row_offset)
    out, m = _run_bda(rows, h, dtype, inp, p, seed, offset, row_offset)
    assert np.array_equal(m, ref["mask"])              # bit-exact mask
    assert err(out, ref["out"], dtype) <= BAR[dtype]
    # no bias, no mask output, in-place residual
    ref2 = oracle.bias_dropout_add(inp["x"], None, inp["resid"], p, seed, offset, row_offset)
    out2, _ = _run_bda(rows, h, dtype, inp, p, seed, offset, row_offset, bias=False, mask=False, inplace=True)
    assert err(out2, ref2["out"], dtype) <= BAR[dtype]


@pytest.mark.parametrize("rows,h,dtype,p,bias", [
    (128, 128, "f32", 0.1, True), (37, 1032, "bf16", 0.25, True), (9, 8, "bf16", 0.0, False), (3, 32768, "bf16", 0.1, True),
    (1024, 6144, "bf16", 0.1, True), (256, 20480, "bf16", 0.1, True), (256, 25600, "bf16", 0.1, False),
])
def test_bias_dropout_add_ln_fwd(rows, h, dtype, p, bias):
    """The fused step equals the composition of the two definitions: out as bias_dropout_add, y = LayerNorm(out)."""
    from gpu_util import BAR, DT, dev, err, host
    inp = rows_inputs(rows, h, dtype, seed=77)
    seed, offset, row_offset = 4321, 12345, 3 * rows
    print(f"bda+ln rows={rows} h={h} {dtype} p={p} bias={bias}", flush=True)
    ref_o = oracle.bias_dropout_add(inp["x"], inp["bias"] if bias else None, inp["resid"], p, seed, offset, row_offset)
    ref_l = oracle.ln_fwd(ref_o["out"], inp["gamma"], inp["beta"], 1e-5)
    tdt, code = DT[dtype]
    desc = sar.RowsDesc.make(rows, h, dtype=code, p=p, seed=seed, offset=offset, row_offset=row_offset)
    x, resid, gamma, beta = (dev(inp[k], dtype) for k in ("x", "resid", "gamma", "beta"))
    b = dev(inp["bias"], dtype) if bias else None
    out, y = torch.empty_like(x), torch.empty_like(x)
    mean = torch.empty(rows, dtype=torch.float32, device="cuda")
    rstd = torch.empty_like(mean)
    sar.bias_dropout_add_ln_fwd(desc, x, b, resid, gamma, beta, out, y, mean, rstd)
    torch.cuda.synchronize()
    assert err(host(out), ref_o["out"], dtype) <= BAR[dtype]
    # y and the statistics belong to the row as stored (rounded to the dtype): the definition applied to exactly
    # those values is the reference at the usual bar ...
    ref_s = oracle.ln_fwd(host(out), inp["gamma"], inp["beta"], 1e-5)
    assert err(host(y), ref_s["y"], dtype) <= BAR[dtype]
    assert err(host(mean), ref_s["mean"], "f32") <= 1e-4
    assert err(host(rstd), ref_s["rstd"], "f32") <= 1e-4
    # ... and against the unrounded fp64 composition y carries two roundings (of out, then of y)
    assert err(host(y), ref_l["y"], dtype) <= 2 * BAR[dtype]
    # the unfused entry points give the same bits for `out`
    out2 = torch.empty_like(x)
    sar.bias_dropout_add(desc, x, b, resid, out2, None)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    # in-place residual
    sar.bias_dropout_add_ln_fwd(desc, x, b, resid, gamma, beta, resid, y, mean, rstd)
    torch.cuda.synchronize()
    assert torch.equal(resid, out2)


@pytest.mark.parametrize("rows,h,dtype,p", [
    (128, 128, "f32", 0.1), (37, 1032, "bf16", 0.25), (9, 8, "bf16", 0.0), (1000, 64, "f32", 0.5),
    (1024, 6144, "bf16", 0.1), (256, 20480, "bf16", 0.1), (256, 25600, "bf16", 0.1),
])
def test_bias_dropout_add_bwd(rows, h, dtype, p):
    from gpu_util import BAR, DT, dev, err, host
    inp = rows_inputs(rows, h, dtype, seed=55)
    seed, offset, row_offset = 1234, (1 << 32) - 3, 7 * rows
    print(f"bda bwd rows={rows} h={h} {dtype} p={p}", flush=True)
    ref = oracle.bias_dropout_add_bwd(inp["dy"], p, seed, offset, row_offset)
    tdt, code = DT[dtype]
    desc = sar.RowsDesc.make(rows, h, dtype=code, p=p, seed=seed, offset=offset, row_offset=row_offset)
    dout = dev(inp["dy"], dtype)
    dx = torch.empty_like(dout)
    dbias = torch.empty(h, dtype=torch.float32, device="cuda")
    ws = torch.empty(max(16, sar.bias_dropout_add_bwd_workspace(desc)), dtype=torch.uint8, device="cuda")
    sar.bias_dropout_add_bwd(desc, dout, dx, dbias, ws)
    torch.cuda.synchronize()
    assert err(host(dx), ref["dx"], dtype) <= BAR[dtype]
    # dbias sums the unrounded fp32 products in fp32
    assert err(host(dbias), ref["dbias"], "f32") <= 1e-4
    # dropped positions are exactly zero and agree with the forward's mask
    m = oracle.bias_dropout_add(inp["x"], None, inp["resid"], p, seed, offset, row_offset)["mask"]
    assert np.array_equal(host(dx) != 0, (m != 0) & (np.asarray(inp["dy"], dtype=np.float64) != 0))
    # without dbias: elementwise kernel, same dx bits, no workspace
    dx2 = torch.empty_like(dout)
    sar.bias_dropout_add_bwd(desc, dout, dx2, None, None)
    torch.cuda.synchronize()
    assert torch.equal(dx, dx2)


@pytest.mark.parametrize("rows,h,dtype,with_bias", [
    (128, 128, "f32", True),        # tiny
    (37, 1032, "bf16", True),       # ragged
    (5, 8, "f32", False),           # smallest row, no bias
    (2048, 10240, "bf16", True),    # 530B MLP on one tensor-parallel rank: s*b rows of 4h/t
    (300, 12800, "bf16", False),    # 1T width, rows split over several slab workgroups
])
def test_bias_gelu(rows, h, dtype, with_bias):
    """bias + GeLU forward and backward (dx, dbias) against the fp64 oracle."""
    from gpu_util import BAR, DT, dev, err, host
    rng = np.random.default_rng(7)
    tdt, code = DT[dtype]
    rnd = (lambda a: a.astype(np.float32)) if dtype == "f32" else (lambda a: torch.from_numpy(a.astype(np.float32)).to(torch.bfloat16).float().numpy())
    x, dy = rnd(rng.normal(size=(rows, h)) * 1.5), rnd(rng.normal(size=(rows, h)))
    bias = rnd(rng.normal(size=h) * 0.5) if with_bias else None
    print(f"bias_gelu rows={rows} h={h} {dtype} bias={with_bias}", flush=True)
    desc = sar.RowsDesc.make(rows, h, dtype=code)
    tx, tdy = dev(x, dtype), dev(dy, dtype)
    tb = dev(bias, dtype) if with_bias else None
    y, dx, dx2 = torch.empty_like(tx), torch.empty_like(tx), torch.empty_like(tx)
    dbias = torch.empty(h, dtype=torch.float32, device="cuda")
    ws = torch.empty(max(16, sar.bias_gelu_bwd_workspace(desc)), dtype=torch.uint8, device="cuda")
    sar.bias_gelu_fwd(desc, tx, tb, y)
    sar.bias_gelu_bwd(desc, tdy, tx, tb, dx, dbias, ws)
    sar.bias_gelu_bwd(desc, tdy, tx, tb, dx2)          # without dbias: the elementwise kernel
    torch.cuda.synchronize()
    ref_y = oracle.bias_gelu_fwd(x, bias)
    ref = oracle.bias_gelu_bwd(dy, x, bias)
    # An elementwise map whose output is rounded once: |x - ref|_e <= 2^-9 |ref_e| in bf16.  The max-over-RMS bar of the
    # other rows kernels cannot hold here at 21 M elements (|y| reaches 8, where half a bf16 unit is 0.03 = 0.035 RMS),
    # so bf16 is judged elementwise with twice that unit plus a small absolute term; fp32 keeps its bar.
    def ok(got, want):
        if dtype == "f32":
            return err(got, want, dtype) < BAR[dtype]
        rms = float(np.sqrt(np.mean(want ** 2)))
        return bool(np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want) + 1e-3 * rms))
    assert ok(host(y), ref_y)
    assert ok(host(dx), ref["dx"])
    assert torch.equal(dx, dx2)
    # dbias is an fp32 sum of fp32 products on both dtypes
    assert err(host(dbias), ref["dbias"], "f32") < 1e-4



@pytest.mark.parametrize("rows,h,dtype", [
    (8192, 1024, "bf16"), (8193, 1016, "bf16"), (4096, 2048, "f32"), (4097, 2056, "bf16"),      # x and dy read once: 128, 256 threads a row
    (2048, 4104, "bf16"), (2049, 20480, "bf16"), (2048, 20480, "f32"), (4096, 28672, "bf16"),   # 512 threads: one chunk more than 512, widest rows
    (2047, 4104, "bf16"), (4095, 20488, "bf16"),                                                # one row too few for that
    (128, 520, "bf16"), (129, 520, "bf16"), (512, 12288, "bf16"), (513, 12288, "bf16"), (512, 12280, "bf16"), (700, 32768, "f32"),
    (256, 1024, "bf16"), (257, 1024, "bf16"), (384, 2048, "f32"), (385, 2048, "f32"), (513, 4096, "bf16"), (385, 4160, "bf16"),  # one split or several: full last blocks
    (320, 16384, "bf16"), (321, 16384, "bf16"), (641, 12352, "f32"), (600, 24576, "bf16"), (520, 20544, "bf16"),                # ... of wide rows
    (300, 28680, "bf16"), (1500, 32768, "bf16"), (1000, 32768, "f32"),                                                          # 1024 threads a row; beyond the last-level cache
    (800, 8200, "bf16"), (801, 8200, "bf16"), (1501, 12288, "bf16"), (1500, 12296, "bf16"), (1024, 8208, "f32"), (1025, 8208, "f32"),  # LayerNorm backward: split on many rows
    (33, 8, "bf16"), (140, 8, "f32"), (300, 72, "bf16"),                                                                         # a column block of one lane
])
def test_column_sums(rows, h, dtype):
    """The passes that sum columns, on both sides of every line of their dispatch: rows split or not, x and dy of the LayerNorm
    backward read once or twice, widths that leave lanes without work.  Reference: the definitions in fp64 on the device;
    tolerances: those of the tests above."""
    from gpu_util import BAR, DT, err, host
    tdt, code = DT[dtype]
    g = torch.Generator(device="cuda").manual_seed(rows + h)
    x, dy = (torch.randn(rows, h, device="cuda", generator=g).to(tdt) for _ in range(2))
    gamma, bias = ((1.0 + 0.1 * torch.randn(h, device="cuda", generator=g)).to(tdt), (0.1 * torch.randn(h, device="cuda", generator=g)).to(tdt))
    print(f"column sums rows={rows} h={h} {dtype}", flush=True)
    desc = sar.RowsDesc.make(rows, h, dtype=code, p=0.1, seed=3, offset=9)
    dx = torch.empty_like(x)
    mean, rstd = (torch.empty(rows, dtype=torch.float32, device="cuda") for _ in range(2))
    c0, c1 = (torch.empty(h, dtype=torch.float32, device="cuda") for _ in range(2))
    def scratch(n):
        return torch.full((max(16, n) // 4,), float("nan"), dtype=torch.float32, device="cuda")
    def close(got, ref, how):
        e = err(host(got), ref.cpu().numpy(), how)
        assert e <= BAR[how], e
    xd, dyd = x.double(), dy.double()
    sar.ln_fwd(desc, x, gamma, bias, dx, mean, rstd)
    sar.ln_bwd(desc, dy, x, mean, rstd, gamma, dx, c0, c1, scratch(sar.ln_bwd_workspace(desc)))
    mu = xd.mean(1, keepdim=True)
    xhat = (xd - mu) * (xd.var(1, unbiased=False, keepdim=True) + desc.eps).rsqrt()
    gg = dyd * gamma.double()
    rs = (xd.var(1, unbiased=False, keepdim=True) + desc.eps).rsqrt()
    close(dx, rs * (gg - gg.mean(1, keepdim=True) - xhat * (gg * xhat).mean(1, keepdim=True)), dtype)
    close(c0, (dyd * xhat).sum(0), "f32")
    close(c1, dyd.sum(0), "f32")
    del xhat, gg
    m = torch.empty(rows, h, dtype=torch.uint8, device="cuda")
    sar.bias_dropout_add(desc, x, None, dy, dx, m)
    sar.bias_dropout_add_bwd(desc, dy, dx, c0, scratch(sar.bias_dropout_add_bwd_workspace(desc)))
    ref = dyd * m.double() / (1.0 - float(np.float32(0.1)))
    close(dx, ref, dtype)
    close(c0, ref.sum(0), "f32")
    sar.bias_gelu_bwd(desc, dy, x, bias, dx, c0, scratch(sar.bias_gelu_bwd_workspace(desc)))
    z = (xd + bias.double())
    ref = dyd * (0.5 * (1.0 + torch.erf(z / 2 ** 0.5)) + z * torch.exp(-z * z / 2) / (2 * np.pi) ** 0.5)
    if dtype == "f32":
        close(dx, ref, dtype)
    else:
        assert bool(((dx.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-3 * ref.square().mean().sqrt()).all())
    close(c0, ref.sum(0), "f32")


@pytest.mark.parametrize("rows,h,dtype,with_bias", [(37, 1032, "bf16", True), (37, 1032, "f32", True), (5, 8, "bf16", False), (5, 8, "f32", False), (300, 12800, "bf16", False),
                                                    (4096, 8200, "bf16", True)])
def test_results_written_past_the_caches(rows, h, dtype, with_bias):
    """The forward of the bias-GeLU with y, and the backward of the dropout-add with dx stored nontemporally, in all their instantiations, forced and (67 MB) as their
    size has it: the reference of every size, and the bits of ordinary stores."""
    from gpu_util import DT
    by_size = rows * h * (2 if dtype == "bf16" else 4) >= 64e6
    try:
        sar.sar_test_force_forms(-1, -1, -1 if by_size else 1, -1)
        test_bias_gelu(rows, h, dtype, with_bias)
        if rows * h < 10 ** 7:
            test_bias_dropout_add_bwd(rows, h, dtype, 0.1)
        tdt, code = DT[dtype]
        g = torch.Generator(device="cuda").manual_seed(rows)
        x, bias = torch.randn(rows, h, device="cuda", generator=g).to(tdt), torch.randn(h, device="cuda", generator=g).to(tdt) if with_bias else None
        y = [torch.full_like(x, float("nan")) for _ in range(2)]
        for stream in (0, 1):
            sar.sar_test_force_forms(-1, -1, stream, -1)
            sar.bias_gelu_fwd(sar.RowsDesc.make(rows, h, dtype=code), x, bias, y[stream])
        desc = sar.RowsDesc.make(rows, h, dtype=code, p=0.1, seed=5)
        ws = torch.empty(max(16, sar.bias_dropout_add_bwd_workspace(desc)), dtype=torch.uint8, device="cuda")
        dx, dbias = [torch.full_like(x, float("nan")) for _ in range(3)], [torch.empty(h, dtype=torch.float32, device="cuda") for _ in range(3)]
        for i, stream in enumerate((0, 1, -1)):
            sar.sar_test_force_forms(-1, -1, stream, -1)
            sar.bias_dropout_add_bwd(desc, x, dx[i], dbias[i], ws)
        torch.cuda.synchronize()
        assert torch.equal(y[0], y[1]) and all(torch.equal(dx[0], dx[i]) and torch.equal(dbias[0], dbias[i]) for i in (1, 2))
    finally:
        sar.sar_test_force_forms(-1, -1, -1, -1)
