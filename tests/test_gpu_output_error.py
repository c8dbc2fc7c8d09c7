"""Layer-output error of the quantized, compensated layer under activation quantization (the metric
of the paper's per-layer error figure, Sec. 5.3) on the device against oracle.layer_output_error.

Inputs of the stage (codes, scales, smoothing diagonal, L_A, L_B) come from the oracle, rounded to
fp32 where the device takes fp32; both sides then evaluate the same function of the same numbers.
Tolerance: the device's products carry about 2^-16 relative error per term with random signs, i.e. a
perturbation of about 1e-5 ||X W^T||_F that is almost orthogonal to the residual; with err = e ||X W^T||_F
the norm moves by about (1e-5 / e)^2 / 2 relative.  The bar is 2e-4 relative, plus 1e-5 ||X W^T||_F for
the nearly exact W8 cases.
"""
import numpy as np
import pytest
import torch

import aser_synth as synth
import paper_2411_07762_amd as aser
from oracle import aser_oracle as orc

from gpu_util import DEV, new_ctx, to_dev_x
from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def run_case(label, spec, sample, variants, packed):
    W = synth.make_weight(spec)
    x_np = synth.make_activations(spec)
    X = synth.activations_as_f32(spec, x_np)
    ref = orc.calibrate_layer(W, X, spec.bits, spec.f, spec.r)
    md = ref.smooth.mdiag
    L_A32, L_B32 = ref.rec.L_A.astype(np.float32), ref.rec.L_B.astype(np.float32)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(spec.m, spec.n, sample, spec.r))
    Wd = torch.from_numpy(W).to(DEV)
    Xd = to_dev_x(spec, x_np[:sample])
    mdd = torch.from_numpy(md).to(DEV)
    if packed:
        codes_d = torch.from_numpy(orc.pack_int4(ref.quant.codes)).to(DEV)
        layout = aser.ASER_CODES_INT4_PACKED
    else:
        codes_d = torch.from_numpy(ref.quant.codes).to(DEV)
        layout = aser.ASER_CODES_INT8
    scales_d = torch.from_numpy(ref.quant.scales).to(DEV)
    LAd, LBd = torch.from_numpy(L_A32).to(DEV), torch.from_numpy(L_B32).to(DEV)
    out = {}
    for act_bits, comp in variants:
        want, ynorm = orc.layer_output_error(W, X[:sample], md, ref.quant.codes, ref.quant.scales,
                                             L_A32 if comp else None, L_B32 if comp else None, act_bits)
        st, err, refn = aser.aser_layer_output_error(ctx, Wd, Xd, mdd, codes_d, layout, scales_d,
                                                     LAd if comp else None, LBd if comp else None,
                                                     spec.r if comp else 0, act_bits or 0)
        ctx.check(st)
        say("%s: act_bits=%s compensated=%s  error oracle %.6g device %.6g (rel %.2e), ||X W^T|| %.6g / %.6g" %
            (label, act_bits, comp, want, err, abs(err - want) / want, ynorm, refn))
        assert abs(refn - ynorm) <= 1e-5 * ynorm
        assert abs(err - want) <= 2e-4 * want + 1e-5 * ynorm
        out[(act_bits, comp)] = err
    return out, ref


VARIANTS = [(None, False), (None, True), (8, False), (8, True), (6, True), (4, True)]

CASES = [
    ("c0", synth.CONFIGS["c0"], 512, False),
    ("ragged_bf16_packed", synth.mini("oe1", 130, 334, 1500, r=24, f=6), 333, True),
    ("tall_f32_w8", synth.mini("oe2", 300, 200, 900, x_dtype="f32", r=16, f=5, bits=8), 257, False),
    ("c1_shape_small", synth.CONFIGS["c1"].with_(m=512, n=768, tokens=3072, r=32, f=16), 1024, True),
]


@pytest.mark.parametrize("name,spec,sample,packed", CASES, ids=[c[0] for c in CASES])
def test_layer_output_error(name, spec, sample, packed):
    say("output error case %s m=%d n=%d sample=%d" % (name, spec.m, spec.n, sample))
    out, ref = run_case(name, spec, sample, VARIANTS, packed)
    # what the paper's figure shows: compensation lowers the error left by RTN, coarser activations raise it
    assert out[(8, True)] < out[(8, False)] and out[(None, True)] < out[(None, False)]
    assert out[(4, True)] > out[(6, True)] > out[(8, True)]


def test_output_error_on_the_calibration_set_is_the_whitened_error():
    """Without activation quantization and over the whole calibration set the output error is the
    whitened error of Eq. 8 (X'^T X' = S S^T): the device's number against the oracle's sigma tail."""
    spec = synth.mini("oe3", 96, 160, 640, r=12, f=4)
    out, ref = run_case("calibration_set", spec, spec.tokens, [(None, True), (None, False)], True)
    assert abs(out[(None, True)] - ref.rec.err) <= 2e-4 * ref.rec.err
    assert abs(out[(None, False)] - ref.rec.err0) <= 2e-4 * ref.rec.err0


def test_headline_layer_output_error_w4a8():
    """The 4096 x 4096 layer of the bench, W4A8 and W4A6 on a sample of 2048 calibration tokens, with
    and without compensation; factors and codes from the device's own calibration of the layer
    (bit-exact codes; factors within the bars of the end-to-end test), the error from both sides."""
    spec = synth.CONFIGS["c1"]
    sample = 2048
    say("output error c1 full size")
    W = synth.make_weight(spec)
    x_np = synth.make_activations(spec, workers=8)
    ctx = new_ctx()
    buf = aser.LayerBuffers(spec.m, spec.n, spec.r, spec.f, spec.bits, packed=True)
    Wd = torch.from_numpy(W).to(DEV)
    Xd = to_dev_x(spec, x_np)
    aser.calibrate_layer(ctx, Wd, Xd, buf)
    torch.cuda.synchronize()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(spec.m, spec.n, sample, spec.r))
    Xs = synth.bf16_to_f32(x_np[:sample])
    md = buf.mdiag.cpu().numpy()
    packed = buf.codes.cpu().numpy()
    codes = np.stack([((packed & 0x0F).astype(np.int8) ^ 8) - 8, ((packed >> 4).astype(np.int8) ^ 8) - 8], axis=-1)
    codes = codes.reshape(spec.m, spec.n).astype(np.int8)
    scales = buf.scales.cpu().numpy()
    L_A, L_B = buf.L_A.cpu().numpy(), buf.L_B.cpu().numpy()
    res = {}
    for act_bits, comp in [(8, False), (8, True), (6, False), (6, True)]:
        want, ynorm = orc.layer_output_error(W, Xs, md, codes, scales, L_A if comp else None, L_B if comp else None, act_bits)
        st, err, refn = aser.aser_layer_output_error(ctx, Wd, Xd[:sample], buf.mdiag, buf.codes, aser.ASER_CODES_INT4_PACKED,
                                                     buf.scales, buf.L_A if comp else None, buf.L_B if comp else None,
                                                     spec.r if comp else 0, act_bits)
        ctx.check(st)
        say("c1 W4A%d compensated=%s: error oracle %.6g device %.6g (rel %.2e), relative to ||X W^T|| %.4f" %
            (act_bits, comp, want, err, abs(err - want) / want, err / refn))
        assert abs(err - want) <= 2e-4 * want
        res[(act_bits, comp)] = err
    assert res[(8, True)] < res[(8, False)] and res[(6, True)] < res[(6, False)]


@pytest.mark.parametrize("rows,m", [(70, 130), (1700, 1800), (2049, 4100)])
@pytest.mark.parametrize("power,act_bits,x_dtype", [(-100, 8, "bf16"), (-80, 8, "f32"), (66, 8, "bf16"), (66, 0, "f32")])
def test_norms_of_tiny_and_huge_outputs(rows, m, power, act_bits, x_dtype):
    """Outputs of about 1e-30, 1e-24 and 1e20, whose squares leave the range of fp32: the sums of squares are fp64, so both norms
    stay what they are for the same activations at unit scale, times the power of two.  Bars as above."""
    rng = np.random.default_rng([9, rows, m])
    n, r = 64, 8
    W = rng.standard_normal((m, n)).astype(np.float32) * 0.5
    X = synth.bf16_to_f32(synth.f32_to_bf16_bits(rng.standard_normal((rows, n)).astype(np.float32)))
    md = np.ones(n, np.float32)
    md[:3] = 2.5
    q = orc.quantize_rtn(W * md[None, :], np.zeros(0, np.int32), np.ones(n, np.float32), 4)
    L_A = rng.standard_normal((m, r)).astype(np.float32) * 0.01
    L_B = rng.standard_normal((r, n)).astype(np.float32) * 0.05
    want, ynorm = orc.layer_output_error(W, X, md, q.codes, q.scales, L_A, L_B, act_bits or None)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(m, n, rows, r))
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    Xd = dev(X * np.float32(2.0 ** power)).to(torch.bfloat16 if x_dtype == "bf16" else torch.float32)
    st, err, ref = aser.aser_layer_output_error(ctx, dev(W), Xd, dev(md), dev(q.codes), aser.ASER_CODES_INT8, dev(q.scales), dev(L_A), dev(L_B),
                                                r, act_bits)
    ctx.check(st)
    err, ref = err * 2.0 ** -power, ref * 2.0 ** -power
    assert abs(ref - ynorm) <= 1e-5 * ynorm
    assert abs(err - want) <= 2e-4 * want + 1e-5 * ynorm


@pytest.mark.parametrize("x_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("act_bits", [0, 8])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_non_finite_activations_are_refused(value, act_bits, x_dtype):
    """One infinite or NaN entry; weights and codes of opposite signs, so that an infinite activation moves both outputs of every
    channel to the same side and no difference of infinities makes it a NaN."""
    W = torch.full((4, 32), 1.001, device=DEV)
    codes = torch.full((4, 32), -7, dtype=torch.int8, device=DEV)
    scales = torch.full((4,), 0.1431, device=DEV)
    X = torch.ones((3, 32), device=DEV)
    X[1, 5] = float(value)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(4, 32, 3, 0))
    st, _, _ = aser.aser_layer_output_error(ctx, W, X.to(torch.bfloat16) if x_dtype == "bf16" else X, None, codes, aser.ASER_CODES_INT8, scales, None, None,
                                            0, act_bits)
    assert st == aser.ASER_ERR_INVALID_ARG and "non-finite" in ctx.last_error()


@pytest.mark.parametrize("m,n,rows,r,bits,x_dtype,act_bits", [
    (70, 96, 33, 0, 8, "bf16", 8), (130, 334, 257, 1, 4, "bf16", 6), (257, 1000, 65, 33, 8, "f32", 8), (64, 64, 1, 64, 4, "bf16", 4),
    (1700, 224, 1800, 97, 4, "bf16", 8), (300, 4128, 129, 128, 8, "bf16", 8), (200, 301, 90, 129, 8, "f32", 8), (5, 3, 7, 2, 8, "bf16", 8)])
def test_second_output_from_codes(m, n, rows, r, bits, x_dtype, act_bits):
    """Channels short of a step of 32 and of 64, code rows used in place and copied, every number of blocks of the rank-r branch, one
    token, every tile size, and the calls that keep the product of planes (r = 129; planes that do not fit), against fp64."""
    g = torch.Generator(device=DEV)
    g.manual_seed(m * n + r)
    W = torch.randn((m, n), generator=g, device=DEV) * 0.05
    X = torch.randn((rows, n), generator=g, device=DEV)
    X = X.to(torch.bfloat16) if x_dtype == "bf16" else X
    md = torch.ones(n, device=DEV)
    md[: n // 3] = 1.5
    qmax = 2 ** (bits - 1) - 1
    q = torch.randint(-qmax, qmax + 1, (m, n), generator=g, device=DEV, dtype=torch.int8)
    packed = bits == 4 and n % 2 == 0
    codes = ((q[:, 0::2] & 15) | (q[:, 1::2] << 4)).view(torch.uint8).contiguous() if packed else q
    scales = (0.5 + torch.rand(m, generator=g, device=DEV)) * 0.1 / qmax
    L_A = torch.randn((m, max(r, 1)), generator=g, device=DEV) * 0.1
    L_B = torch.randn((max(r, 1), n), generator=g, device=DEV) * 0.05
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(m, n, rows, r))
    st, err, ref = aser.aser_layer_output_error(ctx, W, X, md, codes, aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8, scales,
                                                L_A if r else None, L_B if r else None, r, act_bits)
    ctx.check(st)
    xq, xs = orc.quantize_act_rtn(X.float().cpu().numpy(), md.cpu().numpy(), act_bits)
    x = torch.from_numpy(xq.astype(np.float64) * xs.astype(np.float64)[:, None])
    Wt = (q.double() * scales.double()[:, None]).cpu() + ((L_A.double() @ L_B.double()).cpu() if r else 0.0)
    Y = X.double().cpu() @ W.double().cpu().T
    want, ynorm = float(torch.linalg.norm(Y - x @ Wt.T)), float(torch.linalg.norm(Y))
    assert abs(ref - ynorm) <= 1e-5 * ynorm              # 2^-17 per product
    assert abs(err - want) <= 1e-5 * (want + ynorm)


@pytest.mark.parametrize("m,n,rows,r", [(1024, 1024, 500, 64), (300, 4128, 129, 128), (1700, 224, 1800, 33), (96, 512, 64, 16)])
def test_second_output_of_factors_that_cancel(m, n, rows, r):
    """L_A L_B is 1e-4 of its terms, and these are 100 sqrt(r) times the output.  The factors, P and their products keep 24 bits, so an output is off by
    2^-24 of the terms in P and again in L_A P, and by 2^-17 of itself in the planes of W, all with random signs: of the norm over rows m
    outputs that is the same over sqrt(rows m), four standard deviations below, and the square of it."""
    g = torch.Generator(device=DEV)
    g.manual_seed(m + n)
    W = torch.randn((m, n), generator=g, device=DEV) * 0.05
    X = torch.randn((rows, n), generator=g, device=DEV).to(torch.bfloat16)
    q = torch.randint(-127, 128, (m, n), generator=g, device=DEV, dtype=torch.int8)
    scales = (0.5 + torch.rand(m, generator=g, device=DEV)) * 0.1 / 127
    L_A = torch.randn((m, r), generator=g, device=DEV) * 100.0
    L_B = torch.randn((r, n), generator=g, device=DEV) * 0.05
    h = r // 2
    L_A[:, h:2 * h] = -L_A[:, :h]
    L_B[h:2 * h] = L_B[:h] + 1e-6 * torch.randn((h, n), generator=g, device=DEV)
    if r % 2:
        L_A[:, r - 1] *= 1e-4
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(m, n, rows, r))
    st, err, ref = aser.aser_layer_output_error(ctx, W, X, None, q, aser.ASER_CODES_INT8, scales, L_A, L_B, r, 8)
    ctx.check(st)
    xq, xs = orc.quantize_act_rtn(X.float().cpu().numpy(), np.ones(n, np.float32), 8)
    x = torch.from_numpy(xq.astype(np.float64) * xs.astype(np.float64)[:, None])
    Y = X.double().cpu() @ W.double().cpu().T
    D = Y - x @ (q.double() * scales.double()[:, None]).cpu().T - (x @ L_B.double().cpu().T) @ L_A.double().cpu().T
    want = float(torch.linalg.norm(D))
    each = 2 * 2.0 ** -24 * 100 * np.sqrt(r) + 2.0 ** -17
    bound = 4 * each / np.sqrt(rows * m) + each ** 2
    say("output error of factors that cancel %s: %.2e of %.2e" % ((m, n, rows, r), abs(err - want) / want, bound))
    assert abs(err - want) <= bound * want
