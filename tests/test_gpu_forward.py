"""The compensated layer at inference (integer MFMA kernel) against oracle.compensated_forward.

Both sides read the same inputs: W codes and scales, L_A, L_B (fp32) and the smoothing diagonal from the
oracle's calibration of the layer.  The activation codes are bit-exact on both sides (checked), the
integer sums are exact, so what differs is fp32 rounding of the scales (about 1e-7) and the rank-r
branch: about 2^-16 relative per product in the split mode, about 2^-9 per factor in the plain bf16 mode
(three rounded factors, random signs over r terms).  Bars, relative Frobenius over the output:
1e-6 without compensation, 2e-5 split, 4e-3 plain.
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


def forward_case(label, spec, sample, packed, act_bits=8, pad=0):
    W = synth.make_weight(spec)
    x_np = synth.make_activations(spec)
    X = synth.activations_as_f32(spec, x_np)
    ref = orc.calibrate_layer(W, X, spec.bits, spec.f, spec.r)
    md = ref.smooth.mdiag
    L_A32, L_B32 = ref.rec.L_A.astype(np.float32), ref.rec.L_B.astype(np.float32)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(sample, spec.n, spec.m, spec.r))
    Xd = to_dev_x(spec, x_np[:sample])
    mdd = torch.from_numpy(md).to(DEV)
    xq = torch.empty((sample, spec.n), dtype=torch.int8, device=DEV)
    xs = torch.empty(sample, dtype=torch.float32, device=DEV)
    ctx.check(aser.aser_quantize_act_rtn(ctx, Xd, mdd, act_bits, xq, xs))
    q_ref, s_ref = orc.quantize_act_rtn(X[:sample], md, act_bits)
    torch.cuda.synchronize()
    assert np.array_equal(xq.cpu().numpy(), q_ref) and np.array_equal(xs.cpu().numpy(), s_ref)
    if packed:
        wq = torch.from_numpy(orc.pack_int4(ref.quant.codes)).to(DEV)
        layout = aser.ASER_CODES_INT4_PACKED
    else:
        wq = torch.from_numpy(ref.quant.codes).to(DEV)
        layout = aser.ASER_CODES_INT8
    wsd = torch.from_numpy(ref.quant.scales).to(DEV)
    LAd, LBd = torch.from_numpy(L_A32).to(DEV), torch.from_numpy(L_B32).to(DEV)
    for comp, split, bar in ((False, False, 1e-6), (True, True, 2e-5), (True, False, 4e-3)):
        want = orc.compensated_forward(X[:sample], md, ref.quant.codes, ref.quant.scales, L_A32 if comp else None,
                                       L_B32 if comp else None, act_bits)
        Ybuf = torch.full((sample, spec.m + pad), float("nan"), dtype=torch.float32, device=DEV)
        Y = Ybuf[:, :spec.m]
        ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq, layout, wsd, LAd if comp else None, LBd if comp else None,
                                                spec.r if comp else 0, split, Y))
        torch.cuda.synchronize()
        got = Y.cpu().numpy().astype(np.float64)
        rel = np.linalg.norm(got - want) / np.linalg.norm(want)
        say("%s: compensated=%s split=%s  ||Y - Y_oracle|| / ||Y_oracle|| = %.2e (bar %.0e)" % (label, comp, split, rel, bar))
        assert np.isfinite(got).all() and rel <= bar
        if split:
            got_split = got
        if pad:
            assert torch.isnan(Ybuf[:, spec.m:]).all()
    # the output error of the kernel's result is the layer-output error of Sec. 5.3's figure
    e_ref, _ = orc.layer_output_error(W, X[:sample], md, ref.quant.codes, ref.quant.scales, L_A32, L_B32, act_bits)
    Yexact = X[:sample].astype(np.float64) @ W.astype(np.float64).T
    e_kernel = np.linalg.norm(Yexact - got_split)
    e_plain = np.linalg.norm(Yexact - got)                     # got: the plain bf16 run, the last of the loop
    say("%s: output error of the kernel's result %.6g (factors rounded to bf16: %.6g), oracle %.6g" %
        (label, e_kernel, e_plain, e_ref))
    assert abs(e_kernel - e_ref) <= 1e-3 * e_ref + 2e-5 * np.linalg.norm(Yexact)


CASES = [
    ("c0_int8", synth.CONFIGS["c0"], 300, False, 8, 0),
    ("c0_int4", synth.CONFIGS["c0"], 1024, True, 8, 4),
    ("ragged_tokens_outputs", synth.mini("fw1", 333, 320, 1500, r=24, f=6), 777, True, 8, 0),
    ("r_not_multiple_of_32_a6", synth.mini("fw2", 600, 96, 700, r=40, f=4), 129, True, 6, 0),
    ("w8_tall", synth.mini("fw3", 700, 160, 900, x_dtype="f32", r=16, f=5, bits=8), 513, False, 8, 0),
    ("c1_shape_small", synth.CONFIGS["c1"].with_(m=768, n=1024, tokens=4096, r=64, f=16), 2048, True, 8, 0),
    # a few steps of the contraction: a last step of 32 channels with packed int4 and with int8 codes, ragged tokens and
    # outputs, a padded output (these and the cases above run the kernels for a few tokens; the tiles of the prefill kernels
    # are in test_gpu_kernel_paths.py)
    ("w4_half_step_at_the_end", synth.mini("fw4", 300, 352, 1400, r=24, f=5), 600, True, 8, 4),
    ("w4_one_and_a_half_steps", synth.mini("fw5", 260, 96, 900, r=8, f=2), 700, True, 8, 0),
    ("w8_half_a_step", synth.mini("fw6", 257, 32, 600, x_dtype="f32", r=8, f=1, bits=8), 257, False, 8, 0),
    ("w8_two_steps_split_tiles", synth.mini("fw7", 513, 128, 1200, r=16, f=3, bits=8), 1025, False, 8, 0),
]


@pytest.mark.parametrize("name,spec,sample,packed,act_bits,pad", CASES, ids=[c[0] for c in CASES])
def test_compensated_forward(name, spec, sample, packed, act_bits, pad):
    say("forward case %s m=%d n=%d tokens=%d r=%d" % (name, spec.m, spec.n, sample, spec.r))
    forward_case(name, spec, sample, packed, act_bits, pad)


def test_mfma_rate_probe_runs():
    """The measurement aid: a loop of nothing but MFMA instructions must land between a tenth of the nominal peak and
    the nominal peak (2.5 PFLOP/s bf16, 5.0 POP/s int8); with the operand traffic of a tile around the instructions
    it cannot be faster than without (5 % for the clock's wander between launches)."""
    ctx = new_ctx()
    ctx.ensure_workspace((33 << 20) + 4 * 256 * 1024 + 256)
    for kind, peak in ((0, 2500.0), (1, 5000.0)):
        alone = {}
        for wgs in (1, 4):
            st, rate = aser.aser_mfma_rate_probe(ctx, kind, wgs, 2000)
            ctx.check(st)
            say("MFMA-only loop kind %d, %d workgroup(s) per compute unit: %.0f T op/s" % (kind, wgs, rate))
            assert 0.1 * peak < rate <= 1.001 * peak
            alone[wgs] = rate
        st, rate = aser.aser_mfma_rate_probe(ctx, kind + 2, 1, 2000)
        ctx.check(st)
        say("MFMA loop with operand traffic, kind %d: %.0f T op/s" % (kind + 2, rate))
        assert 0.1 * peak < rate <= 1.05 * alone[1]


@pytest.mark.parametrize("rows,n,m,r,split,offset", [
    (2049, 32, 200, 1, True, 0), (2049, 96, 300, 33, False, 1), (2080, 4128, 256, 64, True, 0), (2081, 4096, 257, 65, False, 0),
    (2111, 1056, 128, 97, True, 1), (2112, 224, 512, 128, False, 0),
    # 128 tokens per workgroup: tokens around blocks of 128, steps of 64 channels in threes and twelves, whole and halves
    (16385, 32, 256, 33, True, 0), (16511, 96, 256, 64, False, 1), (16512, 416, 260, 128, True, 0), (16513, 1184, 256, 1, False, 0), (16640, 2080, 300, 96, True, 1),
    (8449, 768, 260, 64, False, 0), (8577, 32, 128, 40, True, 1), (9000, 288, 300, 16, True, 0), (12417, 480, 107, 128, True, 1), (16384, 320, 130, 97, False, 0)])
def test_first_product_of_the_rank_branch_for_many_tokens(rows, n, m, r, split, offset):
    """Token counts around blocks of 32, channels short of and beyond what sixteen wavefronts take at a time, every number of column
    blocks, and an L_B that does not start on 16 bytes, against the same product in fp64 on rounded factors."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + n)
    xq = torch.randint(-127, 128, (rows, n), generator=g, device=DEV, dtype=torch.int8)
    xs = torch.rand(rows, generator=g, device=DEV) * 0.1
    wq = torch.randint(-7, 8, (m, n), generator=g, device=DEV, dtype=torch.int8)
    ws = torch.rand(m, generator=g, device=DEV) * 0.01
    la = torch.randn((m, r), generator=g, device=DEV)
    store = torch.randn(r * n + offset, generator=g, device=DEV)
    lb = store[offset:].view(r, n)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    Y = torch.empty((rows, m), device=DEV)
    ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq, aser.ASER_CODES_INT8, ws, la, lb, r, split, Y))
    torch.cuda.synchronize()
    x = (xq.double() * xs.double()[:, None]).cpu()
    rnd = (lambda t: t.cpu().double()) if split else (lambda t: t.cpu().float().bfloat16().double())
    P = rnd((x @ rnd(lb).T).float())
    ref = x @ (wq.double() * ws.double()[:, None]).cpu().T + P @ rnd(la).T
    # split: 2^-17 per factor and product; plain: P is rounded to 2^-9 from fp32 sums that differ from the reference's, so single values fall on the
    # other side (2^-8 of one of r terms)
    tol = 2e-5 if split else 1e-3
    assert float(torch.linalg.norm(Y.cpu().double() - ref) / torch.linalg.norm(ref)) <= tol


@pytest.mark.parametrize("rows,n,m,w4", [
    (1, 32, 16, True), (16, 96, 33, False), (17, 1056, 100, True), (1, 2080, 4100, False), (33, 3104, 4100, True), (32, 5152, 300, False),
    (3, 4128, 8205, True), (16, 8224, 8205, False), (2, 672, 16500, True), (65, 1568, 500, False), (130, 1120, 700, True)])
def test_integer_sums_of_a_few_tokens(rows, n, m, w4):
    """Contractions that end inside a round of the code stream, inside a step and before the last wavefront's share, tokens and
    outputs that end inside a tile: without factors Y is an exact integer, rounded once, times two scales (four roundings of 2^-24)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows * 7 + n)
    xq = torch.randint(-127, 128, (rows, n), generator=g, device=DEV, dtype=torch.int8)
    xs = torch.rand(rows, generator=g, device=DEV) * 0.1
    q = torch.randint(-7, 8, (m, n), generator=g, device=DEV, dtype=torch.int8)
    codes = ((q[:, 0::2] & 15) | (q[:, 1::2] << 4)).view(torch.uint8).contiguous() if w4 else q
    ws = torch.rand(m, generator=g, device=DEV) * 0.01
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, 0))
    Y = torch.full((rows + 1, m), 7.0, device=DEV)
    ctx.check(aser.aser_compensated_forward(ctx, xq, xs, codes, aser.ASER_CODES_INT4_PACKED if w4 else aser.ASER_CODES_INT8, ws, None, None, 0, True, Y[:rows]))
    torch.cuda.synchronize()
    ref = (xq.cpu().double() @ q.cpu().double().T) * xs.cpu().double()[:, None] * ws.cpu().double()
    assert bool(((Y[:rows].cpu().double() - ref).abs() <= 5 * 2.0 ** -24 * ref.abs()).all())
    assert bool((Y[rows] == 7.0).all())


@pytest.mark.parametrize("rows,n,m,r,offset", [(1, 32, 40, 1, 0), (16, 96, 33, 16, 1), (17, 224, 100, 17, 0), (2, 288, 64, 33, 2), (5, 2080, 8205, 64, 0), (33, 2336, 300, 100, 3),
                                               (16, 4128, 8205, 128, 0), (130, 6176, 48, 7, 0)])
@pytest.mark.parametrize("split", [False, True])
def test_rank_branch_of_a_few_tokens(rows, n, m, r, offset, split):
    """Contractions that end inside a round, a sum of 256 and a workgroup's 2048 channels, ranks around the tiles of 16 and the steps of 32, an L_B that does not
    start on 16 bytes; P in front and beside the codes.  Split: a sum takes eight steps and meets at most 8 + 4 others, 2^-24 each and of the
    largest partial one: 2^-20.  Rounded: P from fp32 sums that differ from the reference's, as for many tokens above.  An infinite factor stays one."""
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + n + r)
    xq = torch.randint(1, 128, (rows, n), generator=g, device=DEV, dtype=torch.int8) * (1 - 2 * (torch.arange(n, device=DEV) % 2)).to(torch.int8)
    xs = 0.01 + torch.rand(rows, generator=g, device=DEV) * 0.1
    wq = torch.randint(-7, 8, (m, n), generator=g, device=DEV, dtype=torch.int8)
    ws = torch.rand(m, generator=g, device=DEV) * 0.01
    la = torch.randn((m, r), generator=g, device=DEV)
    lb = torch.randn(r * n + offset, generator=g, device=DEV)[offset:].view(r, n)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))

    def call():
        Y = torch.empty((rows, m), device=DEV)
        ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq, aser.ASER_CODES_INT8, ws, la, lb, r, split, Y))
        torch.cuda.synchronize()
        return Y.cpu().double()

    x = (xq.double() * xs.double()[:, None]).cpu()
    rnd = (lambda t: t.cpu().double()) if split else (lambda t: t.cpu().float().bfloat16().double())
    ref = x @ (wq.double() * ws.double()[:, None]).cpu().T + rnd((x @ rnd(lb).T).float()) @ rnd(la).T
    assert float(torch.linalg.norm(call() - ref) / torch.linalg.norm(ref)) <= (2.0 ** -20 if split else 1e-3)
    lb[r - 1, n - 2] = float("inf")                       # the codes of even channels are positive
    assert bool((call() == torch.where(la[:, r - 1].cpu() > 0, np.inf, -np.inf)).all())


@pytest.mark.parametrize("n", [8, 504, 2056, 4096, 4097, 4104, 6152, 11008, 16392])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("scaled,offset", [(True, 0), (True, 1), (False, 0)])
def test_activation_quantizer_at_the_ends_of_a_token(n, dt, scaled, offset):
    """Tokens that end inside a thread's groups, in the last one's start and in no group of eight, with M that starts on 16 bytes or not, bit for bit."""
    g = torch.Generator(device=DEV)
    g.manual_seed(n)
    X = (torch.randn((5, n), generator=g, device=DEV) * 3.0).to(dt)
    X[3] = 0.0
    X[4, n - 1] = -500.0                                  # the largest value is the token's last
    md = torch.ones(n + 1, device=DEV)
    md[offset::7] = 1.0 + 30.0 * torch.rand(md[offset::7].shape, generator=g, device=DEV)
    md = md[offset:offset + n] if scaled else None
    q, s = torch.full((6, n), 99, dtype=torch.int8, device=DEV), torch.empty(5, device=DEV)
    ctx = new_ctx()
    ctx.check(aser.aser_quantize_act_rtn(ctx, X, md, 8, q[:5], s))
    torch.cuda.synchronize()
    ref_q, ref_s = orc.quantize_act_rtn(X.float().cpu().numpy(), md.cpu().numpy() if scaled else np.ones(n, np.float32), 8)
    assert np.array_equal(q[:5].cpu().numpy(), ref_q) and np.array_equal(s.cpu().numpy(), ref_s.reshape(-1).astype(np.float32)) and bool((q[5] == 99).all())


@pytest.mark.parametrize("rows,n,m", [(1, 4096, 300), (16, 2080, 8205), (33, 1056, 500)])
@pytest.mark.parametrize("scale", [1e-36, 1e-30, 1e30])
def test_rank_branch_of_a_few_tokens_keeps_its_bits_at_any_scale(rows, n, m, scale):
    """Factors of an uneven size, whose three parts would leave the range of bf16 at one end or the other: the bound of the split factors above."""
    r = 40
    g = torch.Generator(device=DEV)
    g.manual_seed(rows + n)
    xq = torch.randint(-127, 128, (rows, n), generator=g, device=DEV, dtype=torch.int8)
    xs = 0.01 + torch.rand(rows, generator=g, device=DEV) * 0.1
    wq = torch.zeros((m, n), device=DEV, dtype=torch.int8)
    ws = torch.ones(m, device=DEV)
    la = torch.randn((m, r), generator=g, device=DEV) / scale
    lb = torch.randn((r, n), generator=g, device=DEV) * scale
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    Y = torch.empty((rows, m), device=DEV)
    ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq, aser.ASER_CODES_INT8, ws, la, lb, r, True, Y))
    torch.cuda.synchronize()
    ref = ((xq.double() * xs.double()[:, None]).cpu() @ lb.double().cpu().T) @ la.double().cpu().T
    assert float(torch.linalg.norm(Y.double().cpu() - ref) / torch.linalg.norm(ref)) <= 2.0 ** -20
