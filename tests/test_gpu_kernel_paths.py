"""The dispatch borders of single kernels: sizes at the edges of tiles and of the rules that pick a kernel, against
NumPy or the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import aser_synth as synth
import paper_2411_07762_amd as aser
from gpu_util import DEV, lower, new_ctx, run_gram
from oracle import aser_oracle as orc
from test_dispatch_rules import gram_query, rule  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rows", [(1024, 700), (1032, 256), (1280, 255), (1536, 1000), (2304, 2049), (2056, 300), (4096, 777)])
def test_gram_chunks_at_the_borders_of_the_schedules(n, rows):
    """Bound per entry as for every bf16 Gram matrix of this suite: exact products, fp32 sums of at most 32768 terms."""
    spec = synth.mini("gram%d" % n, 64, n, 2 * rows, n_outliers=5, seed_id=950 + n % 50)
    X = synth.make_activations(spec)
    G, abs_sum, count = run_gram(new_ctx(), spec, X, chunks=2)
    ref, ref_abs, _ = orc.gram(synth.activations_as_f32(spec, X))
    d = np.sqrt(np.diag(ref))
    assert np.max(np.abs(lower(G.cpu().numpy()) - np.tril(ref)) / np.outer(d, d)) <= 2e-5
    assert np.max(np.abs(abs_sum.cpu().numpy() - ref_abs) / ref_abs) <= 1e-12
    assert int(count.item()) == 2 * rows


@pytest.mark.parametrize("rows,n,m,r,packed", [
    (1, 32, 17, 1, True), (1, 4096, 8208, 64, True), (15, 96, 500, 40, False), (16, 1056, 8200, 128, True), (17, 2080, 333, 0, False),
    (33, 1024, 64, 8, True), (64, 3104, 8195, 64, False), (65, 11008, 130, 64, True), (128, 160, 8192, 128, False), (128, 4128, 700, 128, True),
    (129, 1056, 260, 64, True), (500, 2080, 96, 72, False), (257, 4096, 8193, 16, True)])
def test_forward_of_a_few_tokens(rows, n, m, r, packed):
    """Integer sums are exact, so without factors only the fp32 scaling remains (two roundings: 1.2e-7, bar 1e-6); the split branch
    carries fp32 sums of n and r terms (bar 2e-5, as for the prefill kernels), the other one bf16 factors (bar 4e-3)."""
    rng = np.random.default_rng([77, rows, n, m, r])
    xq = rng.integers(-127, 128, (rows, n)).astype(np.int8)
    xs = rng.uniform(0.01, 0.05, rows).astype(np.float32)
    q = rng.integers(-7, 8, (m, n)).astype(np.int8) if packed else rng.integers(-127, 128, (m, n)).astype(np.int8)
    ws = rng.uniform(0.001, 0.003, m).astype(np.float32)
    L_A = rng.standard_normal((m, max(r, 1))).astype(np.float32)
    L_B = rng.standard_normal((max(r, 1), n)).astype(np.float32) * 0.01
    X = xq.astype(np.float64) * xs.astype(np.float64)[:, None]
    low = X @ L_B.astype(np.float64).T @ L_A.astype(np.float64).T
    base = X @ (q.astype(np.float64) * ws.astype(np.float64)[:, None]).T
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    wq = torch.from_numpy(orc.pack_int4(q) if packed else q).to(DEV)
    layout = aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8
    lb = torch.zeros(L_B.size + 1, dtype=torch.float32, device=DEV)
    lb[1:] = torch.from_numpy(L_B.reshape(-1)).to(DEV)
    lbs = (lb[1:].view(L_B.shape), torch.from_numpy(L_B).to(DEV))            # 4-byte aligned, 16-byte aligned
    for comp, split, bar in ((False, False, 1e-6), (True, True, 2e-5), (True, False, 4e-3)):
        if comp and r == 0:
            continue
        want = base + low if comp else base
        for lbd in lbs if rows > 1 else lbs[:1]:
            Y = torch.full((rows, m + 3), 7.0, dtype=torch.float32, device=DEV)
            ctx.check(aser.aser_compensated_forward(ctx, torch.from_numpy(xq).to(DEV), torch.from_numpy(xs).to(DEV), wq, layout,
                                                    torch.from_numpy(ws).to(DEV), torch.from_numpy(L_A).to(DEV) if comp else None,
                                                    lbd if comp else None, r if comp else 0, split, Y[:, :m]))
            got = Y.cpu().numpy()
            assert np.all(got[:, m:] == 7.0)
            assert np.linalg.norm(got[:, :m] - want) <= bar * np.linalg.norm(want)


# Sizes that the kernels for a few tokens do not take (tests/test_dispatch_rules.py holds the rule to that): the 256 x 256 tiles with
# fewer steps than their ring has stages and with half a step at the end, the 128 x 256 tiles (fewer than 256 tokens or outputs), and the
# first product of the rank-r branch with one to four blocks of 32 columns; ragged tokens and outputs.
PREFILL = [(2049, 32, 260, 40, False), (2049, 32, 300, 128, True), (2049, 96, 257, 72, True), (2305, 96, 513, 16, False), (2100, 352, 300, 128, False),
           (300, 352, 16500, 40, True), (200, 352, 8250, 72, True), (200, 96, 8250, 16, False), (2100, 96, 200, 128, False), (2100, 32, 130, 24, True),
           (129, 1056, 16400, 0, True), (1, 96, 16500, 128, False)]


@pytest.mark.parametrize("rows,n,m,r,packed", PREFILL)
def test_forward_of_the_prefill_kernels(rows, n, m, r, packed):
    test_forward_of_a_few_tokens(rows, n, m, r, packed)


@pytest.mark.parametrize("rows,n,dtype", [(16385, 2064, "bf16"), (16387, 4096, "bf16"), (65537, 2064, "f32"), (16384, 2064, "bf16"),
                                          (3, 1016, "bf16"), (5, 1032, "f32"), (9, 2048, "bf16"), (7, 2056, "bf16")])
def test_activation_quantizer_at_the_borders_of_its_kernels(rows, n, dtype):
    """Bit-exact.  Tokens are independent, so a sample of them stands for all: the first and last 64 and 300 in between."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(rows + n)
    X = torch.randn((rows, n), generator=gen, device=DEV).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    md = torch.ones(n, device=DEV)
    md[torch.randperm(n, generator=gen, device=DEV)[:32]] = 1.0 + 2.0 * torch.rand(32, generator=gen, device=DEV)
    codes = torch.empty((rows, n), dtype=torch.int8, device=DEV)
    scales = torch.empty(rows, dtype=torch.float32, device=DEV)
    ctx = new_ctx()
    ctx.check(aser.aser_quantize_act_rtn(ctx, X, md, 8, codes, scales))
    pick = np.unique(np.concatenate([np.arange(min(64, rows)), np.arange(max(0, rows - 64), rows), np.random.default_rng(1).integers(0, rows, 300)]))
    at = torch.from_numpy(pick).to(DEV)
    q, s = orc.quantize_act_rtn(X[at].float().cpu().numpy(), md.cpu().numpy(), 8)
    assert np.array_equal(codes[at].cpu().numpy(), q)
    assert np.array_equal(scales[at].cpu().numpy(), s)


@pytest.mark.parametrize("k", [2, 7, 8, 64, 1023, 1025, 2049, 4100])
def test_eigenvalues_at_the_borders_of_the_multisection(k):
    """T = a diagonal matrix (S = none): its singular values are the entries, and the path behind the Gram matrix is fp64, so they
    come back to 60 halvings of the squared range: sigma to 1e-9 of the largest (sqrt of 2^-60)."""
    rng = np.random.default_rng(k)
    sg = np.sort(rng.uniform(0.5, 2.0, k).astype(np.float32))[::-1]
    T = torch.zeros((k, k), dtype=torch.float32, device=DEV)
    T.diagonal().copy_(torch.from_numpy(sg.copy()).to(DEV))
    out = torch.empty(k, dtype=torch.float64, device=DEV)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(k, k, False))
    ctx.check(aser.aser_singular_values(ctx, T, None, out))
    assert np.max(np.abs(out.cpu().numpy() - sg.astype(np.float64))) <= 1e-9 * 2.0
    for alpha in (0.01, 0.4, 0.9999):
        st, r, _ = aser.aser_select_rank(ctx, out, alpha)
        ctx.check(st)
        assert r == orc.rank_from_alpha(out.cpu().numpy(), alpha)


@pytest.mark.parametrize("k", [1, 2, 3, 4, 17, 63, 64, 65, 66, 128, 129, 193, 200, 255, 256, 257, 258, 259, 267, 268, 270, 330, 513])
def test_eigenvalues_of_matrices_that_end_in_one_workgroup(k):
    """Full matrices: the squares within the backward error of the Gram product and of the Householder chain, O(k) roundings of
    the largest (factor 16), against numpy's SVD of the same values in fp64."""
    rng = np.random.default_rng(k)
    A = (rng.standard_normal((k + 5, k)) * np.exp(rng.uniform(-3, 3, k))[None, :]).astype(np.float32)
    out = torch.empty(k, dtype=torch.float64, device=DEV)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(k + 5, k, False))
    ctx.check(aser.aser_singular_values(ctx, torch.from_numpy(A).to(DEV), None, out))
    want = np.linalg.svd(A.astype(np.float64), compute_uv=False)
    assert np.max(np.abs(out.cpu().numpy() ** 2 - want ** 2)) <= 16 * k * 2.0 ** -52 * want[0] ** 2


def known_matrix(m, n, sg, seed):
    """H_1 D H_2 with D the diagonal matrix of sg and H = I - 2 u u^T: a full matrix with known singular values and vectors."""
    rng = np.random.default_rng(seed)
    u, v = rng.standard_normal(m), rng.standard_normal(n)
    u, v = u / np.linalg.norm(u), v / np.linalg.norm(v)
    A = np.zeros((m, n))
    A[np.arange(sg.size), np.arange(sg.size)] = sg
    A -= 2.0 * np.outer(u, u @ A)
    return A - 2.0 * np.outer(A @ v, v)


@pytest.mark.parametrize("k", [1040, 1500, 2300, 3100, 4100])
def test_eigenvalues_of_wide_full_matrices(k):
    """The matrix on the chip from all its sides on, and above 4096 the Sturm counts in pieces, on full matrices (the chain of launches with
    its deferred updates: test_gpu_tridiag_resident.py).  The bar is the rounding
    of the matrix to fp32 (Weyl: at most its Frobenius norm) and the backward error of the fp64 chain as below."""
    sg = np.sort(np.random.default_rng(k).uniform(0.5, 2.0, k))[::-1]
    A = known_matrix(k, k, sg, k).astype(np.float32)
    out = torch.empty(k, dtype=torch.float64, device=DEV)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(k, k, False))
    ctx.check(aser.aser_singular_values(ctx, torch.from_numpy(A).to(DEV), None, out))
    bar = 2.0 ** -24 * np.linalg.norm(sg) + 16 * k * 2.0 ** -52 * sg[0] ** 2 / (2 * sg[-1])
    assert np.max(np.abs(out.cpu().numpy() - sg)) <= bar


@pytest.mark.parametrize("m,n", [(1300, 1200), (2100, 2300), (1100, 3000)])
def test_dense_solver_keeps_its_reflectors_over_deferred_updates(m, n):
    """A rank above the subspace iteration's, S = I (the reflectors of the launches: test_gpu_tridiag_resident.py): T is a known matrix with a gap behind the r-th singular value, so the product of
    the factors is its truncation.  The bars of the other reconstruction tests (error 1e-4, product 1e-3)."""
    r = 130
    rng = np.random.default_rng([m, n])
    sg = np.concatenate([np.sort(rng.uniform(2.0, 3.0, r))[::-1], np.sort(rng.uniform(0.1, 1.0, min(m, n) - r))[::-1]])
    T = known_matrix(m, n, sg, [m, n]).astype(np.float32)
    top = sg.copy()
    top[r:] = 0.0
    want, tail = known_matrix(m, n, top, [m, n]), np.linalg.norm(sg[r:])
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    L_A = torch.empty((m, r), dtype=torch.float32, device=DEV)
    L_B = torch.empty((r, n), dtype=torch.float32, device=DEV)
    sigma = torch.empty(r, dtype=torch.float32, device=DEV)
    st, err, _ = aser.aser_error_reconstruct(ctx, torch.from_numpy(T).to(DEV), torch.eye(n, device=DEV), r, L_A, L_B, sigma)
    ctx.check(st)
    assert abs(err - tail) <= 1e-4 * tail
    assert np.max(np.abs(sigma.cpu().numpy() - sg[:r])) <= 1e-4
    got = L_A.double().cpu().numpy() @ L_B.double().cpu().numpy()
    assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)


@pytest.mark.parametrize("rows,n,m,r,bits,x_dtype,act_bits,pad", [
    (1, 32, 1, 1, 4, "bf16", 8, 0), (65, 100, 70, 9, 4, "bf16", 8, 0), (130, 96, 260, 0, 8, "bf16", 0, 8), (300, 1000, 65, 64, 8, "f32", 6, 0),
    (64, 1026, 200, 33, 4, "f32", 0, 2), (257, 320, 129, 16, 8, "bf16", 8, 1), (1700, 224, 1800, 8, 4, "bf16", 8, 0),
    (2049, 232, 4100, 16, 8, "bf16", 8, 0), (1990, 96, 4096, 0, 4, "f32", 8, 0)])
def test_output_error_at_the_edges_of_its_tiles(rows, n, m, r, bits, x_dtype, act_bits, pad):
    """The bar of the suite's other output-error tests: 2e-4 of the error plus 1e-5 of the output's norm."""
    rng = np.random.default_rng([5, rows, n, m, r])
    W = rng.standard_normal((m, n)).astype(np.float32) * 0.05
    X = rng.standard_normal((rows, n)).astype(np.float32)
    X[:, rng.integers(0, n, 2)] *= 20.0
    if x_dtype == "bf16":
        X = synth.bf16_to_f32(synth.f32_to_bf16_bits(X))
    md = np.ones(n, np.float32)
    md[rng.integers(0, n, 3)] = rng.uniform(1.0, 3.0, 3).astype(np.float32)
    q = orc.quantize_rtn(W * md[None, :], np.zeros(0, np.int32), np.ones(n, np.float32), bits)
    L_A = rng.standard_normal((m, max(r, 1))).astype(np.float32) * 0.01
    L_B = rng.standard_normal((max(r, 1), n)).astype(np.float32) * 0.05
    comp = r > 0
    want, ynorm = orc.layer_output_error(W, X, md, q.codes, q.scales, L_A if comp else None, L_B if comp else None, act_bits or None)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_output_error_workspace_bytes(m, n, rows, r))
    Xd = torch.zeros((rows, n + pad), dtype=torch.bfloat16 if x_dtype == "bf16" else torch.float32, device=DEV)
    Xd[:, :n] = torch.from_numpy(X).to(DEV)
    packed = bits == 4 and n % 2 == 0
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    st, err, ref = aser.aser_layer_output_error(ctx, dev(W), Xd[:, :n], dev(md), dev(orc.pack_int4(q.codes) if packed else q.codes),
                                                aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8, dev(q.scales),
                                                dev(L_A) if comp else None, dev(L_B) if comp else None, r, act_bits)
    ctx.check(st)
    assert abs(ref - ynorm) <= 1e-5 * ynorm
    assert abs(err - want) <= 2e-4 * want + 1e-5 * ynorm


@pytest.mark.parametrize("rows,n,m,r,bits,x_dtype,act_bits,pad", [
    (3, 33, 700, 0, 8, "bf16", 8, 0), (3, 33, 701, 0, 8, "f32", 0, 0), (1000, 1, 1, 0, 8, "f32", 8, 0), (1000, 3, 2, 1, 8, "bf16", 0, 5),
    (16, 1025, 4099, 4, 8, "bf16", 8, 0), (1, 65, 1, 0, 4, "f32", 8, 0), (300, 34, 9, 3, 4, "bf16", 6, 0), (2, 1, 300, 1, 8, "bf16", 8, 0)])
def test_output_error_in_blocks(rows, n, m, r, bits, x_dtype, act_bits, pad):
    """Sizes whose padded planes do not fit the workspace at once (n short of a multiple of 32, few tokens or few channels)."""
    test_output_error_at_the_edges_of_its_tiles(rows, n, m, r, bits, x_dtype, act_bits, pad)


@pytest.mark.parametrize("n,f", [(1, 1), (255, 255), (513, 40), (1024, 1), (1537, 300), (32768, 64)])
def test_outlier_selection_with_many_ties(n, f):
    """Scores of few distinct values, exactly equal on both sides (powers of two): the order is that of the channel index, bit for bit."""
    rng = np.random.default_rng(n)
    W = np.full((4, n), 0.5, np.float32)
    abs_sum = (2.0 ** rng.integers(0, 4, n)).astype(np.float64)
    ref = orc.smooth_outliers(W, abs_sum, 8, f)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(4, n, 0))
    idx = torch.full((f,), 7, dtype=torch.int32, device=DEV)
    mdiag = torch.empty(n, dtype=torch.float32, device=DEV)
    for call in (aser.aser_smooth_outliers, aser.aser_smooth_outliers_noalloc):
        idx.fill_(7)
        ctx.check(call(ctx, torch.from_numpy(W).to(DEV), torch.from_numpy(abs_sum).to(DEV), torch.tensor([8], dtype=torch.int64, device=DEV), f, idx, mdiag))
        assert np.array_equal(idx.cpu().numpy(), ref.idx)
        assert np.array_equal(mdiag.cpu().numpy(), ref.mdiag)


@pytest.mark.parametrize("n,f", [(300, 4), (4096, 4), (4096, 5), (4097, 4), (16384, 19), (16384, 20), (16385, 6), (32768, 57), (32768, 58)])
def test_outlier_selection_on_both_sides_of_its_rule(n, f):
    """The last f that is selected by rounds of an arg-max and the first by the comparison of all pairs, at the widths where the
    former changes its workgroup."""
    test_outlier_selection_with_many_ties(n, f)


@pytest.mark.parametrize("m,n", [(8200, 1100), (8193, 1027), (1025, 8201), (1100, 1028)])
def test_reconstruction_at_the_borders_of_its_tiles(m, n):
    """Sizes around the rules that pick the 256-row tiles (1024 and 8192 rows), with and without 16-byte rows: the bars of the
    other reconstruction tests (error 1e-4, product 1e-3; the gap behind the planted directions is far above 1.05)."""
    rng = np.random.default_rng([m, n])
    r = f = 8
    idx = np.sort(rng.choice(n, f, replace=False)).astype(np.int32)
    T = (rng.random((m, n), dtype=np.float32) - 0.5) * 0.02
    T[:, idx] = rng.standard_normal((m, f)).astype(np.float32) * 0.05
    S = np.tril(rng.standard_normal((n, n)).astype(np.float32), -1) * 0.3
    np.fill_diagonal(S, 20.0 + rng.random(n, dtype=np.float32))
    ref = orc.error_reconstruct(T.astype(np.float64), S.astype(np.float64), r)
    assert ref.gap > 1.05
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    L_A = torch.empty((m, r), dtype=torch.float32, device=DEV)
    L_B = torch.empty((r, n), dtype=torch.float32, device=DEV)
    sigma = torch.empty(r, dtype=torch.float32, device=DEV)
    st, err, _ = aser.aser_error_reconstruct(ctx, torch.from_numpy(T).to(DEV), torch.from_numpy(S).to(DEV), r, L_A, L_B, sigma,
                                             idx=torch.from_numpy(idx).to(DEV), f=f)
    ctx.check(st)
    assert abs(err - ref.err) <= 1e-4 * ref.err
    want = ref.L_A @ ref.L_B
    got = L_A.double().cpu().numpy() @ L_B.double().cpu().numpy()
    assert np.linalg.norm(got - want) <= 1e-3 * np.linalg.norm(want)


@pytest.mark.parametrize("n,pad", [(1, 0), (4, 0), (17, 0), (31, 1), (32, 0), (33, 0), (64, 4), (95, 1), (96, 0), (100, 0), (127, 0), (128, 0),
                                   (129, 3), (164, 0), (256, 8), (300, 0), (388, 0), (1024, 4), (1100, 4), (1283, 0)])
def test_whitening_factor_at_the_edges_of_the_blocks(n, pad):
    """S S^T = G and the triangle against fp64.  Up to 1024 channels every product carries 2^-24 and fp32 sums remain (20 and 8 units of 2^-24; three
    products of two terms instead of six would leave 1.4e-6 to 2.1e-6 and, from 164 channels on, 1.7e-6 to 3.1e-6), behind that 2^-16 per product.
    A block that is not positive definite is reported at its first failing column, wherever that lies in the block."""
    rng = np.random.default_rng([91, n])
    A = rng.standard_normal((2 * n + 8, n)) * rng.uniform(0.5, 4.0, n)
    G = (A.T @ A).astype(np.float32)
    ref = np.linalg.cholesky(G.astype(np.float64))
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(n, n, 0))
    gd = torch.from_numpy(G).to(DEV)
    S = torch.full((n, n + pad), 7.0, dtype=torch.float32, device=DEV)
    st, info = aser.aser_whiten(ctx, gd, None, 0.0, S[:, :n])
    ctx.check(st)
    assert info == 0
    got = S.cpu().numpy().astype(np.float64)
    assert np.all(got[:, n:] == 7.0) and np.all(np.triu(got[:, :n], 1) == 0.0)
    d = np.sqrt(np.diag(G.astype(np.float64)))
    assert np.max(np.abs(got[:, :n] @ got[:, :n].T - G) / np.outer(d, d)) <= (20 * 2.0 ** -24 if n <= 1024 else 1e-5)
    assert np.linalg.norm(got[:, :n] - ref) / np.linalg.norm(ref) <= (8 * 2.0 ** -24 if n <= 1024 else 2e-5)
    for bad in sorted({0, n // 3, n // 2, max(0, n - 14), n - 1}):
        broken = G.copy()
        broken[bad, bad] = -1.0
        st, info = aser.aser_whiten(ctx, torch.from_numpy(broken).to(DEV), None, 0.0, S[:, :n])
        assert st == aser.ASER_ERR_NOT_SPD and info == bad + 1


def gram_diagonal(calls, parts, seg):
    """The diagonal of the Gram matrix of the chunks `calls` as the two-level sums form it: every range of steps (32 tokens) in fp32 chains of
    `seg` steps, eight exact products per rounding, whose results are summed in fp32 and added to G once per range."""
    G = np.zeros(calls[0].shape[1], dtype=np.float32)
    for x in calls:
        products = np.add.reduceat(np.square(x.astype(np.float64)), np.arange(0, len(x), 8), axis=0)
        per = -(-(-(-len(x) // 32)) // parts)
        for a in range(0, len(products), 4 * per):
            total = np.zeros_like(G)
            for b in range(a, min(a + 4 * per, len(products)), 4 * seg):
                chain = np.zeros_like(G)
                for p in products[b:min(b + 4 * seg, a + 4 * per)]:
                    chain = (chain + p).astype(np.float32)
                total = total + chain
            G = G + total
    return G


@pytest.mark.parametrize("n,rows", [(1032, 256), (1032, 287), (1160, 3000), (1288, 4097), (1288, 9001), (2688, 6001), (3080, 4300), (4096, 7503), (4104, 2990)])
def test_gram_chunks_with_two_level_sums(n, rows, rule):
    """Last tiles of one to three quarters, the shortest ranges (8 and 9 steps), ragged last steps.  Bound per entry as above; the diagonal's root mean
    square error against that of the same sums rounded on the CPU (the two agree within 6 %), which without the second level are less accurate."""
    spec = synth.mini("gram%d" % n, 64, n, 2 * rows, n_outliers=5, seed_id=1050 + n % 50)
    X = synth.make_activations(spec)
    G, _, count = run_gram(new_ctx(), spec, X, chunks=2)
    X = synth.activations_as_f32(spec, X)
    ref, _, _ = orc.gram(X)
    d = np.sqrt(np.diag(ref))
    assert np.max(np.abs(lower(G.cpu().numpy()) - np.tril(ref)) / np.outer(d, d)) <= 2e-5 and int(count.item()) == 2 * rows
    tiles, steps, parts, k64 = gram_query(n, rows)
    call = ('AserGramSplit s = aser_gram_dma_split(a[0], a[1], a[2], a[3]), q = aser_gram_seg_split(2 * a[0], a[1], a[2]); '
            'printf("%d %d %d", q.cost < 0.97 * s.cost, q.chunks, q.split);')
    [(taken, chunks, split)] = rule("seg", call, [(tiles, steps, parts, k64)])
    assert taken
    ranges = chunks if 2 * tiles >= 256 // chunks else chunks * split             # the longest ones where there are two kinds
    rms = lambda g: np.sqrt(np.mean((g / np.diag(ref) - 1.0) ** 2))
    calls = [X[:rows], X[rows:]]
    two = rms(gram_diagonal(calls, ranges, -(-steps // (2 * parts))))
    one = rms(gram_diagonal(calls, ranges, steps))
    print("diagonal %d x %d: kernel %.2e, two levels %.2e, one chain per range %.2e" % (n, rows, rms(np.diag(G.cpu().numpy())), two, one))
    assert rms(np.diag(G.cpu().numpy())) <= 1.2 * two < one


@pytest.mark.parametrize("rows,n,m,r,packed", [(1, 2048, 8193, 1, True), (1, 4128, 16384, 64, True), (3, 2080, 8200, 40, False), (16, 2048, 8225, 128, True),
                                               (16, 6176, 9000, 24, False), (2, 2016, 8200, 64, True)])
def test_forward_of_a_few_tokens_with_many_outputs(rows, n, m, r, packed):
    """The rank-r branch beside the codes and on top of them in a second launch; bars as in test_forward_of_a_few_tokens."""
    rng = np.random.default_rng([78, rows, n, m, r])
    xq = rng.integers(-127, 128, (rows, n)).astype(np.int8)
    xs = rng.uniform(0.01, 0.05, rows).astype(np.float32)
    q = rng.integers(-7, 8, (m, n)).astype(np.int8) if packed else rng.integers(-127, 128, (m, n)).astype(np.int8)
    ws = rng.uniform(0.001, 0.003, m).astype(np.float32)
    L_A = rng.standard_normal((m, r)).astype(np.float32)
    L_B = (rng.standard_normal((r, n)) * 0.01).astype(np.float32)
    X = xq.astype(np.float64) * xs.astype(np.float64)[:, None]
    want = X @ (q.astype(np.float64) * ws.astype(np.float64)[:, None]).T + (X @ L_B.astype(np.float64).T) @ L_A.astype(np.float64).T
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    wq = torch.from_numpy(orc.pack_int4(q) if packed else q).to(DEV)
    lb = torch.zeros(L_B.size + 1, dtype=torch.float32, device=DEV)
    lb[1:] = torch.from_numpy(L_B.reshape(-1)).to(DEV)
    for lbd in (lb[1:].view(L_B.shape), torch.from_numpy(L_B).to(DEV)):       # 4-byte aligned, 16-byte aligned
        for split, bar in ((True, 2e-5), (False, 4e-3)):
            Y = torch.full((rows, m + 3), 7.0, dtype=torch.float32, device=DEV)
            ctx.check(aser.aser_compensated_forward(ctx, torch.from_numpy(xq).to(DEV), torch.from_numpy(xs).to(DEV), wq,
                                                    aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8, torch.from_numpy(ws).to(DEV),
                                                    torch.from_numpy(L_A).to(DEV), lbd, r, split, Y[:, :m]))
            got = Y.cpu().numpy()
            assert np.all(got[:, m:] == 7.0)
            assert np.linalg.norm(got[:, :m] - want) / np.linalg.norm(want) <= bar


@pytest.mark.parametrize("rows,n,m,r,packed", [(1, 2048, 8193, 64, True), (16, 4096, 14336, 40, True), (5, 6176, 16384, 16, False), (13, 11008, 8200, 128, False)])
def test_forward_of_a_few_tokens_does_not_depend_on_the_number_of_outputs(rows, n, m, r, packed):
    """The sums behind P and an output are the same, in the same order, whether P is formed in front of the codes or beside them: bit for bit."""
    rng = np.random.default_rng([79, rows, n, m, r])
    xq = torch.from_numpy(rng.integers(-127, 128, (rows, n)).astype(np.int8)).to(DEV)
    xs = torch.from_numpy(rng.uniform(0.01, 0.05, rows).astype(np.float32)).to(DEV)
    q = rng.integers(-7, 8, (m, n)).astype(np.int8) if packed else rng.integers(-127, 128, (m, n)).astype(np.int8)
    wq = torch.from_numpy(orc.pack_int4(q) if packed else q).to(DEV)
    ws = torch.from_numpy(rng.uniform(0.001, 0.003, m).astype(np.float32)).to(DEV)
    L_A = torch.from_numpy(rng.standard_normal((m, r)).astype(np.float32)).to(DEV)
    L_B = torch.from_numpy((rng.standard_normal((r, n)) * 0.01).astype(np.float32)).to(DEV)
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_forward_workspace_bytes(rows, n, m, r))
    layout = aser.ASER_CODES_INT4_PACKED if packed else aser.ASER_CODES_INT8
    for split in (True, False):
        Y, part = (torch.empty((rows, k), dtype=torch.float32, device=DEV) for k in (m, 4096))
        ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq, layout, ws, L_A, L_B, r, split, Y))
        ctx.check(aser.aser_compensated_forward(ctx, xq, xs, wq[:4096], layout, ws[:4096], L_A[:4096], L_B, r, split, part))
        assert np.array_equal(Y[:, :4096].cpu().numpy(), part.cpu().numpy())


@pytest.mark.parametrize("m,n,r", [(3, 5, 1), (16, 33, 3), (64, 64, 7), (65, 130, 9), (256, 256, 17), (256, 300, 18), (257, 200, 40), (300, 257, 3), (700, 513, 20),
                                   (1000, 1040, 5), (40, 2000, 12)])
def test_dense_solver_at_the_edges_of_its_kernels(m, n, r):
    """Factors of small layers against the SVD in fp64: inputs in fp32, everything behind them in fp64, results in fp32 (2^-24 relative, bar 1e-6);
    the residual as a norm of fp64 differences of fp32 factors (bar 1e-5)."""
    rng = np.random.default_rng([93, m, n, r])
    k = min(m, n)
    U, V = np.linalg.qr(rng.standard_normal((m, k)))[0], np.linalg.qr(rng.standard_normal((n, k)))[0]
    S = (np.tril(rng.standard_normal((n, n))) * 0.05 + np.diag(rng.uniform(1.0, 3.0, n))).astype(np.float32)
    A = (U * np.where(np.arange(k) < r, 8.0 + np.arange(k)[::-1] / k, 0.5)) @ V.T          # a gap behind the r-th singular value
    T = np.ascontiguousarray(np.linalg.solve(S.astype(np.float64).T, A.T).T).astype(np.float32)
    A = T.astype(np.float64) @ S.astype(np.float64)
    u, sg, _ = np.linalg.svd(A, full_matrices=False)
    want = u[:, :r] @ (u[:, :r].T @ T.astype(np.float64))
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    L_A, L_B, sigma = (torch.empty(shape, dtype=torch.float32, device=DEV) for shape in ((m, r), (r, n), (r,)))
    st, err, iters = aser.aser_error_reconstruct(ctx, torch.from_numpy(T).to(DEV), torch.from_numpy(S).to(DEV), r, L_A, L_B, sigma)
    ctx.check(st)
    got = L_A.cpu().numpy().astype(np.float64) @ L_B.cpu().numpy().astype(np.float64)
    assert iters == 0 and np.max(np.abs(sigma.cpu().numpy() / sg[:r] - 1.0)) <= 1e-6
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 1e-5
    assert abs(err - np.sqrt(np.sum(sg[r:] ** 2))) <= 1e-5 * np.linalg.norm(sg)


@pytest.mark.parametrize("m,n,r,wanted", [(1100, 1028, 8, "apart"), (1100, 1028, 8, "equal"), (1030, 1200, 1, "apart"), (1029, 1100, 32, "apart"), (1100, 1028, 64, "equal")])
def test_reconstruction_with_equal_singular_values(m, n, r, wanted):
    """A bulk of equal singular values behind the wanted ones, whose pairs nobody asks for, and equal ones among these.  Bars: the product 1e-3 as
    elsewhere; squared singular values 128 * 2^-24 of the largest (fp32 reflectors of a block of 128); columns of L_A orthogonal to twice that,
    measured in their norms, with 2^-17 for the products that form the basis."""
    rng = np.random.default_rng([94, m, n, r])
    k = min(m, n)
    sg = np.full(k, 0.5)
    sg[:r] = np.linspace(3.0, 2.0, r) if wanted == "apart" else 2.0
    sg[0] = 40.0
    U, V = np.linalg.qr(rng.standard_normal((m, k)))[0], np.linalg.qr(rng.standard_normal((n, k)))[0]
    S = (np.tril(rng.standard_normal((n, n)), -1) * 0.01 + np.diag(rng.uniform(1.0, 3.0, n))).astype(np.float32)
    A = (U * sg) @ V.T
    T = np.ascontiguousarray(np.linalg.solve(S.astype(np.float64).T, A.T).T).astype(np.float32)
    want = U[:, :r] @ (U[:, :r].T @ T.astype(np.float64))
    ctx = new_ctx()
    ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    L_A, L_B, sigma = (torch.empty(shape, dtype=torch.float32, device=DEV) for shape in ((m, r), (r, n), (r,)))
    st, err, iters = aser.aser_error_reconstruct(ctx, torch.from_numpy(T).to(DEV), torch.from_numpy(S).to(DEV), r, L_A, L_B, sigma)
    ctx.check(st)
    la, s = L_A.double().cpu().numpy(), sigma.double().cpu().numpy()
    assert iters > 0 and abs(err - 0.5 * np.sqrt(k - r)) <= 1e-4 * err
    assert np.linalg.norm(la @ L_B.double().cpu().numpy() - want) <= 1e-3 * np.linalg.norm(want)
    assert np.max(np.abs(s ** 2 - sg[:r] ** 2)) <= 128 * 2.0 ** -24 * sg[0] ** 2
    u = la / np.linalg.norm(la, axis=0)
    assert np.max(np.abs(u.T @ u - np.eye(r))) <= 256 * 2.0 ** -24 + 2.0 ** -17


def double_well(b, distance, rng):
    """A symmetric tridiagonal matrix of few-bit entries whose two largest eigenvalues (all it has come in pairs) lie `distance`, within a tenth,
    of its radius apart: two mirrored halves that a small entry couples.  Tridiagonal already and exact in fp32, so the solver sees it unrounded."""
    h = b // 2
    for _ in range(100000):
        d, e, c = rng.integers(64, 192, h) / 64.0, rng.integers(8, 64, h - 1) / 64.0, 2.0 ** -float(rng.integers(4, 28))
        half = np.diag(d) + np.diag(e, 1) + np.diag(e, -1)
        w, v = np.linalg.eigh(half)
        rows = d + np.concatenate([[0.0], e]) + np.concatenate([e, [c]])
        guess = 2.0 * c * v[-1, -1] ** 2 / rows.max()
        if not 0.5 * distance < guess < 2.0 * distance:
            continue
        half[-1, -1] += c
        up = np.linalg.eigvalsh(half)[-1]
        half[-1, -1] -= 2.0 * c
        down = np.linalg.eigvalsh(half)[-1]
        if abs((up - down) / rows.max() / distance - 1.0) < 0.1:
            full = np.diag(np.concatenate([d, d[::-1]])).astype(np.float32)
            off = np.concatenate([e, [c], e[::-1]])
            return full + np.diag(off, 1).astype(np.float32) + np.diag(off, -1).astype(np.float32), np.array([up, down])
    raise AssertionError("none found")


@pytest.mark.parametrize("b,need", [(128, 2), (128, 1), (96, 2), (40, 2)])
@pytest.mark.parametrize("distance,apart", [(2e-10, False), (7e-10, False), (1.3e-9, True), (3e-9, True), (8e-9, True), (1e-7, True)])
def test_ritz_pairs_at_the_distance_where_the_fallback_takes_over(b, need, distance, apart):
    """The eigen-solvers of the Ritz problem, called as the reconstruction calls them: from 1e-9 of the radius on the vectors are those of the
    twisted factorisation, below they are the Jacobi solver's, also where only one of the pair is wanted.  Orthogonality: 2^-23 for fp32
    entries, and an error of 2^-52 of the radius in each eigenvalue over their distance (an interval of 3e-15, as after eight rounds of
    the multisection, would leave up to 2.5e-6 at the smallest distance); after about ten sweeps of 127 fp32 rotations 1e-4."""
    M, pair = double_well(b, distance, np.random.default_rng([95, b, need, int(distance * 1e11)]))
    lib, ctx = aser.load_library(), new_ctx()
    Md = torch.from_numpy(M).to(DEV)
    lam, V, refl, tri = (torch.full(shape, 7.0, dtype=torch.float32, device=DEV) for shape in ((b,), (b, b), (b, 128), (384,)))
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    ctx.check(lib["_Z16aser_tridiag_eigP8aser_ctxPKfiPfS3_S3_S3_Pii"](ctx.handle, p(Md), b, p(lam), p(V), p(refl), p(tri), p(flag), need))
    torch.cuda.synchronize()
    before = V.cpu().numpy()
    assert int(flag.item()) == (0 if apart else 1) and np.all(before[:, need:] == 7.0)
    ctx.check(lib["_Z15aser_jacobi_eigP8aser_ctxPKfiPfS3_PKi"](ctx.handle, p(Md), b, p(lam), p(V), p(flag)))
    torch.cuda.synchronize()
    got, pair = V.double().cpu().numpy()[:, :need], pair[:need]
    assert not apart or np.array_equal(V.cpu().numpy(), before)
    off = np.max(np.abs(got.T @ got - np.eye(need)))
    print("distance %.1e: vectors orthogonal to %.1e" % (distance, off))
    assert off <= (2.0 ** -23 + 2.0 * 2.0 ** -52 / distance if apart else 1e-4)
    assert np.max(np.abs(lam.cpu().numpy()[:need] / pair - 1.0)) <= (2.0 ** -23 if apart else 1e-4)
    assert np.max(np.abs(M.astype(np.float64) @ got - got * pair)) <= (2.0 ** -22 if apart else 1e-4) * pair[0]


@pytest.mark.parametrize("b", [2, 3, 16, 17, 18, 49, 97, 127, 128])
@pytest.mark.parametrize("scale", [1e-7, 1.0, 1e9])
def test_ritz_pairs_of_dense_matrices(b, scale):
    """All eigenpairs at the sides around the slots of 16 rows that the tridiagonalisation drops one after the other.  Every one of b - 2 reflections
    moves the matrix by a small multiple of 2^-24 of its norm, in directions of its own: 4 sqrt(b) 2^-24 of the largest eigenvalue
    for the eigenvalues and the residuals, 8 sqrt(b) 2^-24 for the products of vectors that went through b - 2 reflectors."""
    rng = np.random.default_rng([96, b])
    A = rng.standard_normal((b, 2 * b + 3))
    M = (A @ A.T * scale).astype(np.float32)
    sym = 0.5 * (M.astype(np.float64) + M.T)
    want = np.linalg.eigvalsh(sym)[::-1]
    lib, ctx = aser.load_library(), new_ctx()
    Md = torch.from_numpy(M).to(DEV)
    lam, V, refl, tri = (torch.full(shape, 7.0, dtype=torch.float32, device=DEV) for shape in ((b,), (b, b), (b, 128), (384,)))
    flag = torch.ones(1, dtype=torch.int32, device=DEV)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    ctx.check(lib["_Z16aser_tridiag_eigP8aser_ctxPKfiPfS3_S3_S3_Pii"](ctx.handle, p(Md), b, p(lam), p(V), p(refl), p(tri), p(flag), b))
    torch.cuda.synchronize()
    got, v = lam.double().cpu().numpy(), V.double().cpu().numpy()
    eps = 2.0 ** -24 * np.sqrt(b)
    assert int(flag.item()) == 0
    assert np.max(np.abs(got - want)) <= 4 * eps * want[0]
    assert np.max(np.abs(sym @ v - v * want)) <= 4 * eps * want[0]
    assert np.max(np.abs(v.T @ v - np.eye(b))) <= 8 * eps


@pytest.mark.parametrize("diagonal,coupling", [(3e21, 3e17), (1e30, 1e26), (1.0, 1e-4), (1e-22, 1e-26), (1e-30, 1e-34)])
def test_ritz_pairs_of_nearly_diagonal_matrices_at_any_scale(diagonal, coupling):
    """Entries whose products with a column do not fit fp32, or vanish in it, although entries and eigenvalues do.  Tolerances as above."""
    b = 96
    rng = np.random.default_rng(96)
    A = rng.standard_normal((b, b))
    M = (diagonal * np.eye(b) + coupling * (A + A.T)).astype(np.float32)
    sym = 0.5 * (M.astype(np.float64) + M.T)
    want = np.linalg.eigvalsh(sym)[::-1]
    lib, ctx = aser.load_library(), new_ctx()
    Md = torch.from_numpy(M).to(DEV)
    lam, V, refl, tri = (torch.full(shape, 7.0, dtype=torch.float32, device=DEV) for shape in ((b,), (b, b), (b, 128), (384,)))
    flag = torch.ones(1, dtype=torch.int32, device=DEV)
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    ctx.check(lib["_Z16aser_tridiag_eigP8aser_ctxPKfiPfS3_S3_S3_Pii"](ctx.handle, p(Md), b, p(lam), p(V), p(refl), p(tri), p(flag), b))
    torch.cuda.synchronize()
    got, v = lam.double().cpu().numpy(), V.double().cpu().numpy()
    eps = 2.0 ** -24 * np.sqrt(b)
    assert int(flag.item()) == 0
    assert np.max(np.abs(got - want)) <= 4 * eps * want[0]
    assert np.max(np.abs(sym @ v - v * want)) <= 4 * eps * want[0]
    assert np.max(np.abs(v.T @ v - np.eye(b))) <= 8 * eps
