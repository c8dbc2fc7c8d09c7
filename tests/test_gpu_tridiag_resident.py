"""The tridiagonalisation that keeps the matrix on the chip, through the singular values of T alone (S = NULL: T T^T is then formed in fp64
from fp32 entries): matrix sides around its limits (the last 256 rows, chunks of 512 columns, groups of 1024 rows, 4096 rows), odd
ones, and beyond them, where the chain of launches runs first; and that chain alone, which captured calls and layers in flight still take."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2411_07762_amd as aser

from gpu_util import DEV, new_ctx
from test_gpu_kernel_paths import known_matrix

pytestmark = pytest.mark.gpu


def spectrum(ctx, T):
    k = min(T.shape)
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(T.shape[0], T.shape[1], False))
    sig = torch.full((k,), -1.0, dtype=torch.float64, device=DEV)
    ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    torch.cuda.synchronize()
    return sig.cpu().numpy()


def same(got, ref):
    """Two computations of one spectrum: the atomics of the Gram matrix add up in any order and the chain differs, both within the bound below, for
    the eigenvalues, of which a small singular value is the root."""
    return np.abs(got ** 2 - ref ** 2).max() <= 8 * len(ref) * 2.2e-16 * ref[0] ** 2


@pytest.mark.parametrize("k", [326, 517, 519, 1030, 1031, 2054, 3079, 4102])
def test_singular_values_against_lapack(k):
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    T = torch.randn((k, k + 9), generator=g, device=DEV) * torch.logspace(0, -2, k + 9, device=DEV)
    got = spectrum(new_ctx(), T) ** 2
    Td = T.double().cpu()
    ref = torch.linalg.eigvalsh(Td @ Td.T).flip(0).numpy()
    # Householder reduction and bisection are backward stable: every eigenvalue moves by at most a small multiple of k eps |B|
    assert np.abs(got - ref).max() <= 4 * k * 2.2e-16 * ref[0]


@pytest.mark.parametrize("k", [5, 100, 400, 1500])
def test_degenerate_matrices(k):
    ctx = new_ctx()
    T = torch.zeros((k, k), device=DEV)
    assert np.all(spectrum(ctx, T) == 0.0)
    T.diagonal().copy_(torch.arange(k, 0, -1, device=DEV, dtype=torch.float32))      # nothing to reflect: every sub-column is zero
    assert np.allclose(spectrum(ctx, T), np.arange(k, 0, -1.0), rtol=1e-12, atol=0)
    # blocks that do not touch each other, every value many times over, and half of them zero
    T.zero_()
    T.diagonal()[::2] = 3.0
    n3 = (k + 1) // 2
    got = spectrum(ctx, T)
    assert np.allclose(got[:n3], 3.0, rtol=1e-12, atol=0) and np.all(got[n3:] <= 3e-8)     # a square of zero to 1e-16 of 9
    T *= 1e-18                                                                              # squares of 9e-36
    assert np.allclose(spectrum(ctx, T)[:n3], 3e-18, rtol=1e-6, atol=0)
    T[k // 2, k // 3] = float("nan")
    assert np.all(spectrum(ctx, T) == 0.0)               # refused by the rank rule


def graph_nodes(graph):
    count = ctypes.c_size_t(0)
    assert ctypes.CDLL("libamdhip64.so").hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


@pytest.mark.parametrize("k", [600, 1500])
def test_captured_calls_take_the_chain_of_launches(k):
    """A launch per column down to the last 256, and up to two pairs of vectors pending at 1500."""
    T = torch.randn((k, k), device=DEV)
    eager = spectrum(new_ctx(), T)
    stream = torch.cuda.Stream()
    ctx = aser.Context(0, stream.cuda_stream)
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(k, k, False))
    sig = torch.zeros(k, dtype=torch.float64, device=DEV)
    ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph, stream=stream):
        ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    assert graph_nodes(graph) >= k - 256
    for _ in range(3):
        sig.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert same(sig.cpu().numpy(), eager)


def exchange(ctx, gate_attempts, broken=False):
    """The waits of the resident kernel as after `gate_attempts` attempts at its gate, or with an entry that never came."""
    aser.load_library()["_Z17aser_set_exchangeP8aser_ctxib"](ctx.handle, ctypes.c_int(gate_attempts), ctypes.c_bool(broken))
    return ctx


@pytest.mark.parametrize("k", [326, 517, 700, 1031, 2054])
def test_columns_where_the_workgroups_do_not_all_get_in(k):
    """The gate called off by every workgroup: the kernel of one workgroup does the columns instead, to the same bound."""
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    T = torch.randn((k, k + 9), generator=g, device=DEV) * torch.logspace(0, -2, k + 9, device=DEV)
    got = spectrum(exchange(new_ctx(), 0), T) ** 2
    Td = T.double().cpu()
    ref = torch.linalg.eigvalsh(Td @ Td.T).flip(0).numpy()
    assert np.abs(got - ref).max() <= 4 * k * 2.2e-16 * ref[0]


def reconstruct(ctx, T, r):
    m, n = T.shape
    ctx.ensure_workspace(aser.aser_workspace_bytes(m, n, r))
    L_A, L_B, sigma = (torch.empty(shape, device=DEV) for shape in ((m, r), (r, n), (r,)))
    st, err, _ = aser.aser_error_reconstruct(ctx, T, torch.eye(n, device=DEV), r, L_A, L_B, sigma)
    return st, err, L_A.double() @ L_B.double()


@pytest.mark.parametrize("m,n", [(700, 750), (620, 400)])
def test_factors_where_the_workgroups_do_not_all_get_in(m, n):
    """The reflectors that the dense solver carries its vectors back through: the product of the factors is the best approximation whichever
    kernel has made them (neighbouring singular values 1e-3 apart: 2^-24 of the products over that)."""
    rng = np.random.default_rng(m)
    k = min(m, n)
    u, v = np.linalg.qr(rng.standard_normal((m, k)))[0], np.linalg.qr(rng.standard_normal((n, k)))[0]
    s = np.linspace(2.0, 1.0, k)
    T = torch.from_numpy(((u * s) @ v.T).astype(np.float32)).to(DEV)
    uu, sg, vt = np.linalg.svd(T.double().cpu().numpy(), full_matrices=False)
    want = (uu[:, :20] * sg[:20]) @ vt[:20]
    for ctx in (new_ctx(), exchange(new_ctx(), 0)):
        st, err, got = reconstruct(ctx, T, 20)
        ctx.check(st)
        assert abs(err - np.sqrt((sg[20:] ** 2).sum())) <= 1e-6 * err
        assert np.linalg.norm(got.cpu().numpy() - want) <= 2.0 ** -22 * 1e3 * np.linalg.norm(want)


@pytest.mark.parametrize("k", [400, 1500])
def test_a_broken_exchange_is_no_spectrum(k):
    """What the kernels in front have left finite must not come out as one: no singular value, a rank that is refused, factors with an error."""
    T = torch.randn((k, k), device=DEV)
    ctx = exchange(new_ctx(), 1 << 20, broken=True)
    assert np.all(spectrum(ctx, T) == 0.0)
    st, _, _ = aser.aser_select_rank(ctx, torch.zeros(k, dtype=torch.float64, device=DEV), 0.5)
    assert st == aser.ASER_ERR_INVALID_ARG
    if k * k <= 1 << 20:
        st, _, _ = reconstruct(ctx, T, 8)
        assert st == aser.ASER_ERR_NO_CONVERGE
    exchange(ctx, 1 << 20)
    assert spectrum(ctx, T)[0] > 0.0


def test_spectra_beside_work_of_other_streams():
    """Three contexts on streams of their own and products on a fourth: whoever gets in when, the results are those of a call alone."""
    g = torch.Generator(device=DEV)
    g.manual_seed(3)
    Ts = [torch.randn((k, k), generator=g, device=DEV) for k in (700, 900, 1300)]
    alone = [spectrum(new_ctx(), T) for T in Ts]
    streams = [torch.cuda.Stream() for _ in range(4)]
    ctxs = [aser.Context(0, s.cuda_stream) for s in streams[:3]]
    sig = [torch.zeros(T.shape[0], dtype=torch.float64, device=DEV) for T in Ts]
    for c, T in zip(ctxs, Ts):
        c.ensure_workspace(aser.aser_spectrum_workspace_bytes(T.shape[0], T.shape[0], False))
    A = torch.randn((4096, 4096), device=DEV)
    torch.cuda.synchronize()
    for _ in range(2):
        with torch.cuda.stream(streams[3]):
            for _ in range(10):
                B = A @ A
        for c, T, s in zip(ctxs, Ts, sig):
            c.check(aser.aser_singular_values(c, T, None, s))
    torch.cuda.synchronize()
    for s, ref in zip(sig, alone):
        assert same(s.cpu().numpy(), ref)


@pytest.mark.parametrize("k", [40, 300, 700])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_factors_of_a_matrix_that_is_not_finite(k, value):
    T = torch.randn((k, k), device=DEV)
    T[k // 2, k // 3] = value
    st, _, _ = reconstruct(new_ctx(), T, 8)
    assert st == aser.ASER_ERR_NO_CONVERGE


CHAIN_ALONE = -1


@pytest.mark.parametrize("k,gate_attempts", [(1040, CHAIN_ALONE), (1500, CHAIN_ALONE), (2300, CHAIN_ALONE), (3101, CHAIN_ALONE), (4120, CHAIN_ALONE),
                                             (4120, 1 << 20), (4333, 1 << 20)])
def test_eigenvalues_over_deferred_updates(k, gate_attempts):
    """The chain of launches with one, two and four pairs of vectors pending, to its end or, beyond 4096 rows, until the matrix fits the chip.  The bar of the
    wide full matrices: the rounding of the matrix to fp32 and the backward error of the fp64 chain."""
    sg = np.sort(np.random.default_rng(k).uniform(0.5, 2.0, k))[::-1]
    T = torch.from_numpy(known_matrix(k, k, sg, k).astype(np.float32)).to(DEV)
    bar = 2.0 ** -24 * np.linalg.norm(sg) + 16 * k * 2.0 ** -52 * sg[0] ** 2 / (2 * sg[-1])
    assert np.max(np.abs(spectrum(exchange(new_ctx(), gate_attempts), T) - sg)) <= bar


@pytest.mark.parametrize("m,n,gate_attempts", [(1300, 1200, CHAIN_ALONE), (2100, 2300, CHAIN_ALONE), (1100, 3000, CHAIN_ALONE), (4200, 4150, 1 << 20)])
def test_reflectors_over_deferred_updates(m, n, gate_attempts):
    """The dense solver over the same chain: the product of the factors is the truncation behind a gap (error 1e-4, product 1e-3)."""
    r = 130
    rng = np.random.default_rng([m, n])
    sg = np.concatenate([np.sort(rng.uniform(2.0, 3.0, r))[::-1], np.sort(rng.uniform(0.1, 1.0, min(m, n) - r))[::-1]])
    top = sg.copy()
    top[r:] = 0.0
    T = torch.from_numpy(known_matrix(m, n, sg, [m, n]).astype(np.float32)).to(DEV)
    ctx = exchange(new_ctx(), gate_attempts)
    st, err, got = reconstruct(ctx, T, r)
    ctx.check(st)
    tail, want = np.linalg.norm(sg[r:]), known_matrix(m, n, top, [m, n])
    assert abs(err - tail) <= 1e-4 * tail
    assert np.linalg.norm(got.cpu().numpy() - want) <= 1e-3 * np.linalg.norm(want)
