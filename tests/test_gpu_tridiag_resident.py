"""The tridiagonalisation that keeps the matrix on the chip, through the singular values of T alone (S = NULL: T T^T is then formed in fp64
from fp32 entries): matrix sides around its limits (the last 256 rows, chunks of 512 columns, groups of 1024 rows, 4096 rows), odd
ones, and beyond them, where the chain of launches runs first."""
import numpy as np
import pytest
import torch

import paper_2411_07762_amd as aser

from gpu_util import DEV, new_ctx

pytestmark = pytest.mark.gpu


def spectrum(ctx, T):
    k = min(T.shape)
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(T.shape[0], T.shape[1], False))
    sig = torch.full((k,), -1.0, dtype=torch.float64, device=DEV)
    ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    torch.cuda.synchronize()
    return sig.cpu().numpy()


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


def test_captured_calls_take_the_chain_of_launches():
    k = 600
    T = torch.randn((k, k), device=DEV)
    eager = spectrum(new_ctx(), T)
    stream = torch.cuda.Stream()
    ctx = aser.Context(0, stream.cuda_stream)
    ctx.ensure_workspace(aser.aser_spectrum_workspace_bytes(k, k, False))
    sig = torch.zeros(k, dtype=torch.float64, device=DEV)
    ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        ctx.check(aser.aser_singular_values(ctx, T, None, sig))
    for _ in range(3):
        sig.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.abs(sig.cpu().numpy() - eager).max() <= 1e-11 * eager[0]
