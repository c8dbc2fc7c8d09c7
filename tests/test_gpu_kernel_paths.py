"""The dispatch borders of single kernels: sizes at the edges of tiles and of the rules that pick a kernel, against
NumPy or the oracle."""
import numpy as np
import pytest
import torch

import aser_synth as synth
import paper_2411_07762_amd as aser
from gpu_util import DEV, lower, new_ctx, run_gram
from oracle import aser_oracle as orc

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
