"""GPU parity of the one-workgroup selection at the edges of its shape: rows
around the workgroup's 1024 threads, its 8 and 32 keys a thread and its waves,
with heavy ties, all-equal importances, K of one and of all but one row, and
buckets of very different sizes in one launch."""
import numpy as np
import pytest
import torch

from parity_util import log, run_case

pytestmark = pytest.mark.gpu
F32 = np.float32


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# V = ones (r = 1) and small whole numbers: Sigma_p = (worker sum)^2 exactly,
# so every level holds many ties.
def _levels(rows, levels, n):
    vals = np.random.default_rng(rows + levels).integers(0, levels, size=rows).astype(F32)

    def grad(t):
        g = np.zeros((1, rows * n), F32)
        g[0, ::n] = vals
        return g
    return grad


@pytest.mark.parametrize("rows", [2, 63, 65, 1023, 1024, 1025, 8191, 8192, 8193, 31_745, 32_767,
                                  32_768])
@pytest.mark.parametrize("levels", [1, 3, 700])
def test_one_workgroup_selection_ties(rows, levels):
    for K in sorted({1, rows // 3 + 1, rows - 1}):
        log(f"[select] rows={rows} levels={levels} K={K}")
        run_case(label=f"sel_{rows}_{levels}_{K}", d=4 * rows, N=1, n=4, r=1, K=K, eta=1.0,
                 steps=1, grad_fn=_levels(rows, levels, 4), V=np.ones((4, 1), F32))


def test_one_workgroup_selection_uneven_buckets():
    begin = [0, 1, 65, 9_000, 9_002, 41_770, 41_771 + 1024]
    ks = [1, 64, 17, 1, 12_345, 1024]
    log("[select] uneven buckets")
    run_case(label="sel_buckets", d=8 * begin[-1], N=2, n=8, r=4, buckets=(begin, ks), steps=2)
