"""GPU parity of the multi-block selection (over 32,768 rows a bucket) where its
lowest histogram bin decides: more rows kept than have a nonzero importance, all
importances zero, and zeros among denormal and normal importances with the
threshold on a normal, on a denormal and on zero; one block, several blocks and
several tiles a block."""
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


# r = 1, V = 1 in a row's first column and 0 elsewhere: Sigma_p is the square of
# the first value of row p.  2^-70 squared is denormal (2^-140), as are its
# multiples up to 2^7; 2^-75 squared is zero.
def _case(rows, n, n_normal, n_denormal, K, label):
    rng = np.random.default_rng(rows + n_normal + n_denormal)
    first = np.zeros(rows, F32)
    where = rng.permutation(rows)
    normal, denormal = where[:n_normal], where[n_normal:n_normal + n_denormal]
    first[normal] = rng.integers(1, 60, size=n_normal).astype(F32)
    first[denormal] = rng.integers(1, 40, size=n_denormal).astype(F32) * F32(2.0 ** -70)
    some = where[n_normal + n_denormal:][: rows // 10]
    first[some] = F32(2.0 ** -75)
    V = np.zeros((n, 1), F32)
    V[0, 0] = 1.0

    def grad(t):
        g = np.zeros((1, rows * n), F32)
        g[0, ::n] = first
        return g

    log(f"[zeros] {label} rows={rows} normal={n_normal} denormal={n_denormal} K={K}")
    run_case(label=label, d=rows * n, N=1, n=n, r=1, K=K, eta=1.0, steps=1, grad_fn=grad, V=V)


@pytest.mark.parametrize("rows", [32_769, 70_000, 262_145])
def test_lowest_bin_decides(rows):
    some, few = rows // 3, rows // 50
    for K in (1, rows // 2, rows - 1):
        _case(rows, 4, 0, 0, K, "all zero")
    # threshold on zero: ties among zero rows, the nonzero ones all kept
    _case(rows, 4, few, 0, some, "zeros tie")
    _case(rows, 4, few, few, some, "zeros tie below denormals")
    _case(rows, 4, rows, 0, some, "no zeros")
    # threshold on a denormal, and on the first row past them
    _case(rows, 4, few, some, few + some // 2, "denormal threshold")
    _case(rows, 4, 0, some, some, "all denormals kept")
    _case(rows, 4, 0, some, some + 1, "one zero kept")
    _case(rows, 4, few, some, few, "normals only")


# Blocks of more than 8192 rows take several tiles.
def test_lowest_bin_over_several_tiles():
    rows = 2_200_000
    _case(rows, 4, 1000, 0, 700_001, "tiles, zeros tie")
    _case(rows, 4, 1000, 300_000, 200_001, "tiles, denormal threshold")


def test_lowest_bin_in_buckets():
    # A bucket of zeros beside one with few nonzero rows and one without zeros.
    begin, ks = [0, 40_000, 80_000, 120_000], [7, 2_000, 39_999]
    n, rows = 4, 120_000
    first = np.zeros(rows, F32)
    first[40_000:41_500] = np.arange(1, 1_501, dtype=F32)
    first[80_000:] = F32(2.0 ** -70) * np.arange(1, 40_001, dtype=F32)
    V = np.zeros((n, 1), F32)
    V[0, 0] = 1.0

    def grad(t):
        g = np.zeros((1, rows * n), F32)
        g[0, ::n] = first
        return g

    log("[zeros] buckets")
    run_case(label="zeros_buckets", d=rows * n, N=1, n=n, r=1, buckets=(begin, ks), eta=1.0,
             steps=1, grad_fn=grad, V=V)
