"""GPU parity of the payload gather at the edges of its item split: rows of
every remainder modulo four columns, worker counts around the batch of four
that is read together, tensor counts on both sides of the LDS search table,
and payload slots off 16 bytes, with and without the tracker G."""
import pytest
import torch

from parity_util import log, run_case
from test_gpu_model import run_model_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# Four workers at a time up to 8, then eight; rows as single columns and, from
# 12 (one worker) or 128 values on, as quads and single columns.
@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9, 16, 17])
def test_gather_worker_batches_and_remainders(N):
    for n in (1, 3, 4, 5, 6, 7, 8, 11, 13, 31, 127, 129, 130, 131):
        log(f"[gather] N={N} n={n}")
        run_case(label=f"gather_{N}_{n}", d=n * 90 + n // 2, N=N, n=n, K=31, steps=2)
    tensors = [(20, 5, 3), (9, 6, 9), (31, 7, 8), (12, 8, 5), (1, 3, 1), (40, 65, 11)]
    run_model_case(label=f"gather_model_{N}", d=sum(a * b for a, b, _ in tensors), N=N,
                   tensors=tensors, optimizer="msgd", steps=2)


@pytest.mark.parametrize("count", [1023, 1024, 1025, 1500])
def test_gather_many_tensors(count):
    tensors = [(1 + i % 3, 3 + i % 9, 1) for i in range(count)]
    log(f"[gather] {count} tensors")
    run_case(label=f"gather_tensors_{count}", d=sum(a * b for a, b, _ in tensors), N=3,
             tensors=tensors, steps=2)
