"""GPU parity of the dense iteration with its x update in one pass: worker
counts around the batch of four, every optimiser, both gradient types, the
sizes of a partial last workgroup, and any length and element alignment; of the
x update alone likewise; and of Rand-K's momentum where N * d is not a multiple
of four."""
import pytest
import torch

from parity_util import log
from test_gpu_model import run_model_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("N", [1, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("optimizer", ["sgd", "msgd", "adam"])
def test_dense_iterations(N, optimizer):
    for d, dtype, mis in ((4, "f32", 0), (1024 * 4, "bf16", 0), (1024 * 9 + 36, "f32", 0),
                          (5000 + 3, "bf16", 0), (4096, "f32", 1)):
        log(f"[dense] N={N} {optimizer} d={d} {dtype} misalign={mis}")
        run_model_case(label=f"dense_{N}_{optimizer}_{d}", d=d, N=N, n=4, K=1, steps=3,
                       dense_steps=2, optimizer=optimizer, grad_dtype=dtype,
                       family=1 if dtype == "bf16" else 0, weight_decay=5e-4, misalign=mis)


# Dense iterations and, after them, the x update alone, off 16 bytes: fewer
# values than a quad, tails of 1 to 3 values around a tile's end, every
# alignment of the arrays, bf16 gradients in either half of a word.
@pytest.mark.parametrize("optimizer", ["sgd", "msgd", "adam"])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_any_length_and_alignment(optimizer, dtype):
    for d, N, mis in ((1, 1, 0), (2, 2, 1), (3, 5, 0), (5, 3, 2), (1021, 4, 3), (4095, 2, 0),
                      (4096, 3, 1), (4097, 9, 0), (4098, 2, 2), (8192, 1, 3), (10243, 5, 1)):
        log(f"[dense] d={d} N={N} {optimizer} {dtype} misalign={mis}")
        run_model_case(label=f"any_{d}_{N}_{optimizer}_{dtype}", d=d, N=N, n=4, K=1, steps=3,
                       dense_steps=2, optimizer=optimizer, grad_dtype=dtype,
                       family=1 if dtype == "bf16" else 0, weight_decay=5e-4, misalign=mis)


# The x update in tiles where d % 4 != 0, which steps take whose arrays exceed
# the 256 MiB Infinity Cache (20 or 24 bytes a coordinate here; the sizes above
# go one coordinate a thread): tails of 1 to 3 values beside a tile's end.
@pytest.mark.parametrize("optimizer,rest,mis", [("sgd", 1, 0), ("sgd", 4095, 0), ("msgd", 3, 0),
                                                ("msgd", 2, 0), ("msgd", 1, 3)])
def test_x_update_beyond_the_cache(optimizer, rest, mis):
    d = 3296 * 4096 + rest
    assert 20 * d > 256 * 1024 * 1024
    log(f"[dense] x update d={d} {optimizer} misalign={mis}")
    run_model_case(label=f"beyond_{optimizer}_{rest}", d=d, N=1, n=4096, K=1, steps=2,
                   dense_steps=1, optimizer=optimizer, weight_decay=5e-4, misalign=mis)


# The workers' arrays on 16 bytes and the model's off them.
@pytest.mark.parametrize("optimizer,dtype,mis", [("sgd", "f32", 1), ("msgd", "bf16", 2),
                                                 ("adam", "f32", 3), ("adam", "bf16", 1)])
def test_model_arrays_off_16_bytes(optimizer, dtype, mis):
    for d, N in ((4, 1), (1020, 5), (4096 + 36, 3)):
        log(f"[dense] model arrays off 16 bytes d={d} N={N} {optimizer} {dtype} misalign={mis}")
        run_model_case(label=f"model_off_{d}_{N}_{optimizer}_{dtype}", d=d, N=N, n=4, K=1, steps=3,
                       dense_steps=2, optimizer=optimizer, grad_dtype=dtype, misalign_model=mis,
                       family=1 if dtype == "bf16" else 0, weight_decay=5e-4)


@pytest.mark.parametrize("d,N", [(1, 1), (3, 1), (4097, 3), (2051, 2), (1023, 5), (1024, 3)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_randk_momentum_of_any_length(d, N, dtype):
    log(f"[dense] randk momentum d={d} N={N} {dtype}")
    run_model_case(label=f"randk_{d}_{N}", d=d, N=N, n=5, K=1, steps=2, dense_steps=0,
                   optimizer="sgd", compressor="randk", grad_dtype=dtype,
                   family=1 if dtype == "bf16" else 0)
