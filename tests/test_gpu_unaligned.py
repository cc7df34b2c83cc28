"""GPU parity of rows that do not start or end on 16 bytes: widths and worker
bases that are not multiples of 4 values, arrays offset by single elements,
bf16 rows that start in the upper half of a word, every r of the vectorised
kernels, the ragged tail row and Top-K's row norms, against the oracle, bit
for bit."""
import re

import pytest
import torch

import paper_2510_26709_amd as arc
from parity_util import log, run_case
from test_gpu_compare import run_compare_case

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# Rows of one to three values (window kernels), of four to 819 (spans: up to
# 64 rows, down to five) and of more (lines kernel): around whole quads,
# around the 256-column chunks less the line's lag, and whole quads on an odd
# worker base.
WIDTHS = [1, 2, 3, 4, 5, 6, 31, 33, 62, 65, 127, 129, 147, 255, 257, 259, 510, 513, 576, 818, 819,
          820, 821, 990, 992, 993, 1001, 1024, 1026, 2303, 4099]


@pytest.mark.parametrize("n", WIDTHS)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_parity_odd_widths(n, dtype):
    rows = max(3, min(9000 // n, 150)) if n > 1 else 500
    for k, (r, N, extra, mis) in enumerate([(4, 3, 1, 0), (4, 8, n // 2, 1), (8, 2, 0, 3),
                                            (1, 2, 2, 2), (2, 3, 3, 5)]):
        d = n * rows + extra % n
        log(f"[unaligned] n={n} {dtype} r={r} N={N} d={d} misalign={mis}")
        run_case(label=f"odd_{n}_{dtype}_{k}", d=d, N=N, n=n, r=r, K=rows // 7 + 1, steps=2,
                 grad_dtype=dtype, family=1 if dtype == "bf16" else 0, misalign=mis, check_S=True)


# Widths on both sides of the span kernel's forms (3, 5, 7 and 17 loads a lane
# take 737, 1249, 1761 and 4096 values, 64 rows a span): worker bases 31 to 28
# values past a line, the whole quads then starting at any of the four words,
# several full spans, a partial one and a ragged row.
@pytest.mark.parametrize("n,loads", [(4, 3), (7, 3), (11, 3), (12, 5), (19, 5), (20, 7), (27, 7),
                                     (28, 17), (63, 17)])
def test_span_loads_follow_the_rows(n, loads):
    base = n * 330 // 32 * 32
    for k, (dtype, r, mis, res) in enumerate([("f32", 4, 0, 31), ("bf16", 4, 1, 31),
                                              ("f32", 1, 2, 28), ("bf16", 8, 3, 31),
                                              ("f32", 2, 0, 28), ("bf16", 4, 0, 28)]):
        d = base + res
        log(f"[unaligned] span n={n} {dtype} r={r} misalign={mis}")
        run_case(label=f"span_{n}_{k}", d=d, N=4, n=n, r=r, K=20, steps=2, grad_dtype=dtype,
                 family=1 if dtype == "bf16" else 0, misalign=mis, check_S=True)
    comp = arc.Compressor(d=d, N=4, n=n, r=4, K=20, eta=0.1, seed=1)
    try:
        assert f"span_loads={loads} " in comp.describe(), comp.describe()
    finally:
        comp.close()


# Spans of 8 to 32 rows, around the counts where a lane takes one, two, four or
# all of a row's chains (rows * r / chains <= 64), and their partial last spans.
@pytest.mark.parametrize("n", [127, 128, 129, 131, 204, 240, 241, 255, 315, 400, 455, 456, 512])
def test_span_chains_per_lane(n):
    for r, dtype in ((8, "f32"), (4, "bf16"), (8, "bf16"), (2, "f32")):
        log(f"[unaligned] chains n={n} r={r} {dtype}")
        run_case(label=f"chains_{n}_{r}", d=n * 77 + 11, N=2, n=n, r=r, K=9, steps=2,
                 grad_dtype=dtype, family=1 if dtype == "bf16" else 0, check_S=True)


# Wide rows in groups of every 4th row (2307, 5001 values) and of every 4th
# and 2nd at power-of-two widths, with a ragged tail row.
@pytest.mark.parametrize("n,dtype,mis", [(2307, "f32", 1), (2307, "bf16", 0), (5001, "bf16", 3),
                                         (2048, "f32", 0), (4096, "bf16", 1)])
def test_parity_strided_rows_off_lines(n, dtype, mis):
    log(f"[unaligned] strided n={n} {dtype} misalign={mis}")
    run_case(label=f"strided_{n}_{dtype}", d=n * 70 + 1001, N=3, n=n, r=4, K=9, steps=2,
             grad_dtype=dtype, family=1 if dtype == "bf16" else 0, misalign=mis, check_S=True)


# Tensors on either side of a 16-byte boundary in one layout: aligned lists,
# unaligned lists and groups of rows 4 apart side by side.
TENSORS = [(70, 2048, 3), (64, 27, 4), (1, 10, 1), (33, 577, 2), (40, 3072, 2), (9, 3071, 1),
           (130, 64, 9), (2, 3, 1), (129, 300, 5), (1, 1001, 1)]


@pytest.mark.parametrize("dtype,r,mis,pad", [("f32", 4, 0, 0), ("f32", 4, 0, 1), ("bf16", 4, 0, 1),
                                             ("bf16", 2, 1, 3), ("f32", 8, 2, 2),
                                             ("f32", 1, 3, 0)])
def test_tensor_parity_mixed_alignment(dtype, r, mis, pad):
    tensors = TENSORS + [(1, 4 - sum(a * b for a, b, _ in TENSORS) % 4 + pad, 1)]
    log(f"[unaligned] tensors {dtype} r={r} misalign={mis} pad={pad}")
    run_case(label=f"mixed_{dtype}_{r}_{mis}_{pad}", d=sum(a * b for a, b, _ in tensors), N=3, r=r,
             tensors=tensors, steps=2, grad_dtype=dtype, family=1 if dtype == "bf16" else 0,
             misalign=mis, check_S=True)


@pytest.mark.parametrize("n,dtype,mis", [(3, "f32", 0), (33, "bf16", 1), (147, "f32", 1),
                                         (258, "bf16", 0), (1001, "f32", 2), (2050, "bf16", 1)])
def test_topk_norms_unaligned(n, dtype, mis):
    log(f"[unaligned] topk n={n} {dtype} misalign={mis}")
    run_compare_case(compressor="topk", d=n * 70 + n // 2, N=3, n=n, K=6, grad_dtype=dtype,
                     family=1 if dtype == "bf16" else 0, misalign=mis, label=f"topk_{n}_{dtype}")


def _kernel_of(desc):
    """The one list of row groups of a single view."""
    windows = re.search(r"\(64:(\d+) 32:(\d+) 16:(\d+) 8:(\d+) rows\)", desc).groups()
    count = {key: int(re.search(key + r"_groups=(\d+)", desc).group(1))
             for key in ("span", "line", "general")}
    count["window"] = sum(int(c) > 0 for c in windows)
    used = [key for key, c in count.items() if c > 0]
    assert len(used) == 1 and count["window"] <= 1, desc
    return used[0]


# One worker's rows of whole 256-column chunks are on the lines whatever d is;
# several workers' are not.  Spans where six waves' LDS fits a compute unit or
# few waves are needed; the rows of a view are counted, its tail is not.
@pytest.mark.parametrize("n,rows,N,res,r,want", [
    (256, 60, 1, 4, 4, "window"), (512, 60, 1, 8, 4, "window"), (768, 6000, 1, 4, 8, "window"),
    (768, 60, 1, 0, 4, "window"), (768, 60, 4, 0, 4, "window"), (512, 60, 1, 1, 4, "span"),
    (320, 60, 1, 4, 4, "span"), (512, 60, 4, 4, 4, "span"), (2048, 60, 2, 4, 4, "window"),
    (768, 1270, 4, 4, 4, "span"), (768, 1290, 4, 4, 4, "line"), (768, 2580, 2, 4, 2, "span"),
    (640, 2000, 4, 4, 4, "span"), (704, 1400, 4, 8, 4, "span"), (800, 5200, 1, 4, 4, "line"),
    (320, 4000, 4, 4, 8, "span"), (512, 2070, 4, 4, 8, "line"), (819, 2570, 2, 1, 4, "line"),
    (819, 2570, 2, 1, 1, "span")])
def test_kernel_of_the_rows(n, rows, N, res, r, want):
    d = n * rows // 32 * 32 + res
    comp = arc.Compressor(d=d, N=N, n=n, r=r, K=3, eta=0.1, seed=1)
    try:
        assert _kernel_of(comp.describe()) == want, comp.describe()
    finally:
        comp.close()
    log(f"[unaligned] route n={n} rows={rows} N={N} res={res} r={r}")
    run_case(label=f"route_{n}_{N}_{res}_{r}", d=d, N=N, n=n, r=r, K=7, steps=1, check_S=True)


def test_ragged_row_shares_the_launch_of_its_view():
    # Rows on the lines and off them, narrow and wide, on 16 bytes and not:
    # the tail row never adds a list of its own (each non-empty list is one
    # launch of the streaming stage).
    for n, d in ((3904, 3904 * 50 + 36), (2048, 2048 * 50 + 32), (512, 512 * 90 + 40),
                 (333, 333 * 90 + 2), (1001, 1001 * 50 + 3), (4099, 4099 * 40 + 1)):
        comp = arc.Compressor(d=d, N=2, n=n, r=4, K=3, eta=0.1, seed=1)
        try:
            desc = comp.describe()
        finally:
            comp.close()
        _kernel_of(desc)
