"""GPU parity at the edges of the kernels' work splits (against the oracle).

Inputs are dyadic with sums that fit 24 bits, so every fp32 sum is exact in
any order and the comparison is bit for bit; other tolerances are stated
where they are used.
"""
import numpy as np
import pytest

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()
    torch.cuda.empty_cache()


def _offsets(lens):
    off = np.zeros(len(lens) + 1, np.int32)
    off[1:] = np.cumsum(lens)
    return off


def _bf16_bits(x):
    return (np.ascontiguousarray(x, np.float32).view(np.uint32) >> 16).astype(np.uint16)


def _dyadic(rng, shape, dtype):
    """Multiples of 2^-7 below 1 in magnitude (7 bits: exact in bf16 too)."""
    x = (rng.integers(-127, 128, size=shape) / 128.0).astype(np.float32)
    return x if dtype == "fp32" else _bf16_bits(x)


# lane groups of 1 to 64 lanes, with and without lanes past the row's end, and
# rows of several vectors per lane
@pytest.mark.parametrize("dtype,D", [("fp32", 4), ("fp32", 8), ("fp32", 16), ("fp32", 20), ("fp32", 32), ("fp32", 64),
                                     ("fp32", 100), ("fp32", 256), ("fp32", 260), ("fp32", 1024), ("bf16", 8),
                                     ("bf16", 104), ("bf16", 512)])
@pytest.mark.parametrize("B", [3, 4, 37])
def test_forward_short_and_long_bags(dtype, D, B):
    """Neighbouring bags all short (packed one per lane group), a long one
    among short ones, lengths around the packing limit and around the 64 ids
    a wavefront reads at a time; tables ending inside a group of four bags,
    and fewer bags than a group."""
    print(f"case forward bags {dtype} D={D} B={B}", flush=True)
    rng = np.random.default_rng(D * 100 + B)
    rows = [50, 3, 200]
    M = len(rows) * B
    pattern = [0, 1, 8, 1, 9, 1, 1, 2, 63, 64, 65, 7, 8, 8, 8, 8, 0, 0, 0, 0, 128, 129, 1, 1, 1, 1, 1, 31, 33, 4, 5, 6]
    lens = np.array([pattern[(i * 5 + B) % len(pattern)] if B != 37 else pattern[i % len(pattern)] for i in range(M)],
                    np.int32)
    off = _offsets(lens)
    idx = np.concatenate([rng.integers(0, rows[m // B], size=lens[m]) for m in range(M)]).astype(np.int32)
    W = _dyadic(rng, (sum(rows), D), dtype)
    G = (rng.integers(-8, 9, size=(M, D)) / 8.0).astype(np.float32)
    ro = np.concatenate([[0], np.cumsum(rows)])
    for idx64 in (False, True):
        parity.run_case(ro, W, off, idx, G, B, "sum", "sgd", 0.5, 0.0, exact=dtype == "fp32", idx64=idx64)
