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


# rows held by 1, 2, 4 and 16 lane groups of a wavefront, rows of several vectors per lane, and rows in parts (the
# last one partial, or whole)
@pytest.mark.parametrize("dtype,D", [("fp32", 16), ("fp32", 64), ("fp32", 128), ("fp32", 256), ("fp32", 1024),
                                     ("bf16", 128), ("bf16", 512), ("fp32", 1028), ("fp32", 2048), ("bf16", 4096)])
@pytest.mark.parametrize("ids", ["one id", "few rows", "skewed", "any"])
def test_forward_precision_of_long_bags(dtype, D, ids):
    """Bags of up to 20000 ids, of one id over and over, of a table of few
    rows, mostly of a few hot ids, or of any: with rows of one sign, an element's
    relative error is at most one fp32 rounding, 2^-24, for each addition in a
    row's way: a round (3 pairwise and 1 of two rounds; or 8 multiply-adds where
    repeats are merged: rows of one or two lane groups), the lane groups (up to
    2, 6 without a second round, or 1), one for a double sum's conversion and two
    for the mean's scale, 12 in all, and for rows of fewer than 32 lanes one for
    each further chunk of 64 ids."""
    import torch
    import paper_2112_02752_amd as emb
    print(f"case forward precision {dtype} D={D} {ids}", flush=True)
    rng = np.random.default_rng(D)
    R = 20 if ids == "few rows" else 3000
    lens = np.array([1, 7, 30, 64, 65, 200, 1000, 4096, 20000])
    off = _offsets(lens)
    if ids == "one id":
        idx = np.repeat(rng.integers(0, R, size=len(lens)), lens)
    elif ids == "skewed":
        idx = (rng.zipf(1.5, size=off[-1]) - 1) % R
    else:
        idx = rng.integers(0, R, size=off[-1])
    W = torch.from_numpy(rng.uniform(0.5, 1.5, size=(R, D)).astype(np.float32))
    W = W if dtype == "fp32" else W.to(torch.bfloat16)
    t = emb.Tables(W.cuda(), [0, R])
    rows = W.double().numpy()
    for pool in ("sum", "mean"):
        b = emb.Batch(torch.from_numpy(off).cuda(), torch.from_numpy(idx.astype(np.int32)).cuda(), len(lens))
        out = torch.zeros((len(lens), D), device="cuda")
        emb.pool_fwd(t, b, pool, out)
        for m, L in enumerate(lens):
            n = np.bincount(idx[off[m]:off[m + 1]], minlength=R).astype(np.float64)
            ref = (n @ rows) / (L if pool == "mean" else 1)
            err = np.abs(out[m].cpu().numpy().astype(np.float64) - ref) / ref
            wide = D * (4 if dtype == "fp32" else 2) > 256
            assert err.max() <= (12 + (0 if wide else L // 64)) * 2.0 ** -24, (L, pool, err.max())


def _segments_case(rng, seg_lens, M, repeat):
    """A one-table batch of M bags whose sorted keys have the given segment
    lengths; `repeat` positions of a bag carry the same id in a row."""
    N = int(sum(seg_lens))
    ids = np.repeat(np.arange(len(seg_lens)), seg_lens)
    if repeat > 1:
        # whole groups of equal ids move together, so bags hold runs of one id
        groups = [g for L in np.split(ids, np.flatnonzero(np.diff(ids)) + 1)
                  for g in np.array_split(L, max(1, len(L) // repeat))]
        ids = np.concatenate([groups[i] for i in rng.permutation(len(groups))])
    else:
        ids = ids[rng.permutation(N)]
    cuts = np.sort(rng.integers(0, N + 1, size=M - 1))
    off = np.concatenate([[0], cuts, [N]]).astype(np.int32)
    return off, ids.astype(np.int32)


_SEGMENTS = {
    "one": [1],
    "chunk": [64],
    "past a chunk": [65],
    "two long": [65, 65],
    "single positions": [1] * 130,
    "ends at chunk ends": [64, 32, 32, 16, 48, 1, 63],
    "crossing": [40, 40, 40, 64, 64, 2, 63, 64, 1, 65, 15, 17, 16],
    "long after short": [3, 200, 5, 128, 64, 64, 129, 1, 1, 500, 60, 7],
    "across combine ranges": [10, 64 * 64 * 2 + 100, 3, 64 * 64 + 1, 64, 50],
}


@pytest.mark.parametrize("dtype,D", [("fp32", 36), ("fp32", 64), ("bf16", 40), ("fp32", 68), ("fp32", 128),
                                     ("bf16", 104), ("fp32", 256), ("bf16", 264), ("fp32", 1024)])
@pytest.mark.parametrize("name", sorted(_SEGMENTS))
def test_reduce_segment_lengths(dtype, D, name):
    """Segments ending at, before and after the boundaries of chunks, of a
    chunk's parts and of combine ranges, with and without repeated bags; the
    gradient rows are integers, their sums below 2^24, so every order agrees
    bit for bit (fp32 tables: the updated rows too, lr a power of two)."""
    print(f"case reduce segments {name} {dtype} D={D}", flush=True)
    rng = np.random.default_rng(D + len(name))
    for repeat in (1, 5):
        M = max(1, sum(_SEGMENTS[name]) // 9)
        off, idx = _segments_case(rng, _SEGMENTS[name], M, repeat)
        R = len(_SEGMENTS[name]) + 3
        W = _dyadic(rng, (R, D), dtype)
        G = rng.integers(-16, 17, size=(M, D)).astype(np.float32)
        parity.run_case([0, R], W, off, idx, G, M, "sum", "sgd", 0.5, 0.0, exact=dtype == "fp32")
        # unfused, and every optimizer, within the parity tolerance; the unfused
        # update equals the fused one bit for bit
        if repeat == 5:
            for opt in ("adagrad", "adagrad_ew"):
                s0 = np.full(R if opt == "adagrad" else (R, D), 1.0, np.float32)
                got = [parity.run_case([0, R], W, off, idx, G, M, "mean", opt, 0.01, 1e-8, state0=s0.copy(),
                                       fused=fused) for fused in (True, False)]
                keys = got[0][0].unique_keys
                np.testing.assert_array_equal(got[0][2].rows(keys), got[1][2].rows(keys))
                np.testing.assert_array_equal(got[0][2].state_rows(keys), got[1][2].state_rows(keys))


@pytest.mark.parametrize("dtype,D", [("fp32", 36), ("bf16", 72), ("fp32", 132)])
@pytest.mark.parametrize("chunks", [5000, 5001, 8192, 8193, 16384, 16385, 20480, 20481])
def test_reduce_split_of_chunks(dtype, D, chunks):
    """Batches on both sides of the sizes where four, two and one wavefronts
    share a chunk, segments of all lengths around a chunk's and its parts'; the
    gradient rows are integers, their sums exact."""
    print(f"case reduce split {dtype} D={D} chunks={chunks}", flush=True)
    rng = np.random.default_rng(D + chunks)
    N = chunks * 64 - 7
    lens = rng.choice([1, 1, 1, 2, 3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 130, 700, 9000], size=N)
    lens = lens[:int(np.searchsorted(np.cumsum(lens), N)) + 1]
    lens[-1] -= int(lens.sum()) - N
    M = N // 9
    off, idx = _segments_case(rng, lens, M, 1)
    W = _dyadic(rng, (len(lens), D), dtype)
    G = rng.integers(-16, 17, size=(M, D)).astype(np.float32)
    parity.run_case([0, len(lens)], W, off, idx, G, M, "sum", "sgd", 0.5, 0.0, exact=dtype == "fp32")


@pytest.mark.parametrize("D", [36, 48, 64])
@pytest.mark.parametrize("n", [2048 * 64, 2048 * 64 + 1, 5000 * 64 + 1, 10240 * 64 + 1, 16384 * 64 + 1])
def test_unfused_equals_fused_in_both_forms(D, n):
    """Batches on both sides of the sizes where chunks are shared by four, two
    and one wavefronts: a row's sum of squares is formed in one order, whichever
    kernel updates it."""
    print(f"case unfused forms D={D} N={n}", flush=True)
    rng = np.random.default_rng(n + D)
    rows, B = 30000, n // 20
    cuts = np.sort(rng.integers(0, n + 1, size=B - 1))
    off = np.concatenate([[0], cuts, [n]]).astype(np.int32)
    idx = ((rng.zipf(1.2, size=n) - 1) % rows).astype(np.int32)
    W = rng.uniform(-0.1, 0.1, size=(rows, D)).astype(np.float32)
    G = rng.standard_normal((B, D)).astype(np.float32)
    got = [parity.run_case([0, rows], W, off, idx, G, B, "sum", "adagrad", 0.01, 1e-8, fused=f) for f in (True, False)]
    keys = got[0][0].unique_keys
    np.testing.assert_array_equal(got[0][2].rows(keys), got[1][2].rows(keys))
    np.testing.assert_array_equal(got[0][2].state_rows(keys), got[1][2].state_rows(keys))


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1023, 1025, 2047, 2048, 2049, 4096, 4097, 8191, 8192, 8193])
@pytest.mark.parametrize("rows,B", [([2], None), ([1], None), ([70_000], 32768), ([300, 1, 5000], None),
                                    ([9] * 40, 1), ([1 << 20, 1 << 20, 40], 2)])
def test_dedup_of_small_batches(n, rows, B):
    """Batches on both sides of the sizes one workgroup deduplicates, one and
    several tables, one bag a table, and more bags than ids (most of them
    empty); integer outputs are exact (int32 and int64 ids)."""
    T = len(rows)
    B = max(1, n // (3 * T)) if B is None else B
    M = T * B
    print(f"case small dedup N={n} T={T} B={B}", flush=True)
    rng = np.random.default_rng(n + T)
    cuts = np.sort(rng.integers(0, n + 1, size=M - 1)) if M > 1 else np.zeros(0, np.int64)
    off = np.concatenate([[0], cuts, [n]]).astype(np.int32)
    bag = np.repeat(np.arange(M), np.diff(off))
    per = np.asarray(rows)[bag // B]
    idx = np.minimum((per * rng.random(n) ** 3).astype(np.int64), per - 1).astype(np.int32)
    W = _dyadic(rng, (sum(rows), 4), "fp32")
    G = (rng.integers(-8, 9, size=(M, 4)) / 8.0).astype(np.float32)
    ro = np.concatenate([[0], np.cumsum(rows)])
    parity.run_case(ro, W, off, idx, G, B, "sum", "sgd", 0.5, 0.0, exact=True, idx64=bool(n % 2))


def _bags_of(rng, n, M, used):
    """Offsets of M bags that hold n ids in all, in the bags whose number is in `used` only."""
    lens = np.zeros(M, np.int64)
    lens[used] = np.bincount(np.sort(rng.integers(0, len(used), size=n)), minlength=len(used))
    return _offsets(lens)


_LAYOUTS = {
    # one table; bags of about seven ids
    "one table": ([40_000], lambda n: n // 7 + 1, [0]),
    # neighbouring tables share their first positions where no bag of theirs holds an id: first, middle, last
    "empty tables": ([50, 7, 30_000, 11, 3, 900, 1 << 20, 20], lambda n: n // 30 + 1, [2, 5, 6]),
    # so many bags, most of them empty, that the bags around a tile are searched
    "empty bags": ([300, 70_000], lambda n: 200_000, [0, 1]),
    # every bag of one id
    "one id a bag": ([1 << 22], lambda n: max(n, 32_769), [0]),
}


# one partial tile (more bags than one workgroup takes), exact multiples of the
# 2048-key tiles and one key on either side, of a prefix group of 16 tiles, of
# the 2560- and 4096-key tiles of larger batches
_EDGES = [1, 64, 2047, 2048, 2049, 4097, 10_239, 10_240, 10_241, 32_767, 32_768, 32_769, 40_961, 511_999, 512_000,
          512_001, 819_199, 819_200, 819_201, 1_048_577, 1_064_960, 1_064_961]


# (and so many bags, none empty, that the samples around a tile are sampled again)
@pytest.mark.parametrize("layout,n", [(x, n) for x in sorted(_LAYOUTS) for n in _EDGES] +
                         [("one id a bag", 8_400_001), ("one table", 8_400_001),
                          # 1024 and 1025 tiles: the column scan's two forms
                          ("empty tables", 4_194_304), ("empty tables", 4_194_305)])
def test_general_dedup_at_its_edges(layout, n):
    """The dedup by sort passes, co-resident and wait-free: every integer output
    exact, the bags through gradient rows that are sums of integers."""
    import oracle
    import torch
    import paper_2112_02752_amd as emb
    rows, bags, used = _LAYOUTS[layout]
    T, B = len(rows), bags(n)
    M = T * B
    if n <= 8192 and M <= 32_768:
        B = 32_769 // T + 1
        M = T * B
    print(f"case general dedup {layout} N={n} M={M}", flush=True)
    rng = np.random.default_rng(n + M)
    if layout == "one id a bag":
        off = _offsets((np.arange(M) < n).astype(np.int64))
    else:
        off = _bags_of(rng, n, M, np.concatenate([np.arange(t * B, (t + 1) * B) for t in used]))
    bag = np.repeat(np.arange(M), np.diff(off))
    per = np.asarray(rows)[bag // B]
    idx = np.minimum((per * rng.random(n) ** 3).astype(np.int64), per - 1)
    idx = idx if n % 2 else idx.astype(np.int32)
    ro = np.concatenate([[0], np.cumsum(rows)]).astype(np.int64)
    ref = oracle.unique_ids(T, ro, B, off, idx.astype(np.int32))
    G = rng.integers(-8, 9, size=(M, 4)).astype(np.float32)
    o_gr, _ = oracle.grad_reduce(T, B, off, G, "sum", ref)
    tables = emb.Tables(torch.empty((1, 4), dtype=torch.float32, device="cuda"), [int(x) for x in ro])
    b = emb.Batch(torch.from_numpy(off).cuda(), torch.from_numpy(idx).cuda(), B)
    Gd = torch.from_numpy(G).cuda()
    d = emb.DedupBuffers("cuda", n, M, 4)
    gr = torch.zeros((n, 4), device="cuda")
    for concurrent in (False, True):
        emb.unique_ids(tables, b, d.unique_keys, d.counts, d.seg_offsets, d.sort_perm, d.num_unique, d.ws,
                       concurrent=concurrent)
        emb.grad_reduce(tables, b, "sum", Gd, d.sort_perm, d.seg_offsets, d.unique_keys, d.num_unique, d.ws,
                        grad_rows=gr)
        torch.cuda.synchronize()
        assert emb.read_status(d.ws)[0] == 0
        U = int(d.num_unique.item())
        assert U == ref.num_unique
        np.testing.assert_array_equal(d.unique_keys[:U].cpu().numpy().view(np.uint32), ref.unique_keys)
        np.testing.assert_array_equal(d.counts[:U].cpu().numpy(), ref.counts)
        np.testing.assert_array_equal(d.seg_offsets[:U + 1].cpu().numpy(), ref.seg_offsets)
        np.testing.assert_array_equal(d.sort_perm[:n].cpu().numpy(), ref.perm)
        np.testing.assert_array_equal(gr[:U].cpu().numpy(), o_gr)
