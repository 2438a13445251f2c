"""The embedding-bag stage at the edges of its ways of summing: bags of more
ids than the lanes of a bag take in one round, and table rows whose entry
counts lie on both sides of the limits 4 and 64 and of a scan block of 4096
rows."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_parity import _bags, _run_bags, _run_bags_bwd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,M,T", [(4, 70, 3), (8, 33, 9), (16, 129, 2), (32, 17, 8), (64, 1, 11), (256, 21, 2)])
def test_long_bags(dim, M, T):
    dense, offsets, indices, tables = _bags(dim + M, M, T, 200, dim, 3, 150)
    x_ld = (3 + T * dim + 7) // 8 * 8
    x, status = _run_bags(dense, offsets, indices, tables, "f32", x_ld)
    assert status == 0
    ref = oracle.embed_bags(dense.astype(np.float64), offsets, indices, tables.astype(np.float64))
    mag = oracle.embed_bags(dense.astype(np.float64), offsets, indices, np.abs(tables.astype(np.float64)))
    # at most 149 additions in fp32, each half an ulp of at most the sum of magnitudes; log1p a few ulp
    assert np.all(np.abs(x[:, :3 + T * dim] - ref) <= 150 * 2.0 ** -24 * np.abs(mag) + 1e-6 * np.abs(ref))


@pytest.mark.parametrize("dtype,dim,rows", [("f32", 16, 4097), ("bf16", 64, 1030), ("bf16", 256, 65), ("f32", 4, 1023)])
def test_bucket_sizes(dtype, dim, rows):
    """Rows of 0, 1, 3, 4, 5, 63, 64, 65, 130 and 1025 entries, spread over
    two tables and shuffled over the bags; whole numbers, so every sum is exact."""
    rng = np.random.Generator(np.random.PCG64(dim))
    M, T = 61, 2
    offsets, ids, base = np.zeros((T, M + 1), np.int64), [], 0
    for t in range(T):
        at = rng.choice(rows, size=20, replace=False)
        at[:2] = (0, rows - 1) if t else (rows - 1, 0)
        at = np.unique(at)
        some = np.repeat(at, np.resize([1, 4, 5, 64, 65, 3, 63, 130, 1025], at.size))
        rng.shuffle(some)
        cut = np.sort(rng.integers(0, some.size + 1, size=M - 1))
        offsets[t] = base + np.concatenate([[0], cut, [some.size]])
        ids.append(some.astype(np.int32))
        base += some.size
    dx = rng.integers(-8, 9, size=(M, (1 + T * dim + 7) // 8 * 8)).astype(np.float32)
    g, status = _run_bags_bwd(offsets, np.concatenate(ids), dx, 1, rows, dim, dtype)
    assert status == 0
    ref = oracle.embed_bags_backward(offsets, np.concatenate(ids), dx.astype(np.float64), 1, rows, dim)
    assert np.array_equal(g, ref.astype(np.float32))


def _exact(name, counts, M, dim, dtype):
    """One table whose row r has counts[r] entries, shuffled over M bags; whole
    numbers, so every sum is exact."""
    print(f"[bags] {name}", flush=True)
    rng = np.random.Generator(np.random.PCG64(len(counts) + dim))
    ids = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    rng.shuffle(ids)
    cut = np.sort(rng.integers(0, ids.size + 1, size=M - 1))
    offsets = np.concatenate([[0], cut, [ids.size]]).astype(np.int64)[None]
    dx = rng.integers(-8, 9, size=(M, (1 + dim + 7) // 8 * 8)).astype(np.float32)
    g, status = _run_bags_bwd(offsets, ids, dx, 1, len(counts), dim, dtype)
    assert status == 0
    ref = oracle.embed_bags_backward(offsets, ids, dx.astype(np.float64), 1, len(counts), dim)
    assert np.array_equal(g, ref.astype(np.float32))


@pytest.mark.parametrize("dtype,dim", [("bf16", 64), ("f32", 4), ("f32", 16), ("bf16", 256)])
@pytest.mark.parametrize("n", [512, 513])
def test_many_rows_beyond_a_wave(n, dtype, dim):
    """As many rows of more than 64 entries as take a workgroup each, and one
    more, beyond which a wave sums those of up to 512."""
    sizes = [65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1024]
    counts = np.concatenate([np.resize(sizes, n), [0, 1, 4, 5, 63, 64, 0]])
    _exact(f"{n} rows, {dtype}, dim {dim}", counts, 777, dim, dtype)


@pytest.mark.parametrize("dtype,dim", [("bf16", 16), ("f32", 64)])
def test_huge_rows(dtype, dim):
    """Rows of 16384 entries and more: a bitmap after another, dense ranges (the
    row of 90000 in one half of the entries) and sparse ones."""
    counts = [16384, 16385, 90000, 40000, 3, 0, 700, 20000]
    _exact(f"huge, {dtype}, dim {dim}", counts, 3001, dim, dtype)
    _exact(f"dense, {dtype}, dim {dim}", [70000], 5, dim, dtype)
