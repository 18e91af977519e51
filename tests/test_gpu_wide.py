"""Parity of the checks through buckets of ids (plain traces over more than 2^16 ids, k memory
spaces) with the oracle where they can go wrong: one bucket with every event, buckets
without any, ends of chunks and tiles, the numbers of buckets at which the partition
changes, last buckets that are not full."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1910_11110_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1910_11110_amd import vcheck as V
    c = V.Context(0)
    yield c
    c.close()


def ids_of(pattern, n, n_ids, rng):
    if pattern == "uniform":
        return rng.integers(0, n_ids, n)
    if pattern == "last":  # the last ids of the last bucket
        return n_ids - 1 - rng.integers(0, min(3, n_ids), n)
    if pattern == "two-buckets":
        return np.where(rng.random(n) < 0.999, rng.integers(0, min(n_ids, 5000), n), n_ids - 1)
    return np.minimum((rng.pareto(0.4, n) * 2).astype(np.int64) & 0x7FFFFFFF, n_ids - 1)  # skewed


def compare(t, ref, status):
    for _ in range(2):
        t.check()
        assert np.array_equal(status(), ref.status)
        assert np.array_equal(t.final(), ref.final)
        v = t.violations()
        assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


@pytest.mark.parametrize("pattern", ["uniform", "last", "two-buckets", "skewed"])
@pytest.mark.parametrize("n_ids", [65_537, 1 << 20, (1 << 20) + 1, (1 << 22) - 5, 1 << 22])
@pytest.mark.parametrize("n", [1, 4095, 4097, 70_001, 3_000_003])
def test_events(ctx, n, n_ids, pattern):
    from paper_1910_11110_amd import vcheck as V
    print(f"[wide] {pattern} {n} x {n_ids}", flush=True)
    rng = np.random.default_rng(n + n_ids)
    e = gen.pack_events(ids_of(pattern, n, n_ids, rng), rng.integers(0, 5, n), rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8) if n % 2 else None
    t = V.Trace.load(ctx, e, n_ids, init)
    compare(t, O.check(e, n_ids, init), t.status)


@pytest.mark.parametrize("k", [2, 3, 4])
@pytest.mark.parametrize("pattern", ["uniform", "last", "two-buckets", "skewed"])
@pytest.mark.parametrize("n,n_ids", [(1, 1), (4097, 4096), (70_001, 4097), (3_000_003, (1 << 20) + 1), (70_001, 1 << 22),
                                     (70_001, (1 << 22) + 1)])
def test_spaces(ctx, n, n_ids, pattern, k):
    from paper_1910_11110_amd import vcheck as V
    print(f"[wide] spaces k={k} {pattern} {n} x {n_ids}", flush=True)
    rng = np.random.default_rng(n + n_ids + k)
    op, a, b = rng.integers(0, 4, n), rng.integers(0, k, n), rng.integers(0, k, n)
    a, b = np.where(op == 3, 0, a), np.where(op == 2, b, 0)
    e = (ids_of(pattern, n, n_ids, rng) | (op << 24) | (a << 26) | (b << 28)).astype(np.uint32)
    init = rng.integers(0, 1 << k, n_ids).astype(np.uint8) if n % 2 else None
    t = V.Trace.load_spaces(ctx, e, n_ids, k, init)
    compare(t, O.check_spaces(e, n_ids, k, init), t.status16)


@pytest.mark.parametrize("at", [5, 100_000])
def test_malformed(ctx, at):
    import torch
    from paper_1910_11110_amd import vcheck as V
    n, n_ids = 200_000, 70_000
    e = gen.plain_events(n, n_ids, 3)
    e[[at, n - 1]] = [n_ids, 0xFFFFFFFF]
    s = gen.space_events(n, n_ids, 3, 3)
    s[[at, n - 1]] = [3 << 26, 0xFFFFFFFF]  # a location past k
    for words, load in ((e, lambda d: V.Trace.load(ctx, d, n_ids)), (s, lambda d: V.Trace.load_spaces(ctx, d, n_ids, 3))):
        d = torch.from_numpy(words.view(np.int32)).cuda()
        torch.cuda.synchronize()
        t = load(d)
        t.check()
        with pytest.raises(V.VCError) as x:
            ctx.sync()
        assert x.value.code == V.VC_EINVAL and f"index {at}" in str(x.value)
        t.free()
