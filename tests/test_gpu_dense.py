"""Parity of the dense check (statuses of all ids in LDS, 65 to 2^16 ids) with the oracle
where it can go wrong: ends of steps, rounds, tiles and groups of chunks, ids that share a
step in every way, the id spaces at its limits, initial statuses, malformed words."""
import sys

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
    i = np.arange(n)
    if pattern == "uniform":
        return rng.integers(0, n_ids, n)
    if pattern == "one":
        return np.full(n, n_ids - 1)
    if pattern == "runs":  # 1 to 130 events of an id in a row
        return np.repeat(rng.integers(0, n_ids, n), rng.integers(1, 131, n))[:n]
    if pattern == "neighbours":  # different ids of the same few table words
        return (i * 3) % 16
    if pattern == "every-64":  # an id comes back in the next step, at another lane
        return (i % 63) * (n_ids // 63)
    return np.minimum((rng.pareto(1.1, n) * 2).astype(np.int64), n_ids - 1)  # skewed


@pytest.mark.parametrize("pattern", ["uniform", "one", "runs", "neighbours", "every-64", "skewed"])
@pytest.mark.parametrize("n,n_ids", [(1, 65), (63, 65), (64, 66), (511, 72), (513, 4097), (1024, 1 << 16),
                                     (1025, 65_535), (33_000, 300), (100_001, 1 << 15), (1_300_000, 1 << 16)])
def test_dense_shapes(ctx, n, n_ids, pattern):
    from paper_1910_11110_amd import vcheck as V
    print(f"[dense] {pattern} {n} x {n_ids}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(n * 7 + n_ids)
    e = gen.pack_events(ids_of(pattern, n, n_ids, rng), rng.integers(0, 5, n), rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8) if n % 2 else None
    t = V.Trace.load(ctx, e, n_ids, init)
    ref = O.check(e, n_ids, init)
    for _ in range(2):  # the second check finds every buffer used
        t.check()
        assert np.array_equal(t.status(), ref.status)
        assert np.array_equal(t.final(), ref.final)
        v = t.violations()
        assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


@pytest.mark.parametrize("at", [0, 511, 512, 1100, 2099])
def test_dense_malformed(ctx, at):
    """The first malformed word of a device trace, in whole rounds and past them."""
    import torch
    from paper_1910_11110_amd import vcheck as V
    e = gen.plain_events(2100, 1000, 3)
    e[at] = 1000  # id out of range
    e[2099] = 5 << 24
    d = torch.from_numpy(e.view(np.int32)).cuda()
    torch.cuda.synchronize()
    t = V.Trace.load(ctx, d, 1000)
    t.check()
    with pytest.raises(V.VCError) as x:
        ctx.sync()
    assert x.value.code == V.VC_EINVAL and f"index {at}" in str(x.value)
    t.free()
