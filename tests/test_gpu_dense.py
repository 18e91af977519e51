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


@pytest.mark.parametrize("n_ids", [1, 64, 65, 4097, 1 << 16, (1 << 16) + 1, 80_000])
@pytest.mark.parametrize("n", [1, 511, 512, 513, 40_000, 700_001])
def test_overlap_words(ctx, n, n_ids):
    """The combined stream in program order (up to 2^16 arrays) and through the buckets
    (more), at tile ends, with arrays in clusters that all overlap each other."""
    from paper_1910_11110_amd import vcheck as V
    print(f"[dense] overlap {n} x {n_ids}", flush=True)
    rng = np.random.default_rng(n + n_ids)
    lo = (np.arange(n_ids) // 7 * 16 + rng.integers(0, 8, n_ids)).astype(np.uint32)
    hi = lo + rng.integers(1, 12, n_ids).astype(np.uint32)
    op = rng.integers(0, 5, n) if n != 513 else np.zeros(n, np.int64)
    e = gen.pack_events(np.minimum(rng.integers(0, n_ids, n), rng.integers(0, n_ids, n)), op, rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8)
    t = V.Trace.load(ctx, e, n_ids, init)
    t.set_arrays(lo, hi)
    ref = O.check_overlap(e, lo, hi, init)
    for _ in range(2):
        t.check()
        assert np.array_equal(t.status(), ref.status)
        assert np.array_equal(t.final(), ref.final)
        v = t.violations()
        assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
        assert t.induced_stuck() == ref.n_induced_stuck
    t.free()


@pytest.mark.parametrize("nv,npv", [(2, 30), (64, (1 << 16) - 64), (64, (1 << 16) - 63)])
@pytest.mark.parametrize("n", [513, 300_001])
def test_dynamic_words(ctx, n, nv, npv):
    from paper_1910_11110_amd import vcheck as V
    npv = min(npv, n // 4)
    print(f"[dense] dynamic {n} x {nv}+{npv}", flush=True)
    d = gen.dynamic_trace(n, nv, npv, n + npv, space=nv << 14)
    rng = np.random.default_rng(n)
    init = rng.integers(1, 4, d.lo.size).astype(np.uint8)
    ref = O.check_dynamic(d.events, d.lo, d.hi, d.mother, init)
    t = V.Trace.load(ctx, d.events, d.lo.size, init, lifetimes=True)
    t.set_dynamic_arrays(d.lo, d.hi, d.mother)
    for _ in range(2):
        t.check()
        assert np.array_equal(t.status(), ref.status)
        assert np.array_equal(t.final(), ref.final)
        v = t.violations()
        assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


def test_overlap_events_changed(ctx):
    """Device events rewritten after the arrays were set: more induced items than the stream
    holds are refused and reported, and the check stays in bounds; the old events again
    give the old results."""
    import torch
    from paper_1910_11110_amd import vcheck as V
    n, n_ids = 50_000, 300
    rng = np.random.default_rng(3)
    lo = (np.arange(n_ids) // 10 * 16).astype(np.uint32)
    hi = lo + 8
    e = gen.pack_events(rng.integers(0, n_ids, n), rng.integers(0, 5, n), rng.integers(0, 2, n))
    d = torch.from_numpy(e.view(np.int32).copy()).cuda()
    torch.cuda.synchronize()
    t = V.Trace.load(ctx, d, n_ids)
    t.set_arrays(lo, hi)
    t.check()
    want = t.status()
    d.copy_((d & 0x08FFFFFF) | (1 << 24))  # every event a write
    torch.cuda.synchronize()
    t.check()
    with pytest.raises(V.VCError):
        ctx.sync()
    d.copy_(torch.from_numpy(e.view(np.int32)))
    torch.cuda.synchronize()
    t.check()
    assert np.array_equal(t.status(), want)
    t.free()


@pytest.mark.parametrize("n,n_ids", [(1 << 21, 100), ((1 << 21) + 1, 100), (1 << 25, 64), ((1 << 25) + 1, 64),
                                     (1 << 24, 70_000), ((1 << 24) + 1, 70_000)])
def test_list_by_sums_and_by_scan(ctx, n, n_ids):
    """The last traces whose violation list is placed by sums of the tiles' counts, and the
    first ones that take a scan, on each of the three plain checks."""
    from paper_1910_11110_amd import vcheck as V
    print(f"[list] {n} x {n_ids}", flush=True)
    e = gen.plain_events(n, n_ids, n_ids)
    t = V.Trace.load(ctx, e, n_ids)
    t.check()
    ref = O.check(e, n_ids)
    v = t.violations()
    assert v.total == ref.violations.size and np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


@pytest.mark.parametrize("n,n_ids", [(1 << 22, 4097), ((1 << 22) + 511, 1 << 16), ((1 << 22) + 513, 9000)])
@pytest.mark.parametrize("pattern", ["uniform", "skewed", "both"])
def test_dense_forwards(ctx, n, n_ids, pattern):
    """Traces long enough to be folded forwards: of uniform ids, of skewed ones, whose chunks
    are left to the backward fold, and of stretches of either."""
    from paper_1910_11110_amd import vcheck as V
    print(f"[dense] forwards {pattern} {n} x {n_ids}", flush=True)
    rng = np.random.default_rng(n + n_ids)
    ids = ids_of("uniform" if pattern == "uniform" else "skewed", n, n_ids, rng)
    if pattern == "both":
        ids = np.where((np.arange(n) // 100_000) % 2 == 0, rng.integers(0, n_ids, n), ids)
    e = gen.pack_events(ids, rng.integers(0, 5, n), rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8)
    t = V.Trace.load(ctx, e, n_ids, init)
    t.check()
    ref = O.check(e, n_ids, init)
    assert np.array_equal(t.status(), ref.status)
    assert np.array_equal(t.final(), ref.final)
    v = t.violations()
    assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


@pytest.mark.parametrize("word", [5 << 24, 7 << 24, 1 << 28, 1 << 31, 50_000, (1 << 24) - 1])
@pytest.mark.parametrize("at", [0, 70, 511, 4_096, (1 << 22) + 99])
def test_dense_forwards_malformed(ctx, at, word):
    """The first malformed word of a trace folded forwards is reported, wherever it lies."""
    import torch
    from paper_1910_11110_amd import vcheck as V
    n, n_ids = (1 << 22) + 100, 50_000
    e = gen.plain_events(n, n_ids, 3)
    e[at] = word
    e[-1] = 6 << 24
    t = V.Trace.load(ctx, torch.from_numpy(e.view(np.int32)).cuda(), n_ids)
    t.check()
    with pytest.raises(V.VCError) as ex:
        ctx.sync()
    assert str(at) in str(ex.value)
    t.free()


@pytest.mark.parametrize("few", [1, 2, 5, 31, 63])
@pytest.mark.parametrize("ops", ["all", "transfers", "reads"])
def test_dense_steps_that_share(ctx, few, ops):
    """Steps in which most lanes share ids: the functions of an id's lanes composed at once,
    with and without constants among them, from every status."""
    from paper_1910_11110_amd import vcheck as V
    n, n_ids = 20_011, 300
    rng = np.random.default_rng(few)
    ids = rng.permutation(n_ids)[:few][rng.integers(0, few, n)]
    op = {"all": rng.integers(0, 5, n), "transfers": np.where(rng.random(n) < 0.03, 1, rng.integers(2, 4, n)),
          "reads": np.where(rng.random(n) < 0.01, rng.integers(1, 4, n), 0)}[ops]
    e = gen.pack_events(ids, op, rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8)
    t = V.Trace.load(ctx, e, n_ids, init)
    t.check()
    ref = O.check(e, n_ids, init)
    assert np.array_equal(t.status(), ref.status)
    assert np.array_equal(t.final(), ref.final)
    assert np.array_equal(t.violations().indices, ref.violations)
    t.free()


@pytest.mark.parametrize("block", [300, 700, 5000])
@pytest.mark.parametrize("n_ids", [300, 4096, 65_536, 1 << 17])
def test_dense_ids_that_change_their_kind(ctx, n_ids, block):
    """Chunks of several rounds whose blocks are uniform, runs of an id, two ids in turn, skewed
    or a single id, without constants at times: every round goes another way than the last one,
    the first rounds of the chunks too."""
    from paper_1910_11110_amd import vcheck as V
    n = 5_000_011
    rng = np.random.default_rng(n_ids + block)
    i = np.arange(n)
    kind = (i // block) % 5
    ids = np.choose(kind, [rng.integers(0, n_ids, n), np.repeat(rng.integers(0, n_ids, n // 100 + 1), 100)[:n],
                           np.where(i & 1, n_ids - 1, 3), ids_of("skewed", n, n_ids, rng), np.full(n, n_ids // 2)])
    op = np.where((i // (7 * block)) % 3 == 0, rng.integers(0, 5, n), rng.integers(2, 5, n))
    e = gen.pack_events(ids, op, rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8)
    print(f"[dense] changing kinds, {block} x {n_ids}", flush=True)
    t = V.Trace.load(ctx, e, n_ids, init)
    t.check()
    ref = O.check(e, n_ids, init)
    assert np.array_equal(t.status(), ref.status)
    assert np.array_equal(t.final(), ref.final)
    assert np.array_equal(t.violations().indices, ref.violations)
    t.free()


@pytest.mark.parametrize("word", [5 << 24, (1 << 24) - 1])
@pytest.mark.parametrize("n,n_ids", [(70_000, 60), (70_000, 300), ((1 << 22) + 100, 50_000), (70_000, 1 << 17)])
@pytest.mark.parametrize("at", [0, 1, 511, 69_899])
def test_malformed_index_exactly(ctx, n, n_ids, at, word):
    """The index reported is that of the first of two malformed words, digit by digit, on the
    routes of few, many and very many ids and of long traces folded forwards."""
    import re

    import torch

    from paper_1910_11110_amd import vcheck as V
    e = gen.plain_events(n, n_ids, 3)
    e[[at, n - 70]] = word
    t = V.Trace.load(ctx, torch.from_numpy(e.view(np.int32)).cuda(), n_ids)
    t.check()
    with pytest.raises(V.VCError) as ex:
        ctx.sync()
    assert ex.value.code == V.VC_EINVAL and re.search(rf"index {at}\b", str(ex.value)), str(ex.value)
    t.free()
