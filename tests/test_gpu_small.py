"""Parity of the check over at most 64 variables with the oracle where it can go wrong: ends
of strands, tiles and the line between short and long strands, fewer variables than a
word of the look-back holds, traces without writes (no tile's function is constant, so
every look-back runs to the first tile), malformed words of every kind."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_1910_11110_amd import gen

pytestmark = pytest.mark.gpu
LONG = 3 << 21


@pytest.fixture(scope="module")
def ctx():
    from paper_1910_11110_amd import vcheck as V
    c = V.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("ops", ["all", "no-writes", "rare-writes"])
@pytest.mark.parametrize("n_ids", [1, 19, 21, 63, 64])
@pytest.mark.parametrize("n", [15, 17, 4095, 4097, 70_001, LONG - 1, LONG, LONG + 16_385])
def test_strands(ctx, n, n_ids, ops):
    from paper_1910_11110_amd import vcheck as V
    print(f"[small] {n} x {n_ids} {ops}", flush=True)
    rng = np.random.default_rng(n + n_ids)
    op = rng.integers(0, 5, n)
    if ops != "all":
        keep = (rng.random(n) < 1e-4) if ops == "rare-writes" else np.zeros(n, bool)
        op[(op == 1) & ~keep] = 2
    e = gen.pack_events(rng.integers(0, n_ids, n), op, rng.integers(0, 2, n))
    init = rng.integers(0, 4, n_ids).astype(np.uint8)
    t = V.Trace.load(ctx, e, n_ids, init)
    t.check()
    ref = O.check(e, n_ids, init)
    assert np.array_equal(t.status(), ref.status)
    assert np.array_equal(t.final(), ref.final)
    v = t.violations()
    assert np.array_equal(v.indices, ref.violations) and v.first == ref.first
    t.free()


@pytest.mark.parametrize("word", [40, 64, 1 << 23, 5 << 24, 6 << 24, 7 << 24, 1 << 28, 1 << 31])
@pytest.mark.parametrize("n,at", [(5000, 4999), (5000, 17), (LONG + 5, LONG - 100)])
def test_malformed(ctx, n, at, word):
    import torch
    from paper_1910_11110_amd import vcheck as V
    e = gen.plain_events(n, 40, 1)
    e[[at, n - 1]] = word
    d = torch.from_numpy(e.view(np.int32)).cuda()
    torch.cuda.synchronize()
    t = V.Trace.load(ctx, d, 40)
    t.check()
    with pytest.raises(V.VCError) as x:
        ctx.sync()
    assert x.value.code == V.VC_EINVAL and f"index {at}" in str(x.value)
    t.free()


@pytest.mark.parametrize("n", [1, 4097, LONG + 3])
def test_events_off_alignment(ctx, n):
    """Device events that start 4, 8 or 12 bytes past a 16-byte line."""
    import torch
    from paper_1910_11110_amd import vcheck as V
    e = gen.plain_events(n + 3, 20, 2)
    d = torch.from_numpy(e.view(np.int32)).cuda()
    torch.cuda.synchronize()
    for off in (1, 2, 3):
        t = V.Trace.load(ctx, d[off:off + n], 20)
        t.check()
        ref = O.check(e[off:off + n], 20)
        assert np.array_equal(t.status(), ref.status)
        assert np.array_equal(t.final(), ref.final)
        assert np.array_equal(t.violations().indices, ref.violations)
        t.free()
