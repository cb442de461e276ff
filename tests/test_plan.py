"""The planner on the CPU (csrc/mla_plan.h), over calls of every selection
kind: what it picks beside other plans of the same call."""
import random

import pytest

from tests import plan_probe as P


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return P.build(str(tmp_path_factory.mktemp("plan")))


def _calls(seed, n, **kw):
    rng = random.Random(seed)
    return [P.draw(rng, **kw) for _ in range(n)]


def _small(p):
    return p.ws <= P.SCRATCH


def test_no_dearer_than_covering_the_chip(exe):
    """No plan is dearer, at the planner's own prices, than the smallest number
    of splits that covers the chip, in the tile that goes with it, where both
    keep their split rows within the scratch array or neither does.  (A plan of
    several waves has to promise 7 %.)"""
    calls = [P.Call(256, 1, 128, 128, 2048, tokens=True), P.Call(256, 1, 128, 128, 2048, tokens=True, fp8=True),
             P.Call(256, 1, 128, 2048, 2048), P.Call(128, 1, 256, 1500, 1500)] + _calls(1, 6000, kinds=("blocks", "tokens"))
    beside = [P.cover_rule(c) for c in calls]
    over = 0
    for c, both in zip(calls, P.plans(exe, calls, beside)):
        p, q = both
        over += not _small(q)
        if _small(q):
            assert _small(p), (c, p, q)
        if _small(p) == _small(q):
            assert p.us <= q.us / 0.93 + 1e-9, (c, p, q)
    assert over > 100  # the limit is reached


def test_limit_forces_the_tile_by_price(exe):
    # two splits at least, whose rows exceed the scratch array in either tile
    for c in (P.Call(256, 1, 128, 128, 2048, tokens=True), P.Call(256, 1, 128, 2048, 2048),
              P.Call(128, 1, 256, 1500, 1500)):
        one, two = P.plans(exe, [c, c], [(1, 2), (2, 2)])
        assert not _small(one[0])
        assert one[0].us == min(one[1].us, two[1].us)
        assert one[0].row_groups == 2


def test_calls_that_fit_in_covering_splits_fit(exe):
    """What the allocation-free entry takes: every call whose covering splits
    fit its scratch array, per-row selections with long lists among them."""
    calls = [P.Call(300, 4, 16, 500, 400, per_row=True), P.Call(300, 8, 8, 300, 200, per_row=True),
             P.Call(200, 8, 8, 600, 400, per_row=True), P.Call(600, 64, 1, 24, 16, per_row=True),
             P.Call(1, 32768, 1, 24, 12, per_row=True),
             P.Call(1, 2048, 16, 300, 200, per_row=True, row_tile=64)] + _calls(2, 6000)
    beside = [P.cover_rule(c) for c in calls]
    n = 0
    for c, b, both in zip(calls, beside, P.plans(exe, calls, beside)):
        if both is None:
            continue
        p, q = both
        n += c.per_row
        if _small(q):
            assert _small(p), (c, p, q)
        # a tile's rows share the load of a block wherever they did
        assert p.by_id == b[2], (c, p, b)
    assert n > 1000


def test_per_row_lists_hold_their_entries(exe):
    """A split's entries fit the list of the kernel that the plan takes."""
    calls = _calls(3, 4000, kinds=("per_row",))
    for c in calls:
        c.n_splits = random.Random(c.R + c.K).choice([0, 0, 1, 2, 5])
        c.row_tile = random.Random(c.Mq + c.K).choice([0, 64])
    long = 0
    for c, both in zip(calls, P.plans(exe, calls)):
        if both is None:
            continue
        p = both[0]
        entries = p.sps * p.tile_qrows  # (by logical block: sps is K)
        assert entries <= (512 if c.fp8 else 1024), (c, p)
        assert p.S * p.sps >= c.K
        assert p.long_lists == (not c.fp8 and p.row_groups == 1 and entries > 512)
        long += p.long_lists
    assert long > 50
