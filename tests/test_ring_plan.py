"""Choices the planner makes for the direct-load ring with what a compute unit really holds."""
import random
import shutil

import pytest

from tests.ring_plan import ring_plan

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
LDS, LDS_PIECE, CUS = 160 * 1024, 1280, 256          # gfx950 hands LDS out in pieces


def test_wavefronts_that_give_way_are_those_of_the_last_resident_workgroups():
    """Five workgroups of 32 KiB would fill 160 KiB, but each takes 26 pieces of 1280 bytes: four are resident."""
    rng = random.Random(3)
    shares = five = sizes = 0
    for _ in range(20000):
        d, tile, H = rng.choice((32, 64)), rng.choice((64, 128)), rng.choice((1, 3, 4, 6, 8, 12, 16))
        table = rng.choice((0, 976, 9600, 14 * 1024, 15 * 1024, 16 * 1024, 20 * 1024, 24160, 36000, 40960))
        plan = ring_plan((rng.randint(1, 64), H, rng.randint(65, 2100), d), tile, table, qmax=rng.random() < 0.2)
        if not plan.ring:
            continue
        resident = LDS // (-(-plan.lds // LDS_PIECE) * LDS_PIECE)
        if plan.even_from < plan.grid:
            shares += 1
            assert plan.grid - plan.even_from <= resident * CUS, plan
            five += LDS // plan.lds > resident
        sizes |= 1 << plan.waves
    assert shares > 2000 and five > 100
    assert sizes & 0b111111000 == 0b111111000        # three to eight wavefronts


def test_workgroups_of_32_features():
    """Tiles of 64: six wavefronts where a compute unit gets three workgroups at most; of 128: five where it gets two, never six."""
    rng = random.Random(5)
    met = set()
    for _ in range(20000):
        tile = rng.choice((64, 128))
        plan = ring_plan((rng.randint(1, 64), rng.choice((1, 3, 4, 6, 8, 12, 16)), rng.randint(65, 2100), 32), tile,
                         rng.choice((0, 9600, 16 * 1024, 20 * 1024, 30 * 1024, 36000, 40960)))
        if plan.ring:
            met.add((tile, plan.waves))
            assert plan.waves != 6 or (tile == 64 and plan.units <= 3 * CUS), plan
            assert plan.waves != 5 or tile == 64 or plan.units <= 2 * CUS, plan
    assert met >= {(64, 3), (64, 4), (64, 5), (64, 6), (128, 3), (128, 4), (128, 5)}


def test_workgroups_that_do_not_share_the_simds_evenly():
    """64 features: five and six wavefronts with tiles of 64 only alone on a compute unit; with tiles of 128 six, and seven in
    one round, only where LDS holds two workgroups and all heads have a table, and three not with one set of constants per head."""
    rng = random.Random(4)
    met = set()
    for _ in range(30000):
        tile, H, per_head = rng.choice((64, 128)), rng.choice((1, 3, 4, 6, 8, 12, 16)), rng.random() < 0.3
        N = rng.randint(257, 1400)
        plan = ring_plan((rng.randint(1, 64), H, N, 64), tile, rng.choice((0, 9600, 20 * 1024, 24160, 36000, 40960)),
                         per_head=per_head)
        if not plan.ring:
            continue
        met.add((tile, plan.waves, per_head))
        if tile == 64:
            assert plan.waves not in (5, 6) or plan.units <= CUS, plan
        else:
            assert plan.waves != 5 and (plan.waves not in (6, 7) or (not per_head and 3 * plan.lds > LDS)), plan
            assert plan.waves != 7 or plan.units <= 2 * CUS, plan
            blocks = -(-N // 32)
            assert plan.waves != 3 or not per_head or -(-blocks // -(-blocks // 4)) == 3, plan      # (nine: three times three)
    assert {w for t, w, h in met if t == 64} == {3, 4, 5, 6, 7, 8} and {w for t, w, h in met if t == 128 and not h} == {3, 4, 6, 7, 8}
