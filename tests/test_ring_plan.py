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
