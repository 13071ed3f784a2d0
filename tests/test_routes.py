"""The routes a plan chooses for its matrices (host code, no GPU): which short
sides take their whole step in one workgroup, and that the sets of the GPU tests
of the tile edges still reach the edges they are there for."""
import os

import pytest

import test_ns_tiles_gpu as tiles
from paper_2608_05088_amd import libmalt as lm

MATRIX_CORES, THREE_LAUNCHES, WHOLE_STEP = 0, 1, 2


@pytest.fixture(scope="module", autouse=True)
def L():
    if not os.path.exists(lm.LIB_PATH):
        from paper_2608_05088_amd import build
        build.build()
    return lm.lib()


def _routes(shapes, variant="malt"):
    return [r["route"] for r in lm.plan_routes(shapes, variant)]


@pytest.mark.parametrize("shapes,want", [
    # short ones, alone; the largest element count beside many, and one past it
    ([(5, 5)], [WHOLE_STEP]), ([(16, 1024)], [WHOLE_STEP]), ([(3072, 16)], [WHOLE_STEP]), ([(1, 2048)], [WHOLE_STEP]),
    ([(31, 513)], [WHOLE_STEP]), ([(33, 64)], [MATRIX_CORES]),
    ([(32, 2048)] * 64, [WHOLE_STEP] * 64), ([(32, 2049)] * 64, [THREE_LAUNCHES] * 64),
    # one or a few long thin matrices would keep one workgroup busy for 100 to
    # 900 us (1 x 65536: 864 against 63 in three launches), and so would one of 17 to
    # 32 rows with a remainder (1669 x 32: 144 against 73)
    ([(1, 4096)], [THREE_LAUNCHES]), ([(1669, 32)] * 4, [THREE_LAUNCHES] * 4),
    ([(1, 65536)], [THREE_LAUNCHES]), ([(65536, 1)] * 8, [THREE_LAUNCHES] * 8),
    ([(2, 32768), (8192, 3)], [THREE_LAUNCHES] * 2), ([(3, 8192)] * 16, [THREE_LAUNCHES] * 16),
    # many of them fill the chip: whole steps
    ([(3, 8192)] * 64, [WHOLE_STEP] * 64), ([(1, 65536)] * 64, [WHOLE_STEP] * 64), ([(8000, 7)] * 40, [WHOLE_STEP] * 40),
    # of a mixed set only the longest leave
    ([(1, 65536)] + [(3, 5000)] * 60 + [(16, 1024)], [THREE_LAUNCHES] + [WHOLE_STEP] * 61),
    # beside one that has to take three launches they cost no launch more
    ([(32, 40000), (16, 3072)], [THREE_LAUNCHES] * 2),
])
def test_whole_step_only_where_it_is_the_shorter(shapes, want):
    for variant in ("malt", "malter"):
        assert _routes(shapes, variant) == want
        assert lm.check_bounds(shapes, variant) > 0


@pytest.mark.parametrize("name", sorted(tiles.CASES))
def test_tile_cases_reach_their_edges(name):
    tiles.check_edges(name)


def test_routes_reject_bad_arguments(L):
    out = (lm.malt_route_t * 1)()
    assert L.malt_plan_routes(lm._shapes([(8, 8)]), 1, 5, out) == lm.MALT_ERR_INVALID_ARG
    assert L.malt_plan_routes(lm._shapes([(8, 8)]), 1, 0, None) == lm.MALT_ERR_INVALID_ARG
    assert L.malt_plan_routes(lm._shapes([(0, 8)]), 1, 0, out) == lm.MALT_ERR_SHAPE
