"""The Newton-Schulz tile edges (64, 128, 256) and the cut Gram against the
fp64 oracle, at the sizes where a tile, a remainder or a part of a contraction
begins or ends.  The plan chooses the edges from the whole set, so each case is
a set, with the edges that it is meant to reach: they are asserted here and,
without a GPU, in test_routes.py."""
import pytest

from gpu_harness import compare, run_gpu, run_oracle, say
from paper_2608_05088_amd import libmalt as lm
from paper_2608_05088_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = {
    # 64-tiles: one tile, one past it, a remainder on each side, tall and wide
    "edges_64": [(64, 64), (65, 129), (127, 128), (129, 191), (320, 65), (33, 40)],
    # 64-tiles, Gram cut along k: contractions of 141 and 313 stages, one of them
    # of a hi/lo-split matrix, a tall one, and one whose parts are uneven
    "cut_64": [(64, 9001), (200, 20000), (15001, 70)],
    # 64-tiles in Gram and polynomial, 256 in the update, remainders of every kind
    "edges_64_256": [(512, 1536), (512, 512), (513, 2048), (2048, 511)] * 4,
    # the same on 128-tiles throughout, a domain of 640 = 5 x 128 rows among them
    "edges_128": [(512, 1536), (512, 512), (513, 2048), (2048, 511)] * 6,
    # 128-tiles throughout with a hi/lo-split matrix
    "split_128": [(384, 1100), (340, 384), (600, 2048), (100, 2000)] * 12,
    # 256-tiles throughout with a hi/lo-split matrix
    "split_256": [(896, 2600), (896, 896), (100, 3000)] * 12,
    # 128-tiles in the polynomial, 256 elsewhere
    "poly_128": [(768, 2304), (768, 768), (700, 3072), (3072, 768)] * 12,
    # a long matrix beside a small model: its Gram cut on 64-tiles, 128 in the update
    "long_beside_model": [(20000, 348)] + [(348, 1044), (348, 348), (348, 1392), (1392, 348)] * 4,
    # a longer one: cut on 128-tiles, every Gram on 128-tiles
    "cut_128": [(20000, 700)] + [(768, 2304), (768, 768), (768, 3072), (3072, 768)] * 12,
    # the others' Gram on 256-tiles, the long one's cut on 128-tiles beside them
    "cut_beside_256": [(30000, 768)] + [(1280, 3840), (1280, 1280), (1280, 5120), (5120, 1280)] * 4,
}

# Per case: the edge of the Gram (of its first matrix, and of its last), of the
# polynomial and of the update; whether the first matrix's Gram is cut.
EDGES = {
    "edges_64": (64, 64, 64, 64, False),
    "cut_64": (64, 64, 64, 64, True),
    "edges_64_256": (64, 64, 64, 256, False),
    "edges_128": (128, 128, 128, 128, False),
    "split_128": (128, 128, 128, 128, False),
    "split_256": (256, 256, 256, 256, False),
    "poly_128": (256, 256, 128, 256, False),
    "long_beside_model": (64, 64, 64, 128, True),
    "cut_128": (128, 128, 128, 256, True),
    "cut_beside_256": (128, 256, 256, 256, True),
}


def check_edges(name):
    """The plan takes the edges that the case is there for."""
    r = lm.plan_routes(CASES[name], "malter")
    got = (r[0]["gram_tile"], r[-1]["gram_tile"], r[0]["poly_tile"], r[0]["update_tile"], r[0]["gram_parts"] > 1)
    assert got == EDGES[name], f"{name}: the plan takes {got}, the case is there for {EDGES[name]}"
    assert all(x["route"] == 0 for x in r)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lm.lib()


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("abc", [(3.4445, -4.7750, 2.0315), (1.5, -0.5, 0.0)])
def test_tile_edges(name, abc):
    check_edges(name)
    shapes = CASES[name]
    keep = sorted(set(list(range(min(4, len(shapes)))) + [len(shapes) - 1]))
    say(f"[tiles] {name} {len(shapes)} matrices abc={abc} malter x2")
    W0 = [wl.weight(87, i, s) for i, s in enumerate(shapes)]
    grads = [[wl.grad(87, t, i, s, "row_loguniform") for i, s in enumerate(shapes)] for t in (1, 2)]
    hp = dict(lr=3e-3, ns_a=abc[0], ns_b=abc[1], ns_c=abc[2])
    g = run_gpu(shapes, "malter", W0, grads, hp, collect=keep)
    o = run_oracle(shapes, "malter", W0, grads, hp, collect=keep)
    worst = compare(g, o, "malter", label=name)
    say(f"[tiles] {name} worst {worst}")


def test_cubic_iteration_on_256_tiles():
    # c = 0 takes the 256-tile polynomial's reload path, which only sets large
    # enough for 256-tiles reach.
    shapes = [(1280, 1280)] * 36
    assert lm.plan_routes(shapes)[0]["poly_tile"] == 256
    say(f"[tiles] cubic {len(shapes)} matrices")
    W0 = [wl.weight(86, i, s) for i, s in enumerate(shapes)]
    grads = [[wl.grad(86, 1, i, s) for i, s in enumerate(shapes)]]
    hp = dict(lr=3e-3, ns_a=1.5, ns_b=-0.5, ns_c=0.0)
    g = run_gpu(shapes, "malt", W0, grads, hp, collect=[0, 35])
    o = run_oracle(shapes, "malt", W0, grads, hp, collect=[0, 35])
    say(f"[tiles] cubic worst {compare(g, o, 'malt', label='cubic')}")


# Short sides in three launches (the large ones of the set take the others along):
# whole rows and 64-column rounds and their remainders, wide and tall; a
# contraction of several Gram chunks.  Whole steps: test_short_sides_gpu.py.
SHORT = [(8, 64), (64, 8), (16, 1024), (1024, 16), (32, 2048), (2048, 32), (9, 65), (63, 7), (1, 64), (1, 1), (31, 513),
         (16, 4096), (16, 4097), (4097, 16), (32, 40000)]


@pytest.mark.parametrize("variant,ns_steps", [("malt", 5), ("malter", 2), ("malter", 1)])
def test_short_side_edges(variant, ns_steps):
    say(f"[tiles] short sides {SHORT} {variant} ns_steps={ns_steps} x2")
    W0 = [wl.weight(85, i, s) for i, s in enumerate(SHORT)]
    grads = [[wl.grad(85, t, i, s, "row_loguniform") for i, s in enumerate(SHORT)] for t in (1, 2)]
    g = run_gpu(SHORT, variant, W0, grads, dict(lr=1e-2, ns_steps=ns_steps))
    o = run_oracle(SHORT, variant, W0, grads, dict(lr=1e-2, ns_steps=ns_steps))
    # Only the final rounding of O to bf16 (2^-9 per entry at most) is left:
    # 4e-3 covers it in norm, in O and in the update.
    worst = compare(g, o, variant, tol_ns=4e-3, label="short")
    say(f"[tiles] short worst {worst}")
