"""Matrices with a short side of at most 32 (Newton-Schulz in the Gram space, in
float64): whole steps against the oracle at the edges of their workgroup; where
the form can go wrong, gradients of low rank over many
iterations, and sums over a long side, on both routes (whole step in one
workgroup, three launches); gradients that overlap a W which a whole step
writes."""
import numpy as np
import pytest

from gpu_harness import compare, run_gpu, run_oracle, say
from oracle import rel_fro
from paper_2608_05088_amd import libmalt as lm
from paper_2608_05088_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lm.lib()


WHOLE_STEP, THREE_LAUNCHES = 2, 1


def _route(shapes, variant, want):
    assert [r["route"] for r in lm.plan_routes(shapes, variant)] == [want] * len(shapes)


# Sets of whole steps: full and ragged rows and rounds of 64 columns, each register
# size (8, 16, 32 rows), wide and tall, the smallest and the largest.
WHOLE_SETS = {
    "edges": [(8, 64), (64, 8), (16, 1024), (1024, 16), (9, 65), (63, 7), (1, 64), (1, 1), (31, 513), (513, 31),
              (32, 1024), (1024, 32), (5, 512), (17, 1)],
    "many_32_rows": [(32, 2048), (2048, 32), (2047, 32), (29, 2048)] * 16,
    "many_16_rows": [(16, 4096), (4096, 16), (15, 4369), (4097, 9)] * 16,
    "many_long": [(3, 4500), (5000, 2), (7, 4999), (8, 8192)] * 24 + [(16, 1024)],
    "many_longest": [(1, 65536), (65536, 1)] * 32,
}


@pytest.mark.parametrize("name", sorted(WHOLE_SETS))
@pytest.mark.parametrize("variant,ns_steps", [("malt", 5), ("malter", 2), ("malter", 9)])
def test_whole_steps_against_the_oracle(name, variant, ns_steps):
    # Only the final rounding of O to bf16 (2^-9 per entry at most) is left: 4e-3
    # covers it in norm, in O and in the update.
    shapes = WHOLE_SETS[name]
    _route(shapes, variant, WHOLE_STEP)
    keep = list(range(len(shapes))) if name == "edges" else [0, 1, 2, 3, len(shapes) - 1]
    say(f"[short] whole steps {name} {len(shapes)} matrices {variant} ns_steps={ns_steps} x2")
    W0 = [wl.weight(82, i, s) for i, s in enumerate(shapes)]
    grads = [[wl.grad(82, t, i, s, "row_loguniform") for i, s in enumerate(shapes)] for t in (1, 2)]
    hp = dict(lr=1e-2, ns_steps=ns_steps)
    g = run_gpu(shapes, variant, W0, grads, hp, collect=keep)
    o = run_oracle(shapes, variant, W0, grads, hp, collect=keep)
    say(f"[short] whole steps {name} worst {compare(g, o, variant, tol_ns=4e-3, label=name)}")


# By route.  Whole steps: wide, tall, full, ragged, square; three launches: one and
# several Gram chunks.
RANK_SETS = {WHOLE_STEP: [(16, 1024), (1024, 16), (32, 1024), (9, 9), (513, 31)],
             THREE_LAUNCHES: [(16, 4097), (40000, 20), (32, 2048), (9, 9)]}
QUINTIC, CUBIC = (3.4445, -4.7750, 2.0315), (1.5, -0.5, 0.0)


def _low_rank(kind, shape, seed):
    """A gradient of known rank: (G, rank)."""
    rng = np.random.default_rng(seed)
    m, n = shape
    if kind == "constant":
        return np.full(shape, 1e-2, np.float32), 1
    if kind == "repeated":   # rows (columns) in equal pairs and more
        k = (min(shape) + 3) // 4
        base = rng.standard_normal((k, max(shape))) * 1e-2
        g = base[np.arange(min(shape)) % k]
        return np.ascontiguousarray(g if m <= n else g.T).astype(np.float32), k
    r = {"rank1": 1, "rank8": min(8, min(shape))}[kind]
    return (rng.standard_normal((m, r)) @ rng.standard_normal((r, n)) * 1e-2).astype(np.float32), r


@pytest.mark.parametrize("abc,sup", [(QUINTIC, 1.2024), (CUBIC, 1.0)])
@pytest.mark.parametrize("ns_steps", [5, 8, 9, 12, 24, 64])
@pytest.mark.parametrize("route", sorted(RANK_SETS))
def test_low_rank_short_sides_stay_bounded(route, ns_steps, abc, sup):
    # Newton-Schulz maps every singular value of the normalised M~ into [0, sup]
    # at any count (the largest value of the scalar iteration from [0, 1]), so
    # the spectral norm of O exceeds sup by its final rounding only, at most 2^-9
    # ||O||_F <= 2^-9 sup sqrt(32); float32 noise in the null space stays inside
    # the same interval.  On the range of the gradient O is the oracle's up to
    # that rounding (in emulation the iteration itself adds 7e-8).
    kinds = ("constant", "repeated", "rank1", "rank8")
    shapes = [s for s in RANK_SETS[route] for _ in kinds]
    _route(shapes, "malter", route)
    say(f"[short] low-rank {kinds} x {RANK_SETS[route]} ns_steps={ns_steps} abc={abc}")
    made = [_low_rank(kinds[i % len(kinds)], s, 100 + i) for i, s in enumerate(shapes)]
    W0 = [wl.weight(84, i, s) for i, s in enumerate(shapes)]
    hp = dict(lr=1e-2, ns_steps=ns_steps, ns_a=abc[0], ns_b=abc[1], ns_c=abc[2])
    grads = [[g for g, _ in made]]
    st = run_gpu(shapes, "malter", W0, grads, hp)[0]
    orc = run_oracle(shapes, "malter", W0, grads, hp)[0]["inter"]
    worst = 0.0
    for k, s in enumerate(shapes):
        where = f"{kinds[k % len(kinds)]} {s}"
        assert np.isfinite(st.W[k]).all() and np.isfinite(st.O[k]).all(), where
        assert np.linalg.norm(st.O[k], 2) <= sup * (1 + 2.0 ** -9 * np.sqrt(32)) + 1e-6, where
        Mt = orc[k].M_tilde
        if s[0] > s[1]:
            Mt = Mt.T
        U = np.linalg.svd(Mt, full_matrices=False)[0][:, :made[k][1]]
        part = lambda O: U.T @ (O.T if s[0] > s[1] else O)
        # On the range alone: the rounding of the whole O, seen through U.
        err = rel_fro(part(st.O[k]), part(orc[k].O))
        lim = 4e-3 * max(1.0, np.linalg.norm(st.O[k]) / np.linalg.norm(part(orc[k].O)))
        worst = max(worst, err / lim)
        assert err <= lim, f"{where}: rank-{made[k][1]} part of O rel err {err:.3e} > {lim:.1e}"
    say(f"[short] low-rank ns_steps={ns_steps} worst error / bound {worst:.3f}")


# Entries of one magnitude that is not a power of two: float32 partial sums lose
# the same way at every addition, so their error does not average out.
SUM_SHAPES = [(1, 65536), (65536, 1), (1, 4096), (4096, 1), (16, 4096), (4096, 16), (3, 4095), (31, 2111), (2, 100000)]


@pytest.mark.parametrize("shapes,keep,route", [
    (SUM_SHAPES, range(len(SUM_SHAPES)), THREE_LAUNCHES),
    # whole steps of 65536 columns, and of 16 and 32 rows, beside many others
    ([(1, 65536), (65536, 1)] * 32, (0, 1, 63), WHOLE_STEP),
    ([(16, 4096), (4096, 15), (32, 2048), (2048, 31)] * 24, (0, 1, 2, 3), WHOLE_STEP)])
def test_long_side_sums_keep_float64(shapes, keep, route):
    # l and r after one step are (1 - mu2) times sums of G^2 over a long and over
    # a short side.  Rounding: each square (2^-24), the long sums in float64 from
    # float32 partials over at most 256 columns, 32 rows or, in whole steps past
    # 16 rows, 32 columns (sums of equal values: at most 3 additions round, 2^-24 each), the
    # stored float32 (2^-24): 5 * 2^-24 = 3.0e-7 at most.  Float32 over a whole
    # side of 65536 was 1.2e-6 off.
    say(f"[short] sums of equal squares over {shapes[:9]}, {len(shapes)} matrices")
    _route(shapes, "malt", route)
    keep = list(keep)
    W0 = [wl.weight(83, i, s) for i, s in enumerate(shapes)]
    rng = np.random.default_rng(83)
    grads = [[(rng.integers(0, 2, s) * 2 - 1).astype(np.float32) * np.float32(0.0123) for s in shapes]]
    for variant in ("malt", "malter"):
        g = run_gpu(shapes, variant, W0, grads, dict(lr=1e-2), collect=keep)[0]
        o = run_oracle(shapes, variant, W0, grads, dict(lr=1e-2), collect=keep)[0]
        for k, i in enumerate(keep):
            s = shapes[i]
            err = rel_fro(g.l[k], o["l"][k]) if s[0] <= s[1] else rel_fro(g.r[k], o["r"][k])
            say(f"[short] {variant} {s}: long-side sum rel err {err:.2e}")
            assert err <= 3.0e-7, f"{variant} {s}: {err:.2e}"


@pytest.mark.parametrize("variant,ns_steps", [("malt", 5), ("malter", 2), ("malter", 12)])
def test_gradients_overlapping_another_matrix_parameter(variant, ns_steps):
    # Accepted, and every gradient is read before any W is written: the gradient of
    # a whole-step matrix and of a matrix on the matrix cores that lie in the W of
    # whole-step ones.  The same steps with copies of those gradients give the same
    # M (up to the contraction of one expression), l, r and nu (sums in another
    # order: 3e-7) and update (O's last bf16 bit may turn: 4e-3).  A gradient read
    # after its W had been written would be off by about 1e-2, and M with it.
    import torch
    shapes = [(16, 1024), (1024, 16), (256, 512), (16, 1024), (9, 65)]
    assert [r["route"] for r in lm.plan_routes(shapes, variant)] == [2, 2, 0, 2, 2]
    say(f"[short] overlapping gradients {shapes} {variant} ns_steps={ns_steps} x2, then apart")
    hp = lm.make_hparams(lr=1e-2, ns_steps=ns_steps, weight_decay=0.1)
    results = []
    for overlap in (True, False):
        gen = torch.Generator(device="cuda").manual_seed(5)
        flat = torch.randn(200000, device="cuda", generator=gen) * 0.02
        W = [torch.randn(s, device="cuda", generator=gen) * 0.02 for s in shapes]
        W[1] = flat[:16384].view(1024, 16)           # G[2] begins inside it
        G = [torch.randn(s, device="cuda", generator=gen) * 0.01 for s in shapes]
        plan = lm.Plan(shapes, variant)
        steps = []
        for t in range(3):
            g = list(G)
            if t < 2:
                g[0], g[2] = W[3], flat[8192:8192 + 256 * 512].view(256, 512)
                if not overlap:
                    g[0], g[2] = g[0].clone(), g[2].clone()
            before = [w.clone() for w in W]
            plan.step(W, g, hp)
            torch.cuda.synchronize()
            views = [plan.state_views(i) for i in range(len(shapes))]
            steps.append(([w - b for w, b in zip(W, before)], [[x.clone() for x in v if x is not None] for v in views]))
        results.append(steps)
        plan.close()
    err = lambda x, y: float((x.double() - y.double()).norm() / y.double().norm())
    for t, ((da, sa), (db, sb)) in enumerate(zip(*results)):
        for i, s in enumerate(shapes):
            where = f"step {t + 1} matrix {i} {s}"
            # Later gradients are the W that the first step left: 4e-3 of an update
            # of about 1e-2 |W|.
            tol = 1e-6 if t == 0 else 1e-4
            worst = max(err(x, y) for x, y in zip(sa[i], sb[i]))
            say(f"[short] overlap {where}: state {worst:.2e} update {err(da[i], db[i]):.2e}")
            assert worst <= tol, f"{where}: state {worst:.2e}"
            assert err(da[i], db[i]) <= 4e-3, f"{where}: update {err(da[i], db[i]):.2e}"
