"""The neighbour-image search without its table (every octant's
images are the seven towards the vector) and with it (longer lists): random
points, and points of a lattice of eighths of the cell, whose reduced vectors
lie on the octants' faces. binary64 bit for bit against the oracle, which
searches all 27 images of every pair, binary32 within the edge-pair bound."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import fp32_bound_violations, oor_bound_violations, run_gpu

pytestmark = pytest.mark.gpu

CELLS = {"orthogonal": (np.diag([9.0, 10.0, 11.0]), True),
         "skew": (np.array([[10.0, 0, 0], [3.0, 9.5, 0], [2.0, 2.4, 9.0]]), True),
         "skew-back": (np.array([[10.0, 0, 0], [-3.0, 9.5, 0], [2.0, -2.4, 9.0]]), True),
         "face-centred": (np.array([[8.0, 0, 0], [4.0, 6.9, 0], [4.0, 2.3, 6.5]]), False)}


def seven(box):
    """Whether every octant lists only images shifted against its signs."""
    import paper_1808_01478_amd as dh
    lists, _, full = dh.search_images(box)
    if full:
        return False
    for o, images in enumerate(lists):
        for m in images:
            n = (m // 9 - 1, m // 3 % 3 - 1, m % 3 - 1)
            if any(v != 0 and (v > 0) != bool(o >> c & 1) for c, v in enumerate(n)):
                return False
    return True


@pytest.fixture(scope="module")
def ctx():
    import paper_1808_01478_amd as dh
    c = dh.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("points", ["random", "eighths"])
@pytest.mark.parametrize("name", sorted(CELLS))
def test_search_images(ctx, name, points):
    box, plain = CELLS[name]
    assert seven(box) == plain
    rng = np.random.Generator(np.random.PCG64(5))
    f = rng.uniform(-0.2, 1.2, size=(1300, 3))
    if points == "eighths":
        f = rng.integers(0, 8, size=f.shape) / 8.0
    x = np.ascontiguousarray(workloads.rows_combine(f, box))
    for r in (0.55, 0.97):
        fr = workloads.Frame(x, np.array([0, 700, 1300], np.int64), workloads.BOX_TRICLINIC, box,
                             r * workloads.min_width(box), 211, name)
        print(f"\n[case] search {name} {points} r={r}", flush=True)
        w = oracle.edge_window(fr.coords, fr.box, fr.r_max)
        ref = oracle.frame_histogram(fr, edge_window=w)
        h, oor = run_gpu(ctx, fr, 1)
        assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
        h, oor = run_gpu(ctx, fr, 0)
        bad = fp32_bound_violations(h, ref.hist, ref.edges)
        bad += oor_bound_violations(oor, ref.out_of_range, ref.edges)
        assert not bad, bad[:3]


@pytest.mark.parametrize("points", ["random", "eighths", "outliers"])
@pytest.mark.parametrize("name", sorted(CELLS))
def test_searched_pairs_do_not_depend_on_the_staging(ctx, name, points):
    """The pairs the search is defined for, of a frame staged in spatial order
    and of the same frame in a context with a memory budget, which is not; the
    counts as well. Outliers: coordinates that are not finite or too large for
    any bound, whose groups take the canonical sequence throughout."""
    import paper_1808_01478_amd as dh
    box, _ = CELLS[name]
    n = 66_003
    rng = np.random.Generator(np.random.PCG64(n))
    f = rng.uniform(-0.2, 1.2, size=(n, 3))
    if points == "eighths":
        f = rng.integers(0, 40, size=f.shape) / 40.0
    x = np.ascontiguousarray(workloads.rows_combine(f, box))
    if points == "outliers":
        x[rng.integers(0, n, 40), rng.integers(0, 3, 40)] = rng.choice(
            [np.nan, np.inf, -np.inf, 1e18, -3e12, 1e308], 40)
    fr = workloads.Frame(x, np.array([0, 50_001, n], np.int64), workloads.BOX_TRICLINIC, box,
                         0.7 * workloads.min_width(box), 300, name)
    print(f"\n[case] searched pairs {name} {points}", flush=True)
    h, oor = run_gpu(ctx, fr, 1)
    searched, images = ctx.searched_pairs(), ctx.searched_images()
    with dh.Context(0, hbm_budget_bytes=1 << 30) as plain:
        g, oor_g = run_gpu(plain, fr, 1)
        want = plain.searched_pairs()
    assert np.array_equal(h, g) and np.array_equal(oor, oor_g)
    assert 0 < want < fr.total_pairs() and searched == want, (searched, want)
    assert images > 0


@pytest.mark.parametrize("precision", [0, 1])
def test_searched_pairs_of_many_small_items(ctx, precision):
    """The counts of searched pairs add up over waves, items and species: 32
    species against the same points as one."""
    box, _ = CELLS["skew"]
    rng = np.random.Generator(np.random.PCG64(9))
    x = np.ascontiguousarray(workloads.rows_combine(rng.uniform(0, 1, size=(1000, 3)), box))
    got = []
    for k in (32, 1):
        offs = np.linspace(0, 1000, k + 1).astype(np.int64)
        fr = workloads.Frame(x, offs, workloads.BOX_TRICLINIC, box, 0.8 * workloads.min_width(box),
                             128, f"{k} species")
        print(f"\n[case] searched pairs, {k} species", flush=True)
        h, _ = run_gpu(ctx, fr, precision)
        got.append((ctx.searched_pairs(), h.sum()))
        assert 7 * got[-1][0] <= ctx.searched_images() <= 27 * got[-1][0]
    assert got[0] == got[1] and got[0][0] > 0


@pytest.mark.parametrize("n_bins", [60_000, 800_000])
def test_searched_pairs_of_wide_histograms(ctx, n_bins):
    """Wide histograms: bin windows in both stagings, or windows of the sorted
    frame against one pass of atomics."""
    import paper_1808_01478_amd as dh
    box, _ = CELLS["skew"]
    rng = np.random.Generator(np.random.PCG64(11))
    x = np.ascontiguousarray(workloads.rows_combine(rng.uniform(0, 1, size=(66_000, 3)), box))
    fr = workloads.Frame(x, np.array([0, 66_000], np.int64), workloads.BOX_TRICLINIC, box,
                         0.7 * workloads.min_width(box), n_bins, "wide search")
    print(f"\n[case] searched pairs, {n_bins} bins", flush=True)
    h, oor = run_gpu(ctx, fr, 1)
    searched = ctx.searched_pairs()
    with dh.Context(0, hbm_budget_bytes=1 << 30) as plain:
        g, oor_g = run_gpu(plain, fr, 1)
        assert searched == plain.searched_pairs()
    assert np.array_equal(h, g) and np.array_equal(oor, oor_g)
