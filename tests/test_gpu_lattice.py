"""Sorted binary64 frames whose distances lie on bin edges: points of a grid,
several of them coincident or whole cells away, the bin a fraction of the grid's
spacing, so that most passes leave their pairs to the settling pass and the
canonical sequence decides some of each. Bit for bit against the oracle, in one
LDS histogram, in bin windows and with global atomics, and over species sizes
that leave a last single j and partial slices."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

SKEW = np.array([[16.0, 0, 0], [4.0, 16.0, 0], [-4.0, 4.0, 16.0]])
# box type, rows, cut-off (grid spacing 1/2)
KINDS = {"ortho": (workloads.BOX_ORTHO, workloads.ortho_box(16.0, 16.0, 16.0), 7.0),
         "beyond": (workloads.BOX_ORTHO, workloads.ortho_box(16.0, 20.0, 24.0), 11.0),
         "triclinic": (workloads.BOX_TRICLINIC, SKEW, 6.0),
         "search": (workloads.BOX_TRICLINIC, SKEW, 12.0)}
SIZES = [[65_537], [40_000, 25_413, 190, 1]]


@pytest.fixture(scope="module")
def ctx():
    import paper_1808_01478_amd as dh
    c = dh.Context(0)
    yield c
    c.set_config(None)
    c.close()


def grid_frame(kind, sizes, n_bins):
    box_type, rows, r_max = KINDS[kind]
    n = sum(sizes)
    rng = np.random.Generator(np.random.PCG64(n + len(kind)))
    cells = np.rint(np.diag(rows) * 2).astype(int)
    f = np.stack([rng.integers(-m // 4, 2 * m, n) / m for m in cells], axis=1)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return workloads.Frame(np.ascontiguousarray(workloads.rows_combine(f, rows)), offs, box_type,
                           rows, r_max, n_bins, f"grid-{kind}-{len(sizes)}")


@pytest.mark.parametrize("k", range(len(SIZES)))
@pytest.mark.parametrize("kind", list(KINDS))
def test_distances_on_bin_edges(ctx, kind, k):
    for per, shapes in ((64, [None, [4, 1, 128, 1, 0, 4, 1024, 1]]),
                        (8192, [[4, 1, 128, 1, 0, 4, 0, 0]])):
        fr = grid_frame(kind, SIZES[k], int(KINDS[kind][2] * per))
        ref = oracle.frame_histogram(fr)
        for shape in shapes:
            print(f"\n[case] {fr.name} bins={fr.n_bins} shape={shape}", flush=True)
            ctx.set_config(shape)
            h, oor = run_gpu(ctx, fr, 1)
            assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
    ctx.set_config(None)


@pytest.mark.parametrize("points", ["far", "coincident"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_groups_without_a_bound_and_coincident_points(ctx, kind, points):
    """A third of the points 2^26 to 2^40 cells away, where no rounding bound
    decides anything and whole groups are taken from the input, or all at a few
    places, where every distance of a pair is 0 or one of a few."""
    box_type, rows, r_max = KINDS[kind]
    n = 65_700
    rng = np.random.Generator(np.random.PCG64(n))
    f = rng.uniform(0.0, 1.0, size=(n, 3))
    if points == "far":
        f[rng.permutation(n)[:n // 3]] += 2.0 ** rng.integers(26, 41, size=(n // 3, 1))
    else:
        f = f[rng.integers(0, 5, n)]
    fr = workloads.Frame(np.ascontiguousarray(workloads.rows_combine(f, rows)),
                         np.array([0, 40_000, n], np.int64), box_type, rows, r_max, 700, points)
    print(f"\n[case] {points} {kind}", flush=True)
    ref = oracle.frame_histogram(fr)
    h, oor = run_gpu(ctx, fr, 1)
    assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
