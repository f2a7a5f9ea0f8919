"""Points on the faces of the cell in frames that are staged in spatial order:
coordinates a rounding error to either side of a face, on it, and whole cells
away, where the cell of a point and its place in it must come from one
decision. binary64 bit for bit against the oracle, binary32 within the
edge-pair bound."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import fp32_bound_violations, oor_bound_violations, run_gpu

pytestmark = pytest.mark.gpu

SKEW = np.array([[10.0, 0, 0], [3.0, 9.5, 0], [-2.0, 3.5, 9.0]])
ORTHO = workloads.ortho_box(9.0, 10.0, 11.0)
SIZES = [65_500, 101]
# box type, rows, cut-off in smallest widths
KINDS = {"ortho": (workloads.BOX_ORTHO, ORTHO, 0.45),
         "triclinic": (workloads.BOX_TRICLINIC, SKEW, 0.45),
         "search": (workloads.BOX_TRICLINIC, SKEW, 0.8)}


@pytest.fixture(scope="module")
def ctx():
    import paper_1808_01478_amd as dh
    c = dh.Context(0)
    yield c
    c.close()


def face_frame(kind, n_bins=600):
    box_type, rows, r = KINDS[kind]
    n = sum(SIZES)
    rng = np.random.Generator(np.random.PCG64(n))
    f = rng.uniform(0.0, 1.0, size=(n, 3))
    # a third of the points on a face of one axis (as products with the rows:
    # exact zeros and rounding noise of either sign)
    near = [0.0, 1.0, -1.0, 2.0, -1e-17, -1e-16, 1e-16, 1.0 - 2.0 ** -53, 1.0 + 2.0 ** -52]
    for axis in range(3):
        f[axis:n // 3:3, axis] = rng.choice(near, size=len(f[axis:n // 3:3]))
    x = workloads.rows_combine(f, rows)
    # and as coordinates: tiny negative ones and the neighbours of an edge
    for axis in range(3):
        edge = rows[axis, axis]
        values = [-1e-18, -1e-16, -1e-15, -0.0, edge, np.nextafter(edge, 0), np.nextafter(edge, 99),
                  -edge]
        at = rng.integers(0, n, n // 20)
        x[at, axis] = rng.choice(values, size=len(at))
    offs = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int64)
    return workloads.Frame(np.ascontiguousarray(x), offs, box_type, rows,
                           r * workloads.min_width(rows), n_bins, f"faces-{kind}")


@pytest.mark.parametrize("kind", list(KINDS))
def test_points_on_cell_faces(ctx, kind):
    fr = face_frame(kind)
    print(f"\n[case] {fr.name} n={fr.n}", flush=True)
    w = oracle.edge_window(fr.coords, fr.box, fr.r_max)
    ref = oracle.frame_histogram(fr, edge_window=w)
    h, oor = run_gpu(ctx, fr, 1)
    assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
    h, oor = run_gpu(ctx, fr, 0)
    bad = fp32_bound_violations(h, ref.hist, ref.edges)
    bad += oor_bound_violations(oor, ref.out_of_range, ref.edges)
    assert not bad, bad[:3]


@pytest.mark.parametrize("kind", list(KINDS))
def test_scale_of_the_cell_does_not_change_binary64_counts(ctx, kind):
    """Lengths times a power of two leave every step of the canonical sequence
    exact, so the counts: from cells whose squares underflow in binary32 to
    cells whose squares overflow there."""
    fr = face_frame(kind)
    ref, ref_oor = run_gpu(ctx, fr, 1)
    for k in (-300, -71, -45, -38, 55, 62, 300):
        print(f"\n[case] {fr.name} scale 2^{k}", flush=True)
        s = 2.0 ** k
        part = workloads.Frame(fr.coords * s, fr.offsets, fr.box_type, fr.box * s, fr.r_max * s,
                               fr.n_bins, fr.name)
        h, oor = run_gpu(ctx, part, 1)
        assert np.array_equal(h, ref) and np.array_equal(oor, ref_oor), k


def test_binary32_counts_of_extreme_cells(ctx):
    """binary32 lengths times a power of two: exact as well while the squares of
    the pairs' own differences stay normal numbers, so the counts do not change
    where the groups' bounds stop deciding."""
    fr = face_frame("triclinic")
    ref, ref_oor = run_gpu(ctx, fr, 0)
    for k in (-50, -46, -44, 40, 56):
        print(f"\n[case] {fr.name} binary32, scale 2^{k}", flush=True)
        s = 2.0 ** k
        part = workloads.Frame(fr.coords * s, fr.offsets, fr.box_type, fr.box * s, fr.r_max * s,
                               fr.n_bins, fr.name)
        h, oor = run_gpu(ctx, part, 0)
        assert np.array_equal(h, ref) and np.array_equal(oor, ref_oor), k
