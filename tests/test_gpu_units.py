"""Work units of unsorted frames at their edges: slices of 64 R particles with
one lane more or less, j-pieces with remainders against the four j in flight,
diagonal units, species of one particle, items of a single unit. binary64 bit
for bit against the oracle, binary32 within the edge-pair bound."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import fp32_bound_violations, oor_bound_violations, run_gpu

pytestmark = pytest.mark.gpu

SKEW = np.array([[10.0, 0, 0], [3.0, 9.5, 0], [-2.0, 3.5, 9.0]])
SIZES = [[2], [3, 1], [63], [64], [65, 5], [255], [256, 256], [257, 31], [511, 513], [1023],
         [1025, 7, 33], [4097]]
KINDS = {"none": (workloads.BOX_NONE, None, None), "cube": (workloads.BOX_ORTHO,
                                                             workloads.ortho_box(9, 9, 9), 4.5),
         "ortho": (workloads.BOX_ORTHO, workloads.ortho_box(9, 10, 8), 4.0),
         "triclinic": (workloads.BOX_TRICLINIC, SKEW, None),
         "search": (workloads.BOX_TRICLINIC, SKEW, 0.8 * workloads.min_width(SKEW))}


@pytest.fixture(scope="module")
def ctx():
    import paper_1808_01478_amd as dh
    c = dh.Context(0)
    yield c
    c.set_config(None)
    c.close()


@pytest.mark.parametrize("shape", [None, [8, 1, 128, 1, 0, 1, 256, 60], [4, 1, 256, 0, 0, 16, 1024, 0]],
                         ids=["default", "r8", "r4-1024"])
@pytest.mark.parametrize("kind", list(KINDS))
def test_unit_edges(ctx, kind, shape):
    box_type, box, r_max = KINDS[kind]
    ctx.set_config(shape)
    for k, sizes in enumerate(SIZES):
        fr = workloads.random_frame(900 + k, sizes, box_type, r_max=r_max, n_bins=150, box=box)
        print(f"\n[case] units {kind} {sizes} shape={shape}", flush=True)
        w = oracle.edge_window(fr.coords, fr.box, fr.r_max)
        ref = oracle.frame_histogram(fr, edge_window=w)
        h, oor = run_gpu(ctx, fr, 1)
        assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range), sizes
        h, oor = run_gpu(ctx, fr, 0)
        bad = fp32_bound_violations(h, ref.hist, ref.edges)
        bad += oor_bound_violations(oor, ref.out_of_range, ref.edges)
        assert not bad, (sizes, bad[:3])
    ctx.set_config(None)


@pytest.mark.parametrize("n_bins", [1, 37, 4096, (1 << 20) - 3, (1 << 20) - 2, (1 << 20) + 5])
@pytest.mark.parametrize("box_type", [workloads.BOX_NONE, workloads.BOX_ORTHO])
def test_binary64_bin_edges(ctx, box_type, n_bins):
    """binary64 bins at their edges: points of a lattice (coincident ones
    among them) whose distances hit whole bins exactly, and bin counts on both
    sides of the limit of the binary32 root."""
    rng = np.random.Generator(np.random.PCG64(n_bins))
    x = rng.integers(0, 32, size=(1500, 3)) / 4.0
    box = workloads.ortho_box(8, 8, 8) if box_type == workloads.BOX_ORTHO else None
    offs = np.array([0, 900, 1500], np.int64)
    for r_max in (n_bins / 8.0 if n_bins < 100 else 8.0, 6.7):
        fr = workloads.Frame(np.ascontiguousarray(x), offs, box_type, box, r_max, n_bins, "lattice")
        print(f"\n[case] bin edges box={box_type} bins={n_bins} r_max={r_max}", flush=True)
        ref = oracle.frame_histogram(fr)
        h, oor = run_gpu(ctx, fr, 1)
        assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
