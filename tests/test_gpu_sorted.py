"""Spatially sorted frames: group pairs beyond the cut-off or outside a bin
window are skipped. Halving the cut-off and the bins together keeps the scale
and so every pair's bin, so the shorter histogram must be the start of the
longer one, bit for bit, in every accumulation mode; species sizes lie around
multiples of the 64-point groups and the 512-point units."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_util import fp32_bound_violations, oor_bound_violations, run_gpu

pytestmark = pytest.mark.gpu

SKEW = np.array([[10.0, 0, 0], [3.0, 9.5, 0], [-2.0, 3.5, 9.0]])
SIZES = [[65_536], [65_537, 63, 1, 513], [33_000, 32_600, 64], [511, 66_047]]


@pytest.fixture(scope="module")
def ctx():
    import paper_1808_01478_amd as dh
    c = dh.Context(0)
    yield c
    c.set_config(None)
    c.close()


def frame(sizes, box_type, clustered, r_frac, n_bins):
    n = sum(sizes)
    rng = np.random.Generator(np.random.PCG64(n + int(clustered)))
    rows = SKEW if box_type == workloads.BOX_TRICLINIC else workloads.ortho_box(9.0, 10.0, 11.0)
    u = rng.uniform(0.0, 1.0, size=(n, 3))
    if clustered:
        k = (3 * n) // 4
        u[:k] = rng.uniform(0.0, 1.0, (7, 3))[rng.integers(0, 7, k)] + rng.normal(0, 0.03, (k, 3))
        u = rng.permutation(u) + rng.integers(-2, 3, size=(n, 3))  # unwrapped
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return workloads.Frame(np.ascontiguousarray(workloads.rows_combine(u, rows)), offs, box_type,
                           rows, r_frac * workloads.min_width(rows), n_bins, f"sorted-{sizes}")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("box_type", [workloads.BOX_ORTHO, workloads.BOX_TRICLINIC])
@pytest.mark.parametrize("k", range(len(SIZES)))
def test_shorter_cutoff_is_a_prefix(ctx, k, box_type, clustered, precision):
    for n_bins, knobs in ((4096, None), (131_072, [4, 1, 256, 1, 0, 4, 0, 0]),
                          (2048, [8, 1, 128, 1, 0, 8, 256, 1])):
        print(f"\n[case] prefix {SIZES[k]} box={box_type} clustered={clustered} bins={n_bins} "
              f"prec={precision}", flush=True)
        ctx.set_config(knobs)
        full = frame(SIZES[k], box_type, clustered, 0.48, n_bins)
        ref, ref_oor = run_gpu(ctx, full, precision)
        pairs = np.array(full.hist_pairs(), np.uint64)
        assert np.array_equal(ref.sum(1) + ref_oor, pairs)
        for div in (2, 16):
            part = frame(SIZES[k], box_type, clustered, 0.48 / div, n_bins // div)
            h, oor = run_gpu(ctx, part, precision)
            assert np.array_equal(h, ref[:, :n_bins // div]), div
            assert np.array_equal(h.sum(1) + oor, pairs)
    ctx.set_config(None)


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("k", range(len(SIZES)))
def test_search_against_no_search(ctx, k, clustered):
    """binary64 image search of sorted frames: below half the cell the same
    scale needs no search, so the histograms must agree there; beyond it every
    pair is in a bin or out of range; bin windows and global atomics give the
    same counts, and a second species split only moves pairs between rows."""
    full = frame(SIZES[k], workloads.BOX_TRICLINIC, clustered, 0.8, 4096)
    print(f"\n[case] search {SIZES[k]} clustered={clustered}", flush=True)
    ctx.set_config(None)
    ref, ref_oor = run_gpu(ctx, full, 1)
    assert np.array_equal(ref.sum(1) + ref_oor, np.array(full.hist_pairs(), np.uint64))
    for div in (2, 8):
        part = frame(SIZES[k], workloads.BOX_TRICLINIC, clustered, 0.8 / div, 4096 // div)
        h, _ = run_gpu(ctx, part, 1)
        assert np.array_equal(h, ref[:, :4096 // div]), div
    one = workloads.Frame(full.coords, np.array([0, full.n], np.int64), full.box_type, full.box,
                          full.r_max, full.n_bins, "one species")
    h, _ = run_gpu(ctx, one, 1)
    assert np.array_equal(h[0], ref.sum(0))
    for knobs in ([4, 4, 128, 1, 0, 4, 1024, 0], [8, 1, 128, 0, 0, 16, 256, 1]):
        ctx.set_config(knobs)
        h, oor = run_gpu(ctx, full, 1)
        assert np.array_equal(h, ref) and np.array_equal(oor, ref_oor), knobs
    ctx.set_config(None)


def test_search_oracle(ctx):
    fr = frame([66_000, 300], workloads.BOX_TRICLINIC, True, 1.0, 500)
    print(f"\n[case] search oracle {fr.name}", flush=True)
    ref = oracle.frame_histogram(fr)
    h, oor = run_gpu(ctx, fr, 1)
    assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)


@pytest.mark.parametrize("box_type", [workloads.BOX_ORTHO, workloads.BOX_TRICLINIC])
def test_oracle(ctx, box_type):
    fr = frame(SIZES[1], box_type, True, 0.3, 700)
    print(f"\n[case] oracle {fr.name} box={box_type}", flush=True)
    w = oracle.edge_window(fr.coords, fr.box, fr.r_max)
    ref = oracle.frame_histogram(fr, edge_window=w)
    h, oor = run_gpu(ctx, fr, 1)
    assert np.array_equal(h, ref.hist) and np.array_equal(oor, ref.out_of_range)
    h, oor = run_gpu(ctx, fr, 0)
    bad = fp32_bound_violations(h, ref.hist, ref.edges)
    bad += oor_bound_violations(oor, ref.out_of_range, ref.edges)
    assert not bad, bad[:3]


@pytest.mark.parametrize("precision,n_bins", [(1, 800_000), (1, (1 << 20) - 3), (0, 2_600_000)])
def test_wide_windows_against_atomics(ctx, precision, n_bins):
    """Wide histograms of sorted frames run as bin windows, whose skipped group
    pairs must not lose a count: equal to one pass of global atomics."""
    fr = frame(SIZES[1], workloads.BOX_TRICLINIC, True, 0.3, n_bins)
    print(f"\n[case] wide {fr.name} precision={precision} bins={n_bins}", flush=True)
    ctx.set_config(None)
    h, oor = run_gpu(ctx, fr, precision)
    assert ctx.last_config()["mode"] == 1
    ctx.set_config([4, 1, 128 if precision else 256, 1, 0, 4, 0, 1])
    g, oor_g = run_gpu(ctx, fr, precision)
    assert ctx.last_config()["mode"] == 2
    ctx.set_config(None)
    assert np.array_equal(h, g) and np.array_equal(oor, oor_g)
