"""Work lists under a memory budget: items are a matter of speed, so a context
whose budget has little room beside the staged points cuts its work coarser
instead of refusing it. The budgets leave 8 to 100 bytes a point beside the
staged copy and the sort keys; counts equal those of a context without one."""
import numpy as np
import pytest

import workloads
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu

CELL = np.array([[50.0, 0, 0], [15.0, 48.0, 0], [10.0, 12.0, 45.0]])
# box type, rows, species sizes, cut-off, bins, precision, bytes of budget
CALLS = {
    "cube-5k": (workloads.BOX_ORTHO, workloads.ortho_box(40, 40, 40), [5000], 19.0, 1000, 0,
                86_000),
    "cube-20k-f64": (workloads.BOX_ORTHO, workloads.ortho_box(40, 40, 40), [10_000] * 2, 19.0, 1000,
                     1, 692_000),
    "cube-20k-many": (workloads.BOX_ORTHO, workloads.ortho_box(40, 40, 40), [312] * 64, 19.0, 100,
                      0, 471_000),
    "search-60k": (workloads.BOX_TRICLINIC, CELL, [20_000] * 3, 36.0, 4000, 0, 1_103_000),
    "sorted-100k": (workloads.BOX_TRICLINIC, CELL, [33_333] * 3, 20.0, 20_000, 0, 4_323_000),
    "sorted-100k-f64": (workloads.BOX_TRICLINIC, CELL, [33_333] * 3, 20.0, 20_000, 1, 4_334_000),
}


def call_frame(name):
    box_type, rows, sizes, r_max, n_bins, _, _ = CALLS[name]
    rng = np.random.Generator(np.random.PCG64(len(name)))
    x = workloads.rows_combine(rng.uniform(0.0, 1.0, size=(sum(sizes), 3)), rows)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    return workloads.Frame(np.ascontiguousarray(x), offs, box_type, rows, r_max, n_bins, name)


@pytest.mark.parametrize("name", list(CALLS))
def test_small_budget_cuts_coarser(name):
    import paper_1808_01478_amd as dh
    fr = call_frame(name)
    precision, budget = CALLS[name][5:]
    print(f"\n[case] budget {budget} {name}", flush=True)
    with dh.Context(0) as free:
        ref, ref_oor = run_gpu(free, fr, precision)
        plain = free.last_config()["items"]
    with dh.Context(0, hbm_budget_bytes=budget) as ctx:
        for _ in range(2):
            h, oor = run_gpu(ctx, fr, precision)
            assert np.array_equal(h, ref) and np.array_equal(oor, ref_oor)
        assert 0 < ctx.last_config()["items"] < plain


def test_small_budget_of_a_batch():
    import torch
    import paper_1808_01478_amd as dh
    dev = torch.device("cuda")
    frames, refs = [], []
    with dh.Context(0) as free:
        for k in range(6):
            kind = ("cube-5k", "sorted-100k", "search-60k")[k % 3]
            box_type, rows = CALLS[kind][:2]
            n = 30_000 + 25_000 * k
            rng = np.random.Generator(np.random.PCG64(k))
            x = np.ascontiguousarray(workloads.rows_combine(rng.uniform(0.0, 1.0, (n, 3)), rows))
            fr = workloads.Frame(x, np.array([0, n // 2, n], np.int64), box_type, rows, 19.0, 2000,
                                 "batch")
            refs.append(run_gpu(free, fr, 0))
            frames.append({"d_coords": torch.from_numpy(x).to(dev), "offsets": fr.offsets,
                           "box_type": box_type, "box": rows, "r_max": 19.0, "n_bins": 2000,
                           "d_out": torch.empty((3, 2000), dtype=torch.int64, device=dev),
                           "d_out_of_range": torch.empty((3,), dtype=torch.int64, device=dev)})
    staged = sum(len(f["d_coords"]) * (32 if f["box_type"] == workloads.BOX_TRICLINIC and
                                       len(f["d_coords"]) >= 1 << 16 else 16) for f in frames)
    print("\n[case] budget of a batch", flush=True)
    with dh.Context(0, hbm_budget_bytes=staged + (8 << 18) + (60 << 10)) as ctx:
        b = dh.Batch(ctx, frames, 0)
        b.launch()
        torch.cuda.synchronize()
        for f, (h, oor) in zip(frames, refs):
            assert np.array_equal(f["d_out"].cpu().numpy().view(np.uint64), h)
            assert np.array_equal(f["d_out_of_range"].cpu().numpy().view(np.uint64), oor)
        b.close()
