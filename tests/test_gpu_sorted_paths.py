"""Sorted binary64 frames through the other entry points: the allocation-free
call, a batch (launched, and replayed as a graph), the server, the host call and
the trajectory engine give the counts of the single-frame call, with and
without image search, for points on cell faces and coordinates that are not
finite (device buffers only: host entry points refuse those)."""
import numpy as np
import pytest

import workloads
from gpu_util import run_gpu
from test_gpu_faces import KINDS, face_frame

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", list(KINDS))
def test_every_entry_point(kind, tmp_path):
    import torch
    import paper_1808_01478_amd as dh
    from paper_1808_01478_amd import trajfile
    fr = face_frame(kind)
    print(f"\n[case] entry points {fr.name}", flush=True)
    with dh.Context(0) as ctx:
        ref, ref_oor = run_gpu(ctx, fr, 1)
        args = (fr.coords, fr.offsets, fr.box_type, fr.box, fr.r_max, fr.n_bins)
        assert np.array_equal(dh.histo(*args, dh.FP64), ref)
        path, res = str(tmp_path / "t.dhtraj"), str(tmp_path / "r.dhres")
        trajfile.write_trajectory(path, [fr.coords] * 2, fr.box_type, [fr.box] * 2)
        with dh.Trajectory(path) as t:
            assert t.histo(ctx, fr.offsets, fr.r_max, fr.n_bins, 1, res, interval=1) == 2
        _, hist, oor, _ = trajfile.read_results(res, fr.n_hist)
        for k in range(2):
            assert np.array_equal(hist[k], ref) and np.array_equal(oor[k], ref_oor)
        with dh.Server(0, hbm_budget_bytes=1 << 30, max_inflight=2) as srv:
            ids = [srv.submit(*args, 1) for _ in range(2)]
            for i in ids:
                h, o, _ = srv.wait(i)
                assert np.array_equal(h, ref) and np.array_equal(o, ref_oor)
        # device buffers, with a few coordinates that are not finite
        x = fr.coords.copy()
        x[::5000, 1] = np.nan
        x[7::9000, 0] = np.inf
        odd = workloads.Frame(x, fr.offsets, fr.box_type, fr.box, fr.r_max, fr.n_bins, fr.name)
        for f in (fr, odd):
            ref, ref_oor = run_gpu(ctx, f, 1)
            assert np.array_equal(ref.sum(1) + ref_oor, np.array(f.hist_pairs(), np.uint64))
            dev = torch.device("cuda")
            d = torch.from_numpy(f.coords).to(dev)
            out = torch.full(ref.shape, -1, dtype=torch.int64, device=dev)
            oor = torch.full(ref_oor.shape, -1, dtype=torch.int64, device=dev)

            def same():
                torch.cuda.synchronize()
                assert np.array_equal(out.cpu().numpy().view(np.uint64), ref)
                assert np.array_equal(oor.cpu().numpy().view(np.uint64), ref_oor)
                out.fill_(-1)
                oor.fill_(-1)

            dh.histo_noalloc(d, f.offsets, f.box_type, f.box, f.r_max, f.n_bins, 1, out, oor)
            same()
            desc = {"d_coords": d, "offsets": f.offsets, "box_type": f.box_type, "box": f.box,
                    "r_max": f.r_max, "n_bins": f.n_bins, "d_out": out, "d_out_of_range": oor}
            for graph in (False, True):
                batch = dh.Batch(ctx, [desc], 1, graph=graph)
                for _ in range(3):
                    batch.launch()
                    same()
                batch.close()
