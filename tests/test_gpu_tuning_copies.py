"""Tuning caches written when a workgroup counted into several copies of its
histogram: the copies of a cached shape reserve no LDS (which would cost
workgroups per CU or split the histogram into bin windows)."""
import json

import numpy as np
import pytest

import workloads
from gpu_util import run_gpu

pytestmark = pytest.mark.gpu


def test_cached_copies_reserve_no_lds(tmp_path):
    import paper_1808_01478_amd as dh
    fr = workloads.random_frame(77, [6000, 3000], workloads.BOX_ORTHO,
                                box=workloads.ortho_box(20, 20, 20), r_max=9.0, n_bins=20_000)
    print("\n[case] cached copies", flush=True)
    with dh.Context(0) as c:
        c.set_tuning(dh.TUNE_ON, str(tmp_path / "probe.json"))
        run_gpu(c, fr, 0)
        key = next(iter(json.load(open(tmp_path / "probe.json"))["entries"]))
    got = {}
    for copies in (1, 4):
        path = tmp_path / f"hand{copies}.json"
        path.write_text(json.dumps({"version": 3,
                                    "entries": {key: [4, copies, 256, 1, 0, 8, 1024, 0]}}))
        with dh.Context(0) as c:
            c.set_tuning(dh.TUNE_CACHED, str(path))
            h, oor = run_gpu(c, fr, 0)
            got[copies] = (h, oor, c.last_config())
    one, four = got[1][2], got[4][2]
    assert four["copies"] == 4 and four["sweeps"] == 1 and four["mode"] == 0
    assert {**four, "copies": 1} == one
    assert np.array_equal(got[1][0], got[4][0]) and np.array_equal(got[1][1], got[4][1])
