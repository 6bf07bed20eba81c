"""Requests of few rows, whose rows the kernel cuts into more slices than the
plan does: the most slices, counts that are no multiple of the merge's batch,
rows shorter than the slice count, empty rows, compacted lists (cut between
pairs) and every tile height.  Compared with the fp64 oracle at the parity
tests' tolerances; the exported tasks stay the plan's."""
import numpy as np
import pytest

from oracle import attn as oattn
from oracle import plans
from tests.gpu_util import bf16_to_f64, compare, compare_lse, log, run_plan
from workloads import random_case

pytestmark = pytest.mark.gpu

import paper_2609_25869_amd as bsa  # noqa: E402  (fails loudly if libbsa.so is missing)

# (name, B, H, Nq, Nkv, geometry, density, empty query-block rows, plans)
CASES = [
    ("most", 1, 1, 64, 20000, (64, 64), 0.9, 0, (0, 4, 8, 12, 16, 20, 30)),      # 64 slices
    ("odd", 1, 3, 200, 9000, (64, 64), 0.5, 1, (0, 1, 3, 4, 6, 12, 16, 30)),     # 28 slices; Split-K plans too
    ("ragged", 2, 2, 333, 5003, (32, 32), 0.3, 2, (0, 4, 8, 12, 20, 30, 31)),
    ("packed", 1, 2, 77, 6007, (16, 16), 0.2, 1, (0, 8, 24, 30, 33, 4)),         # compacted lists, odd counts
    ("short_rows", 1, 2, 200, 9000, (64, 64), 0.5, 1, (0, 4, 30)),               # one row of a single block
    ("tall_block", 1, 1, 300, 7000, (128, 128), 0.6, 0, (0, 4, 12, 20)),
]


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_sliced_rows_match_oracle(name):
    _, B, H, nq, nkv, geom, dens, empty, ids = [c for c in CASES if c[0] == name][0]
    q, k, v, mask = random_case(sum(map(ord, name)), B, H, nq, nkv, 128, [geom] * H, dens, empty_rows=empty)
    if name == "short_rows":
        mask.head(0, 0)[0, :] = 0
        mask.head(0, 0)[0, 3] = 1
    O_ref, L_ref = oattn.masked_attention(q, k, v, mask)
    segs, _ = plans.mask_stats(mask)
    sliced = 0
    for pid in ids:
        log("case %s plan %d" % (name, pid))
        p, od, lsed, _ = run_plan(bsa, mask, q, k, v, force_plan=pid)
        compare(bf16_to_f64(od), O_ref, "%s plan %d" % (name, pid))
        compare_lse(lsed.cpu().numpy().astype(np.float64), L_ref, "%s plan %d" % (name, pid))
        e, info = bsa.catalog()[pid], p.info()
        tasks = plans.split_tasks(plans.physical_tiles(mask, segs[0].heads, e["tq"], e["tkv"]), e["split"])
        assert np.array_equal(p.export(bsa.EXPORT_TASKS), tasks) and info["n_tasks"] == len(tasks)
        assert np.array_equal(p.export(bsa.EXPORT_DISPATCH), np.arange(len(tasks)))
        sliced += info["workspace_bytes"] > 0
        # the same bits again, and a second pass on the same workspace
        q2, od2, lsed2, devs = run_plan(bsa, mask, q, k, v, force_plan=pid)
        bsa.forward(q2, devs[0], devs[1], devs[2], od2, lsed2)
        assert (od == od2).all().item() and (lsed == lsed2).all().item()
        p.destroy()
        q2.destroy()
    assert sliced >= len(ids) // 2
