"""The dispatch order built per (batch, head) from row hashes, against the
reference written from its definition (exact list equality), at the edges of
its range: the fewest ordered tasks, one workgroup's threads, the most rows
per (batch, head) and the first size beyond it, which takes the general path.
Every mapping writes its own row hashes."""
import numpy as np
import pytest

from tests.gpu_util import expected_dispatch, log, mask_to_dev
from workloads import BlockMask

pytestmark = pytest.mark.gpu

import paper_2609_25869_amd as bsa  # noqa: E402  (fails loudly if libbsa.so is missing)

# (name, batch, heads, query tokens, KV tokens, geometry, plan)
CASES = [
    ("direct", 2, 3, 64 * 129, 64 * 24, (64, 64), 4),
    ("direct_bytes", 1, 2, 64 * 700, 64 * 23 - 5, (64, 64), 25),
    ("refined", 1, 3, 64 * 400, 64 * 24, (64, 64), 0),
    ("refined_q", 1, 1, 64 * 600, 128 * 20, (128, 128), 4),
    ("coarse_q", 1, 1, 64 * 1025, 32 * 40, (32, 32), 30),
    ("coarse_kv", 1, 1, 64 * 520, 32 * 40, (64, 32), 4),
    ("coarse_kv4", 1, 1, 64 * 520, 16 * 40, (16, 16), 4),
    ("compacted", 1, 1, 64 * 520, 16 * 40, (16, 16), 30),
    ("compacted_bytes", 1, 1, 64 * 520, 16 * 41, (16, 16), 33),
    ("most_rows", 1, 2, 64 * 2048, 64 * 12, (64, 64), 4),
    ("beyond", 1, 2, 64 * 2049, 64 * 12, (64, 64), 4),
    ("one_list", 1, 1, 64 * 2048, 64 * 4, (64, 64), 4),
]


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_order_matches_definition(name):
    _, B, H, nq, nkv, (bq, bkv), pid = [c for c in CASES if c[0] == name][0]
    rng = np.random.default_rng(sum(map(ord, name)))
    nqb, nkb = -(-nq // bq), -(-nkv // bkv)
    heads = []
    for _ in range(B):
        row = []
        for _ in range(H):
            # rows drawn from a few patterns, some of them empty, with some rows of their own
            pats = rng.random((1 if name == "one_list" else 17, nkb)) < 0.3
            pats[0] = name == "one_list"
            m = pats[rng.integers(len(pats), size=nqb)]
            own = rng.random(nqb) < (0.0 if name == "one_list" else 0.2)
            m[own] = rng.random((int(own.sum()), nkb)) < 0.3
            row.append(m)
        heads.append(row)
    mask = BlockMask.from_heads(heads, [bq] * H, [bkv] * H, nq, nkv)
    log("case %s: %d rows, plan %d" % (name, nqb, pid))
    p = bsa.plan(mask_to_dev(mask), bq, bkv, bsa.make_shapes(B, H, nq, nkv), head_offset=list(mask.head_offset),
                 stride_b=mask.stride_b, force_plan=pid)
    tasks = p.export(bsa.EXPORT_TASKS)
    member = p.export(bsa.EXPORT_TILE_MEMBER)
    want = expected_dispatch(tasks, p.export(bsa.EXPORT_TILE_KV), member if member.size else None)
    assert np.array_equal(p.export(bsa.EXPORT_DISPATCH), want)
    p.destroy()
