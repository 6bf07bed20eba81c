"""Launches cut into generations (1024 tasks each, the last one short): every
physical query tile has a row compared with the fp64 oracle, and no output is
left unwritten.  Equal row lengths, scattered blocks, 2048 keys a row and K/V
of 32 MiB per head are what the planner cuts launches for; one block less a
row or of K/V is not."""
import numpy as np
import pytest

from oracle import attn as oattn
from tests.gpu_util import bf16_to_f64, compare, compare_lse, log, run_plan
from workloads import BlockMask, bf16_bits_from_f32

pytestmark = pytest.mark.gpu

import paper_2609_25869_amd as bsa  # noqa: E402  (fails loudly if libbsa.so is missing)


@pytest.mark.parametrize("nkv,blocks", [(65536, 32), (65536, 31), (65536 - 64, 32)])
def test_every_generation_matches_oracle(nkv, blocks):
    H, nq, nkb = 3, 64 * 700 - 9, nkv // 64
    rng = np.random.default_rng(nkv + 100 * blocks)
    q, k, v = (bf16_bits_from_f32(rng.standard_normal((1, n, H, 128), dtype=np.float32)) for n in (nq, nkv, nkv))
    heads = []
    for _ in range(H):
        m = np.zeros((700, nkb), dtype=bool)
        for r in range(700):
            m[r, rng.choice(nkb // 2, size=blocks, replace=False) * 2] = True   # no two neighbours
        heads.append(m)
    mask = BlockMask.from_heads([heads], [64] * H, [64] * H, nq, nkv)
    rows = np.array([(0, h, min(nq - 1, 64 * t + int(rng.integers(64)))) for h in range(H) for t in range(700)], dtype=np.int64)
    O_ref, L_ref = oattn.masked_attention(q, k, v, mask, rows=rows)
    for pid in (0, 4, 24, 30, 33, 12):
        log("%d keys, %d blocks, plan %d" % (nkv, blocks, pid))
        p, od, lsed, _ = run_plan(bsa, mask, q, k, v, force_plan=pid)
        assert od.isfinite().all().item() and lsed.isfinite().all().item()
        O, L = bf16_to_f64(od), lsed.cpu().numpy().astype(np.float64)
        compare(O[rows[:, 0], rows[:, 2], rows[:, 1]], O_ref, "plan %d" % pid)
        compare_lse(L[rows[:, 0], rows[:, 1], rows[:, 2]], L_ref, "plan %d" % pid)
        p.destroy()
