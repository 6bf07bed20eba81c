"""The attention kernel's tile lists at the sizes where they can go wrong:
lists of 16-token blocks packed two to a 32-key tile (odd counts, ragged
sequence ends, mask rows that are and are not whole 32-bit words, one and
several query blocks per tile), and lists longer than one and two chunks of
64 entries.  Compared with the fp64 oracle at the tolerances of the parity
tests (unit-variance inputs, bf16 operands and probabilities)."""
import numpy as np
import pytest

from oracle import attn as oattn
from oracle import plans
from tests.gpu_util import bf16_to_f64, compare, compare_lse, log, run_plan
from workloads import bf16_bits_from_f32, random_case

pytestmark = pytest.mark.gpu

import paper_2609_25869_amd as bsa  # noqa: E402  (fails loudly if libbsa.so is missing)

PACKED_PLANS = (0, 8, 24, 26, 30, 31, 33, 34)  # split-free 32-key tiles, one wave per 32 rows

# (name, B, Nq, Nkv, geometry, density, plans)
CASES = [
    ("b16_bytes", 2, 1040, 1040, (16, 16), 0.15, PACKED_PLANS),     # 65 blocks a row: byte-wise mask rows
    ("b16_words", 1, 1088, 1088, (16, 16), 0.15, PACKED_PLANS),     # 68 blocks: word-wise
    ("b16_tail", 1, 300, 1079, (16, 16), 0.25, PACKED_PLANS),       # the last block holds 7 tokens
    ("b64x16", 1, 700, 1100, (64, 16), 0.3, PACKED_PLANS),          # one query block per 64-row tile: no member words
    ("b128x16", 1, 1000, 1271, (128, 16), 0.3, PACKED_PLANS),       # tiles smaller than the query block
    ("b32x16_long", 1, 200, 3000, (32, 16), 0.9, PACKED_PLANS),     # 188 blocks: three chunks
    ("b16_one", 1, 64, 16, (16, 16), 0.7, PACKED_PLANS),            # one block in all
    ("b32_long", 1, 200, 4700, (32, 32), 0.9, (0, 4, 8, 12, 20, 30)),    # 147 tiles with member words
    ("b64_long", 1, 200, 8200, (64, 64), 0.95, (0, 4, 8, 12, 16, 20, 30, 32)),
    ("b64_chunk", 1, 130, 64 * 64, (64, 64), 1.0, (0, 4, 12, 30)),  # exactly one and two chunks
    ("b16_in_64", 1, 300, 1079, (16, 16), 0.25, (4, 12, 20, 32)),   # four blocks along a 64-key tile
    ("b32x16_in_64", 2, 513, 1216, (32, 16), 0.4, (4, 12, 20, 32)),  # whole tiles
    ("b256x16_in_64", 1, 600, 1079, (256, 16), 0.4, (4, 12, 20, 32)),  # one query block and more per tile
    ("b16x8_in_64", 1, 300, 1079, (64, 8), 0.4, (4, 12, 20, 32)),   # eight blocks along a tile
]


@pytest.mark.parametrize("name", [c[0] for c in CASES])
def test_tile_lists_match_oracle(name):
    _, B, nq, nkv, geom, dens, ids = [c for c in CASES if c[0] == name][0]
    q, k, v, mask = random_case(sum(map(ord, name)), B, 2, nq, nkv, 128, [geom] * 2, dens,
                                empty_rows=1 if nq > 64 else 0)
    O_ref, L_ref = oattn.masked_attention(q, k, v, mask)
    segs, _ = plans.mask_stats(mask)
    for pid in ids:
        log("case %s plan %d" % (name, pid))
        p, od, lsed, _ = run_plan(bsa, mask, q, k, v, force_plan=pid)
        compare(bf16_to_f64(od), O_ref, "%s plan %d" % (name, pid))
        compare_lse(lsed.cpu().numpy().astype(np.float64), L_ref, "%s plan %d" % (name, pid))
        e = bsa.catalog()[pid]
        tiles = plans.physical_tiles(mask, segs[0].heads, e["tq"], e["tkv"])
        assert np.array_equal(p.export(bsa.EXPORT_TILE_KV), tiles.kv_tile)
        assert np.array_equal(p.export(bsa.EXPORT_TILE_MEMBER), tiles.member)
        assert np.array_equal(p.export(bsa.EXPORT_TASKS), plans.split_tasks(tiles, e["split"]))
        p.destroy()


# K rows of +inf (scores of +inf, -inf or NaN), and finite ones whose scores
# overflow to +inf and -inf (the queries have one sign)
@pytest.mark.parametrize("fill,one_sign", [(np.inf, False), (3e38, True), (-3e38, True), (np.inf, True)])
def test_infinite_keys_of_inactive_blocks_change_nothing(fill, one_sign):
    """Masking must hold for scores that are not finite: K rows that make them
    so, in blocks a query row does not use, leave its output bitwise unchanged,
    also where a tile shares the block with rows that do use it."""
    for geom, ids in (((16, 16), (0, 4, 8, 12, 20, 30, 32)), ((32, 32), (0, 4, 8, 12, 16, 20, 30)),
                      ((64, 64), (8, 12, 16, 20, 32))):
        q, k, v, mask = random_case(907, 1, 1, 384, 384, 128, [geom], 0.3)
        if one_sign:
            q = q & np.uint16(0x7FFF)
        m = mask.head(0, 0) != 0
        kb = int(np.argmax((~m).sum(0) * m.any(0)))   # used by some rows, not by others
        rows = [r for r in range(m.shape[0]) if not m[r, kb]]
        assert rows and len(rows) < m.shape[0]
        k2 = k.copy()
        k2[0, kb * geom[1]:(kb + 1) * geom[1], 0, :] = bf16_bits_from_f32(np.full((geom[1], 128), fill, np.float32))
        for pid in ids:
            log("geometry %s plan %d" % (geom, pid))
            p, a, la, _ = run_plan(bsa, mask, q, k, v, force_plan=pid)
            p2, b, lb, _ = run_plan(bsa, mask, q, k2, v, force_plan=pid)
            for r in rows:
                sl = slice(r * geom[0], (r + 1) * geom[0])
                assert (a[0, sl] == b[0, sl]).all().item() and (la[0, 0, sl] == lb[0, 0, sl]).all().item(), (pid, r)
            p.destroy()
            p2.destroy()
