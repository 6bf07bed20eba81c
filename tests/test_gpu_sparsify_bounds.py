"""The sparsifier where its fp32 scores cannot decide: equal and nearly equal
scores around the k-th place (more and fewer of them than one wave settles),
zero rows, magnitudes outside fp32's reach, and every row length at which
the selection changes its register layout.  The oracle's masks are met bit
for bit (integer results; no tolerance)."""
import numpy as np
import pytest

from oracle import sparsify as osp
from tests.gpu_util import log, to_dev_bf16
from workloads import bf16_bits_from_f32

pytestmark = pytest.mark.gpu

import paper_2609_25869_amd as bsa  # noqa: E402  (fails loudly if libbsa.so is missing)


def _qk(seed, B, H, nq, nkv):
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((B, nq, H, 128)).astype(np.float32)
    k = rng.standard_normal((B, nkv, H, 128)).astype(np.float32)
    return q, k


def _check(q, k, bq, bkv, topk, diagonal=True, what=""):
    import torch
    qb, kb = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    want, _ = osp.sparsify_topk(qb, kb, bq, bkv, topk, diagonal=diagonal)
    for noalloc in (False, True):
        got = bsa.sparsify_topk(to_dev_bf16(qb), to_dev_bf16(kb), bq, bkv, topk, diagonal=diagonal, noalloc=noalloc)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        assert np.array_equal(got, want), "%s: %d of %d entries differ" % (what, int((got != want).sum()), got.size)


# KV blocks per row around the register counts (64 x 8, 16, 32, 64) and both
# score tile sizes; whole and broken groups of four columns
@pytest.mark.parametrize("nkb", [1, 3, 4, 63, 64, 65, 511, 512, 513, 1024, 1027, 2048, 2052, 4096, 4100])
def test_row_lengths(nkb):
    q, k = _qk(nkb, 1, 2, 200, nkb * 16 - 3 if nkb > 1 else 16)
    for topk in sorted({1, max(1, nkb // 8), max(1, nkb - 1)}):
        log("nkb %d topk %d" % (nkb, topk))
        _check(q, k, 32, 16, topk, what="nkb %d topk %d" % (nkb, topk))


@pytest.mark.parametrize("copies", [2, 40, 64, 65, 300])
def test_ties_across_the_boundary(copies):
    """`copies` equal key blocks straddle the k-th place, and as many that
    differ from them by one bf16 step of one element."""
    q, k = _qk(copies, 1, 1, 256, 1024 * 16)
    q, k = np.abs(q), np.abs(k)
    rng = np.random.default_rng(copies + 1)
    at = rng.permutation(1024)[:2 * copies]
    block = k[0, :16, 0, :].copy()
    for i, kb in enumerate(at):
        k[0, kb * 16:(kb + 1) * 16, 0, :] = block
        if i >= copies:
            k[0, kb * 16, 0, i % 128] *= np.float32(1.0 + 2.0 ** -7)
    _, s = osp.sparsify_topk(bf16_bits_from_f32(q), bf16_bits_from_f32(k), 32, 16, 1)
    above = int(np.median((s[0, 0] > s[0, 0, :, at[0]][:, None]).sum(-1)))
    for topk in (above + 1, above + copies // 2 + 1, above + copies, above + copies + copies // 2):
        topk = min(max(1, topk), 1023)
        log("copies %d topk %d" % (copies, topk))
        _check(q, k, 32, 16, topk, diagonal=False, what="copies %d topk %d" % (copies, topk))


def test_zero_rows_and_zero_keys():
    q, k = _qk(5, 2, 2, 320, 100 * 32)
    q[:, 64:128] = 0.0          # two query blocks of zeros: every score ties
    k[:, 320:1600] = 0.0        # forty zero key blocks
    _check(q, k, 32, 32, 7, diagonal=False, what="zero rows")
    _check(q, k, 32, 32, 60, what="zero rows, more than half")
    _check(q, np.zeros_like(k), 32, 32, 9, what="all keys zero")


@pytest.mark.parametrize("scale_q,scale_k", [(1e18, 1e18), (1e-18, 1e-18), (1e30, 1e-30), (1e-30, 1.0), (1e15, 1e-9)])
def test_magnitudes(scale_q, scale_k):
    q, k = _qk(9, 1, 2, 300, 150 * 16)
    _check(q * np.float32(scale_q), k * np.float32(scale_k), 32, 16, 20, what="scales %g %g" % (scale_q, scale_k))


def test_one_outlier_block_widens_the_bound():
    """A key block 2^14 times the others' size: most columns fall within the
    bound of the k-th score and are settled by their own scores."""
    q, k = _qk(11, 1, 1, 256, 700 * 16)
    k[0, 160:176] *= np.float32(16384.0)
    for topk in (5, 87, 350):
        _check(q, k, 32, 16, topk, what="outlier, topk %d" % topk)


@pytest.mark.parametrize("offset,pad", [(0, 8), (2, 2), (1, 1)])
def test_layouts_of_the_block_means(offset, pad):
    """Rows 16-byte, 4-byte and 2-byte aligned take different load widths."""
    import torch
    q, k = _qk(13, 1, 2, 500, 700)
    qb, kb = bf16_bits_from_f32(q), bf16_bits_from_f32(k)
    want, _ = osp.sparsify_topk(qb, kb, 32, 32, 4)

    def strided(x):
        t = to_dev_bf16(x)
        B, n, H, d = t.shape
        flat = torch.zeros(B * n * H * (d + pad) + 16, dtype=torch.bfloat16, device="cuda")
        v = flat[offset:offset + B * n * H * (d + pad)].view(B, n, H, d + pad)[..., :d]
        v.copy_(t)
        return v
    got = bsa.sparsify_topk(strided(qb), strided(kb), 32, 32, 4)
    torch.cuda.synchronize()
    assert np.array_equal(got.cpu().numpy(), want)


# two heads of seven rows: rows of both in one workgroup, a last one of two
# rows; rows shorter and longer than a wave's and a workgroup's step
@pytest.mark.parametrize("nkb", [2, 63, 65, 257, 1026, 4100, 6144])
def test_undecided_rows_of_every_length(nkb):
    q, k = _qk(nkb + 1, 1, 2, 7 * 16 - 3, nkb * 16)
    log("nkb %d" % nkb)
    _check(q, k * np.float32(1e-14), 16, 16, max(1, nkb // 8), what="out of range, nkb %d" % nkb)
    k[:, nkb // 3 * 16:] = 0.0
    _check(q, k, 16, 16, max(1, nkb // 2), diagonal=False, what="tied, nkb %d" % nkb)


def test_undecided_rows_stay_within_a_few_times_the_usual_cost():
    """Rows that fp32 cannot decide (tied, not finite or out of range) are
    selected in the pinned arithmetic.  With every row such a row the whole
    selection takes 3.3 times the usual at this size; walking the mean keys
    row by row it took 12 times."""
    import torch
    N, H, blk, topk = 65536, 8, 64, 123
    gen = torch.Generator(device="cuda")
    gen.manual_seed(17)
    q, k = (torch.randn((1, N, H, 128), generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    mask = torch.empty((1, H, N // blk, N // blk), dtype=torch.uint8, device="cuda")

    def ms(kk):
        best = float("inf")
        for _ in range(6):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            bsa.sparsify_topk(q, kk, blk, blk, topk, mask=mask)
            e1.record()
            e1.synchronize()
            best = min(best, e0.elapsed_time(e1))
        return best
    usual = ms(k)
    tail = k.clone()
    tail[:, N // 10:] = 0
    nan = k.clone()
    nan[:, 5] = float("nan")
    for name, kk in (("zero tail", tail), ("all zero", torch.zeros_like(k)), ("not a number", nan),
                     ("out of range", k * 1e-14)):
        t = ms(kk)
        log("%s: %.3f ms, usual %.3f ms" % (name, t, usual))
        assert t < 7.0 * usual, (name, t, usual)


def test_more_blocks_than_one_launch_holds():
    """10922 heads of 6144 one-token blocks, 2-byte aligned: more threads than
    one launch of the block means takes, so the heads go in several passes."""
    import torch
    H, n = 10922, 6144
    free = torch.cuda.mem_get_info()[0]
    if free < 40 << 30:
        pytest.skip("needs 40 GB of device memory")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(19)
    q = torch.randn((1, 1, H, 128), generator=gen, device="cuda").to(torch.bfloat16)
    flat = torch.empty(n * H * 128 + 1, dtype=torch.bfloat16, device="cuda")
    k = flat[1:].view(1, n, H, 128)
    for i in range(0, n, 256):
        k[:, i:i + 256].normal_(generator=gen)
    got = bsa.sparsify_topk(q, k, 1, 1, 100)
    for h0 in range(0, H, 4000):
        part = bsa.sparsify_topk(q[:, :, h0:h0 + 4000], k[:, :, h0:h0 + 4000], 1, 1, 100)
        assert torch.equal(got[:, h0:h0 + 4000], part), h0
