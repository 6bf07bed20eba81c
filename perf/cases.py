"""The work whose speed is tracked: requests, forward passes and mask selection
through the package's public entry points (plan, forward, sparsify_topk).

A case names one call pattern ("what"):

  forward   a kept plan run on Q/K/V (warm repeats of a request)
  request   plan + forward of a fresh mask, the plan destroyed afterwards
  sparsify  the device top-k sparsifier alone
  full      sparsify -> plan -> forward, nothing prepared beforehand

and its sizes, block geometry, mask family and options.  Inputs are i.i.d.
normal values in bf16 and seeded masks of the repository's workload families:
Bernoulli blocks with the diagonal, per-row top-k, a 3D window over token
cubes, and a mixture in which every head draws its own family and density.
"""
import math

import torch

import paper_2609_25869_amd as bsa

D = 128
MIX_DENSITIES = (0.02, 0.05, 0.10, 0.25, 0.50)
# block geometries (B_Q, B_KV) that the plan table is profiled for
GEOMETRIES = ((64, 64), (128, 128), (128, 64), (64, 32), (128, 32), (32, 128), (32, 32), (32, 16), (16, 16))


def _case(name, what, B, H, nq, nkv, bq, bkv, mask="topk", rho=0.1, bq2=0, bkv2=0, grid="", half="", lse=False,
          layout="bnhd", noalloc=False):
    c = dict(what=what, B=B, H=H, nq=nq, nkv=nkv, bq=bq, bkv=bkv, mask=mask, rho=rho, bq2=bq2, bkv2=bkv2, grid=grid,
             half=half, lse=lse, layout=layout, noalloc=noalloc)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest request (2 heads, 2048 tokens): launch and planning latency of a complete request,
        # and the same forward repeated on its kept plan (a denoising step that reuses its mask)
        _case("forward_tiny", "forward", 1, 2, 2048, 2048, 64, 64, "bernoulli", 0.3, lse=True),
        _case("request_tiny", "request", 1, 2, 2048, 2048, 64, 64, "bernoulli", 0.3, lse=True),
        # the flagship workload: a five-second 720p clip (115200 tokens, 24 heads), (128,128) blocks under
        # a 3D window of 15.3% density, planning included
        _case("request_window_115k", "request", 1, 24, 115200, 115200, 128, 128, "window", grid="15,6,10",
              half="1,5,5"),
        # the same clip under content-dependent top-k blocks of 64 tokens: attention on a kept plan, and
        # the selection that supplies its mask
        _case("forward_topk_115k", "forward", 1, 24, 115200, 115200, 64, 64, "topk", 0.12),
        _case("sparsify_115k", "sparsify", 1, 24, 115200, 115200, 64, 64, "topk", 0.12),
        # heads with two geometries in one request, densities 5% to 50%
        _case("forward_asym_64k", "forward", 1, 16, 65536, 65536, 128, 32, "bernoulli_range", 0.0, bq2=32, bkv2=128),
        # the largest request: a batch of two 131072-token clips whose heads differ in family and density
        _case("request_mixture_131k", "request", 2, 24, 131072, 131072, 64, 64, "mixture", grid="8,16,16"),
        # the finest blocks, ragged length, with the log-sum-exp
        _case("forward_fine16_30k", "forward", 1, 8, 30011, 30011, 16, 16, "bernoulli", 0.1, lse=True),
        # few query rows against a long ragged context, [B, H, N, d] storage: too few tasks for 256 CUs
        _case("forward_cross_50k", "forward", 1, 8, 777, 50021, 64, 64, "topk", 0.2, lse=True, layout="bhnd"),
        # a medium layer end to end on the device: selection, planning and attention
        _case("full_16k", "full", 1, 12, 16384, 16384, 64, 64, "topk", 0.15, lse=True),
        # selection in a serving loop that may not allocate: batch of two, ragged, different lengths
        _case("sparsify_noalloc_20k", "sparsify", 2, 3, 20011, 17003, 64, 32, "topk", 0.08, noalloc=True),
        # a medium request of 32-token blocks, planning included
        _case("request_32x32_24k", "request", 2, 8, 24576, 24576, 32, 32, "topk", 0.08),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    what = rng.choice(("forward", "request", "forward", "request", "full", "sparsify"))
    mask = "topk" if what in ("full", "sparsify") else rng.choice(("topk", "bernoulli", "mixture"))
    while True:
        bq, bkv = rng.choice(GEOMETRIES)
        B, H = rng.choice((1, 1, 2)), rng.choice((1, 2, 4, 6, 8, 12, 16, 24))
        n = log_int(1000, 131072)
        if rng.random() < 0.5:  # whole numbers of blocks as often as ragged lengths
            n = -(-n // 128) * 128
        nq = n if rng.random() < 0.75 else log_int(64, n)
        rho = math.exp(rng.uniform(math.log(0.02), math.log(0.5)))
        # within the sparsifier's rows, the memory of a mask and the largest listed case's work
        rows, cols = -(-nq // bq), -(-n // bkv)
        density = max(rho, 0.2) if mask == "mixture" else rho
        if cols > 6144 or B * H * rows * cols > 2.5e8 or 4.0 * D * B * H * nq * n * density > 2e13:
            continue
        noalloc = what == "sparsify" and rng.random() < 0.5
        if noalloc and (rows + cols) * 1024 + rows * cols * 8 > (64 << 20):
            continue
        break
    two = mask == "bernoulli" and H > 1 and rng.random() < 0.3
    bq2, bkv2 = rng.choice(GEOMETRIES) if two else (0, 0)
    if two and B * H * (-(-nq // bq2)) * (-(-n // bkv2)) > 2.5e8:
        bq2, bkv2 = 0, 0
    return _case("", what, B, H, nq, n, bq, bkv, mask, round(rho, 4), bq2, bkv2, lse=rng.random() < 0.5,
                 layout=rng.choice(("bnhd", "bnhd", "bhnd")), noalloc=noalloc)


# ---------------------------------------------------------------------------
# Inputs

def _geometry(c, h):
    return (c["bq2"], c["bkv2"]) if c["bq2"] and h % 2 else (c["bq"], c["bkv"])


def _blocks(c, h):
    bq, bkv = _geometry(c, h)
    return -(-c["nq"] // bq), -(-c["nkv"] // bkv)


def _ints(text):
    return [int(x) for x in text.split(",")]


def _tensor(c, n, gen):
    B, H = c["B"], c["H"]
    shape = (B, n, H, D) if c["layout"] == "bnhd" else (B, H, n, D)
    x = torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    return x if c["layout"] == "bnhd" else x.permute(0, 2, 1, 3)


def _diagonal(c, h):
    bq, bkv = _geometry(c, h)
    rows, cols = _blocks(c, h)
    n = min(c["nq"], c["nkv"])
    lo = torch.arange(rows, device="cuda") * bq
    hi = (lo + bq).clamp(max=n)
    kb = torch.arange(cols, device="cuda")
    return (kb[None] >= (lo // bkv)[:, None]) & (kb[None] <= ((hi - 1) // bkv)[:, None]) & (lo < hi)[:, None]


def _window(grid, half):
    ax = [torch.arange(g, device="cuda") for g in grid]
    pos = [p.reshape(-1) for p in torch.meshgrid(*ax, indexing="ij")]
    m = None
    for p, w in zip(pos, half):
        near = (p[:, None] - p[None]).abs() <= w
        m = near if m is None else m & near
    return m


def _topk_count(rho, cols):
    return max(1, int(math.floor(rho * cols + 0.5)))


def _head_mask(c, h, family, rho, gen):
    rows, cols = _blocks(c, h)
    if family == "window":
        if c["grid"]:
            grid = _ints(c["grid"])
            if c["mask"] == "window":
                return _window(grid, _ints(c["half"]))
            return _window(grid, {0.02: (3, 1, 1), 0.05: (1, 3, 3), 0.10: (3, 3, 3), 0.25: (1, 9, 9),
                                  0.50: (6, 7, 7)}[rho])
        q = torch.arange(rows, device="cuda") * cols // rows
        return (q[:, None] - torch.arange(cols, device="cuda")[None]).abs() <= max(1, int(round(rho * cols / 2)))
    x = torch.rand((rows, cols), generator=gen, device="cuda")
    if family == "topk":
        top = torch.topk(x, _topk_count(rho, cols), dim=1).indices
        m = torch.zeros((rows, cols), dtype=torch.bool, device="cuda").scatter_(1, top, True)
    else:
        m = x < rho
    return m | _diagonal(c, h)


def _mask(c, gen, pick):
    """The packed masks, uint8, head by head for each batch."""
    parts = []
    for _ in range(c["B"]):
        for h in range(c["H"]):
            family, rho = c["mask"], c["rho"]
            if family == "bernoulli_range":
                family, rho = "bernoulli", 0.05 + 0.45 * pick.random()
            elif family == "mixture":
                u = pick.random()
                family = "window" if u < 0.4 else "topk" if u < 0.8 else "bernoulli"
                rho = pick.choice(MIX_DENSITIES)
            parts.append(_head_mask(c, h, family, rho, gen).to(torch.uint8).reshape(-1))
    return torch.cat(parts)


def _layout(c):
    """(head offsets, elements of one batch) of the packed masks."""
    off, at = [], 0
    for h in range(c["H"]):
        off.append(at)
        rows, cols = _blocks(c, h)
        at += rows * cols
    return off, at


def _inputs(c, seed):
    import random
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    s = {"q": _tensor(c, c["nq"], gen), "k": _tensor(c, c["nkv"], gen)}
    if c["what"] != "sparsify":
        s["v"] = _tensor(c, c["nkv"], gen)
    if c["what"] in ("forward", "request"):
        s["mask"] = _mask(c, gen, random.Random(seed))
    return s


def prepare(case, seed):
    c = case
    s = _inputs(c, seed)
    s["case"] = c
    s["offsets"], s["stride_b"] = _layout(c)
    H = c["H"]
    s["bq"] = [_geometry(c, h)[0] for h in range(H)] if c["bq2"] else c["bq"]
    s["bkv"] = [_geometry(c, h)[1] for h in range(H)] if c["bq2"] else c["bkv"]
    if c["what"] in ("sparsify", "full"):
        rows, cols = _blocks(c, 0)
        s["topk"] = _topk_count(c["rho"], cols)
        s["mask"] = torch.empty((c["B"], H, rows, cols), dtype=torch.uint8, device="cuda")
    if c["what"] != "sparsify":
        s["o"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty((c["B"], H, c["nq"]), dtype=torch.float32, device="cuda") if c["lse"] else None
        s["shapes"] = bsa.shapes_of(s["q"], s["k"], s["v"], s["o"])
    if c["what"] == "forward":
        s["plan"] = _plan(s)
    return s


def _plan(s):
    return bsa.plan(s["mask"], s["bq"], s["bkv"], s["shapes"], head_offset=s["offsets"], stride_b=s["stride_b"])


def run(state):
    s, what = state, state["case"]["what"]
    out = {}
    if what in ("sparsify", "full"):
        out["mask"] = bsa.sparsify_topk(s["q"], s["k"], s["bq"], s["bkv"], s["topk"], mask=s["mask"],
                                        noalloc=s["case"]["noalloc"])
        if what == "sparsify":
            return out
    p = s["plan"] if what == "forward" else _plan(s)
    out["o"] = p.forward(s["q"], s["k"], s["v"], s["o"], s["lse"])
    if what != "forward":
        p.destroy()
    if s["lse"] is not None:
        out["lse"] = s["lse"]
    return out


# ---------------------------------------------------------------------------
# What a pass cannot do without, and what it should give

def _density(c, h):
    """Expected share of active blocks."""
    rows, cols = _blocks(c, h)
    if c["mask"] == "window":
        share = 1.0
        for g, w in zip(_ints(c["grid"]), _ints(c["half"])):
            share *= sum(min(g - 1, i + w) - max(0, i - w) + 1 for i in range(g)) / (g * g)
        return share
    rho = 0.275 if c["mask"] == "bernoulli_range" else 0.184 if c["mask"] == "mixture" else c["rho"]
    return min(1.0, rho + (1 - rho) / cols)


def work(case):
    c = case
    B, H, nq, nkv = c["B"], c["H"], c["nq"], c["nkv"]
    mask_bytes = B * sum(_blocks(c, h)[0] * _blocks(c, h)[1] for h in range(H))
    qk = 2 * D * B * H * (nq + nkv)
    bytes_, flops = 0, 0
    if c["what"] in ("sparsify", "full"):
        rows, cols = _blocks(c, 0)
        bytes_ += qk + mask_bytes
        flops += B * H * D * (nq + nkv + 2 * rows * cols)
    if c["what"] != "sparsify":
        bytes_ += 2 * qk + (4 * B * H * nq if c["lse"] else 0)
        if c["what"] != "forward":
            bytes_ += mask_bytes
        flops += sum(int(4 * D * B * nq * nkv * _density(c, h)) for h in range(H))
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    # Selected blocks are whole numbers.  O is rounded to bf16, as are the probabilities it is summed from:
    # both together measure about 2.6e-3 from the 64-bit result.
    if case["what"] == "sparsify":
        return "exact"
    return {"rel": 1e-2, "max": 0.15}


def _exact_mask(c, q, k):
    """Mean-pooled top-k blocks with the diagonal, from 64-bit block means."""
    rows, cols = _blocks(c, 0)

    def means(x, blk, nb):
        n = x.shape[1]
        x = torch.nn.functional.pad(x.double(), (0, 0, 0, nb * blk - n))
        s = x.reshape(x.shape[0], nb, blk, D).sum(2)
        cnt = torch.full((nb,), float(blk), dtype=torch.float64, device=x.device)
        cnt[-1] = n - (nb - 1) * blk
        return s / cnt[None, :, None]

    m = torch.empty((c["B"], c["H"], rows, cols), dtype=torch.bool, device="cuda")
    take = _topk_count(c["rho"], cols)
    for b in range(c["B"]):
        for h in range(c["H"]):
            score = means(q[b, :, h][None], c["bq"], rows)[0] @ means(k[b, :, h][None], c["bkv"], cols)[0].T
            top = torch.sort(-score, dim=1, stable=True).indices[:, :take]
            m[b, h] = torch.zeros_like(score, dtype=torch.bool).scatter_(1, top, True) | _diagonal(c, h)
    return m


def exact(case, seed):
    c = case
    if c["what"] == "sparsify":
        s = _inputs(c, seed)
        return {"mask": _exact_mask(c, s["q"], s["k"]).to(torch.uint8)}
    B, H, nq, nkv = c["B"], c["H"], c["nq"], c["nkv"]
    dense = float(B) * H * nq * nkv <= 1e11
    if not dense and B * sum(_blocks(c, h)[0] for h in range(H)) > 60000:
        return None
    s = _inputs(c, seed)
    q, k, v = s["q"], s["k"], s["v"]
    off, per_b = _layout(c)
    masks = _exact_mask(c, q, k) if c["what"] == "full" else None
    o = torch.zeros_like(q, dtype=torch.float64)
    lse = torch.full((B, H, nq), -math.inf, dtype=torch.float64, device="cuda")
    scale = 1.0 / math.sqrt(D)
    for b in range(B):
        for h in range(H):
            bq, bkv = _geometry(c, h)
            rows, cols = _blocks(c, h)
            if masks is not None:
                m = masks[b, h]
            else:
                at = b * per_b + off[h]
                m = s["mask"][at:at + rows * cols].reshape(rows, cols) != 0
            qh, kh, vh = (x[b, :, h].double().contiguous() for x in (q, k, v))
            kt = kh.T.contiguous()
            if dense:
                col = torch.arange(nkv, device="cuda") // bkv
                chunks = range(0, nq, 1024)
            else:
                first, active = m.sum(1).cumsum(0).tolist(), m.nonzero()[:, 1]
                chunks = range(0, nq, bq)
            for r0 in chunks:
                if dense:
                    r1 = min(nq, r0 + 1024)
                    row = torch.arange(r0, r1, device="cuda") // bq
                    z = (qh[r0:r1] @ kt) * scale
                    z.masked_fill_(~m[row][:, col], -math.inf)
                    vv = vh
                else:
                    r1, i = min(nq, r0 + bq), r0 // bq
                    kb = active[(first[i - 1] if i else 0):first[i]]
                    idx = (kb[:, None] * bkv + torch.arange(bkv, device="cuda")).reshape(-1)
                    idx = idx[idx < nkv]
                    if idx.numel() == 0:
                        continue
                    z = (qh[r0:r1] @ kh[idx].T.contiguous()) * scale
                    vv = vh[idx]
                top = z.amax(1, keepdim=True)
                top = torch.where(torch.isinf(top), torch.zeros_like(top), top)
                z.sub_(top).exp_()
                l = z.sum(1, keepdim=True)
                o[b, r0:r1, h] = (z @ vv) / torch.where(l > 0, l, torch.ones_like(l))
                lse[b, h, r0:r1] = (top + l.log())[:, 0]
    out = {"mask": None} if c["what"] == "full" else {}
    out["o"] = o
    if c["lse"]:
        out["lse"] = lse
    return out
