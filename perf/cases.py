"""Performance cases of the attention path: what they call, their inputs, work and tolerances.

A case is one call (or one short run of denoising steps) of one attention
layer of a video diffusion transformer, through the package's public entry
points.  Kinds:

* ``dense``      full attention with its LSE (the warm-up steps of a schedule);
* ``single``     the fresh-LSE search step: attention, LSE, block masses and
                 selection (:func:`single_pass_online_search`);
* ``cached``     the search of a later step from a kept LSE
                 (:func:`block_search`);
* ``select``     a new pattern chosen from masses that the program holds
                 (:func:`block_search` with ``scores``: other per-head counts);
* ``sparse``     block-sparse attention over a kept pattern, the call that
                 nearly every denoising step makes;
* ``denoise``    an ``AdaSpaAttention`` layer over a few steps of a schedule:
                 the search, sparse steps, the LSE-cached search, a sparse step.

Inputs have the frame / patch / text structure of such a sequence: video
tokens share a vector with the tokens of their frame and one with those of
their patch position, text tokens do not.
"""
import math

import torch

import paper_2502_21079_amd as ad
from paper_2502_21079_amd.schedule import AdaSpaAttention, SearchSchedule

DEV = "cuda"
# The long video (720p, 8 s): 256 text tokens and 32 frames of 3,440 patches.
LONG = dict(seqlen=110336, heads=24, head_dim=128, patches=3440, text_len=256, text_first=True)
# The moderate clip: 256 text tokens and 17,664 video tokens, d = 64.
MODERATE = dict(seqlen=17920, heads=48, head_dim=64, patches=1358, text_len=256, text_first=True)
# The smallest shape: a low-resolution preview of four frames.
TINY = dict(seqlen=2048, heads=2, head_dim=64, patches=496, text_len=64, text_first=True)
DENOISE_STEPS = 5
DENOISE_SEARCH = (0, 3)


def _case(name, kind, shape, batch=1, block=128, mode="topk", keep_bp=1000):
    c = dict(kind=kind, batch=batch, block=block, mode=mode, keep_bp=keep_bp, **shape)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # Full attention of the warm-up steps: the smallest preview, the
        # moderate clip, the long video (the largest call of all).
        _case("dense_tiny", "dense", TINY),
        _case("dense_moderate", "dense", MODERATE),
        _case("dense_long", "dense", LONG),
        # The fresh-LSE search step: a short clip of odd length with its text
        # last, coverage selection; and the long video's heads sharded over
        # eight GPUs (three each), the paper's block 64.
        _case("single_ragged", "single", dict(seqlen=9001, heads=12, head_dim=128, patches=880, text_len=226,
                                              text_first=False), mode="coverage", keep_bp=9000),
        _case("single_shard_b64", "single", dict(LONG, heads=3), block=64),
        # The LSE-cached search of a later step: preview and moderate clip.
        _case("cached_tiny", "cached", TINY, block=64, keep_bp=2000),
        _case("cached_moderate", "cached", MODERATE, mode="hierarchical", keep_bp=2000),
        # Another set of per-head counts for the long video's masses, block 64.
        _case("select_long_b64", "select", LONG, block=64, keep_bp=1000),
        # Block-sparse attention of the steps in between: preview, moderate
        # clip, long video.
        _case("sparse_tiny", "sparse", TINY, block=64, keep_bp=2000),
        _case("sparse_moderate", "sparse", MODERATE, keep_bp=1000),
        _case("sparse_long", "sparse", LONG, keep_bp=2000),
        # A whole layer over five steps, two samples side by side (guided and
        # unguided), odd length, block 64.
        _case("denoise_ragged_b64", "denoise", dict(seqlen=5003, heads=8, head_dim=128, patches=477, text_len=226,
                                                    text_first=False), batch=2, block=64, keep_bp=1500),
    ]


def draw(rng):
    """One more case: any kind, lengths over the whole range (odd ones among
    them), every head dimension, block size, selection mode and text order."""
    kind = rng.choice(["dense", "single", "cached", "select", "sparse", "denoise"])
    lo, hi = TINY["seqlen"], LONG["seqlen"]
    L = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if kind == "denoise":
        L = min(L, 32768)
    block = rng.choice([64, 128])
    B = rng.choice([1, 1, 2])
    H = rng.choice([2, 3, 6, 8, 12, 24, 48])
    D = rng.choice([64, 128])
    text = rng.choice([64, 226, 256])
    frames = rng.randint(4, 32)
    mode = rng.choice(["topk", "coverage", "hierarchical"])
    if kind in ("select", "sparse", "denoise"):
        mode = "topk"                      # given counts (the lists then fill their buffers)
    keep = rng.choice([7000, 9000]) if mode == "coverage" else rng.choice([500, 1000, 2000, 4000])
    shape = dict(seqlen=L, head_dim=D, patches=-(-(L - text) // frames), text_len=text,
                 text_first=rng.random() < 0.5)
    # No more work than the long video's full attention, per-row block masses
    # of at most 12 GB and selection buffers of at most 2 GB.
    nb = -(-L // block)
    while H > 1 and (4.0 * B * H * L * L * D * (DENOISE_STEPS if kind == "denoise" else 1) > 7e13
                     or (kind in ("single", "denoise") and 4.0 * B * H * nb * L > 12e9)
                     or (kind != "dense" and 16.0 * B * H * nb * nb > 2e9)):
        H = max(1, H // 2)
    return _case(None, kind, dict(shape, heads=H), batch=B, block=block, mode=mode, keep_bp=keep)


# --- inputs ------------------------------------------------------------------

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + stream) % (1 << 62))
    return g


def _qkv(case, seed):
    """q, k, v as bf16 [B, H, L, D]: N(0, 1) + 0.8 U[frame] + 0.6 W[patch]."""
    B, H, L, D = case["batch"], case["heads"], case["seqlen"], case["head_dim"]
    T, P = case["text_len"], case["patches"]
    v0 = T if case["text_first"] else 0
    vid = torch.arange(L - T, device=DEV)
    out = [torch.empty(B, H, L, D, dtype=torch.bfloat16, device=DEV) for _ in range(3)]
    g = _gen(seed, 1)
    for b in range(B):
        for h in range(H):
            U = torch.randn(int((L - T - 1) // P + 1), D, generator=g, device=DEV)
            W = torch.randn(P, D, generator=g, device=DEV)
            shared = 0.8 * U[vid // P] + 0.6 * W[vid % P]
            for t in out:
                x = torch.randn(L, D, generator=g, device=DEV)
                x[v0:v0 + L - T] += shared
                t[b, h].copy_(x)
    return out


def _text(case):
    start = 0 if case["text_first"] else case["seqlen"] - case["text_len"]
    return start, case["text_len"]


def _text_blocks(case):
    start, n = _text(case)
    return start // case["block"], (start + n - 1) // case["block"]


def _nb(case):
    return -(-case["seqlen"] // case["block"])


def _params(case):
    """Per-head selection parameters in basis points (unused by hierarchical)."""
    H, keep = case["heads"], case["keep_bp"]
    if case["mode"] == "coverage":
        return [keep] * H
    # Heads of unequal density around the mean, as head-adaptive patterns have.
    return [min(10000, max(1, int(keep * (0.6 + 0.8 * h / max(1, H - 1))))) if H > 1 else keep for h in range(H)]


def _counts(case):
    """Kept blocks per video row of each head in top-k mode."""
    nb = _nb(case)
    lo, hi = _text_blocks(case)
    return [max(hi - lo + 1, min(nb, -(-p * nb // 10000))) for p in _params(case)]


def _kept_lse(q, k, scale):
    """The LSE a program kept from an earlier step, [B, H, L] fp32.  It does
    not fit the present q and k exactly: a sixteenth of the keys stands for
    all of them."""
    B, H, L, D = q.shape
    lse = torch.empty(B, H, L, dtype=torch.float32, device=DEV)
    for b in range(B):
        for h in range(H):
            ks = k[b, h, ::16].float()
            for r in range(0, L, 16384):
                s = (q[b, h, r:r + 16384].float() @ ks.t()) * scale
                lse[b, h, r:r + 16384] = torch.logsumexp(s, dim=1) + math.log(L / ks.shape[0])
    return lse


def _blocks_of(x, nb, block):
    """Sums of x's last dimension over blocks of `block` entries."""
    pad = nb * block - x.shape[-1]
    return torch.nn.functional.pad(x, (0, pad)).unflatten(-1, (nb, block)).sum(-1)


def _pattern(case, q, k):
    """A kept block pattern as CSR (int32): text rows complete, every other
    row of a head with the head's count of blocks, the text blocks and those
    with the most attention of a sample of tokens (16 of each block)."""
    B, H, L, D = q.shape
    block, nb = case["block"], _nb(case)
    lo, hi = _text_blocks(case)
    st = block // 16
    masks = []
    for b in range(B):
        for h in range(H):
            qs, ks = q[b, h, ::st].float(), k[b, h, ::st].float()
            mass = torch.empty(nb, nb, device=DEV)
            for p in range(0, nb, 128):
                s = (qs[p * 16:(p + 128) * 16] @ ks.t()) * (D ** -0.5)
                w = _blocks_of(torch.softmax(s, dim=1), nb, 16)
                mass[p:p + 128] = _blocks_of(w.t().contiguous(), -(-w.shape[0] // 16), 16).t()
            mass[:, lo:hi + 1] = float("inf")
            m = torch.zeros(nb, nb, dtype=torch.bool, device=DEV)
            m.scatter_(1, torch.topk(mass, _counts(case)[h], dim=1).indices, True)
            m[lo:hi + 1] = True
            masks.append(m)
    m = torch.cat(masks)
    row_ptr = torch.zeros(B * H * nb + 1, dtype=torch.int32, device=DEV)
    row_ptr[1:] = m.sum(1).cumsum(0)
    return row_ptr, m.nonzero()[:, 1].to(torch.int32).contiguous()


def _masses(case, seed):
    """Block masses with the diagonal, stripes and tails of real heads."""
    B, H, nb = case["batch"], case["heads"], _nb(case)
    per = max(1.0, case["patches"] / case["block"])            # blocks per frame
    i = torch.arange(nb, device=DEV, dtype=torch.float32)
    d = (i[:, None] - i[None, :]).abs()
    stripe = torch.cos(d * (2 * math.pi / per)) * 1.5 - torch.log1p(d / per)
    g = _gen(seed, 2)
    w = torch.empty(B, H, nb, nb, device=DEV)
    for b in range(B):
        for h in range(H):
            x = torch.randn(nb, nb, generator=g, device=DEV) + stripe * (0.5 + 1.5 * h / max(1, H - 1))
            w[b, h] = torch.softmax(x, dim=1) * case["block"]
    return w


def _inputs(case, seed):
    """The inputs alone, made with plain torch."""
    kind = case["kind"]
    s = {}
    if kind == "select":
        s["scores"] = _masses(case, seed)
        return s
    s["q"], s["k"], s["v"] = _qkv(case, seed)
    if kind == "cached":
        s["lse"] = _kept_lse(s["q"], s["k"], case["head_dim"] ** -0.5)
    elif kind == "sparse":
        s["row_ptr"], s["col_idx"] = _pattern(case, s["q"], s["k"])
    elif kind == "denoise":
        # Later steps drift away from the first one.
        g = _gen(seed, 3)
        for n in "qkv":
            e = torch.randn(s[n].shape, generator=g, device=DEV)
            s[n] = [(s[n] + 0.05 * t * e).to(torch.bfloat16) for t in range(DENOISE_STEPS)]
    return s


def _select_args(case):
    ts, tl = _text(case)
    a = dict(block=case["block"], text_start=ts, text_len=tl, mode=case["mode"])
    if case["mode"] == "hierarchical":
        a.update(base_sparsity_bp=10000 - case["keep_bp"], recall_threshold_bp=8000)
    else:
        a.update(head_param_bp=_params(case))
    return a


def _result(case, shape, a):
    """The search result a program keeps and has refilled (zeros past the
    entries in use, so that the whole buffer has defined contents)."""
    B, H, L, D = shape
    nb = _nb(case)
    if case["mode"] == "topk":
        size = ad.block_search_capacity(shape, a["block"], a["text_start"], a["text_len"], "topk", a["head_param_bp"])
    else:
        size = B * H * nb * nb
    return ad.SearchResult(torch.empty(B, H, nb, nb, device=DEV),
                           torch.empty(B * H * nb + 1, dtype=torch.int32, device=DEV),
                           torch.zeros(size, dtype=torch.int32, device=DEV),
                           torch.empty(B, H, dtype=torch.int32, device=DEV),
                           torch.empty(B, H, dtype=torch.float32, device=DEV))


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    shape = (case["batch"], case["heads"], case["seqlen"], case["head_dim"])
    s["kind"], s["shape"] = kind, shape
    if kind == "dense":
        # The work queues' counters are kept, as AdaSpaAttention keeps them.
        s["ws"] = torch.empty(ad.dense_attn_workspace(shape), dtype=torch.uint8, device=DEV)
    elif kind == "sparse":
        s["ws"] = torch.empty(ad.block_sparse_attn_workspace(shape, case["block"]), dtype=torch.uint8, device=DEV)
        ts, tl = _text(case)
        s["args"] = dict(block=case["block"], text_start=ts, text_len=tl)
    elif kind == "denoise":
        a = _select_args(case)
        s["layer"] = AdaSpaAttention(shape, schedule=SearchSchedule(DENOISE_SEARCH), device=DEV + ":0", **a)
    else:
        a = s["args"] = _select_args(case)
        ws_args = (shape, a["block"], a["text_start"], a["text_len"], a["mode"], a.get("head_param_bp"))
        size = (ad.single_pass_online_search_workspace if kind == "single" else ad.block_search_workspace)(*ws_args)
        s["ws"] = torch.empty(size, dtype=torch.uint8, device=DEV)
        if kind != "select":                # with scores given the outputs are new ones
            s["result"] = _result(case, shape, a)
    return s


def _search_out(r):
    return dict(block_mass=r.block_mass, row_ptr=r.row_ptr, col_idx=r.col_idx, head_k=r.head_k,
                head_recall=r.head_recall)


def run(s):
    kind = s["kind"]
    if kind == "dense":
        out, lse = ad.dense_attn_lse(s["q"], s["k"], s["v"], workspace=s["ws"])
        return dict(out=out, lse=lse)
    if kind == "sparse":
        out, lse = ad.block_sparse_attn(s["q"], s["k"], s["v"], s["row_ptr"], s["col_idx"], workspace=s["ws"],
                                        **s["args"])
        return dict(out=out, lse=lse)
    if kind == "single":
        out, lse, r = ad.single_pass_online_search(s["q"], s["k"], s["v"], workspace=s["ws"], result=s["result"],
                                                   **s["args"])
        return dict(out=out, lse=lse, **_search_out(r))
    if kind == "cached":
        return _search_out(ad.block_search(s["q"], s["k"], s["lse"], workspace=s["ws"], result=s["result"],
                                           **s["args"]))
    if kind == "select":
        r = ad.block_search(None, None, None, scores=s["scores"], shape=s["shape"], workspace=s["ws"], **s["args"])
        return dict(row_ptr=r.row_ptr, col_idx=r.col_idx, head_k=r.head_k, head_recall=r.head_recall)
    layer, outs = s["layer"], {}
    for t in range(DENOISE_STEPS):
        outs["out%d" % t], _ = layer.step(t, s["q"][t], s["k"][t], s["v"][t])
    return dict(outs, lse=layer.lse, **_search_out(layer.search))


# --- work and tolerance ------------------------------------------------------

def work(case):
    B, H, L, D, nb = case["batch"], case["heads"], case["seqlen"], case["head_dim"], _nb(case)
    lo, hi = _text_blocks(case)
    nt = hi - lo + 1
    row = 2.0 * B * H * L * D                       # bytes of one of q, k, v, o
    lse = 4.0 * B * H * L
    mass = 4.0 * B * H * nb * nb
    if case["mode"] == "topk":
        nnz = float(B * sum(nt * nb + (nb - nt) * k for k in _counts(case)))
    elif case["mode"] == "hierarchical":
        nnz = float(B * H * (nt * nb + (nb - nt) * nb * case["keep_bp"] / 10000))
    else:                                           # a count that only the search finds
        nnz = 0.1 * B * H * nb * nb
    csr = 4.0 * (nnz + B * H * nb)
    full = 4.0 * B * H * L * L * D
    sparse = 4.0 * D * min(nnz * case["block"] ** 2, float(B * H) * L * L)
    kind = case["kind"]
    if kind == "dense":
        return dict(bytes=4 * row + lse, flops=full)
    if kind == "single":
        return dict(bytes=4 * row + lse + mass + csr, flops=full)
    if kind == "cached":
        return dict(bytes=2 * row + lse + mass + csr, flops=full / 2)
    if kind == "select":
        return dict(bytes=mass + csr, flops=0)
    if kind == "sparse":
        return dict(bytes=4 * row + csr + lse, flops=sparse)
    n_sparse = DENOISE_STEPS - 1
    return dict(bytes=4 * row * DENOISE_STEPS + 2 * lse + 2 * mass + csr * (n_sparse + 2),
                flops=full + full / 2 + n_sparse * sparse)


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    # bf16 outputs are 1.7e-3 off the 64-bit result (one rounding of each
    # weight and one of the result), the LSE of the rounded weights 3e-5.
    if case["kind"] in ("dense", "sparse"):
        return dict(rel=7e-3, max=0.05)
    # Masses are fp32 sums, 1e-7 off; blocks of nearly equal mass may change
    # places in the lists.
    if case["kind"] == "cached":
        return dict(rel=2e-6, max=5e-5, differ=2e-3)
    return dict(rel=7e-3, max=0.1, differ=2e-3)


# --- the same in 64 bits -------------------------------------------------------

def _attn64(case, q, k, v, mask=None, masses=False, rows=2048):
    """Attention of one head in 64 bits: out, lse and (with masses) the block
    masses; mask [NB, NB] keeps blocks."""
    L, D, block, nb = q.shape[0], q.shape[1], case["block"], _nb(case)
    k, v = k.double(), v.double()
    out = torch.empty(L, D, dtype=torch.float64, device=DEV)
    lse = torch.empty(L, dtype=torch.float64, device=DEV)
    mass = torch.empty(nb, nb, dtype=torch.float64, device=DEV) if masses else None
    for r in range(0, L, rows):
        s = (q[r:r + rows].double() * D ** -0.5) @ k.t()
        n = s.shape[0]
        if mask is not None:
            keep = mask[r // block:-(-(r + n) // block)]
            keep = keep.repeat_interleave(block, 0)[:n].repeat_interleave(block, 1)[:, :L]
            s.masked_fill_(~keep, float("-inf"))
        m = s.amax(1, keepdim=True)
        s.sub_(m).exp_()
        t = s.sum(1, keepdim=True)
        out[r:r + n] = (s @ v) / t
        lse[r:r + n] = (m + t.log())[:, 0]
        if masses:
            w = _blocks_of(s.div_(t), nb, block)
            mass[r // block:-(-(r + n) // block)] = _blocks_of(w.t(), -(-n // block), block).t()
    return out, lse, mass


def _mass64(case, q, k, lse, rows=2048):
    L, D, block, nb = q.shape[0], q.shape[1], case["block"], _nb(case)
    k, lse = k.double(), lse.double()
    mass = torch.empty(nb, nb, dtype=torch.float64, device=DEV)
    for r in range(0, L, rows):
        s = ((q[r:r + rows].double() * D ** -0.5) @ k.t()).sub_(lse[r:r + rows, None]).exp_()
        n = s.shape[0]
        w = _blocks_of(s, nb, block)
        mass[r // block:-(-(r + n) // block)] = _blocks_of(w.t(), -(-n // block), block).t()
    return mass


def _kept64(case, mass, sizes):
    """Block masks of top-k selection with the given counts, [heads, NB, NB]."""
    lo, hi = _text_blocks(case)
    masks = []
    for w, n in zip(mass, sizes):
        w = w.clone()
        w[:, lo:hi + 1] = float("inf")
        m = torch.zeros(w.shape, dtype=torch.bool, device=DEV)
        m.scatter_(1, torch.sort(w, dim=1, descending=True, stable=True).indices[:, :n], True)
        m[lo:hi + 1] = True
        masks.append(m)
    return masks


def _recall64(case, mass):
    """Recall of each head [B, H] at the count its mode gives."""
    B, H, nb, _ = mass.shape
    lo, hi = _text_blocks(case)
    curve = torch.empty(B, H, nb, dtype=torch.float64, device=DEV)
    for b in range(B):
        for h in range(H):
            w = mass[b, h].double()
            x = w.clone()
            x[:, lo:hi + 1] = float("inf")
            order = torch.sort(x, dim=1, descending=True, stable=True).indices
            c = torch.gather(w, 1, order).cumsum(1)
            c[lo:hi + 1] = w[lo:hi + 1].sum(1, keepdim=True)
            curve[b, h] = c.sum(0)
    curve /= curve[..., -1:].clone()
    nt = hi - lo + 1
    if case["mode"] == "topk":
        n = torch.tensor(_counts(case), device=DEV).expand(B, H)
    elif case["mode"] == "coverage":
        n = ((curve < case["keep_bp"] / 10000).sum(2) + 1).clamp(max(1, nt), nb)
    else:
        s_bp = 10000 - case["keep_bp"]
        count = lambda bp: min(nb, max(1, nt, -(-bp * nb // 10000)))  # noqa: E731
        base = count(10000 - s_bp)
        few, many = count(10000 - (10000 + s_bp) // 2), count(10000 - max(0, 3 * s_bp - 10000) // 2)
        at = curve[..., base - 1]
        n = torch.full((B, H), base, device=DEV)
        for b in range(B):
            move = min(int((at[b] > 0.8).sum()), H // 2)
            order = torch.sort(at[b], descending=True, stable=True).indices
            n[b, order[:move]] = few
            n[b, order[H - move:]] = many
    return torch.gather(curve, 2, (n - 1).unsqueeze(2))[..., 0]


def exact(case, seed):
    kind = case["kind"]
    B, H, L, D, nb = case["batch"], case["heads"], case["seqlen"], case["head_dim"], _nb(case)
    none = dict(row_ptr=None, col_idx=None, head_k=None)
    s = _inputs(case, seed)
    if kind == "select":
        return dict(none, head_recall=_recall64(case, s["scores"]))
    if kind == "cached":
        mass = torch.stack([torch.stack([_mass64(case, s["q"][b, h], s["k"][b, h], s["lse"][b, h])
                                         for h in range(H)]) for b in range(B)])
        return dict(none, block_mass=mass, head_recall=_recall64(case, mass))

    def layer(q, k, v, masks=None, masses=False):
        out = torch.empty(B, H, L, D, dtype=torch.float64, device=DEV)
        lse = torch.empty(B, H, L, dtype=torch.float64, device=DEV)
        mass = torch.empty(B, H, nb, nb, dtype=torch.float64, device=DEV) if masses else None
        for b in range(B):
            for h in range(H):
                o, l, w = _attn64(case, q[b, h], k[b, h], v[b, h], None if masks is None else masks[b * H + h],
                                  masses)
                out[b, h], lse[b, h] = o, l
                if masses:
                    mass[b, h] = w
        return out, lse, mass

    if kind == "dense":
        out, lse, _ = layer(s["q"], s["k"], s["v"])
        return dict(out=out, lse=lse)
    if kind == "sparse":
        rp, ci = s["row_ptr"].long(), s["col_idx"].long()
        mask = torch.zeros(B * H * nb, nb, dtype=torch.bool, device=DEV)
        mask[torch.repeat_interleave(torch.arange(B * H * nb, device=DEV), rp[1:] - rp[:-1]), ci] = True
        out, lse, _ = layer(s["q"], s["k"], s["v"], mask.view(B * H, nb, nb))
        return dict(out=out, lse=lse)
    if kind == "single":
        out, lse, mass = layer(s["q"], s["k"], s["v"], masses=True)
        return dict(none, out=out, lse=lse, block_mass=mass, head_recall=_recall64(case, mass))
    outs, masks, mass0, lse0 = {}, None, None, None
    for t in range(DENOISE_STEPS):
        q, k, v = s["q"][t], s["k"][t], s["v"][t]
        if t == DENOISE_SEARCH[0]:
            outs["out%d" % t], lse0, mass0 = layer(q, k, v, masses=True)
            masks = _kept64(case, mass0.flatten(0, 1).float(), _counts(case) * B)
            continue
        if t in DENOISE_SEARCH:
            mass0 = torch.stack([torch.stack([_mass64(case, q[b, h], k[b, h], lse0[b, h]) for h in range(H)])
                                 for b in range(B)])
            masks = _kept64(case, mass0.flatten(0, 1).float(), _counts(case) * B)
        outs["out%d" % t], _, _ = layer(q, k, v, masks)
    return dict(none, **outs, lse=lse0, block_mass=mass0, head_recall=_recall64(case, mass0))
