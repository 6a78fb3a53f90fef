"""Key-split attention (four waves share each row's keys) at the edges of its
use: one tile and fewer, every remainder of the 128-key units over the four
splits, ragged lengths, sequences that stop short of a block, rows with fewer
tiles than splits and empty rows, malformed lists, inputs that send single
splits to the exact path, the last items of a launch that run key-split beside
whole ones, and block-sparse patterns on both sides of the choice by density.
Expected values come from the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_21079_amd as ad
from workloads import TINY, make_extreme_qkv, make_qkv, text_blocks
from _helpers import check_lse, check_mass, check_out, f64, oracle_rows, sample_blocks

pytestmark = pytest.mark.gpu


def _w(D, L, heads=2, block=128, text=0):
    return TINY.replace(head_dim=D, seqlen=L, heads=heads, block=block, text_len=min(text, L), frames=4,
                        patches=max(1, (L - min(text, L) + 3) // 4))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("L", [1, 31, 33, 64, 127, 129, 383, 512, 545, 640, 1152, 1663])
def test_dense_every_row(D, L):
    w = _w(D, L)
    q, k, v = make_qkv(w, device="cuda")
    out, lse = ad.dense_attn_lse(q, k, v)
    torch.cuda.synchronize()
    for h in range(w.heads):
        o_ref, l_ref = oracle.dense_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h]), w.scale)
        check_out(out[0, h], o_ref, f"h{h}")
        check_lse(lse[0, h], l_ref, f"h{h}")


@pytest.mark.parametrize("D,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("L", [200, 1090, 1472])
def test_single_pass_masses(D, block, L):
    """Block masses taken by the wave that owns the block's unit: whole and
    partial blocks, with and without a masked tile."""
    w = _w(D, L, block=block, text=64)
    q, k, v = make_qkv(w, device="cuda")
    out, lse, res = ad.single_pass_online_search(q, k, v, block=block, text_start=0, text_len=64, mode="topk",
                                                 head_param_bp=[3000] * w.heads)
    torch.cuda.synchronize()
    for h in range(w.heads):
        qh, kh, vh = f64(q[0, h]), f64(k[0, h]), f64(v[0, h])
        o_ref, l_ref = oracle.dense_attention(qh, kh, vh, w.scale)
        check_out(out[0, h], o_ref, f"h{h}")
        check_mass(res.block_mass[0, h], oracle.block_mass(qh, kh, l_ref, w.scale, block), f"h{h}")


def _csr(lists):
    rp = torch.tensor([0] + list(np.cumsum([len(x) for x in lists])), dtype=torch.int32)
    return rp.cuda(), torch.tensor([c for x in lists for c in x], dtype=torch.int32).cuda()


@pytest.mark.parametrize("D,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
def test_sparse_short_empty_and_malformed_rows(D, block):
    """Rows of 0 to all blocks, the ragged block last, inside a row or alone,
    out-of-range entries, and lists out of order."""
    L = block * 13 + 37
    w = _w(D, L, block=block)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    g = np.random.default_rng(D + block)
    lists = [sorted(g.choice(nb, p % (nb + 1), replace=False).tolist()) for p in range(w.heads * nb)]
    lists[3], lists[4], lists[5] = [nb - 1], [2, nb - 1, 5], [nb - 1, 0]
    lists[6], lists[7] = [-1, 3, nb, 1], [9, 4, 7, 0]
    lists[8] = list(range(nb))[::-1]
    out, lse = ad.block_sparse_attn(q, k, v, *_csr(lists), block=block)
    torch.cuda.synchronize()
    for r, kept in enumerate(lists):
        h, p = divmod(r, nb)
        rows = slice(p * block, min((p + 1) * block, L))
        valid = [c for c in kept if 0 <= c < nb]
        o_ref, l_ref = oracle.masked_attention(f64(q[0, h, rows]), f64(k[0, h]), f64(v[0, h]),
                                               oracle.key_mask_from_blocks(valid, L, block), w.scale)
        check_out(out[0, h, rows], o_ref, f"row {r}")
        check_lse(lse[0, h, rows], l_ref, f"row {r}")


@pytest.mark.parametrize("D", [64, 128])
def test_long_lists_move_the_index_window(D):
    """Lists of more than two chunks of 64 entries, of every length modulo a
    round of the splits: the window of indices moves along the row in each
    wave."""
    L = 64 * 200
    w = _w(D, L, heads=1, block=64)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    g = np.random.default_rng(D)
    lists = [sorted(g.choice(nb, 120 + p % 80, replace=False).tolist()) for p in range(nb)]
    out, lse = ad.block_sparse_attn(q, k, v, *_csr(lists), block=64)
    torch.cuda.synchronize()
    rpn = np.concatenate([[0], np.cumsum([len(x) for x in lists])])
    blocks = sample_blocks(nb, 24, seed=D)
    o_ref, l_ref = oracle.block_sparse_attention(f64(q[0, 0]), f64(k[0, 0]), f64(v[0, 0]), rpn,
                                                 np.concatenate(lists).astype(np.int32), w.scale, 64, qblocks=blocks)
    idx = torch.as_tensor(np.concatenate([np.arange(p * 64, p * 64 + 64) for p in blocks]), device="cuda")
    check_out(out[0, 0, idx], o_ref)
    check_lse(lse[0, 0, idx], l_ref)


@pytest.mark.parametrize("D", [64, 128])
def test_one_split_on_the_exact_path(D):
    """Scores that jump by far more than the lazy reference allows in the keys
    of a single split: that split's waves redo their tiles, the others do
    not, and the merged rows match the oracle."""
    L = 1100
    (q, k, v), scale = make_extreme_qkv("negative", heads=2, seqlen=L, head_dim=D, device="cuda")
    k = k.clone()
    k[:, :, 330:370] *= -0.9                    # the second 64 keys of the third unit of 128
    # The unit's first tile sets its wave's reference, the jump comes after it
    # and passes the 2^100 at which a sum is redone.
    rows = (q[0, :, ::50].float() @ k[0, :, 256:384].float().transpose(1, 2)) * (scale * 1.4427)
    assert float((rows[..., 64:].amax(2) - rows[..., :64].amax(2)).min()) > 110
    out, lse = ad.dense_attn_lse(q, k, v, scale=scale)
    torch.cuda.synchronize()
    for h in range(2):
        o_ref, l_ref = oracle.dense_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h]), scale)
        check_out(out[0, h], o_ref, f"h{h}")
        check_lse(lse[0, h], l_ref, f"h{h}")


# Items of 256 rows: 256 + 64 (the most that run key-split) and + 65 (none) at
# either d, at d 64 just below the length from which they do, + 128, + 129, + 1.
TAILS = [(128, 20, 4090), (128, 107, 700), (64, 107, 700), (64, 24, 4000), (64, 77, 1200), (128, 257, 70),
         (64, 10, 8192), (64, 10, 8191), (64, 3, 27301)]


@pytest.mark.parametrize("D,heads,L", TAILS)
def test_tail_items(D, heads, L):
    """The last items of a launch that fills the chip once: every entry point
    splits the same rows (outputs equal bit for bit), whatever the groups the
    single pass runs in, and the rows match the oracle."""
    w = _w(D, L, heads=heads, text=64)
    q, k, v = make_qkv(w, device="cuda")
    out, lse = ad.dense_attn_lse(q, k, v)
    kw = dict(block=128, text_start=0, text_len=64, mode="topk", head_param_bp=[3000] * heads)
    o0, l0 = ad.dense_attn_lse(q, k, v, balance=False)
    full = ad.single_pass_online_search_workspace(q.shape, 128, 0, 64, "topk", [3000] * heads)
    least = ad.single_pass_online_search_min_workspace(q.shape, 128, 0, 64, "topk", [3000] * heads)
    runs = [ad.single_pass_online_search(q, k, v, workspace=torch.empty(n, dtype=torch.uint8, device="cuda"), **kw)
            for n in (full, least + (full - least) // 3)]
    of, lf, rf = ad.fused_online_search(q, k, v, **kw)
    on, ln, rn = ad.fused_online_search(q, k, v, want_lse=False, **kw)
    two = ad.block_search(q, k, lse, **kw)
    torch.cuda.synchronize()
    assert torch.equal(out, o0) and torch.equal(lse, l0)
    for o, l, _ in runs:
        assert torch.equal(out, o) and torch.equal(lse, l)
    assert torch.equal(runs[0][2].block_mass, runs[1][2].block_mass)
    assert torch.equal(out, of) and torch.equal(lse, lf) and torch.equal(out, on) and ln is None
    assert torch.equal(rf.block_mass, two.block_mass) and torch.equal(rn.block_mass, two.block_mass)
    for h in (0, heads // 2, heads - 1):
        rows = np.unique(np.concatenate([np.arange(min(40, L)), np.arange(max(0, L - 300), L)]))
        o_ref, l_ref = oracle_rows(q, k, v, (0, h), rows, w.scale)
        idx = torch.as_tensor(rows, device="cuda")
        check_out(out[0, h, idx], o_ref, f"h{h}")
        check_lse(lse[0, h, idx], l_ref, f"h{h}")


@pytest.mark.parametrize("D,heads,L", TAILS)
@pytest.mark.parametrize("block", [64, 128])
def test_all_blocks_equal_dense_with_tail_items(D, heads, L, block):
    """Keeping every block is dense attention bit for bit also where dense runs
    its last items key-split: block-sparse attention splits the same rows of
    such a pattern, with and without a text range or a workspace.  A pattern
    that leaves out one block of one row is no such pattern."""
    w = _w(D, L, heads=heads, block=block)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    od, ld = ad.dense_attn_lse(q, k, v)
    rp = torch.arange(heads * nb + 1, dtype=torch.int32, device="cuda") * nb
    ci = torch.arange(nb, dtype=torch.int32, device="cuda").repeat(heads * nb)
    for kw in (dict(), dict(text_start=0, text_len=min(200, L)), dict(balance=False)):
        out, lse = ad.block_sparse_attn(q, k, v, rp, ci, block=block, **kw)
        torch.cuda.synchronize()
        assert torch.equal(out, od) and torch.equal(lse, ld), kw
    if nb > 1:
        rp2 = rp.clone()
        rp2[-1] -= 1                               # the last row without its last block
        out, lse = ad.block_sparse_attn(q, k, v, rp2, ci, block=block)
        torch.cuda.synchronize()
        rows = np.arange((nb - 1) * block, L)
        o_ref, l_ref = oracle.masked_attention(f64(q[0, -1, rows]), f64(k[0, -1]), f64(v[0, -1]),
                                               oracle.key_mask_from_blocks(list(range(nb - 1)), L, block), w.scale)
        check_out(out[0, -1, rows], o_ref)
        check_lse(lse[0, -1, rows], l_ref)
        whole = (nb - 1) * block                   # the other rows keep everything
        check_out(out[0, :, :whole], f64(od[0, :, :whole]))


@pytest.mark.parametrize("D,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("kept,room", [(3, False), (3, True), (40, True), ("all", False)])
def test_sparse_pick_by_density(D, block, kept, room):
    """Mid-size problems with a text range: sparse video rows beside complete
    text rows (key-split), dense ones and all blocks kept (one row per
    workgroup), with a col_idx of the pattern's size and one with room for
    every block."""
    L = 9000
    w = _w(D, L, heads=5, block=block, text=200)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    tb = text_blocks(L, block, 0, 200)
    n = nb if kept == "all" else kept * (128 // block)
    g = np.random.default_rng(block + D)
    lists = [list(range(nb)) if r % nb in tb or n >= nb else
             sorted(set(tb) | set(g.choice(nb, n, replace=False).tolist())) for r in range(w.heads * nb)]
    rp, ci = _csr(lists)
    if room:
        ci = torch.cat([ci, ci.new_full((w.heads * nb * nb - ci.numel(),), -7)])
    out, lse = ad.block_sparse_attn(q, k, v, rp, ci, block=block, text_start=0, text_len=200)
    torch.cuda.synchronize()
    if kept == "all":
        od, ld = ad.dense_attn_lse(q, k, v)
        assert torch.equal(out, od) and torch.equal(lse, ld)
    rpn, cin = rp.cpu().numpy(), ci.cpu().numpy()
    for h in (0, 4):
        blocks = sample_blocks(nb, 6, seed=h, always=(0, 1))
        o_ref, l_ref = oracle.block_sparse_attention(f64(q[0, h]), f64(k[0, h]), f64(v[0, h]),
                                                     rpn[h * nb:(h + 1) * nb + 1], cin, w.scale, block,
                                                     qblocks=blocks)
        rows = np.concatenate([np.arange(p * block, min((p + 1) * block, L)) for p in blocks])
        idx = torch.as_tensor(rows, device="cuda")
        check_out(out[0, h, idx], o_ref, f"h{h}")
        check_lse(lse[0, h, idx], l_ref, f"h{h}")


# (tokens, heads, blocks of 128 kept per video row): patterns that take the key
# split and, the second, one that is too dense for it.
@pytest.mark.parametrize("D,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("L,heads,kept", [(9000, 5, 3), (9000, 5, 30), (16384, 12, 6), (12001, 6, 12)])
@pytest.mark.parametrize("text_first", [True, False])
def test_sparse_results_follow_the_pattern_alone(D, block, L, heads, kept, text_first):
    """A pattern has one result: bit for bit the same whatever text range the
    call names (the right one, none, or one at the other end) and whatever
    room its col_idx has past the last entry."""
    w = _w(D, L, heads=heads, block=block, text=200)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    t0 = 0 if text_first else L - 200
    tb = text_blocks(L, block, t0, 200)
    g = np.random.default_rng(kept + D)
    n = kept * (128 // block)
    lists = [list(range(nb)) if r % nb in tb else
             sorted(set(tb) | set(g.choice(nb, n, replace=False).tolist())) for r in range(heads * nb)]
    rp, ci = _csr(lists)
    roomy = torch.cat([ci, ci.new_full((heads * nb * nb - ci.numel(),), -7)])
    base = None
    for cols in (ci, roomy):
        for start, n_text in ((t0, 200), (0, 0), (L - 200 - t0, 200)):
            res = ad.block_sparse_attn(q, k, v, rp, cols, block=block, text_start=start, text_len=n_text)
            base = base or res
            torch.cuda.synchronize()
            assert torch.equal(res[0], base[0]) and torch.equal(res[1], base[1]), (cols.numel(), start, n_text)


# Without a text range the tiles of 384 rows at both ends come first, from the
# first length with rows between them (769); in blocks of 64 at d 128 up to 1,024
# pairs (128 heads of 8).  The last case has a work queue.
@pytest.mark.parametrize("D,block", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("L,heads", [(768, 48), (769, 48), (900, 43), (1000, 128), (1000, 129), (1025, 300)])
def test_order_without_a_text_range_covers_every_row(D, block, L, heads):
    """Calls with and without a text range run the same rows."""
    w = _w(D, L, heads=heads, block=block, text=100)
    q, k, v = make_qkv(w, device="cuda")
    nb = w.nblocks
    g = np.random.default_rng(L)
    lists = [sorted(g.choice(nb, min(nb, 4), replace=False).tolist()) for _ in range(heads * nb)]
    rp, ci = _csr(lists)
    named = ad.block_sparse_attn(q, k, v, rp, ci, block=block, text_start=0, text_len=100)
    plain = ad.block_sparse_attn(q, k, v, rp, ci, block=block)
    torch.cuda.synchronize()
    assert torch.equal(named[0], plain[0]) and torch.equal(named[1], plain[1])
