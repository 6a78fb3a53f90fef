"""Block selection at the sizes where its kernels change: one key per lane and
one more, every step of the keys a lane holds, the longest row sorted in a
wave's registers and the shortest one sorted in LDS, rows of one block, partial
curves added up by a launch of their own and by the head's workgroup, and more
heads than a row's wave adds up by itself.  Masses hold ties and every
special value (NaN, infinities, zeros of both signs, negatives, subnormals,
masses past the exact sums' cap, halves of the last kept bit).  Everything is
bit-exact against the oracle on the same scores."""
import numpy as np
import pytest
import torch

import oracle
import paper_2502_21079_amd as ad
from workloads import random_block_masses
from test_search_gpu import _compare_selection

pytestmark = pytest.mark.gpu

SPECIAL = [float("nan"), float("inf"), -float("inf"), 0.0, -0.0, -1.0, 1e-40, -1e-40, 1e30, 2.0 ** -33, 3 * 2.0 ** -33,
           2.0 ** -32, (2 ** 24 - 1) * 2.0 ** -56, 2.0 ** 23 + 1, 0.1, 0.1]


def _masses(B, H, nb, seed):
    W = random_block_masses((B, H, nb, nb), seed=seed, ties=False)
    T = random_block_masses((B, H, nb, nb), seed=seed + 1, ties=True)
    W[:, :, 1::3] = T[:, :, 1::3]                       # every third row: a handful of levels
    n = min(nb, len(SPECIAL))
    g = np.random.default_rng(seed)
    for p in range(2, nb, 3):                           # every third row: special values anywhere
        W[:, :, p, torch.as_tensor(g.choice(nb, n, replace=False))] = torch.tensor(SPECIAL[:n])
    return W


# (blocks per row, batch, heads, first text block, text blocks)
CASES = [(1, 1, 3, 0, 0), (1, 1, 2, 0, 1), (2, 1100, 2, 0, 1), (63, 2, 3, 62, 1), (64, 1, 4, 0, 2), (65, 1, 2, 64, 1),
         (128, 1, 2, 3, 4), (129, 1, 2, 0, 3), (257, 1, 3, 250, 7), (513, 1, 2, 0, 4), (897, 1, 1, 0, 2),
         (1281, 1, 1, 1277, 4)]
LONG = [(1729, "coverage"), (2048, "coverage"), (2049, "coverage"), (2049, "hierarchical"), (2689, "topk")]


def _check(nb, B, H, t0, nt, mode):
    L = nb * 64 - (17 if nb > 1 else 0)
    W = _masses(B, H, nb, seed=nb + H)
    tok = (t0 * 64, min(nt * 64, L - t0 * 64))
    kw = dict(head_param_bp=None, base_sparsity_bp=8000, recall_threshold_bp=6000)
    if mode != "hierarchical":
        kw = dict(head_param_bp=[(700 + 2900 * h) % 10001 if mode == "topk" else 9000 - 800 * h for h in range(H)])
    res = ad.block_search(None, None, None, block=64, text_start=tok[0], text_len=tok[1], mode=mode,
                          scores=W.cuda(), shape=(B, H, L, 64), **kw)
    torch.cuda.synchronize()
    if mode == "hierarchical":
        sel = oracle.select_blocks(W.numpy(), L, 64, tok[0], tok[1], mode, [0] * H, base_sparsity_bp=8000,
                                   recall_threshold_bp=6000)
    else:
        sel = oracle.select_blocks(W.numpy(), L, 64, tok[0], tok[1], mode, kw["head_param_bp"])
    _compare_selection(res, sel)


@pytest.mark.parametrize("mode", ["topk", "coverage", "hierarchical"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "nb%d_B%d_H%d" % c[:3])
def test_selection_at_the_kernels_edges(case, mode):
    _check(*case, mode)


@pytest.mark.parametrize("nb,mode", LONG)
def test_selection_of_long_rows(nb, mode):
    _check(nb, 1, 1, 0, 4, mode)


def test_two_long_rows_per_workgroup():
    """Four heads of 2,049 rows are the fewest long rows of which a workgroup of
    the coverage curve takes two (the last one of a head has a single row)."""
    _check(2049, 1, 4, 0, 4, "coverage")
