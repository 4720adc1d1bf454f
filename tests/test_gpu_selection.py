"""The choice of the k best pages, at list lengths on both sides of every rule that divides the work -- rows of candidates per
thread, one block or several per head, what the blocks hand on -- and with ties, which leave the short way of ranking."""
import numpy as np
import pytest
import torch

import paper_2505_13109_amd as fkv
from paper_2505_13109_amd import binding as B

pytestmark = pytest.mark.gpu


def _best(score, k):
    """ids (from 0) of the k largest, ties to the lower id, ascending"""
    order = np.lexsort((np.arange(len(score)), -score.astype(np.float64)))
    return np.sort(order[:k])


@pytest.mark.parametrize("levels", [0, 1, 7])            # values the keys of a page take: random, all pages alike, seven kinds of pages
@pytest.mark.parametrize("G,n_kv,batch,n_cand,k", [
    (4, 2, 1, 5, 5),           # nothing to choose
    (4, 2, 1, 64, 63),         # one wave
    (1, 1, 1, 513, 40),        # one block: two rows, the second with one candidate
    (4, 2, 1, 1537, 97),       # four rows
    # (of more than eight heads; with two, both of these are shared, and test_gpu_selection_rows.py has them with nine)
    (5, 1, 2, 1880, 31),       # 9400 numerators: the most that one block takes
    (5, 1, 2, 1881, 31),       # shared by eight blocks, every key handed on
    (2, 3, 1, 4096, 33),       # eight rows
    (2, 3, 1, 4097, 33),       # sixteen blocks, each hands on its best
    (3, 1, 1, 2563, 700),      # ... eight blocks, which hand on everything, more than the last one's registers hold
    (8, 1, 1, 2400, 150),      # eight blocks of 300 with 150 each: in registers
    (8, 1, 1, 5100, 200),      # sixteen, 200 of 319 each: more than the registers hold
    (6, 40, 1, 2300, 20),      # many heads: two blocks each
    (1, 16, 16, 600, 50),      # selection in a launch of its own
    (4, 16, 8, 2600, 40),      # ... and two blocks per head
])
def test_the_best_pages_of_a_list(G, n_kv, batch, n_cand, k, levels):
    _check(G, n_kv, batch, n_cand, k, levels, "MeanS")


@pytest.mark.parametrize("levels", [0, 1, 7])
@pytest.mark.parametrize("pooling", ["MeanQK", "MaxQ"])  # scores of either sign, hundreds of them of one exponent
@pytest.mark.parametrize("G,n_kv,batch,n_cand,k", [
    (4, 2, 1, 64, 63),         # one wave
    (4, 2, 1, 150, 20),        # three: fewer threads than counters
    (4, 2, 1, 992, 32),
    (5, 1, 2, 1880, 500),
    (2, 3, 1, 4097, 33),       # sixteen blocks, each hands on its best
    (8, 1, 1, 2400, 150),
    (8, 1, 1, 5100, 200),      # more than the registers hold
    (1, 16, 16, 600, 50),      # selection in a launch of its own
])
def test_the_best_pages_by_other_scores(G, n_kv, batch, n_cand, k, pooling, levels):
    _check(G, n_kv, batch, n_cand, k, levels, pooling)


def _check(G, n_kv, batch, n_cand, k, levels, pooling):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_cand + levels)
    pages = n_cand + 4
    ctx = pages * 32
    if levels:
        kind = torch.randint(0, levels, (batch, pages, 1, n_kv, 1), device="cuda", generator=gen).to(torch.bfloat16)
        K = (1.0 + 0.25 * kind).expand(batch, pages, 32, n_kv, 128).reshape(batch, ctx, n_kv, 128).contiguous()
    else:
        K = torch.randn((batch, ctx, n_kv, 128), dtype=torch.bfloat16, device="cuda", generator=gen)
    q = torch.randn((batch, G * n_kv, 128), device="cuda", generator=gen).to(torch.bfloat16)
    g = fkv.FreeKV(n_layers=1, batch=batch, n_q_heads=G * n_kv, n_kv_heads=n_kv, max_ctx=ctx + 32, budget=128 + 32 * k, sink=64, window=64,
                   tau=0.8, dtype="bf16", select_pooling=pooling)
    g.load_prefix(0, K, K)
    new = torch.zeros((batch, n_kv, 128), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((batch, G * n_kv, 128), device="cuda")
    ids = torch.full((batch, n_kv, k), -1, dtype=torch.int32, device="cuda")
    g.page_select(0, q, ids)
    score, own = g.debug_read(0, B.DBG_SCORES), ids.cpu().numpy()
    for b in range(batch):
        for m in range(n_kv):
            assert np.array_equal(own[b, m], 2 + _best(score[b, m, 2:2 + n_cand], k)), (b, m)
    # the layer-step, in one launch where the shape takes one, scores and chooses alike
    g.decode_step(0, q, new, new, out)
    assert np.array_equal(g.debug_read(0, B.DBG_SCORES)[..., 2:2 + n_cand], score[..., 2:2 + n_cand])
    assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS), own)
    g.health(0)
    g.close()
