"""The choice of the k best pages where its code differs: rows of candidates per thread, waves that are not full, keys that are ranked
against each other or not, scores below the last counter's reach, and what several blocks hand on.  Against the numbers' definition:
the ids by the scores that the library reports, the scores by those of the same list in a launch of another shape."""
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


def _select(G, n_cand, k, K, q, batch=1):
    g = fkv.FreeKV(n_layers=1, batch=batch, n_q_heads=G, n_kv_heads=1, max_ctx=K.shape[1] + 32, budget=128 + 32 * k, sink=64, window=64, tau=0.8)
    g.load_prefix(0, K.expand(batch, -1, -1, -1).contiguous(), K.expand(batch, -1, -1, -1).contiguous())
    ids = torch.full((batch, 1, k), -1, dtype=torch.int32, device="cuda")
    g.page_select(0, q.expand(batch, -1, -1).contiguous(), ids)
    score = g.debug_read(0, B.DBG_SCORES)[:, 0, 2:2 + n_cand]
    g.health(0)
    g.close()
    return ids.cpu().numpy()[:, 0], score


@pytest.mark.parametrize("scale", [0.0, 1.0, 12.0])      # all alike; a softmax over many pages; one whose k-th best is next to nothing
@pytest.mark.parametrize("G,n_cand,k", [
    (4, 1, 1), (4, 63, 7), (4, 65, 64),                   # one wave, two
    (4, 511, 32), (4, 512, 32), (4, 513, 512),            # one row; a second of one candidate
    # (one head: what has more than 16 rows times G is shared; in one block in test_rows_of_one_block)
    (7, 1024, 96), (7, 1025, 3), (7, 1342, 100),          # two rows, three of four, the most that one block has
    (3, 2048, 500), (3, 2049, 64), (3, 3133, 40),         # four rows, eight
    (8, 1300, 65), (5, 2100, 33), (4, 4096, 300),         # in several blocks: every key handed on
    (4, 5000, 32), (4, 8160, 1), (6, 9000, 129),          # ... each block's best
])
def test_rows_waves_and_ranks(G, n_cand, k, scale):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_cand + k)
    K = torch.randn((1, (n_cand + 4) * 32, 1, 128), dtype=torch.bfloat16, device="cuda", generator=gen)
    q = (scale * torch.randn((1, G, 128), device="cuda", generator=gen)).to(torch.bfloat16)
    ids, score = _select(G, n_cand, k, K, q)
    assert np.array_equal(ids[0], 2 + _best(score[0], k))
    # 320 requests with the same list, in a scan and a selection of their own where that is what so many take: the same bits
    if n_cand in (63, 513, 1025):
        many, scores = _select(G, n_cand, k, K, q, batch=320)
        assert np.array_equal(scores, np.broadcast_to(score[0], scores.shape)) and np.array_equal(many, np.broadcast_to(ids[0], many.shape))


@pytest.mark.parametrize("G,n_cand,heads", [
    (3, 2048, 2), (3, 2049, 2), (3, 2300, 9),             # the longest list that one block has, the shortest that several share, heads too many for it
    (2, 2049, 4), (4, 1025, 5), (5, 1024, 1), (5, 1025, 1), (5, 1100, 8), (5, 1100, 9),
    (8, 1025, 3), (8, 1150, 40), (7, 1342, 8),
])
def test_alone_and_shared(G, n_cand, heads):
    """One list per head, cut by the number of heads and candidates: the same scores, bit for bit, as in 96 heads, which have a block each."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_cand * 64 + heads)
    k = 37
    K = torch.randn((1, (n_cand + 4) * 32, 1, 128), dtype=torch.bfloat16, device="cuda", generator=gen)
    q = torch.randn((1, G, 128), device="cuda", generator=gen).to(torch.bfloat16)
    ids, score = _select(G, n_cand, k, K, q, batch=heads)
    many, scores = _select(G, n_cand, k, K, q, batch=96)
    want = 2 + _best(score[0], k)
    assert np.array_equal(ids, np.broadcast_to(want, ids.shape)) and np.array_equal(many, np.broadcast_to(want, many.shape))
    assert np.array_equal(score, np.broadcast_to(score[0], score.shape)) and np.array_equal(scores, np.broadcast_to(score[0], scores.shape))


@pytest.mark.parametrize("scale", [0.0, 1.0, 12.0])
@pytest.mark.parametrize("G,n_cand,k", [
    (7, 1024, 96), (7, 1025, 3), (7, 1342, 100),          # two rows, three of four, the most that one of more than eight heads has
    (3, 2048, 500), (3, 2049, 64), (3, 3133, 40),         # four rows, eight
    (5, 1880, 31), (5, 1881, 31),                         # 9400 softmax numerators; shared
    (4, 2048, 97), (2, 4096, 33),                         # all of the rows there are
])
def test_rows_of_one_block(G, n_cand, k, scale):
    """The same with nine heads, whose lists stay with one block longer than those of up to eight."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_cand + k)
    K = torch.randn((1, (n_cand + 4) * 32, 1, 128), dtype=torch.bfloat16, device="cuda", generator=gen)
    q = (scale * torch.randn((1, G, 128), device="cuda", generator=gen)).to(torch.bfloat16)
    ids, score = _select(G, n_cand, k, K, q, batch=9)
    want = 2 + _best(score[0], k)
    assert np.array_equal(score, np.broadcast_to(score[0], score.shape)) and np.array_equal(ids, np.broadcast_to(want, ids.shape))


@pytest.mark.parametrize("G,n_cand,heads", [
    (8, 1024, 8), (8, 1025, 8), (4, 2048, 8), (4, 2049, 8), (2, 4096, 8), (2, 4097, 8), (3, 2048, 8), (3, 2049, 8),      # rows times G of 16 and above
    (5, 1024, 8), (5, 1025, 8), (5, 1025, 9), (5, 1500, 8), (5, 1500, 9),                                                # eight heads and nine
    (8, 1175, 9), (8, 1176, 9), (3, 3133, 9), (3, 3134, 9),                                                              # 9400 numerators
    (5, 1500, 1), (5, 1500, 3), (5, 1568, 2), (5, 1569, 2), (5, 1800, 6), (5, 1800, 7),                                  # few heads, at home and away
])
def test_either_side_of_the_rules(G, n_cand, heads):
    """A layer-step's ids and scores, one list per head, against those of the same list in page_select with 96 heads."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n_cand * 64 + heads)
    k = 33
    K = torch.randn((1, (n_cand + 4) * 32, 1, 128), dtype=torch.bfloat16, device="cuda", generator=gen)
    q = torch.randn((1, G, 128), device="cuda", generator=gen).to(torch.bfloat16)
    many, scores = _select(G, n_cand, k, K, q, batch=96)
    g = fkv.FreeKV(n_layers=1, batch=heads, n_q_heads=G, n_kv_heads=1, max_ctx=K.shape[1] + 32, budget=128 + 32 * k, sink=64, window=64, tau=0.8)
    full = K.expand(heads, -1, -1, -1).contiguous()
    g.load_prefix(0, full, full)
    new, out = torch.zeros((heads, 1, 128), dtype=torch.bfloat16, device="cuda"), torch.empty((heads, G, 128), device="cuda")
    g.decode_step(0, q.expand(heads, -1, -1).contiguous(), new, new, out)
    ids, score = g.debug_read(0, B.DBG_ACTIVE_IDS)[:, 0], g.debug_read(0, B.DBG_SCORES)[:, 0, 2:2 + n_cand]
    assert np.array_equal(score, np.broadcast_to(scores[0], score.shape)) and np.array_equal(ids, np.broadcast_to(many[0], ids.shape))
    assert g.test_by_itself(0)[0] == 0                       # no block had to do without the others
    g.health(0)
    g.close()


@pytest.mark.parametrize("n_cand,k", [(61, 48), (70, 48), (100, 48), (130, 70)])
def test_weights_next_to_nothing(n_cand, k):
    """A few pages have it all, and fewer than are chosen: the others' scores, of which there are 64 and fewer or more, are below the last
    counter's reach."""
    values = 0.15 + 0.4 * (np.arange(n_cand) * 29 % 64) / 64.0
    high = np.arange(0, n_cand, 2)[:k - 8]
    values[high] = 8.0
    K = torch.zeros((1, (n_cand + 4) * 32, 1, 128), dtype=torch.bfloat16, device="cuda")
    K[0, 64:(n_cand + 2) * 32, 0, 0] = torch.tensor(values, device="cuda").to(torch.bfloat16).repeat_interleave(32)
    q = torch.zeros((1, 4, 128), dtype=torch.bfloat16, device="cuda")
    q[..., 0] = torch.tensor([32.0, 31.0, 31.5, 32.5], device="cuda")
    ids, score = _select(4, n_cand, k, K, q)
    low = np.delete(score[0], high)
    assert (low < 2.0 ** -32).all() and len(np.unique(low)) > 2
    assert np.array_equal(ids[0], 2 + _best(score[0], k))
