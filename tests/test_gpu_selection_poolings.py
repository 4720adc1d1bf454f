"""The choice of the k best pages by the poolings without a softmax, whose scores have no largest value that is known beforehand: lists
shared by several blocks, with the best pages in other blocks than the one that puts them in order."""
import numpy as np
import pytest
import torch

import paper_2505_13109_amd as fkv
from paper_2505_13109_amd import binding as B

pytestmark = pytest.mark.gpu

EDGE = 2                                                 # sink and window pages


def _best(score, k):
    """ids (from 0) of the k largest, ties to the lower id, ascending"""
    order = np.lexsort((np.arange(len(score)), -score.astype(np.float64)))
    return np.sort(order[:k])


def _context(G, n_cand, k, pooling, n_kv=1, batch=1):
    """One channel of the keys decides: a page's weight is its value there, times 7 / sqrt(128) or so."""
    return fkv.FreeKV(n_layers=1, batch=batch, n_q_heads=G * n_kv, n_kv_heads=n_kv, max_ctx=(n_cand + 2 * EDGE + 1) * 32, budget=(2 * EDGE + k) * 32,
                      sink=EDGE * 32, window=EDGE * 32, tau=0.8, select_pooling=pooling)


def _select(G, values, k, pooling, batch=1):
    """ids and scores of a list of pages with these values"""
    n = len(values)
    K = torch.zeros((batch, (n + 2 * EDGE) * 32, 1, 128), dtype=torch.bfloat16, device="cuda")
    K[:, EDGE * 32:(EDGE + n) * 32, 0, 3] = torch.tensor(values, device="cuda").to(torch.bfloat16).repeat_interleave(32)
    q = torch.zeros((batch, G, 128), dtype=torch.bfloat16, device="cuda")
    q[..., 3] = 7.0
    g = _context(G, n, k, pooling, batch=batch)
    g.load_prefix(0, K, K)
    ids = torch.full((batch, 1, k), -1, dtype=torch.int32, device="cuda")
    out = torch.empty((batch, G, 128), device="cuda")
    new = torch.zeros((batch, 1, 128), dtype=torch.bfloat16, device="cuda")
    g.page_select(0, q, ids)
    score = g.debug_read(0, B.DBG_SCORES)[:, 0, EDGE:EDGE + n]
    g.decode_step(0, q, new, new, out)
    stepped = g.debug_read(0, B.DBG_ACTIVE_IDS)[:, 0]
    g.health(0)
    g.close()
    ids = ids.cpu().numpy()[:, 0]
    assert np.array_equal(ids, stepped)
    return ids - EDGE, score


# in several blocks, of which each hands on its best (5000 candidates) or all it has, and in one
@pytest.mark.parametrize("pooling", ["MeanQK", "MaxQK", "MeanQ", "MaxQ", "MaxS", "MeanS"])
@pytest.mark.parametrize("end", [-1.0, 1.0])             # the list's last quarter below zero, or above the rest of it
@pytest.mark.parametrize("G,n_cand,k,high", [
    (4, 5000, 32, 40), (4, 5000, 32, 33), (1, 5000, 32, 64), (4, 5000, 3, 63),
    (8, 2400, 150, 190), (8, 1300, 20, 60), (4, 992, 32, 40), (4, 97, 20, 30),
])
def test_high_pages_far_from_the_last_block(G, n_cand, k, high, end, pooling):
    """The best pages are in the first half of the list, the later the better, and far above all of its end."""
    gen = np.random.default_rng(n_cand + high)
    values = gen.integers(-64, 64, n_cand) / 64.0                                      # (bf16 holds these)
    values[3 * n_cand // 4:] += end
    at = np.sort(gen.permutation(n_cand // 2)[:high])
    values[at] = 4.0 + np.arange(high) / 32.0
    ids, score = _select(G, values, k, pooling)
    assert np.array_equal(ids[0], _best(score[0], k))
    assert set(ids[0]) <= set(at)


@pytest.mark.parametrize("pooling", ["MeanQK", "MaxQK", "MeanQ", "MaxQ"])
@pytest.mark.parametrize("G,n_cand,k", [(4, 5000, 32), (8, 1300, 20), (4, 992, 32), (1, 97, 40)])
def test_scores_far_below_the_largest(G, n_cand, k, pooling):
    """One page high, no more than k - 1 within eight octaves of it: the last of the chosen are among those of the last counter."""
    values = np.full(n_cand, -3.0)
    few = np.arange(5, n_cand, n_cand // (k + 12))[:k + 10]
    values[few] = 2.0 ** -9 * (1.0 + (np.arange(len(few)) * 37 % 64) / 64.0)
    values[few[: k // 2]] = 1.0
    values[7] = 3.0
    ids, score = _select(G, values, k, pooling)
    assert np.array_equal(ids[0], _best(score[0], k))


@pytest.mark.parametrize("pooling", ["MaxS", "MeanQK", "MaxQK", "MeanQ", "MaxQ"])
@pytest.mark.parametrize("G,n_cand,k,batch", [
    (4, 1, 1, 1), (4, 63, 7, 1), (7, 65, 64, 1),          # one wave, two
    (4, 512, 32, 1), (4, 513, 512, 1),                    # one row of candidates a thread, a second of one candidate
    (8, 1024, 96, 1), (8, 1025, 3, 1), (5, 1537, 33, 1),  # two, three, four
    (3, 2049, 64, 1), (2, 3073, 40, 1), (2, 4096, 500, 1),           # five, seven, eight
    (4, 2400, 33, 1), (4, 6000, 32, 1), (1, 9000, 600, 1),           # several blocks: every key handed on, each block's best, too many for registers
    (4, 513, 32, 320), (2, 2100, 32, 256),                # in a launch of their own
])
def test_rows_in_use(G, n_cand, k, batch, pooling):
    """Random pages: the ids are those of the scores, and the scores of one request the same bits in a launch of any shape."""
    gen = np.random.default_rng(n_cand + k)
    values = (gen.standard_normal(n_cand) * 0.5).astype(np.float32)
    ids, score = _select(G, values, k, pooling, batch=batch)
    one, s1 = _select(G, values, k, pooling, batch=12)
    assert np.array_equal(score, np.broadcast_to(s1[0], score.shape)) and np.array_equal(s1, np.broadcast_to(s1[0], s1.shape))
    want = _best(s1[0], k)
    assert np.array_equal(ids, np.broadcast_to(want, ids.shape)) and np.array_equal(one, np.broadcast_to(want, one.shape))


@pytest.mark.parametrize("pooling", ["MaxS", "MeanQK", "MaxQ"])
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("placement,layers", [
    (0, 64), (0, 80),                                     # 277 MB of pages that the layers attend, 346: summaries, and pages too, read past the caches
    (1, 1), (1, 64),                                      # the KV in a host pool
])
def test_the_layer_step_in_larger_contexts_and_with_a_host_pool(placement, layers, dtype, pooling):
    """Three steps of one layer against a context of that layer alone in HBM: page ids and scores are the same, outputs up to how they are split."""
    n_kv, G, ctx, k, tokens = 8, 2, 5000, 16, 3
    dt = torch.bfloat16 if dtype == "bf16" else torch.float16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layers + placement)
    K, V = (torch.randn((1, ctx, n_kv, 128), dtype=dt, device="cuda", generator=gen) for _ in range(2))
    q = [torch.randn((1, n_kv * G, 128), device="cuda", generator=gen).to(dt) for _ in range(tokens)]
    new = [torch.randn((2, 1, n_kv, 128), device="cuda", generator=gen).to(dt) for _ in range(tokens)]
    seen = []
    for where, n_layers in ((placement, layers), (0, 1)):
        g = fkv.FreeKV(n_layers=n_layers, batch=1, n_q_heads=n_kv * G, n_kv_heads=n_kv, max_ctx=ctx + 120, budget=1024, sink=256, window=256, tau=0.8,
                       dtype=dtype, placement=where, select_pooling=pooling)
        g.load_prefix(0, K, V)
        out = torch.empty((tokens, 1, n_kv * G, 128), device="cuda")
        steps = []
        for t in range(tokens):
            g.decode_step(0, q[t], new[t][0], new[t][1], out[t])
            steps.append((g.debug_read(0, B.DBG_ACTIVE_IDS), g.debug_read(0, B.DBG_SCORES)[..., 8:156], g.debug_read(0, B.DBG_FLAGS)))
        assert g.step_launches(0) == 1
        g.flush()
        g.health(0)
        g.close()
        seen.append((steps, out.cpu()))
    for one, other in zip(seen[0][0], seen[1][0]):
        assert all(np.array_equal(a, b) for a, b in zip(one, other))
    assert (seen[0][1] - seen[1][1]).abs().max() <= 1e-4 * seen[1][1].abs().max()
