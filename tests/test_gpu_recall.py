"""The recall kernel where its division of the work changes: from one missing unit to more than the launch has waves, heads
without a miss among the others, more heads than a block has threads."""
import numpy as np
import pytest
import torch

import paper_2505_13109_amd as fkv
from paper_2505_13109_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,n_kv,per_head", [
    (1, 1, [1]),                                   # a single unit
    (1, 8, [0, 3, 0, 0, 5, 1, 0, 8]),              # fewer units than waves: eight waves to a unit
    (2, 8, [16, 0, 7, 16, 9, 0, 16, 1] * 2),       # ... two to a unit
    (2, 8, [16] * 15 + [15]),                      # 255: one short of a unit a wave
    (3, 8, [16, 13, 0, 16, 16, 16, 11, 16] * 3),   # more units than waves
    (137, 8, [1, 0, 2, 0, 1, 1, 0, 1] * 137),      # more heads than a block has threads
])
def test_every_missing_unit_is_recalled_once(batch, n_kv, per_head):
    ctx, k = 20 * 32 + 9, 16
    gen = torch.Generator(device="cuda")
    gen.manual_seed(len(per_head) + per_head[0])
    K, V = (torch.randn((batch, ctx, n_kv, 128), device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2))
    g = fkv.FreeKV(n_layers=1, batch=batch, n_q_heads=n_kv, n_kv_heads=n_kv, max_ctx=704, budget=64 + k * 32, sink=32, window=32,
                   tau=0.8, dtype="bf16", placement=fkv.FKV_PLACE_HOST)
    g.load_prefix(0, K, V)
    rng = np.random.default_rng(3)
    ids = np.full((batch, n_kv, k), -1, dtype=np.int32)
    for h, n in enumerate(per_head):
        ids[h // n_kv, h % n_kv, :n] = np.sort(rng.choice(np.arange(1, 19), n, replace=False))
    cached = g.dev_arena.clone()
    g.recall_pages(0, torch.from_numpy(ids).cuda())
    assert np.array_equal(g.debug_read(0, B.DBG_MISS)[..., 0].reshape(-1), per_head)
    n_slots = k + 3
    pool = torch.zeros((batch, n_slots, 2, 32, n_kv, 128), dtype=torch.bfloat16, device="cuda")
    pages = torch.zeros((batch, n_kv, n_slots), dtype=torch.int32, device="cuda")
    g.export_nhd(0, pool, pages, use=fkv.FKV_USE_PENDING)
    torch.cuda.synchronize()
    assert torch.equal(pages[:, :, 1:1 + k].cpu(), torch.from_numpy(ids))
    for b in range(batch):
        for m in range(n_kv):
            n = per_head[b * n_kv + m]
            if n == 0:
                continue
            at = torch.from_numpy(ids[b, m, :n].astype(np.int64)).cuda()
            for x, which in ((K, 0), (V, 1)):
                want = x[b, :, m][: 20 * 32].reshape(20, 32, 128)[at]
                assert torch.equal(pool[b, 1:1 + n, which, :, m], want), (b, m, which)
    # nothing else of the page pool is written: a head without a miss keeps its bytes
    per = (1 + 3 + 2 * k) * 16384
    before, after = (t[: batch * n_kv * per].view(batch * n_kv, per) for t in (cached, g.dev_arena))
    same = (before == after).all(dim=1).cpu().numpy()
    assert np.array_equal(same, np.array(per_head) == 0)
    g.close()


@pytest.mark.parametrize("own_copy_stream", [False, True])
@pytest.mark.parametrize("batch,ctx,launches", [(1, 4000, 1), (32, 4000, 3)])        # the layer-step in one launch, and in separate ones
def test_a_captured_step_with_the_host_pool(batch, ctx, launches, own_copy_stream):
    """Four steps of two layers, captured right behind the prompts, with heads that are not corrected and miss pages from the second
    step on: what a captured recall moves is what the layer's next captured step attends.  (That the recall lies between the two
    whatever the timing: test_host_order.py.)  Every replay against eager steps."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(29)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen)

    layers, steps = 2, 4
    kv = [[normal(batch, ctx, 8, 128).to(torch.bfloat16) for _ in range(2)] for _ in range(layers)]
    q = [[normal(batch, 32, 128)] for _ in range(layers)]
    for x in q:
        while len(x) < steps:
            x.append(0.9 * x[-1] + 0.436 * normal(batch, 32, 128))
    q = [[y.to(torch.bfloat16) for y in x] for x in q]
    new = [[normal(2, batch, 8, 128).to(torch.bfloat16) for _ in range(steps)] for _ in range(layers)]
    results = []
    for captured in (False, True):
        g = fkv.FreeKV(n_layers=layers, batch=batch, n_q_heads=32, n_kv_heads=8, max_ctx=4096, budget=1024, sink=64, window=64,
                       tau=0.8, dtype="bf16", placement=fkv.FKV_PLACE_HOST)
        out = torch.zeros((steps, layers, batch, 32, 128), device="cuda")
        copy = torch.cuda.Stream()

        deferred = []                                      # units that a step's deferred recall moves, in the eager run

        def decode():
            for t in range(steps):
                for l in range(layers):
                    g.decode_step(l, q[l][t], new[l][t][0], new[l][t][1], out[t, l], copy_stream=copy if own_copy_stream else None)
                    if not captured:
                        deferred.append(int(g.debug_read(l, B.DBG_MISS)[..., 0][g.debug_read(l, B.DBG_FLAGS) == 0].sum()))
            if own_copy_stream:
                torch.cuda.current_stream().wait_stream(copy)

        for l in range(layers):
            g.load_prefix(l, *kv[l])
        torch.cuda.synchronize()
        if captured:
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                decode()
            for _ in range(3):
                out.zero_()
                graph.replay()
                torch.cuda.synchronize()
                results.append(out.clone())
            out.zero_()
            for l in range(layers):                        # outside of the graph once more: from the prompts on
                g.load_prefix(l, *kv[l])
            decode()
            torch.cuda.synchronize()
            results.append(out.clone())
        else:
            decode()
            torch.cuda.synchronize()
            results.append(out.clone())
            assert g.step_launches(0) == launches
            assert min(deferred[layers:]) > 0, deferred
        for l in range(layers):
            g.health(l)
        g.close()
    for r in results[1:]:
        assert torch.equal(r, results[0])
