"""Reads past the caches: contexts whose layers together hold more than the memory-side cache take other variants of the kernels
than small ones, with the same results bit for bit."""
import numpy as np
import pytest
import torch

import paper_2505_13109_amd as fkv
from paper_2505_13109_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n_q", [("bf16", 32), ("fp16", 56)])
@pytest.mark.parametrize("placement,layers,steps", [
    (0, 36, "decode"),         # 36 x 8 heads x 65 pages: 307 MB, the summaries go past
    (0, 50, "decode"),         # 426 MB: the pages too
    (1, 36, "decode"),         # the same with the KV in a host pool
    (0, 36, "primitives"),
    (0, 50, "primitives"),
])
def test_a_layer_of_many_against_a_layer_by_itself(placement, layers, steps, dtype, n_q):
    torch_dtype = getattr(torch, {"bf16": "bfloat16", "fp16": "float16"}[dtype])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(layers + n_q)
    ctx = 100 * 32 + 5

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=gen).to(torch_dtype)

    K, V = normal(1, ctx, 8, 128), normal(1, ctx, 8, 128)
    q = [normal(1, n_q, 128)]
    for _ in range(3):
        q.append((0.8 * q[-1].float() + 0.6 * normal(1, n_q, 128).float()).to(torch_dtype))
    new = [normal(2, 1, 8, 128) for _ in q]
    got = []
    for n in (1, layers):
        g = fkv.FreeKV(n_layers=n, batch=1, n_q_heads=n_q, n_kv_heads=8, max_ctx=104 * 32, budget=2048, sink=512, window=512, tau=0.8, dtype=dtype,
                       placement=placement)
        layer = n - 1
        g.load_prefix(layer, K, V)
        out = torch.zeros((1, n_q, 128), device="cuda")
        for t, x in enumerate(q):
            if steps == "decode":
                g.decode_step(layer, x, new[t][0], new[t][1], out)
            else:
                g.kv_append(layer, new[t][0], new[t][1])
                g.corr_check(layer, x)
                g.page_select(layer, x)
                g.sparse_decode_attn(layer, x, out, use=fkv.FKV_USE_BY_FLAG)
                g.commit(layer)
            got.append((g.debug_read(layer, B.DBG_WEIGHTS)[..., 16:84], g.debug_read(layer, B.DBG_ACTIVE_IDS), out.clone()))
        g.health(layer)
        g.close()
    for (w0, ids0, out0), (w1, ids1, out1) in zip(got[:len(q)], got[len(q):]):
        assert np.array_equal(w0, w1) and np.array_equal(ids0, ids1) and torch.equal(out0, out1)


def test_a_scan_of_many_layers_against_a_layer_by_itself():
    """256 heads of 346 candidates: 46 MB of summaries and 72 MB of pages a layer, which one layer leaves in the cache."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    batch, ctx = 32, 348 * 32 + 5
    K, V = (torch.randn((batch, ctx, 8, 128), dtype=torch.bfloat16, device="cuda", generator=gen) for _ in range(2))
    q = torch.randn((3, batch, 32, 128), device="cuda", generator=gen).to(torch.bfloat16)
    got = []
    for n in (1, 3):
        g = fkv.FreeKV(n_layers=n, batch=batch, n_q_heads=32, n_kv_heads=8, max_ctx=350 * 32, budget=512, sink=32, window=32, tau=0.8, dtype="bf16")
        g.load_prefix(n - 1, K, V)
        out = torch.zeros((batch, 32, 128), device="cuda")
        for t in range(3):
            g.decode_step(n - 1, q[t], K[:, t].contiguous(), V[:, t].contiguous(), out)
            assert g.step_launches(n - 1) == 3
            got.append((g.debug_read(n - 1, B.DBG_WEIGHTS)[..., 1:347], g.debug_read(n - 1, B.DBG_ACTIVE_IDS), out.clone()))
        g.health(n - 1)
        g.close()
    for (w0, ids0, out0), (w1, ids1, out1) in zip(got[:3], got[3:]):
        assert np.array_equal(w0, w1) and np.array_equal(ids0, ids1) and torch.equal(out0, out1)
