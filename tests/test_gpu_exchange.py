"""What the blocks of a launch tell each other, where it could go wrong: launches that are captured and replayed."""
import numpy as np
import pytest
import torch

import paper_2505_13109_amd as fkv
from paper_2505_13109_amd import binding as B

pytestmark = pytest.mark.gpu

DT = torch.bfloat16


def _normal(gen, *shape):
    return torch.randn(shape, dtype=torch.float32, device="cuda", generator=gen)


class _Inputs:
    """A prompt and decode inputs for one layer; consecutive queries similar enough that some heads are corrected."""

    def __init__(self, seed, batch, n_q, n_kv, ctx, tokens):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        self.batch, self.n_q, self.n_kv, self.ctx = batch, n_q, n_kv, ctx
        self.K, self.V = (_normal(gen, batch, ctx, n_kv, 128).to(DT) for _ in range(2))
        first = _normal(gen, batch, n_q, 128)
        self.q = [first.to(DT)] + [(0.8 * first + 0.6 * _normal(gen, batch, n_q, 128)).to(DT) for _ in range(tokens - 1)]
        self.k, self.v = ([_normal(gen, batch, n_kv, 128).to(DT) for _ in range(tokens)] for _ in range(2))

    def context(self, max_ctx=None, **kw):
        args = dict(n_layers=1, batch=self.batch, n_q_heads=self.n_q, n_kv_heads=self.n_kv, budget=1024, sink=64, window=64,
                    max_ctx=max_ctx or -(-(self.ctx + 64) // 32) * 32, tau=0.8, dtype="bf16")
        args.update(kw)
        return fkv.FreeKV(**args)

    def out(self):
        return torch.zeros((self.batch, self.n_q, 128), dtype=torch.float32, device="cuda")


def _step(g, q, k, v, out):
    g.decode_step(0, q, k, v, out)


def _primitives(g, q, k, v, out):
    g.kv_append(0, k, v)
    g.corr_check(0, q)
    g.page_select(0, q)
    g.sparse_decode_attn(0, q, out, use=fkv.FKV_USE_BY_FLAG)
    g.commit(0)


@pytest.mark.parametrize("call,batch,n_q,n_kv,ctx,launches", [
    (_step, 1, 32, 8, 20000, 1),          # the one-launch layer-step: a head's selection and attention each in several blocks
    (_step, 1, 16, 2, 40000, 1),          # G = 8, selection in four slices
    (_step, 66, 16, 4, 1500, 2),          # separate launches
    (_primitives, 1, 32, 8, 20000, None),
])
def test_a_captured_step_is_right_at_every_replay(call, batch, n_q, n_kv, ctx, launches):
    """A replay repeats the captured step -- same position, same ACTIVE selection, same previous query -- on whatever
    the input buffers hold by then.  Every replay against an eager context brought to the same state, with eager work
    on that context and synchronisations in between."""
    x = _Inputs(17 + ctx, batch, n_q, n_kv, ctx, 6)
    g, e = x.context(), x.context()
    q, k, v, out, ref = x.q[0].clone(), x.k[0].clone(), x.v[0].clone(), x.out(), x.out()
    g.load_prefix(0, x.K, x.V)
    _step(g, q, k, v, out)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(g, q, k, v, out)
    if launches is not None:
        assert g.step_launches(0) == launches
    corrected = 0
    for t in (1, 2, 3, 4, 5, 2, 1):
        e.load_prefix(0, x.K, x.V)
        _step(e, x.q[0], x.k[0], x.v[0], ref)
        call(e, x.q[t], x.k[t], x.v[t], ref)
        flags, ids = e.debug_read(0, B.DBG_FLAGS), e.debug_read(0, B.DBG_ACTIVE_IDS)
        corrected += int(flags.sum())
        q.copy_(x.q[t])
        k.copy_(x.k[t])
        v.copy_(x.v[t])
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(g.debug_read(0, B.DBG_FLAGS), flags)
        assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS), ids), t
        assert torch.equal(out, ref), t
    assert 0 < corrected < 7 * batch * n_kv
    g.health(0)
    g.close()
    e.close()
