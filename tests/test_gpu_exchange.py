"""What the blocks of a launch tell each other, where it could go wrong: launches that are captured and replayed, numbers
that come round again, waits for blocks that do not come, several contexts at once."""
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


def _same_as_a_fresh_context(g, x, tokens):
    """`g` decodes `tokens` of x (its prompt just loaded) exactly as a context that did nothing before."""
    e = x.context()
    out, ref = x.out(), x.out()
    e.load_prefix(0, x.K, x.V)
    for t in range(tokens):
        _step(g, x.q[t], x.k[t], x.v[t], out)
        _step(e, x.q[t], x.k[t], x.v[t], ref)
        assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS), e.debug_read(0, B.DBG_ACTIVE_IDS)), t
        assert torch.equal(out, ref), t
    e.close()


def test_weights_of_separate_launches_are_no_tags():
    """A long prompt is scored in a launch of its own, as plain fp32; the short prompt that follows in the same context
    takes one launch, whose blocks know each other's weights by a launch number.  With every plain weight the same odd bit
    pattern and the launch numbered to match, no plain weight may be taken for one of the new prompt's."""
    x = _Inputs(5, 30, 8, 8, 3000, 3)                                     # 240 KV heads
    long_ctx = (800 + 4) * 32                                             # 7 blocks of 128 pages to score per head
    g = x.context(max_ctx=long_ctx + 32)
    ones = torch.ones((30, long_ctx, 8, 128), dtype=DT, device="cuda")
    g.load_prefix(0, ones, ones)
    q = torch.zeros((30, 8, 128), dtype=DT, device="cuda")
    q[..., 0] = 7.0                                                       # 7 * fl32(1 / sqrt(128)): an odd bit pattern
    _step(g, q, x.k[0], x.v[0], x.out())
    assert g.step_launches(0) == 3
    bits = int(g.debug_read(0, B.DBG_WEIGHTS)[0, 0, 2:300].view(np.uint32).min())
    assert bits & 1 and (g.debug_read(0, B.DBG_WEIGHTS)[:, :, 2:300].view(np.uint32) == bits).all()
    g.load_prefix(0, x.K, x.V)
    g.test_launch_number((bits >> 1) - 1)                                 # tag of the next launch: 2 * number + 1 = bits
    _same_as_a_fresh_context(g, x, 2)
    assert g.step_launches(0) == 1
    g.health(0)
    g.close()


def test_launch_numbers_starting_over():
    """After 2^31 launches the numbers repeat.  Words left by the launches of the first time round carry the same numbers:
    none of them may be taken for a new one's."""
    x, y = _Inputs(7, 1, 32, 8, 20000, 4), _Inputs(8, 1, 32, 8, 20000, 4)
    g = x.context()
    g.load_prefix(0, y.K, y.V)
    _step(g, y.q[0], y.k[0], y.v[0], y.out())                             # number 1
    g.load_prefix(0, x.K, x.V)
    g.test_launch_number(0x7fffffff)
    _same_as_a_fresh_context(g, x, 4)
    g.health(0)
    g.close()


# Between the two ways attention is computed: weights carried to 16 bits or more (two 8-bit halves: 2^-17 each) against fp32,
# for outputs about a tenth of the values they average; sums of up to 2100 terms in fp32.
ALONE_TOL = 1e-4


def _close(out, ref):
    err = (out - ref).abs().amax(-1) / ref.abs().amax(-1)
    return bool(torch.isfinite(out).all()) and float(err.max()) <= ALONE_TOL


def _everything(g):
    return {what: g.debug_read(0, what) for what in (B.DBG_ACTIVE_IDS, B.DBG_FLAGS, B.DBG_WEIGHTS, B.DBG_SCORES)}


@pytest.mark.parametrize("call,batch,n_q,n_kv,ctx,kw,launches", [
    (_step, 1, 32, 8, 20000, {}, 1),                                      # one selecting block per head
    (_step, 1, 16, 2, 40000, {}, 1),                                      # four slices
    (_step, 1, 7, 1, 290000, {}, 1),                                      # sixteen, the last one short
    (_step, 1, 16, 2, 40000, dict(select_pooling="MaxQK"), 1),            # no softmax: keys are all that is exchanged
    (_step, 1, 10, 2, 40000, dict(select_pooling="MeanQ"), 1),
    (_step, 1, 16, 2, 40000, dict(placement=1), 1),                       # with a recall plan
    (_step, 64, 32, 4, 2500, {}, 2),                                      # separate launches, scoring and selection in one
    (_primitives, 1, 16, 2, 40000, {}, None),                             # the same, four slices
    (_primitives, 4, 4, 4, 170000, {}, None),                             # selection in a launch of its own, two slices
])
@pytest.mark.parametrize("kinds", [B.FKV_WAIT_WEIGHTS, B.FKV_WAIT_MAXIMA, B.FKV_WAIT_SUMS,
                                   B.FKV_WAIT_KEYS, 15])
def test_a_selecting_block_that_waits_in_vain(call, batch, n_q, n_kv, ctx, kw, launches, kinds):
    """Every wait of the given kinds inside the selection runs out at once.  No block may hand on what it did not get: ids and
    scores are, bit for bit, those of a context whose waits end, and outputs to fp32 rounding (a selection made alone takes
    longer than attention waits for it)."""
    x = _Inputs(31 + ctx, batch, n_q, n_kv, ctx, 3)
    g, e = x.context(**kw), x.context(**kw)
    out, ref = x.out(), x.out()
    g.load_prefix(0, x.K, x.V)
    e.load_prefix(0, x.K, x.V)
    g.test_impatience(kinds)
    for t in range(3):
        call(g, x.q[t], x.k[t], x.v[t], out)
        _step(e, x.q[t], x.k[t], x.v[t], ref)                             # (the primitives' separate kernels against one launch)
        assert launches is None or g.step_launches(0) == launches
        got, want = _everything(g), _everything(e)
        lo, hi = 2, g.context_len(0) // 32 - 2                            # candidate pages
        for what in got:
            a, b = (z[what][..., lo:hi] if what in (B.DBG_WEIGHTS, B.DBG_SCORES) else z[what] for z in (got, want))
            assert np.array_equal(a, b), (t, what)
        if kw.get("placement"):
            assert np.array_equal(g.debug_read(0, B.DBG_MISS)[..., 0], e.debug_read(0, B.DBG_MISS)[..., 0])
        assert _close(out, ref), t
    g.health(0)
    g.close()
    e.close()


def _static(g, q, k, v, out):
    g.kv_append(0, k, v)
    g.corr_check(0, q)
    g.page_select(0, q)
    g.sparse_decode_attn_static(0, q, out, use=fkv.FKV_USE_BY_FLAG)
    g.commit(0)


@pytest.mark.parametrize("call,batch,n_q,n_kv,ctx,kw", [
    (_step, 1, 32, 8, 20000, {}),
    (_step, 1, 16, 2, 40000, dict(budget=4096)),                          # G = 8, seventeen pages to a block
    (_step, 1, 32, 8, 20000, dict(tau=1.5)),                              # every head corrected
    (_step, 3, 14, 2, 1250, dict(budget=512)),                            # a new page begins; few candidates
    (_step, 2, 10, 2, 9000, dict(placement=1)),                           # pages fetched from the host pool
    (_step, 1, 5, 5, 2111, dict(placement=1, tau=1.5)),                   # the new token fills its page
    (_primitives, 7, 40, 8, 5003, {}),
    (_static, 1, 32, 8, 20000, {}),
])
@pytest.mark.parametrize("kinds", [B.FKV_WAIT_SPLITS, B.FKV_WAIT_IDS, 63])
def test_an_attention_block_that_waits_in_vain(call, batch, n_q, n_kv, ctx, kw, kinds):
    """Every wait of the given kinds in attention runs out at once: the block makes the ids, and its outputs, itself.  Ids are
    the same bit for bit, outputs to fp32 rounding, and what the step leaves behind serves the next one, which waits as usual."""
    x = _Inputs(47 + ctx, batch, n_q, n_kv, ctx, 4)
    g, e = x.context(**kw), x.context(**kw)
    out, ref = x.out(), x.out()
    g.load_prefix(0, x.K, x.V)
    e.load_prefix(0, x.K, x.V)
    for t in range(4):
        g.test_impatience(kinds if t < 3 else 0)
        call(g, x.q[t], x.k[t], x.v[t], out)
        call(e, x.q[t], x.k[t], x.v[t], ref)
        assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS), e.debug_read(0, B.DBG_ACTIVE_IDS)), t
        assert _close(out, ref) if t < 3 else torch.equal(out, ref), t
    if kw.get("placement"):
        ids = e.debug_read(0, B.DBG_ACTIVE_IDS)
        for head in range(n_kv):
            for page in ids[0, head][ids[0, head] >= 0][::5]:
                assert np.array_equal(g.debug_read_page(0, 0, head, int(page), 2), e.debug_read_page(0, 0, head, int(page), 2))
    g.health(0)
    g.close()
    e.close()


@pytest.mark.parametrize("call,kinds", [(_step, B.FKV_WAIT_KEYS), (_step, B.FKV_WAIT_SPLITS), (_step, B.FKV_WAIT_IDS), (_primitives, B.FKV_WAIT_WEIGHTS),
                                        (_primitives, B.FKV_WAIT_SPLITS)])
def test_what_blocks_make_by_themselves_is_counted(call, kinds):
    """Four slices a head, every head corrected: none as long as waits end, and some for every kind that does not; once read, none again."""
    x = _Inputs(3, 1, 16, 2, 40000, 4)
    g, out = x.context(tau=1.5), x.out()
    g.load_prefix(0, x.K, x.V)
    for t, k in enumerate((0, kinds, 0)):
        g.test_impatience(k)
        call(g, x.q[t], x.k[t], x.v[t], out)
        assert (g.test_by_itself(0)[0] > 0) == (k != 0), t
    g.health(0)
    g.close()


@pytest.mark.parametrize("n_ctx", [2, 6])
def test_contexts_decoding_at_once_on_streams_of_their_own(n_ctx):
    """Contexts of different shapes, each with a stream of its own and nothing waited for until all steps are enqueued, decode
    what they decode one after the other."""
    shapes = [(4, 32, 8, 3000, {}), (1, 16, 2, 40000, {}), (8, 16, 4, 2500, dict(tau=1.5)), (1, 32, 8, 20000, dict(tau=1.5)),
              (31, 64, 8, 2200, {}), (2, 40, 8, 9000, dict(placement=1))][:n_ctx]
    xs = [_Inputs(100 + i, b, n_q, n_kv, ctx, 8) for i, (b, n_q, n_kv, ctx, _) in enumerate(shapes)]
    want, ids = [], []
    for x, s in zip(xs, shapes):
        g = x.context(**s[4])
        g.load_prefix(0, x.K, x.V)
        outs = [x.out() for _ in range(8)]
        for t in range(8):
            _step(g, x.q[t], x.k[t], x.v[t], outs[t])
        ids.append(g.debug_read(0, B.DBG_ACTIVE_IDS))
        want.append(outs)
        g.health(0)
        g.close()
    gs = [x.context(**s[4]) for x, s in zip(xs, shapes)]
    streams = [torch.cuda.Stream() for _ in gs]
    for rounds in range(10):
        for x, g in zip(xs, gs):
            g.load_prefix(0, x.K, x.V)
        got = [[x.out() for _ in range(8)] for x in xs]
        torch.cuda.synchronize()
        for t in range(8):
            for i, (x, g) in enumerate(zip(xs, gs)):
                g.decode_step(0, x.q[t], x.k[t], x.v[t], got[i][t], stream=streams[i], copy_stream=streams[i])
        torch.cuda.synchronize()
        for i, g in enumerate(gs):
            g.health(0)
            assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS), ids[i]), (rounds, i)
            assert all(_close(a, b) for a, b in zip(got[i], want[i])), (rounds, i)
    for g in gs:
        g.close()


def test_contexts_of_few_heads_at_once_find_room_on_the_xcds_they_share():
    """Four contexts, as many as a process has launches on the machine at once, of one to seven heads each cut into as many blocks as may
    wait for each other on one XCD, on streams of their own and with every head corrected: no wait runs out."""
    shapes = [(1, 4, 1, 12000, 3072), (1, 8, 4, 30000, 6144), (1, 16, 2, 20000, 4096), (1, 28, 7, 20000, 4096)]
    xs = [_Inputs(200 + i, b, n_q, n_kv, ctx, 12) for i, (b, n_q, n_kv, ctx, _) in enumerate(shapes)]
    gs = [x.context(budget=s[4], tau=1.5) for x, s in zip(xs, shapes)]
    streams = [torch.cuda.Stream() for _ in gs]
    runs = []
    for at_once in (False, True):
        for x, g in zip(xs, gs):
            g.load_prefix(0, x.K, x.V)
        got = [[x.out() for _ in range(12)] for x in xs]
        torch.cuda.synchronize()
        for t in range(12):
            for x, g, o, s in zip(xs, gs, got, streams):
                g.decode_step(0, x.q[t], x.k[t], x.v[t], o[t], stream=s, copy_stream=s)
                if not at_once:
                    torch.cuda.synchronize()
        torch.cuda.synchronize()
        for i, g in enumerate(gs):
            assert g.step_launches(0) == 1
            assert g.test_by_itself(0) == (0, True), (at_once, i)
        runs.append((got, [g.debug_read(0, B.DBG_ACTIVE_IDS) for g in gs]))
    (want, ids), (got, ids_then) = runs
    for i, g in enumerate(gs):
        assert np.array_equal(ids[i], ids_then[i]), i
        assert all(_close(a, b) for a, b in zip(got[i], want[i])), i
        g.health(0)
        g.close()


def test_more_heads_than_a_grid_dimension_holds():
    """65600 (request, KV head) pairs, with scoring, selection and attention each a launch of its own: the requests on both
    sides of the 32768th and 65536th pair against a context of those requests alone."""
    batch, n_kv = 8200, 8
    x = _Inputs(3, batch, n_kv, n_kv, 130, 2)
    kw = dict(budget=96, sink=32, window=32, max_ctx=160)
    pick = [0, 4095, 4096, 8191, 8192, 8199]
    g, e = x.context(**kw), x.context(batch=len(pick), **kw)
    out, ref = x.out(), torch.zeros((len(pick), n_kv, 128), dtype=torch.float32, device="cuda")
    g.load_prefix(0, x.K, x.V)
    e.load_prefix(0, x.K[pick].contiguous(), x.V[pick].contiguous())
    for t in range(2):
        _step(g, x.q[t], x.k[t], x.v[t], out)
        _step(e, *(z[t][pick].contiguous() for z in (x.q, x.k, x.v)), ref)
        assert g.step_launches(0) == 3
        assert np.array_equal(g.debug_read(0, B.DBG_ACTIVE_IDS)[pick], e.debug_read(0, B.DBG_ACTIVE_IDS)), t
        assert torch.isfinite(out).all() and _close(out[pick], ref), t
    g.health(0)
    g.close()
    e.close()
