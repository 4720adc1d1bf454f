"""Which kernels the library launches and in which order it hands work to streams, on the CPU: the HIP runtime's calls are taken by
a recorder (hip_recorder.c), nothing runs, and what is recorded is read as a graph of what has to wait for what.  Here a missing
wait between the compute stream and the copy stream shows whatever the timing; results on a GPU show it only when a recall
happens to be late."""
import ctypes as C
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COMPUTE, COPY = 0x100, 0x200


def _play(recorder, library, config, calls):
    """(In a process of its own: the recorder's symbols come before the HIP runtime's.)  For each call its return code and how many
    lines the log had when it began."""
    rec = C.CDLL(recorder, mode=C.RTLD_GLOBAL)
    rec.rec_log.restype = C.c_char_p
    lib = C.CDLL(library)
    dims = ("n_layers", "batch", "n_q_heads", "n_kv_heads", "head_dim", "page_size", "max_ctx", "budget_tokens", "sink_tokens", "window_tokens", "dtype",
            "placement")

    class Config(C.Structure):
        _fields_ = [(n, C.c_int32) for n in dims] + [("tau", C.c_float)] + [(n, C.c_int32) for n in ("recall_mode", "select_pooling", "corr_pooling")]

    ctx, some = C.c_void_p(), C.c_void_p(0x10000000)                  # (no address is looked at)
    where = config.pop("where", 0)
    rec.rec_where(where)
    left = 98 if where == 4 else 0
    st, cs, copy = C.c_void_p(COMPUTE), C.c_void_p(COPY), C.c_void_p(config.pop("copy", COPY))
    rc = lib.fkv_create(C.byref(Config(**config)), some, C.c_size_t(1 << 50), some, C.c_size_t(1 << 50), C.byref(ctx))
    assert rc == 0, rc
    assert rec.hipGetLastError() == left                              # (the program's own error is still there, and none of the library's)
    done = []
    for call, *args in calls:
        at = rec.rec_log().count(b"\n")
        if call == "load":
            rc = lib.fkv_load_prefix(ctx, args[0], some, some, args[1], st)
        elif call == "step":
            rc = lib.fkv_decode_step(ctx, args[0], some, some, some, some, st, copy)
        elif call == "select":
            rc = lib.fkv_page_select(ctx, args[0], some, None, st)
        elif call == "attend":
            rc = lib.fkv_sparse_decode_attn(ctx, args[0], some, some, 0, st)
        elif call == "append":
            rc = lib.fkv_kv_append(ctx, args[0], some, some, st, copy)
        elif call == "capture":
            rc = rec.rec_capture(st) and 0
        elif call == "end_capture":
            rc = rec.rec_end_capture() and 0
        done.append((rc, at))
    return rec.rec_log().decode().splitlines(), done


@pytest.fixture(scope="module")
def play(tmp_path_factory):
    recorder = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", recorder, os.path.join(ROOT, "tests", "hip_recorder.c")], check=True)
    library = os.environ.get("FKV_LIB") or os.path.join(ROOT, "paper_2505_13109_amd", "libfreekv.so")

    def run(calls, **config):
        base = dict(n_layers=2, batch=1, n_q_heads=32, n_kv_heads=8, head_dim=128, page_size=32, max_ctx=8192, budget_tokens=1024, sink_tokens=64,
                    window_tokens=64, dtype=1, placement=1, tau=0.8, recall_mode=0, select_pooling=0, corr_pooling=0)
        base.update(config)
        out = subprocess.run([sys.executable, os.path.abspath(__file__), json.dumps([recorder, library, base, calls])], check=True, capture_output=True, text=True)
        lines, done = json.loads(out.stdout.splitlines()[-1])
        return Order(lines, calls, done)

    return run


class Order:
    def __init__(self, lines, calls, done):
        self.ops = [line.split() for line in lines]
        self.calls = calls
        self.rc = [rc for rc, _ in done]
        self.span = [(at, done[i + 1][1] if i + 1 < len(done) else len(lines)) for i, (_, at) in enumerate(done)]
        last_of, recorded, sync, self.after = {}, {}, None, []        # after[i]: what op i directly waits for
        for i, op in enumerate(self.ops):
            if op[0] == "sync":
                self.after.append(list(range(i)))
                sync = i
                continue
            stream, captured = op[2], op[-1]
            before = [last_of.get(stream), sync]
            if op[0] == "wait" and recorded.get(op[1], (0, None))[1] == captured:      # (a record in a capture means nothing outside of it)
                before.append(recorded[op[1]][0])
            self.after.append([b for b in before if b is not None])
            last_of[stream] = i
            if op[0] == "record":
                recorded[op[1]] = (i, captured)
            if op[0] == "launch" and op[3] != "(nil)":
                recorded[op[3]] = (i, "0")                            # a stop event is never part of a capture

    def before(self, a, b):
        """op a is over before op b begins, whatever the timing"""
        seen, todo = set(), [b]
        while todo:
            i = todo.pop()
            if i == a:
                return True
            if i not in seen and i > a:
                seen.add(i)
                todo.extend(self.after[i])
        return False

    def launches(self, call, kernel, stream=None):
        """ops of the call that launch the kernel"""
        lo, hi = self.span[call]
        return [i for i in range(lo, hi) if self.ops[i][0] == "launch" and kernel in self.ops[i][1] and (stream is None or int(self.ops[i][2], 16) == stream)]

    def first_launch(self, call):
        return self.launches(call, "")[0]

    def recall_of(self, call):
        """the deferred recall of a step's uncorrected heads: the first gather on the copy stream from there on"""
        return next(i for i in range(self.span[call][0], len(self.ops)) if self.ops[i][0] == "launch" and "gather_kernel" in self.ops[i][1]
                    and int(self.ops[i][2], 16) == COPY)


def _index(calls, *wanted):
    return [i for i, c in enumerate(calls) if tuple(c) == wanted]


@pytest.mark.parametrize("captured", [False, True])
@pytest.mark.parametrize("batch,layers", [(1, 1), (1, 2), (1, 5), (1, 18), (32, 2)])      # one launch a layer-step, and separate ones
def test_a_deferred_recall_lies_between_its_step_and_the_next(play, batch, layers, captured):
    loads = [("load", l, 4000) for l in range(layers)]
    steps = [("step", l) for _ in range(4) for l in range(layers)]
    calls = loads + ([("capture",)] if captured else []) + steps
    o = play(calls, n_layers=layers, batch=batch)
    assert set(o.rc) == {0}
    for l in range(layers):
        mine = _index(calls, "step", l)
        for now, then in zip(mine, mine[1:]):
            chosen = [i for k in ("layer_kernel", "step_kernel", "select_kernel") for i in o.launches(now, k)]
            recall = o.recall_of(now)
            assert chosen and o.before(chosen[-1], recall)
            assert o.before(recall, o.first_launch(then)), f"layer {l}: nothing orders the next step behind the recall"


@pytest.mark.parametrize("batch,layers", [(1, 1), (1, 2), (1, 5), (32, 2)])
def test_a_new_prompt_lies_behind_what_the_old_context_left_on_the_copy_stream(play, batch, layers):
    """A recall writes page-cache slots, an offload (here of the page that the first step fills) the host pool: both would land in
    the new context."""
    before = [("load", l, 4031) for l in range(layers)] + [("step", l) for _ in range(3) for l in range(layers)]
    calls = before + [("load", l, 4000) for l in range(layers)]
    o = play(calls, n_layers=layers, batch=batch)
    assert set(o.rc) == {0}
    for l in range(layers):
        again = o.launches(_index(calls, "load", l, 4000)[0], "load_prefix_kernel")[0]
        steps = _index(calls, "step", l)
        offloads = o.launches(steps[0], "offload_kernel", COPY)
        assert len(offloads) == 1
        assert o.before(o.recall_of(steps[-1]), again), f"layer {l}: nothing orders the new prompt behind the recall"
        assert o.before(offloads[0], again), f"layer {l}: nothing orders the new prompt behind the offload"


@pytest.mark.parametrize("calls", [
    [("step", 0), ("capture",), ("load", 0, 4000)],                        # a captured load behind eager steps
    [("capture",), ("step", 0), ("end_capture",), ("load", 0, 4000)],      # ... the other way round
    [("capture",), ("step", 0), ("end_capture",), ("capture",), ("load", 0, 4000)],      # ... in two captures
])
def test_a_new_prompt_does_not_wait_across_the_edge_of_a_capture(play, calls):
    """(An event of the one side has no meaning on the other.)  Nor does the first step after it."""
    o = play([("load", 0, 4031)] + calls + [("step", 0)], n_layers=1)
    assert set(o.rc) == {0}
    lo, hi = o.span[-2]
    assert [op[0] for op in o.ops[lo:hi]] == ["launch"]
    lo, hi = o.span[-1]
    first = o.first_launch(len(o.calls) - 1)
    assert all(op[0] == "launch" for op in o.ops[lo:first])


@pytest.mark.parametrize("step", ["append", "step"])
@pytest.mark.parametrize("window", [0, 64])
def test_a_page_is_offloaded_before_a_later_one_takes_its_place(play, window, step):
    """The window pages and the open one live in a ring of units: the token that opens page p goes where page p - n_ring was, which the copy
    stream has to have read by then."""
    n_ring, start = window // 32 + 2, 4000
    calls = [("load", 0, start)] + [(step, 0)] * 300
    o = play(calls, n_layers=1, window_tokens=window)
    assert set(o.rc) == {0}
    opens, fills = {}, {}
    for i in range(1, len(calls)):
        page, at = divmod(start + i - 1, 32)
        if at == 0:
            opens[page] = o.first_launch(i)
        if at == 31:
            fills[page] = o.launches(i, "offload_kernel", COPY)[0]
    pairs = [(p, p + n_ring) for p in fills if p + n_ring in opens]
    assert len(pairs) >= 5
    for old, new in pairs:
        assert o.before(fills[old], opens[new]), f"page {new} may be written over page {old} before that is offloaded"


@pytest.mark.parametrize("kernel,past,layers,batch,ctx,budget", [
    ("layer_kernelILi1ELi4ELb0E", "Li0E", 32, 1, 1500, 4096),        # 47 pages a head, 201 MB, though the budget is 129
    ("layer_kernelILi1ELi4ELb0E", "Li3E", 32, 1, 2600, 4096),        # 82: 344 MB
    ("layer_kernelILi1ELi4ELb0E", "Li3E", 40, 1, 32768, 2048),       # 341 MB
    ("layer_kernelILi1ELi4ELb0E", "Li1E", 32, 1, 32768, 2048),       # 277 MB of pages, 130 MB of summaries
    ("scan_kernelILi1ELi4E", "Lb0E", 1, 32, 16640, 1024),            # 138 MB of pages, 65 MB of summaries
    ("scan_kernelILi1ELi4E", "Lb1E", 2, 32, 16640, 1024),
    ("attn_kernelILi1ELi4E", "Lb0E", 2, 32, 16640, 1024),
    ("attn_kernelILi1ELi4E", "Lb1E", 3, 32, 16640, 1024),            # 415 MB of pages
])
def test_reads_past_the_cache_are_for_what_does_not_fit_it(play, kernel, past, layers, batch, ctx, budget):
    """By the bytes that a context's layers attend and score (template arguments of the kernel's name: past the caches or not)."""
    o = play([("load", 0, ctx), ("step", 0)], n_layers=layers, batch=batch, max_ctx=33280, budget_tokens=budget, sink_tokens=256, window_tokens=256, placement=0)
    assert o.rc == [0, 0]
    (op,) = o.launches(1, kernel)
    assert kernel + past + "E" in o.ops[op][1]


@pytest.mark.parametrize("batch,ctx,scoring,selecting,splits", [
    (16, 33300, 8, 1, 2),      # 1024 candidates
    (16, 33312, 9, 1, 1),      # 1025
    (8, 49000, 12, 1, 2),      # 1515
    (8, 33300, 8, 1, 4),
    (10, 40000, 10, 1, 2),     # three would fit
    (6, 49000, 12, 1, 3),      # five would
    (5, 49000, 12, 1, 5),
    (1, 49000, 48, 1, 9),
])
def test_attention_beside_long_lists_of_many_heads_is_cut_half_as_fine(play, batch, ctx, scoring, selecting, splits):
    o = play([("load", 0, ctx), ("step", 0)], n_layers=1, batch=batch, max_ctx=65536, budget_tokens=2048, sink_tokens=256, window_tokens=256, placement=0)
    (op,) = o.launches(1, "layer_kernel")
    assert o.ops[op][4] == f"{8 * batch}x{2 + scoring + selecting + splits}x1"


@pytest.mark.parametrize("where,wide", [
    (0, 16),      # blocks go to the XCDs in turn: twelve heads by eight
    (1, 12),      # they do not
    (2, 12),      # the kernel that looks was not launched, (3) or has written nothing: not known, whatever the memory held
    (3, 12),
    (4, 16),      # they do, whatever the program called before
])
def test_heads_are_put_on_xcds_only_where_blocks_are_known_to_go(play, where, wide):
    o = play([("load", 0, 2000), ("step", 0)], n_layers=1, batch=3, n_q_heads=16, n_kv_heads=4, max_ctx=4096, placement=0, where=where)
    assert o.rc == [0, 0]
    (op,) = o.launches(1, "layer_kernel")
    assert o.ops[op][4].split("x")[0] == str(wide)
    assert ("home_layer_kernel" in o.ops[op][1]) == (wide == 16)                     # (what the kernel was compiled for is what its grid says)


@pytest.mark.parametrize("where,step,wide", [(0, "Lb1EE", 16), (1, "Lb0EE", 12)])
def test_launches_of_the_primitives_at_home(play, where, step, wide):
    """Twelve heads of 16 pages, at home if blocks are known to go there: the same of the step kernel, and of attention in its two grids."""
    o = play([("load", 0, 2000), ("select", 0), ("attend", 0)], n_layers=1, batch=3, n_q_heads=16, n_kv_heads=4, max_ctx=4096, placement=0, where=where,
             budget_tokens=512)
    assert o.rc == [0, 0, 0]
    (op,) = o.launches(1, "step_kernel")
    assert step in o.ops[op][1] and o.ops[op][4].split("x")[0] == str(wide)
    (op,) = o.launches(2, "attn_kernel")
    n = 512 // 32 + 1                                                                # pages, four to a block
    assert (("home_attn_kernel" in o.ops[op][1]), o.ops[op][4]) == ((True, f"8x{-(-n // 4)}x2") if where == 0 else (False, f"{-(-n // 4)}x12x1"))


def _decode(play, heads, candidates, pages, call="step", **config):
    """One call of `heads` KV heads with so many candidates and attended pages, the open one included: its launches"""
    ctx = (candidates + 8) * 32 + 5
    o = play([("load", 0, ctx), (call, 0)], **dict(dict(n_layers=1, batch=heads, n_q_heads=4, n_kv_heads=1, max_ctx=ctx + 59, budget_tokens=(pages - 1) * 32,
                                                        sink_tokens=128, window_tokens=128, placement=0), **config))
    assert o.rc == [0, 0]
    lo, hi = o.span[1]
    return [op for op in o.ops[lo:hi] if op[0] == "launch"]


@pytest.mark.parametrize("heads,candidates,pages,home", [
    (1, 100, 33, True), (1, 992, 65, True), (1, 992, 129, False),            # 0.5, 1.4 and 2.3 MB more than an even share for one XCD
    (4, 992, 129, True), (4, 992, 257, False),               # 1.3, 2.4
    (4, 90, 1000, True),                                     # a budget that the context has no pages for does not count: 0.8
    (7, 992, 129, True),                                     # 0.3
    (12, 992, 65, True), (12, 100, 129, False),              # 0.8, 0.9
    (9, 992, 129, False),                                    # 2.3
    (14, 480, 129, False), (14, 480, 65, True),              # two heads' 66 blocks do not fit an XCD at once; 50 do
    (28, 992, 33, True), (100, 480, 65, True), (100, 992, 129, False),      # 0.5, 0.7, 1.3
    (8, 992, 129, True), (120, 992, 129, True),              # they go round evenly
])
def test_heads_at_home_by_what_their_xcd_has_to_read(play, heads, candidates, pages, home):
    (op,) = _decode(play, heads, candidates, pages)
    assert ("home_layer_kernel" in op[1], int(op[4].split("x")[0])) == (home, -(-heads // 8) * 8 if home else heads)


@pytest.mark.parametrize("heads,pages,home", [(1, 65, True), (1, 129, False), (4, 65, True), (4, 129, False), (12, 33, True), (12, 65, False), (28, 129, False),
                                              (16, 257, True)])
def test_attention_by_itself_at_home(play, heads, pages, home):
    """(0.9, 1.8, 0.5, 1.1, 0.3, 0.5 and 1.1 MB; two heads to each)"""
    (op,) = _decode(play, heads, 992, pages, call="attend")
    assert ("home_attn_kernel" in op[1]) == home


@pytest.mark.parametrize("batch,home", [(65535, True), (65536, False)])
def test_attention_by_itself_of_more_heads_than_its_grid_at_home_can_have(play, batch, home):
    """Eight KV heads a request, a budget of two blocks a head: at home a grid dimension counts the heads by eight and ends at 65535."""
    o = play([("load", 0, 40), ("attend", 0)], n_layers=1, batch=batch, n_q_heads=8, n_kv_heads=8, max_ctx=64, budget_tokens=300 * 32, placement=0)
    assert o.rc == [0, 0]
    (op,) = o.launches(1, "attn_kernel")
    x, y, z = (int(v) for v in o.ops[op][4].split("x"))
    assert ("home_attn_kernel" in o.ops[op][1]) == home and x * y * z >= batch * 8 * 2 and max(y, z) <= 65535


@pytest.mark.parametrize("heads,candidates,pages,scoring,splits", [
    (36, 480, 129, 4, 7), (40, 480, 129, 8, 8),              # 504 blocks are there at once, 520 are not
    (72, 100, 65, 1, 3), (76, 100, 65, 4, 4),                # 504, 532
    (136, 100, 39, 2, 1), (136, 100, 40, 2, 2),              # a block has pages enough from 40 on
    (136, 240, 65, 4, 3), (136, 241, 65, 2, 1),              # few heads of one block each behind many scoring blocks
    (176, 344, 65, 3, 1), (184, 344, 65, 3, 2),              # no longer few
    (96, 480, 96, 8, 5), (96, 480, 97, 4, 2),                # long streams: 192 blocks have a unit each
    (104, 480, 97, 4, 4),                                    # 208 just miss that
    (64, 480, 129, 8, 4), (68, 480, 129, 4, 7),              # 256 do not; 204 do
    (196, 992, 80, 8, 2), (200, 992, 80, 8, 1),              # 2548 blocks; 2600 would be too many for one launch
    (128, 1023, 65, 8, 4), (128, 1024, 65, 8, 2),            # beside long lists it is not cut finer
])
def test_attention_of_many_heads_is_cut_into_as_many_blocks_as_fit(play, heads, candidates, pages, scoring, splits):
    (op,) = _decode(play, heads, candidates, pages)
    assert "layer_kernel" in op[1] and int(op[4].split("x")[1]) == 2 + scoring + 1 + splits


@pytest.mark.parametrize("heads,pages,placement,splits", [
    (8, 65, 0, 9), (8, 129, 0, 16), (8, 257, 0, 16), (8, 1000, 0, 16),
    (8, 129, 1, 15),                                         # runs of nine
    (16, 129, 0, 9),
    (1, 129, 0, 17),                                         # spread over the XCDs
])
def test_no_more_blocks_of_a_head_wait_on_an_xcd_than_four_launches_leave_room_for(play, heads, pages, placement, splits):
    (op,) = [op for op in _decode(play, heads, 992, pages, placement=placement) if "layer_kernel" in op[1]]
    rows = int(op[4].split("x")[1])
    scoring = [-(-992 // (32 * passes)) for passes in (1, 2, 4)]
    assert rows - 3 - splits in scoring, rows


@pytest.mark.parametrize("placement", [0, 1])
@pytest.mark.parametrize("pooling", range(6))
def test_the_poolings_beside_the_methods_have_kernels_of_their_own(play, pooling, placement):
    """In each of the launches that pick pages: with the layer-step, by themselves, and after a scan of their own."""
    (op,) = [op for op in _decode(play, 8, 480, 33, placement=placement, select_pooling=pooling) if "layer_kernel" in op[1]]
    kind = int(op[1].split("layer_kernelILi1ELi4ELb" + str(placement) + "ELi")[1].split("E")[0])
    assert (kind & 4 != 0) == (pooling != 0)
    (op,) = _decode(play, 8, 480, 33, call="select", placement=placement, select_pooling=pooling)
    assert "step_kernelILi1ELi4ELb" + ("1" if pooling == 0 else "0") + "E" in op[1]
    op = _decode(play, 256, 480, 33, call="select", placement=placement, select_pooling=pooling)[-1]
    assert "select_kernelILi4ELb" + ("1" if pooling == 0 else "0") + "E" in op[1]


@pytest.mark.parametrize("heads", [1, 2, 3])
@pytest.mark.parametrize("candidates,selecting,home", [
    (1440, 8, True),                                         # 2 + 45 + 8 + 9 blocks are an XCD's slots
    (1441, 4, True), (1568, 4, True),                        # 46 to 49 scoring blocks: half as many select
    (1569, 8, False),                                        # nor would those fit
])
def test_few_heads_share_a_list_among_as_many_blocks_as_fit_their_xcd(play, heads, candidates, selecting, home):
    (op,) = _decode(play, heads, candidates, 65, n_q_heads=5)
    assert ("home_layer_kernel" in op[1]) == home
    assert int(op[4].split("x")[1]) == 2 + -(-candidates // 32) + selecting + 9


@pytest.mark.parametrize("heads,G,candidates,selecting,config", [
    (8, 8, 1024, 1, {}), (8, 8, 1025, 4, {}), (8, 3, 2048, 1, {}), (8, 3, 2049, 8, {}), (8, 5, 1024, 1, {}), (8, 5, 1025, 4, {}),   # rows times G of 16
    (8, 4, 2048, 1, {}), (8, 4, 2049, 8, {}), (8, 2, 4096, 1, {}), (8, 2, 4097, 16, {}),                                            # the registers
    (9, 5, 1880, 1, {}), (9, 5, 1881, 8, {}), (9, 8, 1175, 1, {}), (9, 8, 1176, 4, {}),                                             # more than eight heads
    (8, 8, 1175, 1, dict(select_pooling=2)), (8, 8, 1176, 4, dict(select_pooling=2)),                                               # other poolings
    (8, 8, 1175, 1, dict(placement=1)), (8, 8, 1176, 4, dict(placement=1)),                                                         # a host pool
])
def test_how_many_blocks_have_a_list(play, heads, G, candidates, selecting, config):
    (op,) = _decode(play, heads, candidates, 33, call="select", n_q_heads=G, **config)
    rows = int(op[4].split("x")[1])
    assert "step_kernel" in op[1] and rows - selecting in [-(-candidates // (32 * passes)) for passes in (1, 2, 4)]


@pytest.mark.parametrize("heads,G,candidates,home,rows", [
    (7, 5, 1100, True, 2 + 35 + 4 + 9),                                                                              # one pass a scoring block fits
    (6, 5, 1800, True, 2 + 29 + 8 + 9), (4, 7, 2000, True, 2 + 32 + 8 + 9), (7, 5, 1700, True, 2 + 27 + 8 + 9),      # two
    (4, 4, 4000, True, 2 + 32 + 16 + 9),                                                                             # four
    (4, 4, 2000, False, 2 + 63 + 1 + 9), (3, 5, 1800, False, 2 + 57 + 8 + 9),        # a block each; fewer than four heads: one pass, and away
])
def test_few_heads_with_shared_lists_come_home_by_more_passes(play, heads, G, candidates, home, rows):
    (op,) = _decode(play, heads, candidates, 65, n_q_heads=G)
    assert ("home_layer_kernel" in op[1], int(op[4].split("x")[1])) == (home, rows)


@pytest.mark.parametrize("placement,layers,kind", [(0, 1, 4), (0, 64, 5), (0, 80, 7), (1, 1, 4), (1, 64, 5)])
def test_other_poolings_read_past_the_cache_by_the_same_rule(play, placement, layers, kind):
    (op,) = [op for op in _decode(play, 1, 140, 33, n_layers=layers, n_q_heads=16, n_kv_heads=8, placement=placement, select_pooling=2) if "layer_kernel" in op[1]]
    assert f"layer_kernelILi1ELi2ELb{placement}ELi{kind}EE" in op[1]


if __name__ == "__main__":
    print(json.dumps(_play(*json.loads(sys.argv[1]))))
