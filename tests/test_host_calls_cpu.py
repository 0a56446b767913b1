"""The library's host side (plans, workspaces, launches) on a HIP runtime that
records instead of running: no GPU needed."""
import os
import threading

import pytest

import host_calls
from host_calls import BF16, F32


@pytest.fixture(scope="module")
def so(tmp_path_factory):
    if not os.path.exists(host_calls.LIB):
        pytest.skip("libquan.so not built")
    return host_calls.build(tmp_path_factory.mktemp("fakehip"))


# ---- host threads on one stream ----

# (call, shape (n, c_in, h, w, c_out, k, stride, pad)): launches around a shared buffer
SHARED = [("forward_packed", (8, 12, 20, 20, 20, 3, 1, 1)),   # a padded copy
          ("forward_packed", (8, 20, 33, 31, 16, 3, 1, 1)),   # a larger one: the buffer grows
          ("forward_packed", (1, 128, 7, 7, 64, 3, 1, 1)),    # partial tiles
          ("forward_packed", (1, 256, 14, 14, 256, 3, 1, 1)),
          ("forward", (4, 16, 16, 16, 32, 3, 1, 1)),          # packed kernels
          ("inference", (4, 12, 16, 16, 32, 3, 1, 1)),
          ("iqbn_layer", (16, 64, 56, 56, 64, 3, 1, 1)),      # statistics
          ("backward_data", (4, 16, 16, 16, 32, 3, 2, 1)),
          ("backward_weight", (4, 16, 16, 16, 32, 3, 1, 1))]


def _threads(q, streams):
    """Two threads, each its own order of the calls; what they launched."""
    for name, shape in SHARED:      # each call's launches by itself
        getattr(q, name)(shape, stream=streams[0])
    alone = {}
    for name, shape in SHARED:
        q.clear()
        getattr(q, name)(shape, stream=streams[0])
        alone[(name, shape)] = [e.name for e in q.events() if e.what == "L"]
    q.lib.quan_release()
    q.clear()
    q.fake.fake_delay(100)
    failed = []

    def run(tag):
        try:
            q.fake.fake_tag(tag)
            for name, shape in (SHARED if tag == 1 else SHARED[::-1]) * 4:
                getattr(q, name)(shape, stream=streams[tag - 1])
        except Exception as e:  # noqa: BLE001
            failed.append(repr(e))

    threads = [threading.Thread(target=run, args=(t,)) for t in (1, 2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    return alone, q.events(), failed


def test_calls_of_two_threads_on_one_stream_do_not_interleave(so):
    """Calls that hand data from one launch to the next through a buffer of the
    stream: with two threads on one stream, each call's launches stay
    together, and a buffer that a call has taken is not freed before its last
    launch."""
    alone, events, failed = host_calls.in_child(_threads, so, (0, 0))
    assert not failed, failed
    assert all(len(v) > 1 for k, v in alone.items()), alone
    per = {1: list(SHARED) * 4, 2: SHARED[::-1] * 4}
    launches = [e for e in events if e.what == "L"]
    i = 0
    while i < len(launches):
        tag = launches[i].tag
        want = alone[per[tag].pop(0)]
        got = launches[i:i + len(want)]
        assert [(e.tag, e.name) for e in got] == [(tag, n) for n in want], f"launch {i}"
        i += len(want)
    assert not per[1] and not per[2]
    # a launch whose first argument lies in a buffer finds it allocated
    live = {}
    for e in events:
        if e.what == "M":
            live[e.ptr] = e.bytes
        elif e.what == "F":
            del live[e.ptr]
        elif e.what == "L" and 0x600000000000 <= e.ptr < 0x700000000000:
            assert any(p <= e.ptr < p + b for p, b in live.items()), e


def test_threads_on_different_streams_run_side_by_side(so):
    """Streams have their own buffers and wait for nobody."""
    _, events, failed = host_calls.in_child(_threads, so, (0x11, 0x22))
    assert not failed, failed
    tags = [e.tag for e in events if e.what == "L"]
    changes = sum(a != b for a, b in zip(tags, tags[1:]))
    assert changes > len(SHARED) * 8, "one thread waited for the other's calls"


# ---- calls under graph capture, after a warm-up on another size ----

S = 0x33  # the stream


def _captured(q, call, warm, shape, kw):
    getattr(q, call)(warm, stream=S, **kw)
    q.clear()
    q.fake.fake_capture(S, 1)
    try:
        getattr(q, call)(shape, stream=S, **kw)
    finally:
        q.fake.fake_capture(S, 0)
    return q.events()


def check_captured(so, call, warm, shape, **kw):
    events = host_calls.in_child(_captured, so, call, warm, shape, kw)
    assert any(e.what == "L" for e in events)
    assert all(e.what == "L" and e.in_capture for e in events), [e for e in events if e.what != "L"]


ONE, FEW, MANY = (1, 64, 14, 14), (4, 64, 28, 28), (64, 64, 28, 28)


@pytest.mark.parametrize("dtype", [BF16, F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("c_out", [32, 64, 200, 600])
@pytest.mark.parametrize("warm,shape", [(ONE, FEW), (ONE, MANY), (FEW, MANY), (MANY, ONE), (MANY, FEW)])
def test_inference_captured_after_another_size(so, dtype, k, c_out, warm, shape):
    """An inference layer that has run on the stream, with any batch, is
    captured without an allocation: whichever form the new size takes."""
    tail = (c_out, k, 1, k // 2)
    check_captured(so, "inference", warm + tail, shape + tail, dtype=dtype)


def test_inference_captured_after_another_layer(so):
    """A layer of another kernel size and as many output channels is warm-up enough."""
    check_captured(so, "inference", (16, 64, 56, 56, 64, 1, 1, 0), (16, 64, 56, 56, 64, 3, 1, 1))


# ---- buffers that a captured graph holds ----

# (call, captured, the larger call after it)
OUTGROWN = [("forward", (2, 16, 12, 12, 16, 3, 1, 1), (2, 128, 12, 12, 128, 3, 1, 1)),       # packed kernels
            ("forward_packed", (1, 128, 7, 7, 64, 3, 1, 1), (1, 256, 14, 14, 256, 3, 1, 1)),  # partial tiles
            ("forward_packed", (2, 12, 20, 20, 16, 3, 1, 1), (8, 12, 40, 40, 16, 3, 1, 1)),   # a padded copy
            ("backward_data", (2, 16, 12, 12, 16, 3, 1, 1), (2, 128, 12, 12, 128, 3, 1, 1)),  # packed kernels
            ("backward_weight", (8, 16, 32, 32, 16, 3, 1, 1), (8, 128, 32, 32, 128, 3, 1, 1)),
            ("inference", (16, 64, 28, 28, 64, 3, 1, 1), (16, 64, 28, 28, 128, 3, 1, 1)),     # folded maps
            ("iqbn_layer", (2, 64, 12, 12, 64, 3, 1, 1), (16, 64, 56, 56, 512, 1, 1, 0)),     # statistics
            ("iqbn", (2, 64, 40, 40), (16, 512, 56, 56)),
            ("iqbn_backward", (2, 64, 40, 40), (16, 512, 56, 56))]


def _outgrown(q, call, shape, larger):
    getattr(q, call)(*(shape if call in FLAT else (shape,)), stream=S)
    q.fake.fake_capture(S, 1)
    getattr(q, call)(*(shape if call in FLAT else (shape,)), stream=S)
    q.fake.fake_capture(S, 0)
    q.clear()
    getattr(q, call)(*(larger if call in FLAT else (larger,)), stream=S)
    grown = q.events()
    q.clear()
    q._ok(q.lib.quan_release())
    return grown, q.events()


FLAT = ("iqbn", "iqbn_backward")


@pytest.mark.parametrize("call,shape,larger", OUTGROWN, ids=[f"{c}-{s}" for c, s, _ in OUTGROWN])
def test_captured_buffers_outlive_a_larger_call(so, call, shape, larger):
    """Whatever buffer a captured call took, its replays still find it after a
    larger call on the stream; quan_release gives all of them back."""
    grown, released = host_calls.in_child(_outgrown, so, call, shape, larger)
    assert any(e.what == "M" for e in grown), "the larger call grew nothing"
    assert not [e for e in grown if e.what == "F"]
    assert len([e for e in released if e.what == "F"]) > len([e for e in grown if e.what == "M"])


# ---- captures of a smaller batch than the stream has run ----

def _smaller(q, cases):
    """The cases whose capture allocated or failed."""
    bad = []
    for i, (call, shape, batch, kw) in enumerate(cases):
        stream = 0x1000 + 16 * i

        def go(n):
            args = (n, *shape) if call in FLAT else ((n, *shape),)
            getattr(q, call)(*args, stream=stream, **kw)

        go(batch[0])
        q.clear()
        q.fake.fake_capture(stream, 1)
        try:
            go(batch[1])
        except RuntimeError as e:
            bad.append((call, shape, batch, kw, str(e)))
        q.fake.fake_capture(stream, 0)
        q.fake.hipGetLastError()
        bad += [(call, shape, batch, kw, e.what) for e in q.events() if e.what != "L"]
    return bad


BATCHES = [(64, 4), (64, 1), (8, 1), (8, 5), (4, 3), (16, 5), (3, 2), (1, 1)]


@pytest.mark.parametrize("stats", [0, 1, 2], ids=["auto", "epilogue", "pass"])
@pytest.mark.parametrize("dtype", [BF16, F32], ids=["bf16", "fp32"])
def test_training_layer_captured_on_a_smaller_batch(so, dtype, stats):
    """A convolution with IQBN behind it that has run on the stream is captured
    with any smaller batch without an allocation, whichever place its
    statistics then come from."""
    layers = [(20, 8, 8, 8, 3, 1, 1), (48, 32, 32, 32, 3, 2, 1), (32, 16, 16, 32, 3, 1, 1), (64, 28, 28, 64, 3, 1, 1),
              (256, 14, 14, 256, 3, 1, 1), (400, 8, 8, 32, 3, 1, 1), (64, 28, 28, 128, 1, 1, 0), (16, 32, 32, 16, 5, 1, 2)]
    cases = [("iqbn_layer", s, b, dict(dtype=dtype, stats=stats)) for s in layers for b in BATCHES]
    assert host_calls.in_child(_smaller, so, cases) == []


@pytest.mark.parametrize("dtype", [BF16, F32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("call", ["backward_weight", "backward_data", "forward", "iqbn", "iqbn_backward"])
def test_other_calls_captured_on_a_smaller_batch(so, call, dtype):
    """So are the other calls that need a buffer."""
    sizes = [(c, h, w) for c in (1, 12, 16, 32, 48, 69, 128) for h, w in ((32, 32), (14, 14), (9, 11), (5, 40))]
    layers = sizes if call in FLAT else [(c, h, w, o, k, s, k // 2) for c, h, w in sizes for o in (8, 16, 20, 70)
                                         for k, s in ((1, 1), (3, 1), (3, 2), (5, 1))]
    cases = [(call, s, b, dict(dtype=dtype)) for s in layers for b in BATCHES]
    assert host_calls.in_child(_smaller, so, cases) == []


# ---- where the statistics of a convolution + IQBN come from ----

def _stats_launches(q, shapes, stats, dtype):
    out = []
    for i, shape in enumerate(shapes):
        q.iqbn_layer(shape, dtype=dtype, stats=stats, stream=0x5000 + 16 * i)
        q.clear()
        q.iqbn_layer(shape, dtype=dtype, stats=stats, stream=0x5000 + 16 * i)
        out.append([e.name for e in q.events() if e.what == "L"])
    return out


# few tiles and many stages: layers whose convolution splits K where it may
SPLIT = [(1, 256, 14, 14, 256, 3, 1, 1), (1, 64, 28, 28, 64, 3, 1, 1), (4, 128, 7, 7, 32, 3, 1, 1),
         (1, 64, 40, 40, 48, 3, 1, 1)]


def test_epilogue_statistics_are_the_epilogues(so):
    """A caller that asks for statistics in the convolution's epilogue gets them
    there wherever the layer's tiles can gather them, also on a layer that
    would split K otherwise."""
    for names in host_calls.in_child(_stats_launches, so, SPLIT, 1, BF16):
        assert len(names) == 3, names
        assert any("iqbn_finalize_tiles" in n for n in names) and not any("add_splits" in n for n in names), names
    for names in host_calls.in_child(_stats_launches, so, SPLIT[:2], 0, BF16):
        assert any("add_splits" in n for n in names), names
    # fp32 tiles cannot: the pass, behind a split convolution
    for names in host_calls.in_child(_stats_launches, so, SPLIT[:2], 1, F32):
        assert any("add_splits" in n for n in names) and not any("tiles" in n for n in names), names


# ---- calls beside another stream's capture ----

def _beside(q, calls):
    for name, args in calls:        # the stream's other buffers
        getattr(q, name)(*args, stream=S)
    q.clear()
    q.fake.fake_capture(0x99, 1)    # by another thread
    for name, args in calls:
        args = tuple((a[0] * 16,) + a[1:] if isinstance(a, tuple) else a for a in args)
        getattr(q, name)(*args, stream=S)
    q.fake.fake_capture(0x99, 0)
    return q.events()


def test_growing_buffers_leave_other_streams_captures_alone(so):
    """A call that allocates or outgrows its buffers while another thread
    captures another stream makes no call that would break that capture."""
    calls = [(name, (shape,)) for name, shape in SHARED]
    events = host_calls.in_child(_beside, so, calls)
    assert any(e.what == "M" for e in events) and any(e.what == "F" for e in events)
    assert not [e for e in events if e.name == "refused"]


# ---- the padded copy of partial channel chunks ----

def _pads(q, cases):
    out = []
    for i, (call, shape, dtype) in enumerate(cases):
        q.clear()
        getattr(q, call)(shape, dtype=dtype, stream=0x7000 + 16 * i)
        ev = q.events()
        out.append((any("pad_channels" in e.name for e in ev), max([e.bytes for e in ev if e.what == "M"], default=0)))
    return out


def test_padded_copy_is_made_where_it_pays(so):
    """The rule's two sides at sizes that were measured (one launch more and a
    pass over both copies, against element loads in every stage)."""
    no = [((32, 3, 112, 112, 16, 1, 1, 0), BF16), ((32, 9, 112, 112, 16, 1, 1, 0), BF16),
          ((64, 5, 56, 56, 32, 1, 1, 0), BF16), ((64, 12, 56, 56, 32, 1, 1, 0), BF16),
          ((16, 18, 56, 56, 16, 1, 1, 0), BF16), ((16, 60, 56, 56, 16, 1, 1, 0), BF16),
          ((20, 92, 40, 40, 13, 1, 1, 0), BF16), ((8, 100, 56, 56, 16, 1, 1, 0), BF16),
          ((16, 9, 56, 56, 16, 1, 1, 0), F32), ((16, 33, 56, 56, 16, 1, 1, 0), F32),
          ((32, 1, 112, 112, 16, 1, 1, 0), F32)]
    yes = [((32, 12, 112, 112, 16, 1, 1, 0), BF16), ((64, 28, 56, 56, 32, 1, 1, 0), BF16),
           ((16, 100, 56, 56, 16, 1, 1, 0), BF16), ((8, 7, 112, 112, 128, 1, 1, 0), BF16),
           ((8, 1, 64, 64, 16, 3, 1, 1), BF16), ((1, 1, 32, 32, 16, 3, 1, 1), BF16),
           ((64, 1, 224, 224, 16, 3, 1, 1), BF16), ((8, 12, 75, 77, 20, 3, 1, 1), BF16),
           ((64, 9, 56, 56, 32, 1, 1, 0), F32), ((64, 33, 56, 56, 32, 1, 1, 0), F32),
           ((32, 1, 112, 112, 16, 3, 1, 1), F32)]
    got = host_calls.in_child(_pads, so, [("forward_packed", s, t) for s, t in no + yes])
    wrong = [(s, t) for (s, t), (padded, _) in zip(no + yes, got) if padded != ((s, t) in yes)]
    assert not wrong


def test_padded_copy_is_bounded(so):
    """No call keeps more than 512 MiB for a padded copy, though one bf16 channel
    becomes eight."""
    cases = [("forward_packed", (16, 1, 700, 700, 8, 3, 1, 1), BF16), ("forward_packed", (64, 1, 512, 512, 8, 3, 1, 1), BF16),
             ("forward_packed", (64, 3, 512, 512, 4, 3, 1, 1), F32), ("backward_data", (64, 4, 512, 512, 1, 3, 1, 1), BF16)]
    for (padded, largest), case in zip(host_calls.in_child(_pads, so, cases), cases):
        assert largest <= 512 << 20, (case, largest)
        assert padded == (case[1][0] == 16), case


# ---- the stem's work-groups ----

def _stem_groups(q, cases):
    out = []
    for case in cases:
        q.clear()
        q.stem(*case)
        out.append([e.bytes for e in q.events() if e.what == "L"])
    return out


def test_stem_work_groups_have_pixels_for_their_table(so):
    """Every work-group builds the layer's weight table, so beyond two per compute
    unit (512), which build theirs side by side, none is launched for a short
    row of a narrow image: 64 output pixels or more each."""
    cases = [(n, h, h, c, k, s) for n in (1, 8, 64) for h in (9, 14, 27, 37, 56, 86, 138, 224) for s in (1, 2)
             for c, k in ((4, 3), (16, 3), (24, 5), (36, 3), (64, 1), (64, 3), (16, 7))]
    for case, groups in zip(cases, host_calls.in_child(_stem_groups, so, cases)):
        n, h, _, c, k, s = case
        pixels = n * ((h - 1) // s + 1) ** 2
        assert len(groups) == 1 and groups[0] <= max(512, n, pixels / 64), (case, groups)


# ---- forms by size ----

def _names(q, cases):
    out = []
    for i, (call, args, kw) in enumerate(cases):
        q.clear()
        getattr(q, call)(*args, stream=0x9000 + 16 * i, **kw)
        ev = q.events()
        out.append(([(e.name, e.bytes) for e in ev if e.what == "L"], [e.bytes for e in ev if e.what == "M"]))
    return out


def test_wide_fp32_rows_take_the_merged_form(so):
    """A tensor of few pixels takes one launch, but fp32 rows above 4 MiB, of
    which a column group reads half lines, the merged two."""
    cases = [("iqbn", (1, c, 32, 32), dict(dtype=t)) for c, t in ((256, F32), (260, F32), (1024, F32), (512, BF16), (1024, BF16))]
    small = [any("iqbn_small" in n for n, _ in names) for names, _ in host_calls.in_child(_names, so, cases)]
    assert small == [True, False, False, True, True]


def test_partials_of_rows_read_by_element(so):
    """Rows that are no whole 16-byte pieces, few side by side in a block, leave
    partials for at least 24 rows each."""
    cases = [("iqbn_backward", (1, c, 1, px), dict(relu=False)) for c in (55, 231, 291) for px in (1024, 2000, 5000)]
    for (call, args, _), (names, _) in zip(cases, host_calls.in_child(_names, so, cases)):
        assert "iqbn_bwd_reduce" in names[0][0]
        assert names[0][1] <= args[3] // 24 + 1, (args, names[0])


def test_blocks_of_wide_rows(so):
    """Passes without partials go to about four blocks per compute unit over all
    column groups, however many those are; the statistics to one."""
    cases = [("iqbn_backward", (1, 401, 1, 11135), dict(relu=False)), ("iqbn", (1, 401, 1, 11135), dict()),
             ("iqbn", (1, 24, 1, 36469), dict(dtype=F32))]
    (gradient, _), (forward, _), (narrow, _) = host_calls.in_child(_names, so, cases)
    assert "iqbn_bwd_apply" in gradient[-1][0] and gradient[-1][1] <= 11135 // 24 + 1
    assert "iqbn_affine" in forward[-1][0] and forward[-1][1] <= 11135 // 24 + 1
    assert "iqbn_stats" in narrow[0][0] and narrow[0][1] <= 256
