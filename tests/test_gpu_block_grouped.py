"""fff_forward_block's grouped launches (levels from the root on the matrix cores, bucketing, subtree launch) against the oracle, on several
streams, captured, and where there is no scratch for them."""
import ctypes

import numpy as np
import pytest

import fff_workloads as W
import oracle
from fff_testlib import ROUTING_MARGIN, TOL, out_to_f64
from test_gpu_block import _check, _inputs, _upload

pytestmark = pytest.mark.gpu
F32, BF16, RELU, GELU = W.DTYPE_F32, W.DTYPE_BF16, W.ACT_RELU, W.ACT_GELU


@pytest.fixture
def forced():
    """forced(k): grouped launches, k of the last levels with the leaves, at any batch size."""
    import paper_2308_14711_amd as F
    old = F.fff_debug_option("token_max_T")

    def to(k):
        F.fff_debug_option("token_max_T", 0)
        F.fff_debug_option("subtree", k + 2)
    yield to
    F.fff_debug_option("token_max_T", old)
    F.fff_debug_option("subtree", 0)


CASES = [
    # name,        T,    D,    O,    depth, n, L,  act,  dtype, norm, residual, k
    ("vit",        3000, 768,  768,  8,     4, 8,  GELU, BF16,  True,  True,  3),        # 124 columns from the root
    ("one",        1,    64,   64,   3,     2, 3,  RELU, BF16,  True,  True,  1),
    ("tile_more",  65,   8,    8,    2,     1, 1,  GELU, BF16,  True,  True,  1),        # rows of one piece
    ("seven",      1500, 1024, 264,  9,     1, 5,  GELU, BF16,  True,  False, 2),        # seven levels from the root; the longest row
    ("two_steps",  2000, 136,  136,  8,     8, 4,  RELU, BF16,  True,  True,  2),        # 8 neurons a node: levels in two launches
    ("wide16",     1000, 200,  200,  4,     16, 16, GELU, BF16, True,  True,  1),        # 48 columns with the leaves
    ("whole",      1500, 1024, 1040, 9,     1, 5,  GELU, BF16,  True,  False, 2),        # output rows of more than 1024: rows in three parts
    ("whole_two",  1300, 136,  1032, 8,     8, 4,  RELU, BF16,  True,  False, 2),        # the same, levels in two launches, an odd stage
    ("whole_one",  65,   8,    1032, 2,     1, 1,  GELU, BF16,  True,  False, 1),
    ("stages2",    700,  128,  128,  4,     3, 4,  GELU, BF16,  True,  True,  1),        # two and three whole stages, nothing behind them
    ("stages3",    700,  192,  192,  5,     2, 6,  RELU, BF16,  True,  True,  2),
    ("plain",      1100, 2056, 40,   5,     3, 6,  RELU, BF16,  False, False, 2),        # no normalisation: rows of any length
    ("f32",        1300, 512,  512,  6,     4, 8,  GELU, F32,   True,  True,  1),
    ("f32_two",    1200, 100,  68,   9,     2, 3,  RELU, F32,   True,  False, 2),        # 100 features: three pieces and a quarter of a stage
    ("f32_plain",  900,  1000, 1000, 4,     5, 2,  GELU, F32,   False, True,  1),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_against_the_oracle(case, forced):
    import paper_2308_14711_amd as F
    print("\n[case] grouped block %s T=%d D=%d O=%d depth=%d n=%d L=%d act=%d dtype=%d norm=%s residual=%s k=%d seed 5" % case, flush=True)
    forced(case[-1])
    _check(case[:-1])
    assert "subtree_kernel" in F.fff_last_launch() and F.fff_last_launch().endswith("k=%d" % case[-1]), F.fff_last_launch()
    _check(case[:-1], want_idx=False)
    if case[2] == case[3]:
        _check(case[:-1], in_place=True)


def _call(F, d, case, out, idx=None):
    _, T, D, O, depth, n, L, act, dtype, norm, residual = case
    F.fff_forward_block(d[0], d[1], d[2], 1e-5, *d[3:], depth, n, L, act, residual, out, idx)


def _state(case, seed):
    _, T, D, O, depth, n, L, act, dtype, norm, residual = case
    x, ln, nodes, leaves = _inputs(*case[:-1], seed)
    return [_upload(x)] + [_upload(a) for a in ln] + [_upload(a) for a in nodes] + [_upload(a) for a in leaves]


STREAMS = ("streams", 6000, 256, 256, 7, 4, 6, GELU, BF16, True, True)


def _rows(F, d, case=STREAMS):
    import torch
    out = torch.empty((case[1], case[3]), dtype=torch.bfloat16, device="cuda")
    _call(F, d, case, out)
    torch.cuda.synchronize()
    return out


def _grouped_and_not(F, d):
    """The call's rows through the grouped launches and through the one launch that needs no scratch."""
    grouped = _rows(F, d)
    assert "subtree_kernel" in F.fff_last_launch()
    F.fff_debug_option("subtree", 1)
    plain = _rows(F, d)
    assert "subtree_kernel" not in F.fff_last_launch()
    F.fff_debug_option("subtree", 5)
    return grouped, plain


def test_last_block_top_is_of_the_last_call(forced):
    import paper_2308_14711_amd as F
    case = ("top", 32768) + STREAMS[2:]
    print("\n[case] grouped block, last_block_top after a call with levels in LDS T=32768 D=256 depth=7 n=4 L=6", flush=True)
    d = _state(case, 40)
    forced(3)
    for option, staged in ((1, True), (5, False)):
        F.fff_debug_option("subtree", option)
        _rows(F, d, case)
        assert ("subtree_kernel" not in F.fff_last_launch()) == staged and (F.fff_get_option("last_block_top") > 0) == staged


def test_calls_overlap_on_several_streams(forced):
    """Calls of different inputs in flight together on six streams (and on one given by its handle), three times: every result is that of
    the call alone, bit for bit."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block on six streams T=6000 D=256 depth=7 n=4 L=6", flush=True)
    forced(3)
    states = [_state(STREAMS, 20 + i) for i in range(6)]
    alone = [_rows(F, d) for d in states]
    streams = [torch.cuda.Stream() for _ in states]
    outs = [[torch.empty_like(alone[0]) for _ in range(3)] for _ in states]
    torch.cuda.synchronize()
    for rep in range(3):
        for s, d, o in zip(streams, states, outs):
            if s is streams[0]:
                F.fff_forward_block(d[0], d[1], d[2], 1e-5, *d[3:], 7, 4, 6, GELU, True, o[rep], None, s.cuda_stream)
            else:
                with torch.cuda.stream(s):
                    _call(F, d, STREAMS, o[rep])
            assert "subtree_kernel" in F.fff_last_launch()
    torch.cuda.synchronize()
    for want, o in zip(alone, outs):
        assert all(torch.equal(got, want) for got in o)


def test_same_bits_eager_captured_and_beside_a_callers_workspace(forced):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block captured, and with a caller's workspace; T=6000 D=256 depth=7 n=4 L=6", flush=True)
    d, other = _state(STREAMS, 31), _state(STREAMS, 32)
    forced(3)
    grouped, _ = _grouped_and_not(F, d)
    want_other = _rows(F, other)
    out, out2 = torch.empty_like(grouped), torch.empty_like(grouped)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _call(F, d, STREAMS, out)
        assert "subtree_kernel" in F.fff_last_launch()
        _call(F, other, STREAMS, out2)
    for _ in range(3):
        out.fill_(float("nan"))
        out2.fill_(float("nan"))
        scribble = [torch.full((1 << 20,), 255, dtype=torch.uint8, device="cuda") for _ in range(8)]     # eager work between the replays
        assert torch.equal(_rows(F, other), want_other)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, grouped) and torch.equal(out2, want_other)
        del scribble
    buf = torch.full((1 << 20,), 77, dtype=torch.uint8, device="cuda")
    F.fff_set_workspace(buf)
    try:
        assert torch.equal(_rows(F, d), grouped) and "subtree_kernel" in F.fff_last_launch()
        assert (buf[256:] == 77).all()
    finally:
        F.fff_set_workspace(None)


def test_a_call_beside_another_threads_capture(forced):
    """An eager call for whose scratch the allocator has to ask the device, while another thread captures: both are what they are alone."""
    import threading
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block beside another thread's capture T=6000 D=256 depth=7 n=4 L=6", flush=True)
    d, other = _state(STREAMS, 35), _state(STREAMS, 36)
    forced(3)
    want, want_other = _rows(F, d), _rows(F, other)
    out, out_other = torch.full_like(want, float("nan")), torch.full_like(want, float("nan"))
    side, failed = torch.cuda.Stream(), []

    def eager():
        try:
            F.fff_forward_block(other[0], other[1], other[2], 1e-5, *other[3:], 7, 4, 6, GELU, True, out_other, None, side)
        except Exception as e:
            failed.append(e)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        t = threading.Thread(target=eager)
        t.start()
        t.join()
        _call(F, d, STREAMS, out)
    assert not failed, failed
    torch.cuda.synchronize()
    assert torch.equal(out_other, want_other)
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want)


def test_without_scratch_the_one_launch_runs(forced):
    """A stream captured by other means than torch's graphs, no memory left, and the entry point of the C ABI that takes no scratch."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block without scratch: captured outside torch, out of memory, C ABI; T=6000 D=256 depth=7 n=4 L=6", flush=True)
    d = _state(STREAMS, 33)
    forced(3)
    grouped, plain = _grouped_and_not(F, d)
    out = torch.full_like(plain, float("nan"))
    hip = ctypes.CDLL("libamdhip64.so")
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    s, graph, execution = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    torch.cuda.synchronize()
    assert hip.hipStreamBeginCapture(s, 1) == 0                  # thread-local
    try:
        F.fff_forward_block(d[0], d[1], d[2], 1e-5, *d[3:], 7, 4, 6, GELU, True, out, None, side)
    finally:
        ended = hip.hipStreamEndCapture(s, ctypes.byref(graph))
    assert ended == 0 and "subtree_kernel" not in F.fff_last_launch()
    assert hip.hipGraphInstantiate(ctypes.byref(execution), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(execution, s) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, plain)
    assert hip.hipGraphExecDestroy(execution) == 0 and hip.hipGraphDestroy(graph) == 0
    out.fill_(float("nan"))
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-6)
    try:
        keep = []
        try:                                                     # what the allocator still holds free
            while True:
                keep.append(torch.empty(1 << 19, dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:
            pass
        _call(F, d, STREAMS, out)
        assert "subtree_kernel" not in F.fff_last_launch()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    assert torch.equal(out, plain)
    L, p = F.lib(), lambda t: ctypes.c_void_p(t.data_ptr())
    args = lambda o: [p(t) for t in d[:3]] + [1e-5] + [p(t) for t in d[3:]] + [7, 4, 6, GELU, 1, p(o), None, None, 6000, 256, 256, 1]
    need = F.fff_block_scratch_bytes(6000, 256, 256, 7, 4, 6, True, BF16)
    scratch = torch.empty(need, dtype=torch.uint8, device="cuda")
    for entry, more, want in ((L.fff_forward_block, [], plain), (L.fff_forward_block_scratch, [None, 0], plain),
                              (L.fff_forward_block_scratch, [p(scratch), need], grouped)):
        out.fill_(float("nan"))
        assert entry(*args(out), *more) == 0
        torch.cuda.synchronize()
        assert torch.equal(out, want)
    assert L.fff_forward_block_scratch(*args(out), p(scratch), need - 1) == 6
    assert L.fff_forward_block_scratch(*args(out), ctypes.c_void_p(scratch.data_ptr() + 16), need) == 6
    assert L.fff_forward_block_scratch(*args(out), p(out), need) == 8


@pytest.mark.parametrize("T,D,O,depth,n,L,dtype,expect", [
    (50432, 768, 768, 8, 4, 8, BF16, True), (30000, 768, 768, 8, 4, 8, BF16, True), (16384, 768, 768, 8, 4, 8, BF16, False),      # by estimate
    (20000, 512, 1600, 7, 4, 8, BF16, True), (2000, 512, 1600, 7, 4, 8, BF16, False),
    (45000, 64, 64, 3, 1, 2, BF16, False), (20000, 1032, 1032, 7, 4, 8, BF16, False),      # few rows met; a normalised row of more than 1024
    (50000, 768, 768, 8, 4, 17, BF16, False),                                               # leaves of more than 16 neurons
], ids=str)
def test_which_batches_take_them(T, D, O, depth, n, L, dtype, expect):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block rule T=%d D=%d O=%d depth=%d n=%d L=%d" % (T, D, O, depth, n, L), flush=True)
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    nodes, leaves = (1 << depth) - 1, 1 << depth
    out = torch.empty((T, O), dtype=torch.bfloat16, device="cuda")
    F.fff_forward_block(z(T, D), z(D), z(D), 1e-5, z(nodes, n, D), z(nodes, n), z(nodes, n), z(nodes), z(leaves, L, D), z(leaves, L), z(leaves, L, O),
                        z(leaves, O), depth, n, L, RELU, O == D, out)
    torch.cuda.synchronize()
    assert ("subtree_kernel" in F.fff_last_launch()) == expect, F.fff_last_launch()
    assert not out.any()


@pytest.mark.parametrize("what", ["gamma", "nodes", "leaves"])
def test_infinite_gammas_and_weights_on_normalised_bf16_rows(what, forced):
    """An infinite scale of one feature, or infinite weights: routing, infinities and NaN as the oracle has them (both bf16 rows of a
    token meet an infinite weight, the second with any sign or zero).  The same for calls of rows of up to 1024 features with longer output
    rows, whose launch without scratch has the token in fp32."""
    import torch
    import paper_2308_14711_amd as F
    case = ("inf", 700, 512, 1040, 5, 3, 4, RELU, BF16, True, False)
    name, T, D, O, depth, n, L, act, dtype, norm, residual = case
    print("\n[case] grouped block bf16 infinities in %s T=%d D=%d O=%d depth=%d n=%d L=%d seed 41" % ((what,) + case[1:7]), flush=True)
    forced(2)
    x, ln, nodes, leaves = _inputs(*case[:-1], 41)
    ln, nodes, leaves = [a.copy() for a in ln], [a.copy() for a in nodes], [a.copy() for a in leaves]
    inf, minus_inf = np.uint16(0x7F80), np.uint16(0xFF80)
    if what == "gamma":
        ln[0][17] = inf
    elif what == "nodes":
        nodes[0][0, 0, -1], nodes[0][1:3, 1, 30] = inf, minus_inf
    else:
        leaves[0][::2, 1, -1], leaves[0][1::2, 2, 100] = inf, minus_inf
    d = [_upload(x)] + [_upload(a) for a in ln] + [_upload(a) for a in nodes] + [_upload(a) for a in leaves]
    out = torch.full((T, O), 7.0, dtype=torch.bfloat16, device="cuda")
    idx = torch.full((T,), -9, dtype=torch.int32, device="cuda")
    _call(F, d, case, out, idx)
    torch.cuda.synchronize()
    assert "subtree_kernel" in F.fff_last_launch()
    ref, ref_idx, margin = oracle.forward_block(x, *ln, 1e-5, *nodes, *leaves, depth, n, L, act, residual)
    same = idx.cpu().numpy() == ref_idx
    assert (margin[~same] < ROUTING_MARGIN).all() and same.sum() > T // 2, "routing differs from the oracle"
    got, want = out_to_f64(out)[same], ref[same]
    assert not np.isfinite(want).all() or what == "nodes"
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
    assert np.array_equal(got[np.isinf(got)], want[np.isinf(want)])
    fin = np.isfinite(want)
    scale = np.where(fin, np.abs(want), 0).max(axis=1, keepdims=True) + 1e-30
    assert (np.abs(np.where(fin, got, 0) - np.where(fin, want, 0)) <= TOL[dtype] * scale).all()
