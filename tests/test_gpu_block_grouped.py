"""fff_forward_block's grouped launches (levels from the root on the matrix cores, bucketing, subtree launch) against the oracle, on several
streams, and where they must not run: during capture and with a caller's workspace."""
import numpy as np
import pytest

import fff_workloads as W
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


def test_calls_overlap_on_several_streams(forced):
    """More streams than scratch blocks, calls of different inputs in flight together, twice: every result is that of the call alone (the
    calls that find no block take the launch without scratch, within its rounding)."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block on six streams T=6000 D=256 depth=7 n=4 L=6", flush=True)
    forced(3)
    states = [_state(STREAMS, 20 + i) for i in range(6)]
    alone, ungrouped = [], []
    for grouped, results in ((True, alone), (False, ungrouped)):
        F.fff_debug_option("subtree", 5 if grouped else 1)
        for d in states:
            results.append(torch.empty((6000, 256), dtype=torch.bfloat16, device="cuda"))
            _call(F, d, STREAMS, results[-1])
            torch.cuda.synchronize()
    F.fff_debug_option("subtree", 5)
    streams = [torch.cuda.Stream() for _ in states]
    outs = [[torch.empty_like(alone[0]) for _ in range(3)] for _ in states]
    torch.cuda.synchronize()
    for rep in range(3):
        for s, d, o in zip(streams, states, outs):
            with torch.cuda.stream(s):
                _call(F, d, STREAMS, o[rep])
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        for got in o:
            assert torch.equal(got, alone[i]) or torch.equal(got, ungrouped[i])


def test_no_scratch_during_capture_or_with_a_callers_workspace(forced):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped block captured, with a caller's workspace, after a release; T=6000 D=256 depth=7 n=4 L=6", flush=True)
    d = _state(STREAMS, 31)
    forced(3)
    out = torch.empty((6000, 256), dtype=torch.bfloat16, device="cuda")
    _call(F, d, STREAMS, out)
    torch.cuda.synchronize()
    assert "subtree_kernel" in F.fff_last_launch()
    grouped = out.clone()
    F.fff_debug_option("subtree", 1)
    _call(F, d, STREAMS, out)
    torch.cuda.synchronize()
    plain = out.clone()
    F.fff_debug_option("subtree", 5)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        _call(F, d, STREAMS, out)
    assert "subtree_kernel" not in F.fff_last_launch()
    for _ in range(3):
        out.fill_(float("nan"))
        _call(F, d, STREAMS, torch.empty_like(out))         # eager work between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, plain)
    buf = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    F.fff_set_workspace(buf)
    try:
        _call(F, d, STREAMS, out)
        torch.cuda.synchronize()
        assert "subtree_kernel" not in F.fff_last_launch() and torch.equal(out, plain)
    finally:
        F.fff_set_workspace(None)
    F.fff_release_workspace()
    _call(F, d, STREAMS, out)
    torch.cuda.synchronize()
    assert "subtree_kernel" in F.fff_last_launch() and torch.equal(out, grouped)


@pytest.mark.parametrize("T,D,O,depth,n,L,dtype,expect", [
    (40961, 768, 768, 8, 4, 8, BF16, True), (40960, 768, 768, 8, 4, 8, BF16, False),      # rows that 16 lanes hold: 160 tokens a compute unit
    (20000, 512, 1600, 7, 4, 8, BF16, True), (2000, 512, 1600, 7, 4, 8, BF16, False),      # longer rows: by estimate
    (45000, 64, 64, 3, 1, 2, BF16, False), (20000, 1032, 1032, 7, 4, 8, BF16, False),      # few rows met; a normalised row of more than 1024
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
