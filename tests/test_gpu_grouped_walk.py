"""The grouped walk (tokens grouped by the node they reach after the top levels, then the rest of the fused launch in that order):
the fused launch's bits for every kernel it has, at the edges of its tiles, and what a call does where no workspace is to be had."""
import pytest

import fff_workloads as W
from fff_testlib import check_against_oracle, run_forward, to_device

pytestmark = pytest.mark.gpu

# T, D, O, depth, L, dtype: rows of 4, 6, 8 pieces a lane of 16 and 3, 4, 8, 16 of 64, whole and checked ones; a tile holds 32 tokens
# (16 lanes each), 8 or 4: one more, one less, a single token
CASES = [
    (1, 768, 768, 7, 1, W.DTYPE_BF16), (31, 512, 512, 2, 3, W.DTYPE_BF16), (33, 768, 768, 8, 2, W.DTYPE_BF16),
    (257, 8, 16, 9, 1, W.DTYPE_BF16), (2049, 1024, 520, 8, 8, W.DTYPE_BF16), (9, 2048, 2048, 7, 4, W.DTYPE_BF16),
    (4097, 1800, 600, 9, 1, W.DTYPE_BF16), (7, 4096, 4096, 8, 4, W.DTYPE_BF16), (3001, 4000, 4000, 9, 3, W.DTYPE_BF16),
    (515, 8192, 2048, 8, 2, W.DTYPE_BF16), (1030, 384, 384, 10, 8, W.DTYPE_F32), (517, 1024, 1000, 8, 1, W.DTYPE_F32),
    (130, 2000, 500, 7, 2, W.DTYPE_F32), (5, 4096, 4096, 7, 1, W.DTYPE_F32),
    (7, 1032, 1032, 7, 2, W.DTYPE_BF16), (1001, 1528, 768, 9, 1, W.DTYPE_BF16), (9, 1536, 1536, 8, 3, W.DTYPE_BF16),     # 129, 191, 192 pieces
    (9, 764, 764, 8, 4, W.DTYPE_F32), (1030, 768, 768, 9, 1, W.DTYPE_F32),
]


@pytest.mark.parametrize("case", CASES, ids=["T%d_D%d_O%d_d%d_L%d_%s" % (c[:5] + (("f32", "bf16")[c[5]],)) for c in CASES])
@pytest.mark.parametrize("node_b", ["uniform", "zipf"])
def test_same_bits_as_the_fused_launch(case, node_b):
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, L, dtype = case
    print("\n[case] grouped walk T=%d D=%d O=%d depth=%d L=%d dtype=%d %s seed 71" % (case + (node_b,)), flush=True)
    w = W.make_layer("grouped", T, D, O, depth, L, W.ACT_GELU, dtype, seed=71, node_b=node_b)
    dev = to_device(w)
    res = {}
    try:
        for path in (1, 6):
            F.fff_set_option("path", path)
            res[path] = run_forward(w, dev)
            assert F.fff_get_option("last_path") == path
        assert "grouped" in F.fff_last_launch()
        out, _ = run_forward(w, dev, want_idx=False)
    finally:
        F.fff_set_option("path", 0)
    bits = torch.int16 if dtype == W.DTYPE_BF16 else torch.int32
    assert torch.equal(res[1][0].view(bits), res[6][0].view(bits)) and torch.equal(res[1][1], res[6][1])
    assert torch.equal(out.view(bits), res[6][0].view(bits))
    check_against_oracle(w, *res[6])




@pytest.mark.parametrize("T, D, O, depth, L, dtype, expect", [
    (65536, 768, 768, 13, 1, W.DTYPE_BF16, 6),       # in the place of the split launch
    (65536, 768, 768, 11, 1, W.DTYPE_BF16, 5),       # whose tables are not yet large enough here
    (30000, 360, 360, 13, 4, W.DTYPE_F32, 6),        # of the staged path's gather kernel
    (30000, 768, 768, 8, 8, W.DTYPE_BF16, 2),        # not of its subtree launch
    (8192, 1024, 1024, 13, 4, W.DTYPE_BF16, 1),      # up to 32 tokens a compute unit: fused
    (12753, 2080, 2080, 8, 6, W.DTYPE_BF16, 2),      # rows that fill half of the lanes stay with the tile kernels,
    (13000, 2080, 2080, 11, 8, W.DTYPE_BF16, 2),     # with the gather kernel
    (13000, 2104, 2104, 11, 2, W.DTYPE_BF16, 5),     # and with the split launch
    (9000, 2048, 2048, 14, 8, W.DTYPE_BF16, 1),      # few token rows, fewer than leaves: fused
])
def test_which_calls_take_it(T, D, O, depth, L, dtype, expect):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] route T=%d D=%d O=%d depth=%d L=%d dtype=%d" % (T, D, O, depth, L, dtype), flush=True)
    dt = torch.bfloat16 if dtype == W.DTYPE_BF16 else torch.float32
    n = 1 << depth
    new = lambda *s: torch.zeros(s, dtype=dt, device="cuda")
    F.fff_forward_hard(new(T, D), new(n - 1, D), new(n - 1), new(n, L, D), new(n, L), new(n, L, O), new(n, O), depth, L, W.ACT_RELU, new(T, O))
    torch.cuda.synchronize()
    assert F.fff_get_option("last_path") == expect, F.fff_last_launch()


@pytest.mark.parametrize("T, D, depth, L, other", [(8200, 768, 12, 1, 5), (9000, 768, 8, 8, 2), (700, 256, 6, 4, 1)], ids=["split", "staged", "medium"])
def test_asked_for_without_a_workspace_it_is_the_fused_launch(T, D, depth, L, other):
    """Option path = 6 with a caller's workspace that is too short, whatever launch the sizes take by themselves."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] path 6 without a workspace T=%d D=O=%d depth=%d L=%d bf16 seed 74" % (T, D, depth, L), flush=True)
    w = W.make_layer("grouped_no_ws", T, D, D, depth, L, W.ACT_RELU, W.DTYPE_BF16, seed=74)
    dev = to_device(w)
    run_forward(w, dev)
    assert F.fff_get_option("last_path") == other
    try:
        F.fff_set_option("path", 1)
        out, idx = run_forward(w, dev)
        F.fff_set_option("path", 6)
        short = torch.empty(256, dtype=torch.uint8, device="cuda")
        F.fff_set_workspace(short)
        got, got_idx = run_forward(w, dev)
        assert F.fff_get_option("last_path") == 1 and "grouped" not in F.fff_last_launch()
    finally:
        F.fff_set_workspace(None)
        F.fff_set_option("path", 0)
    assert torch.equal(got, out) and torch.equal(got_idx, idx)


def _deep():
    """A call that the fused launch would take, and whose tables outgrow the L2s: its arguments and its output."""
    import torch
    g0 = torch.Generator(device="cuda").manual_seed(73)
    new = lambda *s: torch.empty(s, device="cuda").uniform_(-.05, .05, generator=g0).to(torch.bfloat16)
    T, D, depth, L, n = 16385, 4096, 14, 3, 1 << 14
    args = (new(T, D), new(n - 1, D), new(n - 1), new(n, L, D), new(n, L), new(n, L, D), new(n, D), depth, L, W.ACT_GELU)
    return args, torch.full((T, D), float("nan"), dtype=torch.bfloat16, device="cuda")


def test_in_the_place_of_the_fused_launch_the_workspace_is_left_alone():
    """The fused launch needs no memory.  What takes its place neither grows the library's workspace nor works in it or in the caller's, so
    that a captured graph of such a call holds neither: it has scratch of torch's, and calls through the C ABI that bring none are fused.  The same
    bits each way."""
    import ctypes
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped walk without workspace T=16385 D=4096 depth=14 L=3 bf16", flush=True)
    args, ref = _deep()
    T, D = ref.shape
    depth, L = args[7:9]
    out = torch.full_like(ref, float("nan"))
    same = lambda: torch.equal(out.view(torch.int16), ref.view(torch.int16))
    F.fff_set_option("path", 1)
    try:
        F.fff_forward_hard(*args, ref)
    finally:
        F.fff_set_option("path", 0)
    torch.cuda.synchronize()
    F.fff_release_workspace()
    F.fff_debug_option("fail_workspace_growth", 1)          # (a call that grows it uses this up)
    try:
        F.fff_forward_hard(*args, out)
        torch.cuda.synchronize()
        assert F.fff_debug_option("fail_workspace_growth") == 1 and F.fff_get_option("last_path") == 6 and same()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            F.fff_forward_hard(*args, out)
        assert F.fff_get_option("last_path") == 6
        p = lambda t: ctypes.c_void_p(t.data_ptr())
        raw = [p(t) for t in args[:7]] + [depth, L, W.ACT_GELU, p(out), None, None, T, D, D, W.DTYPE_BF16]
        call = lambda entry, *more: (out.fill_(float("nan")), entry(*raw, *more), torch.cuda.synchronize())[1]
        need = F.fff_hard_scratch_bytes(T, D, D, depth, L, W.DTYPE_BF16)
        scratch = torch.empty(need, dtype=torch.uint8, device="cuda")
        lib = F.lib()
        for entry, more, path in ((lib.fff_forward_hard, (), 1), (lib.fff_forward_hard_scratch, (None, 0), 1),
                                  (lib.fff_forward_hard_scratch, (p(scratch), need), 6), (lib.fff_forward_hard_static, (), 1)):
            assert call(entry, *more) == 0 and F.fff_get_option("last_path") == path and same()
        assert F.fff_debug_option("fail_workspace_growth") == 1
    finally:
        F.fff_debug_option("fail_workspace_growth", 0)
    buf = torch.full((F.fff_workspace_bytes(T, depth),), 77, dtype=torch.uint8, device="cuda")
    for b in (buf[:256], buf):                              # too short for a layer that needs it, and large enough
        F.fff_set_workspace(b)
        try:
            out.fill_(float("nan"))
            F.fff_forward_hard(*args, out)
            torch.cuda.synchronize()
            assert F.fff_get_option("last_path") == 6 and same()
            with torch.cuda.graph(torch.cuda.CUDAGraph()):
                F.fff_forward_hard(*args, out)
            assert F.fff_get_option("last_path") == 6
        finally:
            F.fff_set_workspace(None)
    assert (buf[256:] == 77).all()
    for _ in range(3):
        out.fill_(float("nan"))
        scribble = [torch.full((1 << 20,), 255, dtype=torch.uint8, device="cuda") for _ in range(8)]     # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        assert same()
        del scribble


def test_streams_other_captures_and_no_memory():
    """Overlapping calls on several streams have scratch of their own; a stream that is captured by other means than torch's graphs, whose
    replays would work in memory of a later owner, and a full device get the fused launch."""
    import ctypes
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped walk on four streams, captured outside torch, out of memory T=16385 D=4096 depth=14 L=3 bf16", flush=True)
    args, ref = _deep()
    F.fff_forward_hard(*args, ref)
    torch.cuda.synchronize()
    assert F.fff_get_option("last_path") == 6
    streams, outs = [torch.cuda.Stream() for _ in range(4)], [torch.full_like(ref, float("nan")) for _ in range(4)]
    torch.cuda.synchronize()
    for rep in range(2):
        for s, o in zip(streams, outs):
            F.fff_forward_hard(*args, o, None, s)
            assert F.fff_get_option("last_path") == 6
    torch.cuda.synchronize()
    assert all(torch.equal(o.view(torch.int16), ref.view(torch.int16)) for o in outs)
    out, side = outs[0], streams[0]
    hip = ctypes.CDLL("libamdhip64.so")
    s, graph, execution = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(s, 1) == 0                  # thread-local
    try:
        F.fff_forward_hard(*args, out, None, side)
    finally:
        ended = hip.hipStreamEndCapture(s, ctypes.byref(graph))
    assert ended == 0 and F.fff_get_option("last_path") == 1
    assert hip.hipGraphInstantiate(ctypes.byref(execution), graph, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        assert hip.hipGraphLaunch(execution, s) == 0
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
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
        F.fff_forward_hard(*args, out)
        assert F.fff_get_option("last_path") == 1
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
