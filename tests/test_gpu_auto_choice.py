"""The launch path chosen by shape and batch size against the forced ones, on shapes that none of the
rules in fff_api.hip was fitted on (row lengths other than 768 and 4096, inputs and outputs of different
width, fp32): the automatic choice must be within 30 % of the fastest path that takes the shape.  A
timing test, so with a wide margin: what it catches is a rule that sends a shape to a path that is half
as fast as another one, not a few percent."""
import numpy as np
import pytest

import fff_workloads as W

pytestmark = pytest.mark.gpu

SHAPES = [
    # T,      D,    O,    depth, L, dtype
    (20000,  1024, 1024, 9,  1,  W.DTYPE_BF16),
    (20000,  1024, 1024, 9,  6,  W.DTYPE_BF16),
    (100000, 512,  512,  10, 2,  W.DTYPE_BF16),
    (30000,  2048, 512,  12, 1,  W.DTYPE_BF16),
    (12000,  384,  1536, 8,  8,  W.DTYPE_BF16),
    (9000,   3072, 768,  9,  2,  W.DTYPE_BF16),
    (50000,  768,  3072, 5,  8,  W.DTYPE_BF16),
    (40000,  640,  640,  11, 2,  W.DTYPE_BF16),
    (1500,   768,  768,  8,  4,  W.DTYPE_BF16),
    (30000,  512,  512,  9,  2,  W.DTYPE_F32),
    # a wave a token against a block a token on element-wise output rows of wide leaves, and against the staged path's full tiles
    (2547,   32,   958,  5,  32, W.DTYPE_BF16),
    (6366,   544,  544,  1,  32, W.DTYPE_BF16),
    (8128,   872,  872,  9,  16, W.DTYPE_BF16),
    # the grouped walk against the tile kernels, with rows that fill half of its lanes
    (12753,  2080, 2080, 8,  6,  W.DTYPE_BF16),
    (14111,  2272, 2272, 9,  8,  W.DTYPE_BF16),
]


@pytest.mark.parametrize("shape", SHAPES, ids=["T%d_D%d_O%d_d%d_L%d_%s" % (s[0], s[1], s[2], s[3], s[4], "bf16" if s[5] else "f32")
                                               for s in SHAPES])
def test_automatic_choice_is_close_to_the_fastest_path(shape):
    import torch
    import paper_2308_14711_amd as F
    from fff_testlib import to_device
    T, D, O, depth, L, dtype = shape
    print("\n[case] auto choice T=%d D=%d O=%d depth=%d L=%d dtype=%d seed 71" % (T, D, O, depth, L, dtype), flush=True)
    w = W.make_layer("auto", T, D, O, depth, L, W.ACT_GELU, dtype, seed=71, keep_f32=False)
    dev = to_device(w)
    es = 2 if dtype == W.DTYPE_BF16 else 4
    n = max(2, min(6, int(6.0e8 / (T * (D + O) * es))))          # rotate buffers: no run finds its rows cached
    xs = [dev["x"]] + [dev["x"].clone() for _ in range(n - 1)]
    outs = [torch.empty((T, O), dtype=dev["x"].dtype, device="cuda") for _ in range(n)]
    idx = torch.empty((T,), dtype=torch.int32, device="cuda")
    times, took = {}, {}
    try:
        for path in (0, 1, 2, 4, 5):
            F.fff_set_option("path", path)

            def step(i):
                F.fff_forward_hard(xs[i % n], dev["node_w"], dev["node_b"], dev["leaf_w1"], dev["leaf_b1"], dev["leaf_w2"],
                                   dev["leaf_b2"], depth, L, w.act, outs[i % n], idx)

            for i in range(5):
                step(i)
            torch.cuda.synchronize()
            if path and F.fff_get_option("last_path") != path:
                continue                                   # the shape does not take this path
            best = float("inf")
            for rep in range(3):                           # best of three batches of 20 calls
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                for i in range(20):
                    step(i)
                e1.record()
                torch.cuda.synchronize()
                best = min(best, e0.elapsed_time(e1) * 1000 / 20)
            times[path] = best
            took[path] = F.fff_get_option("last_path")
    finally:
        F.fff_set_option("path", 0)
    fastest = min(v for k, v in times.items() if k != 0)
    print("  auto -> path %d: %.1f us; forced: %s" % (took[0], times[0], {k: round(v, 1) for k, v in times.items() if k}), flush=True)
    assert times[0] <= 1.3 * fastest + 2.0, "auto took path %d at %.1f us, the fastest path needs %.1f us" % (took[0], times[0], fastest)


def _best(step):
    """Best of three batches of 20 calls, us a call."""
    import torch
    for _ in range(5):
        step()
    best = float("inf")
    for rep in range(3):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record()
        for _ in range(20):
            step()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 1000 / 20)
    return best


# the two kernels of one block a token, and the element-wise kernel for leaves that nothing else takes: T, D, O, depth, L, dtype
TOKEN_SHAPES = [(4500, 456, 456, 3, 120, W.DTYPE_BF16), (40, 1096, 1096, 3, 300, W.DTYPE_BF16), (1900, 344, 2900, 3, 90, W.DTYPE_BF16),
                (90, 904, 904, 6, 20, W.DTYPE_BF16), (1300, 200, 200, 8, 20, W.DTYPE_F32), (900, 328, 23, 6, 14, W.DTYPE_BF16),
                (500, 480, 113, 4, 300, W.DTYPE_BF16), (9000, 33, 33, 4, 100, W.DTYPE_BF16)]


@pytest.mark.parametrize("shape", TOKEN_SHAPES, ids=["T%d_D%d_O%d_d%d_L%d_%s" % (s[:5] + ("bf16" if s[5] else "f32",)) for s in TOKEN_SHAPES])
def test_one_block_a_token_takes_the_faster_kernel(shape):
    import torch
    import paper_2308_14711_amd as F
    from fff_testlib import to_device
    T, D, O, depth, L, dtype = shape
    print("\n[case] token kernels T=%d D=%d O=%d depth=%d L=%d dtype=%d seed 72" % shape, flush=True)
    w = W.make_layer("auto", T, D, O, depth, L, W.ACT_GELU, dtype, seed=72, keep_f32=False)
    dev = to_device(w)
    out, idx = torch.empty((T, O), dtype=dev["x"].dtype, device="cuda"), torch.empty((T,), dtype=torch.int32, device="cuda")
    times = {}
    try:
        for name, path, kernel in (("auto", 0, 0), ("block", 4, 1), ("rows", 4, 2), ("element-wise", 3, 0)):
            F.fff_set_option("path", path)
            F.fff_debug_option("token_kernel", kernel)
            times[name] = _best(lambda: F.fff_forward_hard(dev["x"], dev["node_w"], dev["node_b"], dev["leaf_w1"], dev["leaf_b1"],
                                                           dev["leaf_w2"], dev["leaf_b2"], depth, L, w.act, out, idx))
    finally:
        F.fff_set_option("path", 0)
        F.fff_debug_option("token_kernel", 0)
    print("  us a call:", {k: round(v, 1) for k, v in times.items()}, flush=True)
    assert times["auto"] <= 1.3 * min(times.values()) + 2.0, times


# fff_forward_block's small batches against its kernels of large ones: T, D, depth, n, L, dtype
BLOCK_SHAPES = [(900, 88, 2, 2, 3, W.DTYPE_F32), (1000, 56, 3, 3, 6, W.DTYPE_BF16), (480, 776, 7, 4, 8, W.DTYPE_BF16), (1000, 504, 8, 8, 16, W.DTYPE_BF16),
                (700, 1544, 6, 4, 8, W.DTYPE_BF16), (950, 27, 2, 1, 3, W.DTYPE_BF16), (900, 333, 6, 4, 4, W.DTYPE_F32)]


@pytest.mark.parametrize("shape", BLOCK_SHAPES, ids=["T%d_D%d_d%d_n%d_L%d_%s" % (s[:5] + ("bf16" if s[5] else "f32",)) for s in BLOCK_SHAPES])
def test_norm_block_takes_the_faster_side(shape):
    import torch
    import paper_2308_14711_amd as F
    from fff_testlib import to_device
    T, D, depth, n, L, dtype = shape
    print("\n[case] block auto T=%d D=%d depth=%d n=%d L=%d dtype=%d seed 73" % shape, flush=True)
    w = W.make_layer("auto", T, D, D, depth, L, W.ACT_GELU, dtype, seed=73, keep_f32=False)
    dev = to_device(w)

    def up(a):
        return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16) if a.dtype == np.uint16 else torch.from_numpy(a).cuda()

    ln = [up(a) for a in W.layer_norm_params(D, dtype, seed=73)]
    nodes = [up(a) for a in W.wide_nodes(depth, n, D, dtype, seed=73)]
    out, idx = torch.empty((T, D), dtype=dev["x"].dtype, device="cuda"), torch.empty((T,), dtype=torch.int32, device="cuda")
    times, old = {}, F.fff_debug_option("token_max_T")
    try:
        for name, limit in (("auto", old), ("large", 0), ("small", 4 * T)):
            F.fff_debug_option("token_max_T", limit)
            times[name] = _best(lambda: F.fff_forward_block(dev["x"], *ln, 1e-5, *nodes, dev["leaf_w1"], dev["leaf_b1"], dev["leaf_w2"],
                                                            dev["leaf_b2"], depth, n, L, w.act, True, out, idx))
    finally:
        F.fff_debug_option("token_max_T", old)
    print("  us a call:", {k: round(v, 1) for k, v in times.items()}, flush=True)
    assert times["auto"] <= 1.3 * min(times.values()) + 2.0, times
