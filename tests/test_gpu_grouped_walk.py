"""The grouped walk (tokens grouped by the node they reach after the top levels, then the rest of the fused launch in that order):
the fused launch's bits for every kernel it has, at the edges of its tiles, and what a call does where no workspace is to be had."""
import pytest

import fff_workloads as W
from fff_testlib import check_against_oracle, run_forward, to_device

pytestmark = pytest.mark.gpu

# T, D, O, depth, L, dtype: rows of 1, 4, 6, 8 pieces a lane of 16 and 4, 8, 16 of 64, whole and checked ones; a tile holds 32 tokens
# (16 lanes each), 8 or 4: one more, one less, a single token
CASES = [
    (1, 768, 768, 7, 1, W.DTYPE_BF16), (31, 512, 512, 2, 3, W.DTYPE_BF16), (33, 768, 768, 8, 2, W.DTYPE_BF16),
    (257, 8, 16, 9, 1, W.DTYPE_BF16), (2049, 1024, 520, 8, 8, W.DTYPE_BF16), (9, 2048, 2048, 7, 4, W.DTYPE_BF16),
    (4097, 1800, 600, 9, 1, W.DTYPE_BF16), (7, 4096, 4096, 8, 4, W.DTYPE_BF16), (3001, 4000, 4000, 9, 3, W.DTYPE_BF16),
    (515, 8192, 2048, 8, 2, W.DTYPE_BF16), (1030, 384, 384, 10, 8, W.DTYPE_F32), (517, 1024, 1000, 8, 1, W.DTYPE_F32),
    (130, 2000, 500, 7, 2, W.DTYPE_F32), (5, 4096, 4096, 7, 1, W.DTYPE_F32),
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


def test_without_a_workspace_the_fused_launch_runs():
    """A call whose other route is the fused launch, which needs no workspace, still needs none: captured where the library's would have to
    grow, or with a caller's that is too short, it is the fused launch, with the same bits."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] grouped walk without workspace T=16385 D=4096 depth=14 L=3 bf16", flush=True)
    g0 = torch.Generator(device="cuda").manual_seed(73)
    new = lambda *s: torch.empty(s, device="cuda").uniform_(-.05, .05, generator=g0).to(torch.bfloat16)
    T, D, depth, L, n = 16385, 4096, 14, 3, 1 << 14
    args = (new(T, D), new(n - 1, D), new(n - 1), new(n, L, D), new(n, L), new(n, L, D), new(n, D), depth, L, W.ACT_GELU)
    ref, out = (torch.zeros((T, D), dtype=torch.bfloat16, device="cuda") for _ in range(2))
    F.fff_forward_hard(*args, ref)
    torch.cuda.synchronize()
    assert F.fff_get_option("last_path") in (1, 6)
    taken = F.fff_get_option("last_path") == 6
    buf = torch.empty(256, dtype=torch.uint8, device="cuda")
    F.fff_set_workspace(buf)
    try:
        F.fff_forward_hard(*args, out)
        torch.cuda.synchronize()
        assert F.fff_get_option("last_path") == 1 and torch.equal(out.view(torch.int16), ref.view(torch.int16))
    finally:
        F.fff_set_workspace(None)
    F.fff_release_workspace()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        F.fff_forward_hard(*args, out)
    assert F.fff_get_option("last_path") == 1
    F.fff_reserve_workspace(T, depth)
    again = torch.cuda.CUDAGraph()
    out2 = torch.zeros_like(out)
    with torch.cuda.graph(again):
        F.fff_forward_hard(*args, out2)
    assert F.fff_get_option("last_path") == (6 if taken else 1)
    for _ in range(3):
        for g, o in ((graph, out), (again, out2)):
            o.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(o.view(torch.int16), ref.view(torch.int16))
    out.zero_()
    F.fff_forward_hard_static(*args, out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), ref.view(torch.int16))
    assert taken
