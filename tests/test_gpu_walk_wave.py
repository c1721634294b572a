"""A wave a token (medium batches): every kernel of it against the oracle, at the edges of its rows, trips, blocks and output units."""
import pytest

import fff_workloads as W
from fff_testlib import check_against_oracle, run_forward, to_device

pytestmark = pytest.mark.gpu

# T, D, O, depth, L, dtype
CASES = [
    (1, 8, 8, 1, 1, W.DTYPE_BF16), (257, 512, 512, 2, 8, W.DTYPE_BF16), (600, 520, 1, 3, 9, W.DTYPE_BF16),          # a piece a lane, one more
    (1025, 768, 768, 11, 1, W.DTYPE_BF16), (2047, 768, 520, 10, 5, W.DTYPE_BF16), (4097, 1024, 77, 6, 4, W.DTYPE_BF16),
    (4095, 1032, 513, 5, 3, W.DTYPE_BF16), (2049, 2048, 2048, 7, 17, W.DTYPE_BF16), (300, 2056, 72, 4, 64, W.DTYPE_BF16),
    (1030, 4096, 4096, 9, 2, W.DTYPE_BF16), (3000, 4088, 10, 6, 7, W.DTYPE_BF16), (8193, 64, 64, 8, 32, W.DTYPE_BF16),
    (4096, 784, 10, 6, 4, W.DTYPE_F32), (513, 4, 3, 12, 1, W.DTYPE_F32), (2500, 260, 260, 5, 16, W.DTYPE_F32),
    (700, 2048, 31, 3, 6, W.DTYPE_F32), (12289, 128, 128, 6, 8, W.DTYPE_F32),
]


@pytest.mark.parametrize("case", CASES, ids=["T%d_D%d_O%d_d%d_L%d_%s" % (c[:5] + (("f32", "bf16")[c[5]],)) for c in CASES])
@pytest.mark.parametrize("act", [W.ACT_RELU, W.ACT_GELU], ids=["relu", "gelu"])
def test_against_the_oracle(case, act):
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, L, dtype = case
    print("\n[case] wave a token T=%d D=%d O=%d depth=%d L=%d dtype=%d act=%d seed 81" % (case + (act,)), flush=True)
    w = W.make_layer("wave", T, D, O, depth, L, act, dtype, seed=81)
    dev = to_device(w)
    F.fff_set_option("path", 7)
    try:
        out, idx = run_forward(w, dev)
        assert F.fff_get_option("last_path") == 1 and "walk_wave_kernel" in F.fff_last_launch()
        again, _ = run_forward(w, dev, want_idx=False)
    finally:
        F.fff_set_option("path", 0)
    check_against_oracle(w, out, idx)
    assert torch.equal(out, again)


@pytest.mark.parametrize("dtype", [W.DTYPE_BF16, W.DTYPE_F32], ids=["bf16", "f32"])
@pytest.mark.parametrize("moved", ["out", "leaf_w2", "leaf_b2"])
def test_output_rows_off_a_piece(moved, dtype):
    """Output rows of whole pieces whose tensors start one element behind a 16-byte boundary: stored and read element by element, and
    nothing beside them is touched."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] wave a token, %s off a boundary T=1500 D=O=256 depth=6 L=3 dtype=%d seed 85" % (moved, dtype), flush=True)
    w = W.make_layer("wave_off", 1500, 256, 256, 6, 3, W.ACT_GELU, dtype, seed=85)
    dev = to_device(w)
    dev["out"] = torch.full((w.T, w.O), 7.0, dtype=dev["x"].dtype, device="cuda")
    room = torch.full((dev[moved].numel() + 9,), 7.0, dtype=dev["x"].dtype, device="cuda")
    dev[moved] = room[1:-8].view(dev[moved].shape).copy_(dev[moved])
    assert dev[moved].data_ptr() % 16 != 0
    idx = torch.empty((w.T,), dtype=torch.int32, device="cuda")
    for path in (7, 0):
        F.fff_set_option("path", path)
        try:
            F.fff_forward_hard(dev["x"], dev["node_w"], dev["node_b"], dev["leaf_w1"], dev["leaf_b1"], dev["leaf_w2"], dev["leaf_b2"], w.depth,
                               w.leaf_width, w.act, dev["out"], idx)
        finally:
            F.fff_set_option("path", 0)
        torch.cuda.synchronize()
        assert "walk_wave_kernel" in F.fff_last_launch() and "elements" in F.fff_last_launch()
        check_against_oracle(w, dev["out"], idx)
        assert (room[:1] == 7).all() and (room[-8:] == 7).all()


def test_captured_and_replayed():
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] wave a token, captured T=2048 D=O=768 depth=11 L=1 bf16 seed 86", flush=True)
    w = W.make_layer("wave_graph", 2048, 768, 768, 11, 1, W.ACT_GELU, W.DTYPE_BF16, seed=86)
    dev = to_device(w)
    ref, ref_idx = run_forward(w, dev)
    assert "walk_wave_kernel" in F.fff_last_launch()
    out, idx = torch.empty_like(ref), torch.empty_like(ref_idx)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        F.fff_forward_hard(dev["x"], dev["node_w"], dev["node_b"], dev["leaf_w1"], dev["leaf_b1"], dev["leaf_w2"], dev["leaf_b2"], w.depth,
                           w.leaf_width, w.act, out, idx)
    for _ in range(3):
        out.fill_(float("nan"))
        idx.fill_(-1)
        again, _ = run_forward(w, dev)                      # eager work between the replays
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(idx, ref_idx) and torch.equal(again, ref)


@pytest.mark.parametrize("where", ["leaf_w1", "node_w"])
def test_infinite_weights_and_nan_tokens_stay_with_their_tokens(where):
    """Lanes past a row multiply nothing: an infinite last weight (of one leaf's neuron, or of a node) reaches the tokens that meet it and
    no other, and is not turned into NaN."""
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] wave a token, infinite weights T=1500 D=72 O=16 depth=5 L=3 fp32 in %s" % where, flush=True)
    w = W.make_layer("wave_inf", 1500, 72, 16, 5, 3, W.ACT_RELU, W.DTYPE_F32, seed=82)
    dev = to_device(w)
    dev["x"][7] = float("nan")
    F.fff_set_option("path", 7)
    try:
        ref, leaf = run_forward(w, dev)
        if where == "leaf_w1":
            dev["leaf_w1"][int(leaf[20]), 1, -1] = float("inf")
            got, now = run_forward(w, dev)
            assert torch.equal(now, leaf)
            hit = leaf == leaf[20]
        else:
            dev["node_w"][0, -1] = float("inf")
            got, now = run_forward(w, dev)
            right = dev["x"][:, -1] > 0
            assert torch.equal(now[dev["x"][:, -1] != 0] >= 16, right[dev["x"][:, -1] != 0])
            hit = (now != leaf)
    finally:
        F.fff_set_option("path", 0)
    hit[7] = True
    assert torch.equal(got[~hit], ref[~hit]) and int((~hit).sum()) > 500
    if where == "leaf_w1":
        only = hit.clone()
        only[7] = False
        x_last, h = dev["x"][only][:, -1], got[only]
        assert not bool(torch.isnan(h[x_last > 0]).any()) and not bool(torch.isinf(h[x_last < 0]).any())
    assert int(leaf[7]) == 0            # NaN logits go left


@pytest.mark.parametrize("T, D, O, L, dtype, expect", [
    (512, 768, 768, 4, W.DTYPE_BF16, False), (513, 768, 768, 8, W.DTYPE_BF16, True), (1024, 768, 768, 9, W.DTYPE_BF16, False),
    (1024, 4096, 4096, 8, W.DTYPE_BF16, True), (2048, 768, 768, 1, W.DTYPE_BF16, True), (2048, 128, 128, 1, W.DTYPE_BF16, False),
    (2048, 768, 768, 16, W.DTYPE_BF16, True), (4096, 2048, 2048, 32, W.DTYPE_BF16, True), (4096, 4096, 4096, 8, W.DTYPE_BF16, False),
    (4096, 784, 10, 4, W.DTYPE_F32, True), (4097, 768, 768, 1, W.DTYPE_BF16, False), (8192, 256, 250, 16, W.DTYPE_BF16, True),
    (12288, 512, 512, 4, W.DTYPE_BF16, True), (12289, 512, 512, 4, W.DTYPE_BF16, False),
    # bf16 leaves of full tiles go to the staged path's matrix launches, fp32 ones not
    (8192, 256, 256, 16, W.DTYPE_BF16, False), (8192, 256, 256, 16, W.DTYPE_F32, True), (6144, 256, 256, 16, W.DTYPE_BF16, True),
    (8192, 256, 256, 12, W.DTYPE_BF16, True), (6144, 256, 256, 24, W.DTYPE_BF16, True), (6145, 256, 256, 24, W.DTYPE_BF16, False),
    (6144, 256, 256, 32, W.DTYPE_BF16, False),
    # element-wise output rows of wide leaves: a block a token
    (2500, 64, 437, 16, W.DTYPE_BF16, True), (2500, 64, 439, 16, W.DTYPE_BF16, False), (3073, 64, 439, 16, W.DTYPE_BF16, True),
    # short rows
    (3072, 64, 64, 6, W.DTYPE_BF16, True), (3073, 64, 64, 6, W.DTYPE_BF16, False), (3073, 64, 7, 6, W.DTYPE_BF16, False),
    (3073, 200, 7, 6, W.DTYPE_BF16, True),
    (6144, 320, 320, 6, W.DTYPE_BF16, True), (6145, 320, 320, 6, W.DTYPE_BF16, False), (6145, 320, 19, 6, W.DTYPE_BF16, False),
    (6145, 320, 21, 6, W.DTYPE_BF16, True), (9000, 256, 256, 4, W.DTYPE_BF16, False), (9000, 256, 21, 4, W.DTYPE_BF16, True),
])
def test_which_calls_take_it(T, D, O, L, dtype, expect):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] route T=%d D=%d O=%d depth=6 L=%d dtype=%d" % (T, D, O, L, dtype), flush=True)
    dt = torch.bfloat16 if dtype == W.DTYPE_BF16 else torch.float32
    depth, n = 6, 64
    new = lambda *s: torch.zeros(s, dtype=dt, device="cuda")
    F.fff_forward_hard(new(T, D), new(n - 1, D), new(n - 1), new(n, L, D), new(n, L), new(n, L, O), new(n, O), depth, L, W.ACT_RELU, new(T, O))
    torch.cuda.synchronize()
    assert ("walk_wave_kernel" in F.fff_last_launch()) == expect, F.fff_last_launch()


@pytest.mark.parametrize("T, top", [(2000, 0), (4000, 5), (8000, 6)])
def test_last_walk_top_is_of_this_call(T, top):
    """Levels in LDS as the kernel's note has them, after a call that kept other ones; 0 after a call that kept none."""
    import paper_2308_14711_amd as F
    print("\n[case] wave a token, last_walk_top T=%d D=128 O=40 depth=7 L=3 bf16 seed 84" % T, flush=True)
    w = W.make_layer("wave_top", T, 128, 40, 7, 3, W.ACT_RELU, W.DTYPE_BF16, seed=84)
    dev = to_device(w)
    try:
        for path, want in ((1, None), (7, top), (1, None), (4, 0)):
            F.fff_set_option("path", path)
            run_forward(w, dev)
            note = F.fff_last_launch()
            assert ("walk_wave_kernel" in note) == (path == 7)
            if want is None:
                want = int(note.split("top=")[1])
                assert want not in (0, top)
            assert F.fff_get_option("last_walk_top") == want and (path != 7 or note.endswith("top=%d" % want)), note
    finally:
        F.fff_set_option("path", 0)


# option, value, T, L: an option that picks among the launches of another path, and what the call's launches are named then
OTHERS = [
    ("leaf_path", 1, 4000, 16, "leaf_gather_kernel"), ("leaf_path", 2, 4000, 16, "leaf_hidden_kernel"), ("bucketing", 0, 4000, 16, "leaf_gather_kernel"),
    ("bucket_kernel", 3, 4000, 16, "bucket_hist_kernel"), ("leaf_split", 4, 4000, 16, "leaf_gather_kernel"), ("subtree", 2, 4000, 16, "subtree_kernel"),
    ("subtree", 1, 4000, 16, "leaf_hidden_kernel"), ("token_kernel", 2, 2000, 16, "token_rows_kernel"), ("walk_top", 1, 4000, 4, "walk_kernel"),
    ("walk_bpc", 2, 4000, 4, "walk_kernel"), ("walk_tpg", 1, 4000, 4, "walk_kernel"),
]


@pytest.mark.parametrize("option, value, T, L, name", OTHERS, ids=["%s%d" % o[:2] for o in OTHERS])
def test_options_of_the_other_launches_reach_them(option, value, T, L, name):
    import paper_2308_14711_amd as F
    print("\n[case] wave a token, option %s=%d T=%d D=256 O=128 depth=6 L=%d bf16 seed 83" % (option, value, T, L), flush=True)
    w = W.make_layer("wave_options", T, 256, 128, 6, L, W.ACT_GELU, W.DTYPE_BF16, seed=83)
    dev = to_device(w)
    run_forward(w, dev)
    assert "walk_wave_kernel" in F.fff_last_launch()
    public = option in ("leaf_path", "bucketing")
    (F.fff_set_option if public else F.fff_debug_option)(option, value)
    try:
        out, idx = run_forward(w, dev)
        assert "walk_wave_kernel" not in F.fff_last_launch() and name in F.fff_last_launch(), F.fff_last_launch()
        assert ("bucket" in F.fff_last_launch()) == (L > 8 and T > 3072 and option != "bucketing")
    finally:
        (F.fff_set_option if public else F.fff_debug_option)(option, 1 if option == "bucketing" else 0)
    check_against_oracle(w, out, idx)
