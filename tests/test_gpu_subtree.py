"""The launch that takes the last k levels, the leaf and the output rows of grouped tokens (subtree_kernel), against
the oracle: at the edges of its tiles (64 tokens, 64 output columns, blocks of 16 columns, 128 bytes of a row), for every k it has, and the
rules that choose it."""
import numpy as np
import pytest

import fff_workloads as W
from fff_testlib import check_against_oracle, out_to_f64, run_forward, to_device

pytestmark = pytest.mark.gpu
F32, BF16, RELU, GELU = W.DTYPE_F32, W.DTYPE_BF16, W.ACT_RELU, W.ACT_GELU


@pytest.fixture
def forced():
    """forced(k): the staged path, with k of the last levels in the subtree launch."""
    import paper_2308_14711_amd as F

    def to(k):
        F.fff_set_option("path", 2)
        F.fff_debug_option("subtree", k + 2)
    yield to
    F.fff_set_option("path", 0)
    F.fff_debug_option("subtree", 0)


CASES = [
    # name,       T,     D,    O,    depth, L,  act,  dtype, k
    ("one",       1,     64,   64,   3,     4,  RELU, BF16,  0),       # one token; groups without any
    ("tile_less", 63,    72,   8,    1,     1,  GELU, BF16,  0),       # rows of nine pieces, one output range of 8
    ("tile",      64,    64,   72,   1,     2,  RELU, BF16,  1),       # one group of all tokens
    ("tile_more", 65,    8,    64,   2,     3,  GELU, BF16,  2),       # rows of one piece; a leaf width that does not divide 16
    ("wide16",    1000,  136,  264,  4,     16, GELU, BF16,  2),       # 67 columns, 64 pairs and 4 biases: five steps
    ("steps9",    900,   200,  136,  5,     7,  GELU, BF16,  4),       # 127 columns; 112 pairs and 16 biases: two batches of steps
    ("cols96",    700,   768,  768,  5,     11, RELU, BF16,  3),       # 95 columns
    ("long",      500,   4104, 40,   4,     5,  RELU, BF16,  1),       # 65 stages of the ring, the last of one piece
    ("out_long",  300,   64,   1096, 3,     8,  GELU, BF16,  1),       # 18 ranges, the last of 8 columns
    ("groups1k",  3000,  64,   64,   10,    3,  RELU, BF16,  0),       # 1024 groups, most tiles nearly empty
    ("deep",      2500,  128,  128,  12,    2,  GELU, BF16,  2),
    ("f32_one",   1,     64,   64,   3,     4,  RELU, F32,   0),
    ("f32_tile",  65,    4,    4,    2,     1,  GELU, F32,   2),
    ("f32_l16",   1000,  68,   132,  4,     16, GELU, F32,   2),
    ("f32_l5",    700,   768,  260,  5,     5,  RELU, F32,   4),       # 95 columns
    ("f32_l8",    3000,  256,  512,  7,     8,  GELU, F32,   0),
    ("f32_long",  400,   2052, 40,   3,     9,  RELU, F32,   1),
]


@pytest.mark.parametrize("node_b", ["uniform", "zipf"])
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_against_the_oracle(case, node_b, forced):
    import paper_2308_14711_amd as F
    name, T, D, O, depth, L, act, dtype, k = case
    print("\n[case] subtree %s T=%d D=%d O=%d depth=%d L=%d act=%d dtype=%d k=%d node_b=%s seed 7" % (case + (node_b,)), flush=True)
    w = W.make_layer("subtree_" + name, T, D, O, depth, L, act, dtype, seed=7, node_b=node_b)
    forced(k)
    out, idx = run_forward(w)
    assert F.fff_get_option("last_leaf_path") == 4 and "k=%d" % k in F.fff_last_launch(), F.fff_last_launch()
    check_against_oracle(w, out, idx)
    again, _ = run_forward(w, want_idx=False)        # the order of tokens inside a group does not show
    bits = out.view(out.dtype).contiguous().view(-1)
    assert bits.equal(again.contiguous().view(-1))


@pytest.mark.parametrize("dtype,k", [(BF16, 0), (BF16, 1), (BF16, 3), (F32, 0), (F32, 2)])
def test_weights_that_are_not_finite_stay_with_their_leaf(dtype, k, forced):
    """Infinite and NaN output weights show in the rows of their own leaf's tokens, at their own columns, and nowhere else."""
    import torch
    T, D, O, depth, L = 3000, 128, 136, 5, 6
    print("\n[case] subtree non-finite weights dtype=%d k=%d seed 9" % (dtype, k), flush=True)
    w = W.make_layer("subtree_inf", T, D, O, depth, L, GELU, dtype, seed=9)
    forced(k)
    dev = to_device(w)
    plain, idx = run_forward(w, dev)
    dev["leaf_w2"][5, 3, 7] = float("inf")
    dev["leaf_b2"][9, 100] = float("-inf")
    dev["leaf_w2"][11, 2, 135] = float("nan")
    out, _ = run_forward(w, dev)
    got, ref, leaf = out_to_f64(out), out_to_f64(plain), idx.cpu().numpy()
    special = np.zeros(got.shape, bool)
    special[leaf == 5, 7] = special[leaf == 9, 100] = special[leaf == 11, 135] = True
    assert special.sum() > 30 and not np.isfinite(got[special]).any()
    assert (got[leaf == 9, 100] == -np.inf).all() and np.isnan(got[leaf == 11, 135]).all()
    tol = 2e-2 if dtype == BF16 else 1e-5
    assert (np.abs(got - ref)[~special] <= tol * np.abs(ref).max()).all()


def test_leaf_stage_alone(forced):
    """fff_leaf_forward: the leaves are given (k = 0)."""
    import torch
    import oracle
    import paper_2308_14711_amd as F
    from fff_testlib import oracle_inputs
    print("\n[case] subtree leaf_forward T=2000 D=96 O=200 depth=4 L=12 seed 3", flush=True)
    w = W.make_layer("subtree_leaf", 2000, 96, 200, 4, 12, RELU, BF16, seed=3)
    dev, ins = to_device(w), oracle_inputs(w)
    leaf = np.random.default_rng(3).integers(0, 16, 2000).astype(np.int32)
    forced(0)
    out = torch.full((2000, 200), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.fff_leaf_forward(dev["x"], dev["leaf_w1"], dev["leaf_b1"], dev["leaf_w2"], dev["leaf_b2"], torch.from_numpy(leaf).cuda(), 4, 12, RELU, out)
    torch.cuda.synchronize()
    assert "subtree_kernel" in F.fff_last_launch()
    ref = oracle.leaf_forward(ins[0], ins[3], ins[4], ins[5], ins[6], leaf, 4, 12, RELU)
    err = np.abs(out_to_f64(out) - ref).max(axis=1) / np.abs(ref).max(axis=1)
    assert err.max() <= 2e-2


@pytest.mark.parametrize("T,D,O,depth,L,dtype,expect", [
    (16384, 768, 768, 8, 8, BF16, "k=1"), (16383, 768, 768, 8, 8, BF16, "leaf_hidden_kernel"),         # a tile a compute unit
    (8193, 512, 512, 5, 12, BF16, "k=0"), (8193, 2304, 256, 5, 12, BF16, "leaf_hidden_kernel"),        # wider leaves: rows of up to 4 KB
    (16384, 128, 520, 6, 16, BF16, "leaf_hidden_kernel"),                                                # output rows four times the input rows
    (16384, 128, 392, 6, 16, BF16, "leaf_hidden_kernel"), (16384, 128, 384, 6, 16, BF16, "k=0"),        # and three times
    (8193, 768, 768, 6, 4, F32, "k=0"), (8193, 1024, 1024, 6, 3, F32, "leaf_gather_kernel"),            # fp32: four neurons
    (9000, 128, 128, 6, 8, F32, "k=0"), (9000, 124, 124, 6, 8, F32, "leaf_gather_kernel"),              # fp32: 8 KB of leaf rows
    (20000, 192, 192, 10, 9, F32, "leaf_gather_kernel"),                                                 # fp32: 32 tokens a group
    (8193, 512, 512, 6, 8, F32, "k=0"), (8192, 512, 512, 9, 8, F32, "fused"), (20000, 512, 512, 11, 8, F32, "leaf_gather_kernel"),
], ids=str)
def test_which_batches_take_it(T, D, O, depth, L, dtype, expect):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] subtree rule T=%d D=%d O=%d depth=%d L=%d dtype=%d" % (T, D, O, depth, L, dtype), flush=True)
    dt = torch.bfloat16 if dtype == BF16 else torch.float32
    z = lambda *s: torch.zeros(s, dtype=dt, device="cuda")
    n = 1 << depth
    out = torch.empty((T, O), dtype=dt, device="cuda")
    staged = D * L < 2000                               # (would go to the fused launch)
    F.fff_set_option("path", 2 if staged else 0)
    try:
        F.fff_forward_hard(z(T, D), z(n - 1, D), z(n - 1), z(n, L, D), z(n, L), z(n, L, O), z(n, O), depth, L, RELU, out)
    finally:
        F.fff_set_option("path", 0)
    torch.cuda.synchronize()
    assert expect in F.fff_last_launch(), F.fff_last_launch()
    assert not out.any()


@pytest.mark.parametrize("T,D,O,depth,L,dtype,expect", [
    (16384, 512, 512, 8, 8, BF16, True), (16383, 512, 512, 8, 8, BF16, False), (16384, 512, 512, 9, 8, BF16, False),      # 64 tokens a leaf
    (65536, 256, 256, 10, 8, BF16, True), (65536, 248, 248, 10, 8, BF16, False),                                           # 1024 leaves: 8 KB
    (16384, 512, 512, 7, 8, F32, True), (16383, 512, 512, 7, 8, F32, False), (30000, 900, 900, 5, 2, F32, False),
    (30000, 904, 904, 5, 2, BF16, False), (30000, 904, 904, 5, 3, BF16, True),
], ids=str)
def test_which_batches_of_given_leaves_take_it(T, D, O, depth, L, dtype, expect):
    import torch
    import paper_2308_14711_amd as F
    print("\n[case] subtree rule, leaves given T=%d D=%d O=%d depth=%d L=%d dtype=%d" % (T, D, O, depth, L, dtype), flush=True)
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16 if dtype == BF16 else torch.float32, device="cuda")
    n = 1 << depth
    out = z(T, O).fill_(float("nan"))
    F.fff_leaf_forward(z(T, D), z(n, L, D), z(n, L), z(n, L, O), z(n, O), torch.arange(T, dtype=torch.int32, device="cuda") % n, depth, L, RELU, out)
    torch.cuda.synchronize()
    assert ("subtree_kernel" in F.fff_last_launch()) == expect, F.fff_last_launch()
    assert not out.any()


def _both_launches(call, shape):
    """(rows, leaves, launch) of a call through the subtree launch and through the launches it stands for."""
    import torch
    import paper_2308_14711_amd as F
    res = []
    for option in (None, 1):
        old = F.fff_debug_option("subtree")
        if option:
            F.fff_debug_option("subtree", option)
        out = torch.full(shape, 7.0, dtype=torch.float32, device="cuda")
        idx = torch.full(shape[:1], -9, dtype=torch.int32, device="cuda")
        call(out, idx)
        torch.cuda.synchronize()
        F.fff_debug_option("subtree", old)
        res.append((out_to_f64(out), idx.cpu().numpy(), F.fff_last_launch()))
    assert "subtree_kernel" in res[0][2] and "subtree_kernel" not in res[1][2], (res[0][2], res[1][2])
    return res


def _same_infinities(a, b):
    (got, gi, _), (ref, ri, _) = a, b
    assert np.array_equal(gi, ri), "leaves differ at %s" % np.nonzero(gi != ri)[0][:5]
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    scale = np.where(fin, np.abs(ref), 0).max(axis=1, keepdims=True)
    assert (np.abs(np.where(fin, got, 0) - np.where(fin, ref, 0)) <= 1e-5 * scale).all()


def _plant(what, x, nodes, w1):
    """Infinities of both signs in tokens, node weights ([NN, D]) or leaf weights, or finite values whose sums overflow."""
    if what == "tokens":
        x[3, 5], x[40, 0], x[77, -1], x[100, 17] = np.inf, -np.inf, np.inf, -np.inf
    elif what == "nodes":
        nodes[0, -1] = nodes[2:7:2, 7] = np.inf
        nodes[1:7:2, 2] = -np.inf
    elif what == "leaves":
        w1[::2, 0, -1], w1[1::2, 1, 0], w1[1::4, 2, 30] = np.inf, -np.inf, np.inf
    else:                                                  # the first two products are finite, their sum is not
        x[:400, 0] = x[:400, 33] = 1.5
        x[400:, 33] = 0
        for a in (nodes[0], w1[::2, 1]):
            a[..., 0] = a[..., 33] = 2e38
        for a in (nodes[1], nodes[2], w1[1::2, 2]):
            a[..., 0] = a[..., 33] = -2e38


@pytest.mark.parametrize("what", ["tokens", "nodes", "leaves", "overflow"])
@pytest.mark.parametrize("act", [RELU, GELU], ids=["relu", "gelu"])
@pytest.mark.parametrize("k", [0, 2])
def test_infinite_pre_activations_in_fp32(what, act, k, forced):
    """fp32 pre-activations that are infinite, or overflow, stay infinities: routing, infinities and NaN as in the launches before."""
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, L = 1500, 132, 68, 4, 6
    print("\n[case] subtree fp32 infinities in %s act=%d k=%d seed 15" % (what, act, k), flush=True)
    w = W.make_layer("subtree_pre_inf", T, D, O, depth, L, act, F32, seed=15)
    host = [np.array(w.device_array(t)) for t in W.TENSORS]
    _plant(what, host[0], host[1], host[3])
    dev = [torch.from_numpy(a).cuda() for a in host]
    forced(k)
    call = lambda out, idx: F.fff_forward_hard(*dev, depth, L, act, out, idx)
    new, old = _both_launches(call, (T, O))
    assert what == "nodes" or not np.isfinite(old[0]).all()
    _same_infinities(new, old)
    if k == 0:
        given = torch.from_numpy(old[1]).cuda()
        leaf = lambda out, idx: F.fff_leaf_forward(dev[0], *dev[3:], given, depth, L, act, out)
        _same_infinities(*_both_launches(leaf, (T, O)))


@pytest.mark.parametrize("what", ["tokens", "nodes", "leaves", "overflow"])
@pytest.mark.parametrize("act", [RELU, GELU], ids=["relu", "gelu"])
def test_infinite_pre_activations_in_the_grouped_block(what, act, forced):
    """The same for fff_forward_block without a norm: levels from the root, last levels and leaves.  (Rows of 128 features: whole
    pieces for every lane of the launch before, whose idle lanes would multiply an infinite weight by zero.)"""
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, n, L = 1500, 128, 68, 5, 3, 4
    print("\n[case] grouped block fp32 infinities in %s act=%d seed 16" % (what, act), flush=True)
    w = W.make_layer("block_pre_inf", T, D, O, depth, L, act, F32, seed=16)
    nodes = [np.array(a) for a in W.wide_nodes(depth, n, D, F32, seed=16)]
    host = [np.array(w.device_array(t)) for t in ("x", "leaf_w1", "leaf_b1", "leaf_w2", "leaf_b2")]
    _plant(what, host[0], nodes[0][:, 0], host[1])
    x, *leaves = [torch.from_numpy(a).cuda() for a in host]
    d_nodes = [torch.from_numpy(a).cuda() for a in nodes]
    forced(2)
    old_T = F.fff_debug_option("token_max_T")
    F.fff_debug_option("token_max_T", 0)
    try:
        call = lambda out, idx: F.fff_forward_block(x, None, None, 0.0, *d_nodes, *leaves, depth, n, L, act, False, out, idx)
        new, old = _both_launches(call, (T, O))
    finally:
        F.fff_debug_option("token_max_T", old_T)
    _same_infinities(new, old)


def _whole_numbers(T, D, O, depth, L, shape_of_nodes):
    """Tokens, nodes and leaves of small whole numbers whose sums are exact in fp32.  A leaf's first two neurons have up to 22 bits and
    differ in the lowest 13; their output weights are 1 and -1, so an output is that difference."""
    import torch
    g = torch.Generator().manual_seed(17)
    r = lambda shape, low, high: torch.randint(low, high + 1, shape, generator=g).to(torch.bfloat16)
    nodes, leaves, half = (1 << depth) - 1, 1 << depth, D // 2
    x = r((T, D), -2, 2)
    x[:, :half] = x[:, :half].abs()
    w1 = torch.zeros((leaves, L, D), dtype=torch.bfloat16)
    w1[:, 0, :half] = r((leaves, half), 1, 63) * 1024
    w1[:, 1, :half] = w1[:, 0, :half]
    w1[:, :2, half:] = r((leaves, 2, D - half), -63, 63)
    w2 = torch.zeros((leaves, L, O), dtype=torch.bfloat16)
    w2[:, 0], w2[:, 1] = 1, -1
    node_w = r((nodes,) + shape_of_nodes + (D,), -3, 3)
    return x, node_w, w1, torch.zeros((leaves, L), dtype=torch.bfloat16), w2, torch.zeros((leaves, O), dtype=torch.bfloat16)


def _bits(t):
    import torch
    return np.ascontiguousarray(t.contiguous().view(torch.int16).numpy().view(np.uint16))


@pytest.mark.parametrize("T,depth,L,k", [(1000, 6, 9, 0), (1000, 6, 16, 1), (1500, 7, 12, 2), (700, 5, 2, 0), (700, 5, 2, 3)])
def test_hidden_activations_keep_all_bits_where_the_gather_kernel_does(T, depth, L, k, forced):
    """The batches of 8 to 31 tokens a leaf (and leaves of two neurons) that go to the gather kernel otherwise, in fp32: exact."""
    import oracle
    import torch
    import paper_2308_14711_amd as F
    D, O = 64, 72
    print("\n[case] subtree whole numbers T=%d depth=%d L=%d k=%d seed 17" % (T, depth, L, k), flush=True)
    x, node_w, w1, b1, w2, b2 = _whole_numbers(T, D, O, depth, L, ())
    node_b = torch.zeros(len(node_w), dtype=torch.bfloat16)
    forced(k)
    out = torch.full((T, O), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.fff_forward_hard(*[t.cuda() for t in (x, node_w, node_b, w1, b1, w2, b2)], depth, L, RELU, out)
    torch.cuda.synchronize()
    assert "subtree_kernel" in F.fff_last_launch()
    ref, _, _ = oracle.forward_hard(*[_bits(t) for t in (x, node_w, node_b, w1, b1, w2, b2)], depth, L, RELU)
    want = torch.from_numpy(ref).to(torch.bfloat16)
    assert (want != 0).float().mean() > 0.9 and torch.equal(out.cpu(), want)


def test_hidden_activations_keep_all_bits_in_the_grouped_block(forced):
    import oracle
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, n, L = 1000, 64, 72, 6, 2, 5
    print("\n[case] grouped block whole numbers T=%d depth=%d n=%d L=%d k=2 seed 17" % (T, depth, n, L), flush=True)
    x, node_w, w1, b1, w2, b2 = _whole_numbers(T, D, O, depth, L, (n,))
    nodes = [node_w, torch.zeros(node_w.shape[:2], dtype=torch.bfloat16), torch.ones(node_w.shape[:2], dtype=torch.bfloat16),
             torch.full(node_w.shape[:1], -20, dtype=torch.bfloat16)]
    forced(2)
    old_T = F.fff_debug_option("token_max_T")
    F.fff_debug_option("token_max_T", 0)
    out = torch.full((T, O), float("nan"), dtype=torch.bfloat16, device="cuda")
    F.fff_forward_block(x.cuda(), None, None, 0.0, *[t.cuda() for t in nodes + [w1, b1, w2, b2]], depth, n, L, RELU, False, out)
    torch.cuda.synchronize()
    F.fff_debug_option("token_max_T", old_T)
    assert "subtree_kernel" in F.fff_last_launch()
    ref, idx, _ = oracle.forward_block(_bits(x), None, None, 0.0, *[_bits(t) for t in nodes + [w1, b1, w2, b2]], depth, n, L, RELU, False)
    want = torch.from_numpy(ref).to(torch.bfloat16)
    assert len(set(idx.tolist())) > 8 and (want != 0).float().mean() > 0.9 and torch.equal(out.cpu(), want)


def test_a_finite_activation_beyond_the_largest_bf16_value_stays_finite(forced):
    import torch
    import paper_2308_14711_amd as F
    T, D, O, depth, L = 300, 64, 72, 4, 9
    print("\n[case] subtree activations between the largest bf16 and fp32 values T=%d depth=%d L=%d k=1" % (T, depth, L), flush=True)
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    most = torch.finfo(torch.bfloat16).max
    x, node_w, w1, b1, w2 = z(T, D) + 1, z(15, D), z(16, L, D), z(16, L), z(16, L, O)
    node_w[0::2, 3], node_w[1::2, 3] = 1, -1
    w1[:, 2, 5], b1[:, 2], w2[:, 2] = most, 1e36, 2.0 ** -20
    outs = []
    forced(1)
    for option in (3, 1):
        F.fff_debug_option("subtree", option)
        out = z(T, O).fill_(float("nan"))
        if option == 1:
            F.fff_set_option("leaf_path", 1)                     # the gather kernel
        F.fff_forward_hard(x, node_w, z(15), w1, b1, w2, z(16, O), depth, L, RELU, out)
        F.fff_set_option("leaf_path", 0)
        torch.cuda.synchronize()
        assert ("subtree_kernel" if option == 3 else "leaf_gather_kernel") in F.fff_last_launch(), F.fff_last_launch()
        outs.append(out)
    assert torch.isfinite(outs[1]).all() and (outs[1] > 3e32).all() and torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("D", [512, 1024, 136])
def test_normalised_rows_keep_all_bits_where_output_rows_are_longer(D, forced):
    """Output rows of more than 1024 features, whose launch without scratch has the normalised token in fp32.  A leaf neuron of
    ones sums a token's normalised elements, which is zero but for rounding: about sqrt(D) 2^-25 from fp32 elements (measured here: the
    launch without scratch), sqrt(D) 2^-18 from pairs of bf16 ones, a hundred times that.  Twice the former is allowed."""
    import torch
    import paper_2308_14711_amd as F
    T, O, depth, n, L = 600, 1032, 2, 1, 2
    print("\n[case] grouped block sums of normalised rows T=%d D=%d O=%d k=1 seed 18" % (T, D, O), flush=True)
    g = torch.Generator().manual_seed(18)
    bf = lambda t: t.to(torch.bfloat16).cuda()
    ones, zeros = (lambda *s: bf(torch.ones(s))), (lambda *s: bf(torch.zeros(s)))
    x, node_w = bf(torch.randn(T, D, generator=g)), bf(torch.randn(3, n, D, generator=g))
    w1 = ones(4, L, D)
    w1[:, 1] = -1
    w2 = ones(4, L, O)
    forced(1)
    old_T = F.fff_debug_option("token_max_T")
    F.fff_debug_option("token_max_T", 0)
    rms = []
    for option in (3, 1):
        F.fff_debug_option("subtree", option)
        out = torch.full((T, O), float("nan"), dtype=torch.bfloat16, device="cuda")
        F.fff_forward_block(x, ones(D), zeros(D), 1e-5, node_w, zeros(3, n), ones(3, n), zeros(3), w1, zeros(4, L), w2, zeros(4, O), depth, n, L,
                            RELU, False, out)
        torch.cuda.synchronize()
        assert ("subtree_kernel" in F.fff_last_launch()) == (option == 3), F.fff_last_launch()
        rms.append(out.double().pow(2).mean().sqrt().item())
    F.fff_debug_option("token_max_T", old_T)
    print("   rms %.3e, launch without scratch %.3e" % tuple(rms), flush=True)
    assert 0 < rms[0] <= 2 * rms[1]


@pytest.mark.parametrize("T,D,O,depth,n,L,act,dtype,k", [
    (6000, 768, 768, 4, 0, 8, GELU, BF16, 0), (3000, 392, 392, 7, 0, 12, GELU, BF16, 1),          # in the place of the tile kernels, the gather kernel
    (4000, 768, 768, 5, 0, 8, GELU, F32, 0), (4000, 256, 392, 6, 0, 4, RELU, F32, 1),
    (3000, 768, 768, 6, 4, 8, GELU, BF16, 2), (3000, 272, 1536, 4, 4, 16, RELU, BF16, 1), (3000, 512, 512, 6, 4, 8, GELU, F32, 1)], ids=str)
def test_error_against_64_bits_is_no_larger_than_without_it(T, D, O, depth, n, L, act, dtype, k, forced):
    """2-norm of the difference from the oracle (64 bits) through the subtree launch, and through the launches it stands for.  A bf16 call's
    error is its last rounding's: results that differ by less than that round alike but for ties (1e-4 allowed); sums in fp32 differ by
    their order (5 % allowed)."""
    import oracle
    import torch
    import paper_2308_14711_amd as F
    from fff_testlib import oracle_inputs
    print("\n[case] subtree error T=%d D=%d O=%d depth=%d n=%d L=%d act=%d dtype=%d k=%d seed 19" % (T, D, O, depth, n, L, act, dtype, k), flush=True)
    w = W.make_layer("subtree_error", T, D, O, depth, L, act, dtype, seed=19)
    dev, ins = to_device(w), oracle_inputs(w)
    up = lambda a: torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16) if dtype == BF16 else torch.from_numpy(a).cuda()
    forced(k)
    old_T = F.fff_debug_option("token_max_T")
    F.fff_debug_option("token_max_T", 0)
    errors = []
    if n:
        nodes, ln = W.wide_nodes(depth, n, D, dtype, seed=19), W.layer_norm_params(D, dtype, seed=19)
        ref, ref_idx, _ = oracle.forward_block(ins[0], *ln, 1e-5, *nodes, *ins[3:], depth, n, L, act, False)
        args = [up(np.ascontiguousarray(a)) for a in list(ln) + list(nodes)]
    else:
        ref, ref_idx, _ = oracle.forward_hard(*ins, depth, L, act)
    for option in (k + 2, 1):
        F.fff_debug_option("subtree", option)
        out = torch.empty((T, O), dtype=dev["x"].dtype, device="cuda")
        idx = torch.empty((T,), dtype=torch.int32, device="cuda")
        if n:
            F.fff_forward_block(dev["x"], *args[:2], 1e-5, *args[2:], *[dev[t] for t in W.TENSORS[3:]], depth, n, L, act, False, out, idx)
        else:
            F.fff_forward_hard(*[dev[t] for t in W.TENSORS], depth, L, act, out, idx)
        torch.cuda.synchronize()
        assert ("subtree_kernel" in F.fff_last_launch()) == (option > 1), F.fff_last_launch()
        same = idx.cpu().numpy() == ref_idx
        assert same.mean() > 0.99
        errors.append(np.linalg.norm(out_to_f64(out)[same] - ref[same]) / np.linalg.norm(ref[same]))
    F.fff_debug_option("token_max_T", old_T)
    print("   %.5e, without it %.5e" % tuple(errors), flush=True)
    assert errors[0] <= errors[1] * (1.0001 if dtype == BF16 else 1.05)
