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
    F.fff_forward_hard(z(T, D), z(n - 1, D), z(n - 1), z(n, L, D), z(n, L), z(n, L, O), z(n, O), depth, L, RELU, out)
    torch.cuda.synchronize()
    assert expect in F.fff_last_launch(), F.fff_last_launch()
    assert not out.any()
