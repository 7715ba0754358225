"""Kernels that contract split operands (three bf16 planes) on the bf16 matrix
units: batch sizes on both sides of every rule that selects them, tiles with
remainders, groups whose tile list runs in several chunks, deep batches with few
rows per level, operands and weights that cannot be split, and the accuracy of
the sums themselves (tests/test_split_planes.py shows that the bound finds a lost
or misplaced plane).  GPU."""
import dataclasses

import numpy as np
import pytest

from tests.gpu_helpers import announce, compare_states, need_gpu

torch = pytest.importorskip("torch")

from oracle import cortex_oracle as O
from paper_2011_01383_amd import cortex as C
from paper_2011_01383_amd import inputs as I
from paper_2011_01383_amd.runner import DeviceWorkload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()


def run(wl):
    dw = DeviceWorkload(wl)
    dw.step()
    assert dw.status_code() == 0
    return dw


def tree_rnn(seed, batch, lo, hi, H):
    return I.tree_rnn_forest_workload(seed, batch=batch, H=H, leaf_lo=lo, leaf_hi=hi)


def childsum(seed, batch, lo, hi, max_arity=4):
    return I.childsum_treelstm_workload(seed, batch=batch, H=256, node_lo=lo, node_hi=hi, max_arity=max_arity)


# the last size of one rule and the first of the next (a binary tree of n leaves
# has 2n - 1 nodes), odd sizes, and chains whose groups hold more tiles than one
# list chunk
SIZES = {
    "nary_h256_1535": lambda: I.nary_treelstm_workload(1, batch=1, H=256, leaf_lo=768, leaf_hi=768),
    "nary_h256_1537": lambda: I.nary_treelstm_workload(2, batch=1, H=256, leaf_lo=769, leaf_hi=769),
    "nary_h256_4001": lambda: I.nary_treelstm_workload(3, batch=1, H=256, leaf_lo=2001, leaf_hi=2001),
    "tree_rnn_h256_2559": lambda: I.tree_rnn_workload(4, n_leaves=1280, H=256),
    "tree_rnn_h256_2561": lambda: I.tree_rnn_workload(5, n_leaves=1281, H=256),
    "tree_rnn_h256_6143": lambda: I.tree_rnn_workload(6, n_leaves=3072, H=256),
    "tree_rnn_h256_6145": lambda: I.tree_rnn_workload(7, n_leaves=3073, H=256),
    "tree_rnn_h256_forest": lambda: tree_rnn(8, 211, 3, 61, 256),
    "tree_rnn_h512_2561": lambda: I.tree_rnn_workload(9, n_leaves=1281, H=512),
    "childsum_h256_1199": lambda: childsum(13, 1, 1199, 1199),
    "childsum_h256_1200": lambda: childsum(14, 1, 1200, 1200),
    "childsum_h256_arity2": lambda: childsum(15, 40, 30, 90, max_arity=2),
    "childsum_h256_all_leaves": lambda: childsum(16, 1201, 1, 1),
    "childsum_h256_forest": lambda: childsum(17, 333, 1, 60),
    "mvrnn_d128_one_leaf": lambda: I.mvrnn_workload(29, batch=1, d=128, leaf_lo=1, leaf_hi=1),
    "mvrnn_d128_forest": lambda: I.mvrnn_workload(30, batch=23, d=128, leaf_lo=1, leaf_hi=50),
    "dag_h256_1x1": lambda: I.dagrnn_workload(10, n_grids=1, rows=1, cols=1, H=256),
    "dag_h256_6143": lambda: I.dagrnn_workload(25, n_grids=1, rows=1, cols=6143, H=256),
    "dag_h256_29x31": lambda: I.dagrnn_workload(55, n_grids=7, rows=29, cols=31, H=256),
    "dag_h256_6144": lambda: I.dagrnn_workload(26, n_grids=2, rows=48, cols=64, H=256),
    "dag_h256_36863": lambda: I.dagrnn_workload(27, n_grids=191, rows=1, cols=193, H=256),
    "dag_h256_36865": lambda: I.dagrnn_workload(28, n_grids=365, rows=1, cols=101, H=256),
    "dag_h512_33x17": lambda: I.dagrnn_workload(11, n_grids=5, rows=33, cols=17, H=512),
}


@pytest.mark.parametrize("name", sorted(SIZES))
def test_sizes(name):
    wl = SIZES[name]()
    announce("split %s N=%d" % (name, wl.N))
    compare_states(run(wl).states_by_node(), O.forward_workload(wl), name)


def _caterpillars(seed, batch, n_leaves):
    """N-ary TreeLSTM over chain-shaped trees: one node per tree and level."""
    wl = I.nary_treelstm_workload(seed, batch=1, H=256, leaf_lo=batch * n_leaves, leaf_hi=batch * n_leaves)
    children, is_leaf = I.forest_to_children([I.caterpillar(n_leaves, left_spine=bool(i & 1)) for i in range(batch)], 2)
    x_index = np.full(is_leaf.size, -1, dtype=np.int32)
    x_index[is_leaf] = np.random.default_rng(seed).integers(0, 1000, size=int(is_leaf.sum()))
    return dataclasses.replace(wl, children=children, x_index=x_index)


@pytest.mark.parametrize("groups", [0, 1, 3])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_childsum_schedules_agree(mode, groups):
    """Node groups and level orderings change the schedule only: bitwise the
    default's states; one group has more tiles and leaves than its list."""
    wl = childsum(18, 60, 20, 80)
    announce("split childsum mode %d groups %d N=%d" % (mode, groups, wl.N))
    ref = run(wl).states_by_node()
    C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, mode)
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, groups)
    try:
        got = run(wl).states_by_node()
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, 0)
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, 0)
    for key in ref:
        assert np.array_equal(ref[key], got[key]), key
    if mode == 0 and groups == 0:
        compare_states(ref, O.forward_workload(wl), "childsum")


@pytest.mark.parametrize("groups", [0, 1])
def test_more_tiles_than_the_list(groups):
    """450 levels of one tile each: with one node group its 449 tiles take
    four chunks of the list (128 tiles)."""
    wl = _caterpillars(12, 4, 450)
    announce("split caterpillars groups %d N=%d" % (groups, wl.N))
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, groups)
    try:
        got = run(wl).states_by_node()
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, 0)
    compare_states(got, O.forward_workload(wl), "caterpillars")


@pytest.mark.parametrize("groups,units", [(32, 32), (33, 64), (64, 64)])
def test_dag_node_groups(groups, units):
    """Every group count that some slice width has room for (256 compute units)
    runs, on the narrowest such slices."""
    wl = I.dagrnn_workload(33, n_grids=2, rows=48, cols=64, H=256)
    announce("split dag groups %d N=%d" % (groups, wl.N))
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, groups)
    try:
        got = run(wl).states_by_node()
        assert C.cortex_last_grid(1) == groups * (256 // units)
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, 0)
    compare_states(got, O.forward_workload(wl), "dag")


@pytest.mark.parametrize("groups", [1, 3])
def test_mvrnn_node_groups(groups):
    """One node group holds more nodes than its list (512); the states are
    bitwise those of the default."""
    wl = I.mvrnn_workload(31, batch=8, d=128, leaf_lo=90, leaf_hi=90)
    announce("split mvrnn groups %d N=%d" % (groups, wl.N))
    ref = run(wl).states_by_node()
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, groups)
    try:
        got = run(wl).states_by_node()
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, 0)
    for key in ref:
        assert np.array_equal(ref[key], got[key]), key
    compare_states(ref, O.forward_workload(wl), "mvrnn")


def _binary(wl, trees):
    """The workload's cell, weights and inputs over other binary trees."""
    children, is_leaf = I.forest_to_children(trees, 2)
    rows = wl.x_table.shape[0]
    x_index = np.full(is_leaf.size, -1, dtype=np.int32)
    x_index[is_leaf] = np.arange(int(is_leaf.sum())) % rows
    return dataclasses.replace(wl, children=children, x_index=x_index)


def _childsum_trees(trees):
    wl = childsum(47, 1, 9, 9)
    children, is_leaf = I.forest_to_children(trees, 4)
    return dataclasses.replace(wl, children=children, x_index=(np.arange(is_leaf.size) % 1000).astype(np.int32))


def _cats(n, leaves):
    return [I.caterpillar(leaves, left_spine=bool(i & 1)) for i in range(n)]


def _chains(n, nodes):
    out = []
    for _ in range(n):
        t = []
        for _ in range(nodes - 1):
            t = [t]
        out.append(t)
    return out


# batches with few rows per level, for every kernel that holds the form for them,
# and what CORTEX_KNOB_FWD_NODE_GROUPS makes of the same grid in the wide form
DEEP = {
    "nary_in_lds": (lambda: _binary(I.nary_treelstm_workload(48, batch=1, H=256), _cats(3, 400)), 8),
    "nary": (lambda: _binary(I.nary_treelstm_workload(49, batch=1, H=256), _cats(2, 900)), 8),
    "tree_rnn_h256": (lambda: _binary(I.tree_rnn_workload(50, n_leaves=64, H=256), _cats(3, 500)), 16),
    "tree_rnn_h256_wide": (lambda: _binary(I.tree_rnn_workload(51, n_leaves=64, H=256), _cats(17, 200)), 64),
    "tree_rnn_h512": (lambda: _binary(I.tree_rnn_workload(52, n_leaves=64, H=512), _cats(17, 90)), 16),
    "childsum_in_lds": (lambda: _childsum_trees(_chains(3, 500)), 8),
    "childsum": (lambda: _childsum_trees(_chains(2, 900)), 8),
}


def _best_us(dw, repeats=7):
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(repeats):
        start.record()
        dw.step()
        end.record()
        torch.cuda.synchronize()
        best = min(best, start.elapsed_time(end))
    assert dw.status_code() == 0
    return 1e3 * best


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("name", sorted(DEEP))
def test_deep_narrow_batches(name, mode):
    """Deep, narrow batches take the form with the shorter tile: its states are
    the oracle's under every level ordering, bitwise the same."""
    wl = DEEP[name][0]()
    announce("split deep %s mode %d N=%d" % (name, mode, wl.N))
    C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, mode)
    try:
        got = run(wl).states_by_node()
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, 0)
    if mode == 0:
        compare_states(got, O.forward_workload(wl), name)
    else:
        ref = run(wl).states_by_node()
        for key in ref:
            assert np.array_equal(ref[key], got[key]), key


@pytest.mark.parametrize("name", sorted(DEEP))
def test_deep_narrow_batches_are_faster(name):
    """...and it is the faster one there: the same grid held to the wide form
    (by its node groups) takes 1.07 to 1.4 times as long."""
    wl, groups = DEEP[name][0](), DEEP[name][1]
    announce("split deep times %s N=%d" % (name, wl.N))
    dw = run(wl)
    us = _best_us(dw)
    grid = C.cortex_last_grid(1)
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, groups)
    try:
        dw.step()
        assert C.cortex_last_grid(1) == grid
        wide = _best_us(dw)
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_NODE_GROUPS, 0)
    assert us < wide, (us, wide)


@pytest.mark.parametrize("leaves,value,status", [
    (320, "N", C.CORTEX_ST_BAD_LINEARIZATION), (320, -2, C.CORTEX_ST_BAD_LINEARIZATION), (2, "N", C.CORTEX_ST_BAD_LINEARIZATION),
    (320, 0, C.CORTEX_ST_OK), (321, "N", C.CORTEX_ST_OK)])
def test_mvrnn_checks_child_rows(leaves, value, status):
    """Up to 640 nodes every entry of child_rows has to be a row or -1, also
    those of leaf rows, which no node reads."""
    wl = I.mvrnn_workload(45, batch=1, d=128, leaf_lo=leaves, leaf_hi=leaves)
    announce("split mvrnn child_rows N=%d %s" % (wl.N, value))
    dw = DeviceWorkload(wl)
    dw.linearize()
    dw.lin.child_rows[2] = wl.N if value == "N" else value          # row 1 is a leaf
    dw.forward()
    assert dw.status_code() == status


@pytest.mark.parametrize("leaves,status", [(24, C.CORTEX_ST_INPUT_RANGE), (25, C.CORTEX_ST_OK)])
def test_mvrnn_checks_input_indexes(leaves, status):
    """cortex_tree_infer up to 47 nodes refuses an input index out of range at
    any node; beyond, MV-RNN reads them at leaves only."""
    wl = I.mvrnn_workload(46, batch=1, d=128, leaf_lo=leaves, leaf_hi=leaves)
    x_index = wl.x_index.copy()
    x_index[np.nonzero(x_index < 0)[0][0]] = leaves                 # an inner node; the table has `leaves` rows
    announce("split mvrnn x_index N=%d" % wl.N)
    dw = DeviceWorkload(dataclasses.replace(wl, x_index=x_index))
    dw.infer()
    assert dw.status_code() == status


UNSPLITTABLE = {
    # (one level: P is linear, and deeper products of huge finite values leave the fp32 range)
    "mvrnn": lambda: I.mvrnn_workload(32, batch=9, d=128, leaf_lo=2, leaf_hi=2),
    "nary": lambda: I.nary_treelstm_workload(20, batch=60, H=256, leaf_lo=20, leaf_hi=20),
    "childsum": lambda: childsum(24, 80, 20, 20),
    "tree_rnn": lambda: tree_rnn(21, 60, 30, 30, 256),
    "tree_rnn_wide": lambda: tree_rnn(56, 104, 30, 30, 256),
    "tree_rnn_h512": lambda: tree_rnn(57, 60, 30, 30, 512),
    "dag_h256": lambda: I.dagrnn_workload(22, n_grids=3, rows=5, cols=4, H=256),
    "dag_h256_32": lambda: I.dagrnn_workload(58, n_grids=128, rows=7, cols=7, H=256),
    "dag_h256_64": lambda: I.dagrnn_workload(59, n_grids=3, rows=5, cols=4, H=256),
    "dag_h512": lambda: I.dagrnn_workload(23, n_grids=2, rows=5, cols=4, H=512),
}
UNITS = {"dag_h256_64": 64}                  # slice width held by the knob


@pytest.fixture
def units(name):
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_SLICE_UNITS, UNITS.get(name, 0))
    yield
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_SLICE_UNITS, 0)


@pytest.mark.parametrize("value", [float("inf"), 3.4e38, -3.397e38, float("nan")])
@pytest.mark.parametrize("where", ["input", "weight"])
@pytest.mark.parametrize("name", sorted(UNSPLITTABLE))
def test_unsplittable_values(name, where, value, units):
    """One infinite, NaN or near-overflow input element or weight: the states
    are those of the definition (the gates saturate; NaN spreads to the same
    nodes and units)."""
    wl = UNSPLITTABLE[name]()
    announce("split %s %s %r N=%d" % (name, where, value, wl.N))
    if where == "input":
        key = "x" if wl.x is not None else "leaf_mat" if wl.leaf_mat is not None else "x_table"
        arr = getattr(wl, key).copy()
        arr.reshape(arr.shape[0], -1)[3, 5] = value
    else:
        # (child-sum: an input weight; its leaves have no recurrent product to meet one of U)
        key = "U" if wl.U is not None and wl.cell != I.CELL_CHILDSUM_TREELSTM else "W"
        key = "W_M" if wl.W_M is not None else key
        arr = getattr(wl, key).copy()
        arr.reshape(-1, wl.H)[7, 9] = value
    wl = dataclasses.replace(wl, **{key: arr})
    got = run(wl).states_by_node()
    with np.errstate(all="ignore"):
        ref = O.forward_workload(wl)
    for key in ref:
        r32 = ref[key].astype(np.float32).astype(np.float64)       # fp64 states beyond the fp32 range
        assert np.array_equal(np.isnan(got[key]), np.isnan(r32)), key
        fine = np.isfinite(r32)
        assert np.array_equal(got[key][~fine & ~np.isnan(r32)], r32[~fine & ~np.isnan(r32)]), key
        assert float(np.abs(got[key][fine] - r32[fine]).max()) <= 1e-4 * max(1.0, float(np.abs(r32[fine]).max())), key


ACCURACY = {
    # name: (workload, slice-width knob), one for each kernel and slice width
    "nary_8": (lambda: I.nary_treelstm_workload(62, batch=60, H=256), 0),
    "nary_2": (lambda: I.nary_treelstm_workload(63, batch=60, H=256), 2),
    "tree_rnn_16": (lambda: tree_rnn(64, 60, 30, 30, 256), 0),
    "tree_rnn_64": (lambda: tree_rnn(65, 110, 30, 30, 256), 0),
    "tree_rnn_h512_32": (lambda: tree_rnn(66, 60, 30, 30, 512), 0),
    "dag_16_one_launch": (lambda: I.dagrnn_workload(67, n_grids=4, rows=9, cols=9, H=256), 0),
    "dag_16": (lambda: I.dagrnn_workload(68, n_grids=30, rows=9, cols=9, H=256), 0),
    "dag_32": (lambda: I.dagrnn_workload(69, n_grids=80, rows=9, cols=9, H=256), 0),
    "dag_64": (lambda: I.dagrnn_workload(70, n_grids=10, rows=9, cols=9, H=256), 64),
    "dag_h512": (lambda: I.dagrnn_workload(71, n_grids=30, rows=9, cols=9, H=512), 0),
    "childsum": (lambda: childsum(72, 60, 20, 80), 0),
    "mvrnn": (lambda: I.mvrnn_workload(73, batch=20, d=128), 0),
    "mvrnn_one_launch": (lambda: I.mvrnn_workload(74, batch=1, d=128, leaf_lo=20, leaf_hi=20), 0),
}


@pytest.mark.parametrize("name", sorted(ACCURACY))
def test_accuracy_of_the_sums(name):
    """The computed states are off from 64 bits by at most 5e-7 of their
    2-norm: fp32 rounding (0.9e-7 to 2.6e-7 with every plane product in place;
    without any one of the six, 1e-6 or more)."""
    make, units = ACCURACY[name]
    wl = make()
    announce("split accuracy %s N=%d" % (name, wl.N))
    C.cortex_set_knob(C.CORTEX_KNOB_FWD_SLICE_UNITS, units)
    try:
        got = run(wl).states_by_node()
    finally:
        C.cortex_set_knob(C.CORTEX_KNOB_FWD_SLICE_UNITS, 0)
    ref = O.forward_workload(wl)
    inner = (wl.children.reshape(wl.N, wl.K) >= 0).any(1)        # (leaves copy their inputs)
    for key in ref:
        err = float(np.linalg.norm(got[key][inner] - ref[key][inner]) / np.linalg.norm(ref[key][inner]))
        print("%s %s %.2g" % (name, key, err))
        assert err <= 5e-7, key


def test_mvrnn_tiny_matrices():
    """P is linear in the children's matrices, so a column of tiny elements gives
    a column of P with its own relative accuracy: elements of 1e-35, where three
    bf16 planes hold 18 bits, leave an error of fp32 size (1e-6; with the planes it
    is 2.8e-6)."""
    wl = I.mvrnn_workload(53, batch=30, d=128, leaf_lo=2, leaf_hi=2)
    wl = dataclasses.replace(wl, leaf_mat=np.ascontiguousarray(np.random.default_rng(53).normal(size=wl.leaf_mat.shape)
                                                               .astype(np.float32)))
    wl.leaf_mat[:, :, 70] *= np.float32(1e-35)
    announce("split mvrnn tiny N=%d" % wl.N)
    got, ref = run(wl).states_by_node()["P"], O.forward_workload(wl)["P"]
    inner = wl.x_index < 0
    for col in (69, 70, 71):
        g, r = got[inner][:, :, col], ref[inner][:, :, col]
        assert np.linalg.norm(g - r) <= 1e-6 * np.linalg.norm(r), col


MANY = {
    "nary": lambda: I.nary_treelstm_workload(36, batch=100, H=256),
    "childsum": lambda: childsum(37, 100, 20, 80),
    "tree_rnn_h256": lambda: tree_rnn(38, 60, 32, 32, 256),
    "tree_rnn_h256_wide": lambda: tree_rnn(39, 200, 32, 32, 256),
    "tree_rnn_h512": lambda: tree_rnn(40, 60, 32, 32, 512),
    "mvrnn": lambda: I.mvrnn_workload(41, batch=20, d=128),
    "dag_h256": lambda: I.dagrnn_workload(42, n_grids=10, rows=10, cols=10, H=256),
    "dag_h256_wide": lambda: I.dagrnn_workload(43, n_grids=20, rows=32, cols=32, H=256),
    "dag_h512": lambda: I.dagrnn_workload(44, n_grids=10, rows=10, cols=10, H=512),
}


@pytest.mark.parametrize("name", sorted(MANY))
def test_cost_of_an_infinite_weight(name):
    """With an infinite weight every tile of one slice forms its sums in fp32:
    the batch takes 1.6 to 4.4 times as long as with finite weights, not tens of
    times (16 to 55 with scalar fp32 sums)."""
    wl = MANY[name]()
    key = "W_M" if wl.W_M is not None else "U" if wl.U is not None and wl.cell != I.CELL_CHILDSUM_TREELSTM else "W"
    arr = getattr(wl, key).copy()
    arr.reshape(-1, wl.H)[7, 9] = np.inf
    us = []
    for case in (wl, dataclasses.replace(wl, **{key: arr})):
        announce("split cost %s N=%d" % (name, wl.N))
        dw = run(case)
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        best = float("inf")
        for _ in range(5):
            start.record()
            dw.step()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end))
        assert dw.status_code() == 0
        us.append(1e3 * best)
    assert us[1] <= 8 * us[0], us


BEYOND = dict(
    UNSPLITTABLE,
    # (one level: further up the huge weight would magnify the rounding of the states below)
    nary=lambda: I.nary_treelstm_workload(34, batch=520, H=256, leaf_lo=2, leaf_hi=2),
    tree_rnn=lambda: tree_rnn(35, 900, 2, 2, 256),
    tree_rnn_wide=lambda: tree_rnn(60, 2049, 2, 2, 256),
    tree_rnn_h512=lambda: tree_rnn(61, 860, 2, 2, 512),
)


@pytest.mark.parametrize("x,w", [(3e38, 2001.3), (-3e38, 2001.3), (2e30, 3e12), (1.0009e30, -3.003e12)])
@pytest.mark.parametrize("name", sorted(BEYOND))
def test_products_beyond_the_fp32_range(name, x, w, units):
    """Finite inputs and weights, each of which can be split, whose product
    leaves the fp32 range: the sum is an infinity of that sign, as in fp32
    arithmetic (a gate saturates), and never NaN from two plane products that
    overflow with opposite signs."""
    wl = BEYOND[name]()
    announce("split %s x %r w %r N=%d" % (name, x, w, wl.N))
    H, new = wl.H, {}
    if wl.leaf_mat is not None:
        # (vectors that keep B a and A b finite)
        new = {"leaf_mat": wl.leaf_mat.copy(), "x_table": wl.x_table.copy(), "W_M": wl.W_M.copy()}
        new["leaf_mat"][:, 9, 5] = x
        new["x_table"][:, 5] = 0.5
        new["W_M"].reshape(H, 2, H)[7, :, 9] = w
    else:
        key = "x" if wl.x is not None else "x_table"
        new[key] = getattr(wl, key).copy()
        new[key][:, 9] = x
        if wl.cell == I.CELL_TREE_RNN:
            new["W"] = wl.W.copy()
            new["W"].reshape(H, 2, H)[7, :, 9] = w
        else:
            wkey = "U" if wl.cell == I.CELL_NARY_TREELSTM else "W"       # the weights that meet an input row
            new[wkey] = getattr(wl, wkey).copy()
            new[wkey].reshape(-1, H, H)[:, 7, 9] = w
    wl = dataclasses.replace(wl, **new)
    got = run(wl).states_by_node()
    with np.errstate(all="ignore"):
        ref = O.forward_workload(wl)
        for key in ref:
            r32 = ref[key].astype(np.float32).astype(np.float64)
            assert not np.isnan(got[key]).any(), key
            inf, small = np.isinf(r32), np.abs(r32) <= 16
            assert np.array_equal(got[key][inf], r32[inf]), key
            assert float(np.abs(got[key][small] - r32[small]).max()) <= 1e-4, key
            # input rows (copied), and P's sums of two products of at most 0.1 |x|, which
            # may cancel: each product and each of eight partial sums rounds once
            rest = ~inf & ~small
            atol = 10 * 2.0 ** -24 * 0.1 * abs(x) if key == "P" else 0.0
            assert np.allclose(got[key][rest], r32[rest], rtol=2e-7, atol=atol), key
