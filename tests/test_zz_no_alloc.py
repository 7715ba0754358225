"""cortex_tree_infer_noalloc (the entry point for callers that cannot
allocate): the same path as cortex_tree_infer with the workspace in the
library's own device array.  Its results must be bitwise those of
cortex_tree_infer and within the oracle bound, on consecutive calls whose
batches shrink (the array keeps the previous call's contents), after a call
that failed, and it must reject batches beyond its limits on the host."""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import cortex_oracle as O
from paper_2011_01383_amd import cortex as C
from paper_2011_01383_amd import inputs as I
from paper_2011_01383_amd.runner import DeviceWorkload
from tests.gpu_helpers import announce, compare_lin, compare_states, need_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    need_gpu()
    yield


def noalloc(dw):
    return C.cortex_tree_infer_noalloc(dw.cell, dw.H, dw.children, dw.lin, dw.x_table, dw.x_rows, dw.x_index,
                                       dw.leaf_mat, W=dw.W, U=dw.U, b=dw.b, W_M=dw.W_M, h=dw.h, c_or_P=dw.c,
                                       status=dw.status)


def poison(dw):
    dw.h.fill_(float("nan"))
    if dw.c is not None:
        dw.c.fill_(float("nan"))
    dw.lin.level_nodes.fill_(-7)


def run_both(wl):
    """(no-alloc lin, states) and (cortex_tree_infer lin, states)."""
    a = DeviceWorkload(wl)
    poison(a)
    C.check(noalloc(a), "cortex_tree_infer_noalloc")
    assert a.status_code() == 0
    b = DeviceWorkload(wl)
    poison(b)
    b.infer()
    assert b.status_code() == 0
    return (a.lin_host(), a.states_by_node()), (b.lin_host(), b.states_by_node())


PAIRS = {
    # (larger batch, smaller batch) per cell; the first calls the fused
    # instances, "nary_two_launch" a batch beyond the fused range
    "nary": (lambda: I.nary_treelstm_workload(101, batch=10, H=256),
             lambda: I.nary_treelstm_workload(102, batch=3, H=256)),
    "childsum": (lambda: I.childsum_treelstm_workload(103, batch=10, H=256),
                 lambda: I.childsum_treelstm_workload(104, batch=2, H=256)),
    "tree_rnn_h256": (lambda: I.tree_rnn_workload(105, n_leaves=60, H=256),
                      lambda: I.tree_rnn_workload(106, n_leaves=9, H=256)),
    "treegru": (lambda: I.childsum_treegru_workload(107, batch=6, H=256),
                lambda: I.childsum_treegru_workload(108, batch=2, H=256)),
    "mvrnn": (lambda: I.mvrnn_workload(109, batch=6, d=64),
              lambda: I.mvrnn_workload(110, batch=2, d=64)),
    # the most nodes the staging of P takes at d = 128 (256), then a small batch
    "mvrnn_d128": (lambda: I.mvrnn_workload(117, batch=2, d=128, leaf_lo=64, leaf_hi=64),
                   lambda: I.mvrnn_workload(118, batch=2, d=128)),
    "nary_two_launch": (lambda: I.nary_treelstm_workload(111, batch=90, H=256),
                        lambda: I.nary_treelstm_workload(112, batch=40, H=256)),
}


@pytest.mark.parametrize("name", sorted(PAIRS))
def test_matches_tree_infer_on_shrinking_calls(name):
    for k, make in enumerate(PAIRS[name]):
        wl = make()
        announce("noalloc %s call %d N=%d" % (name, k, wl.N))
        (lin_a, st_a), (lin_b, st_b) = run_both(wl)
        compare_lin(lin_a, lin_b, wl.K)
        compare_lin(lin_a, O.linearize(wl.children, wl.K), wl.K)
        for key in st_b:
            assert np.array_equal(st_a[key], st_b[key]), (name, k, key)
        compare_states(st_a, O.forward_workload(wl), "%s call %d" % (name, k))


def test_call_after_a_failed_call():
    bad = I.nary_treelstm_workload(113, batch=2, H=256)
    ch = bad.children.copy()
    ch[np.nonzero(ch >= 0)[0][0]] = bad.N + 5                  # a child index out of range
    bad = I.Workload(bad.name, bad.cell, bad.H, bad.K, ch, x_index=bad.x_index, x_table=bad.x_table,
                     U=bad.U, b=bad.b)
    announce("noalloc after a failed call N=%d" % bad.N)
    dw = DeviceWorkload(bad)
    dw.h.fill_(7.0)
    C.check(noalloc(dw), "cortex_tree_infer_noalloc")
    assert dw.status_code() == C.CORTEX_ST_CHILD_RANGE
    assert bool((dw.h == 7.0).all())
    good = I.nary_treelstm_workload(114, batch=4, H=256)
    (_, st_a), (_, st_b) = run_both(good)
    for key in st_b:
        assert np.array_equal(st_a[key], st_b[key]), key
    compare_states(st_a, O.forward_workload(good), "after a failed call")


def test_left_over_treegru_values_are_no_exchanged_pairs():
    """TreeGRU with a barrier between its exchanges leaves plain floats in the
    array; here their bits are every small integer, so also the tag of the next
    launch.  MV-RNN at d = 128, whose workgroups exchange tagged pairs, must not
    take them for published values.  One column of matrices holds a value that
    cannot be split, so the workgroups of that column run late and the others
    do look before the values are there (its products meet zero weights in p)."""
    gru = I.childsum_treegru_workload(119, batch=20, H=512, node_lo=50, node_hi=50)
    W, b = gru.W.copy(), gru.b.copy()
    W.reshape(3, 512, 512)[2] = 0.0                            # kept: W_h x + b_h = b_h
    b.reshape(3, 512)[2] = (np.arange(512, dtype=np.uint32) // 2 + 1).view(np.float32)
    dw = DeviceWorkload(dataclasses.replace(gru, W=W, b=b))
    wl = I.mvrnn_workload(120, batch=85, d=128, leaf_lo=2, leaf_hi=2)
    leaf_mat, x_table, Wv = wl.leaf_mat.copy(), 0.1 * wl.x_table, wl.W.copy()
    leaf_mat[:, 3, 5] = 3.4e38
    Wv.reshape(128, 2, 128)[:, :, 3] = 0.0
    wl = dataclasses.replace(wl, leaf_mat=leaf_mat, x_table=x_table, W=Wv)
    announce("noalloc MV-RNN d=128 N=%d after TreeGRU N=%d with kept values" % (wl.N, dw.N))
    mv, ref = DeviceWorkload(wl), O.forward_workload(wl)["h"]
    for _ in range(4):
        C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, 3)
        try:
            C.check(noalloc(dw), "cortex_tree_infer_noalloc")
        finally:
            C.cortex_set_knob(C.CORTEX_KNOB_LEVEL_SYNC, 0)
        assert dw.status_code() == 0
        poison(mv)
        C.check(noalloc(mv), "cortex_tree_infer_noalloc")
        assert mv.status_code() == 0
        compare_states({"h": mv.states_by_node()["h"]}, {"h": ref}, "after kept values")


def test_rejects_batches_beyond_its_limits():
    # N * H beyond the h staging region (2,097,152 elements)
    big = I.nary_treelstm_workload(115, batch=1, H=256, leaf_lo=4200, leaf_hi=4200)
    assert big.N * big.H > 2097152
    announce("noalloc too large N=%d" % big.N)
    dw = DeviceWorkload(big)
    dw.h.fill_(7.0)
    assert noalloc(dw) == C.CORTEX_E_WORKSPACE
    assert dw.status_code() == 0
    assert bool((dw.h == 7.0).all())
    # N * H * H beyond the staging of P (4,194,304 elements)
    dw = DeviceWorkload(I.mvrnn_workload(121, batch=2, d=128, leaf_lo=65, leaf_hi=65))
    assert dw.N == 258
    assert noalloc(dw) == C.CORTEX_E_WORKSPACE
    assert dw.status_code() == 0
    # an unsupported hidden size is rejected as by cortex_tree_infer
    small = I.nary_treelstm_workload(116, batch=2, H=64)
    dw = DeviceWorkload(small)
    assert C.cortex_tree_infer_noalloc(C.CORTEX_NARY_TREELSTM, 100, dw.children, dw.lin,
                                       torch.zeros(dw.x_rows * 100, device="cuda"), dw.x_rows,
                                       dw.x_index, None, U=torch.zeros(10 * 100 * 100, device="cuda"),
                                       b=torch.zeros(500, device="cuda"), h=torch.zeros(dw.N * 100, device="cuda"),
                                       c_or_P=torch.zeros(dw.N * 100, device="cuda"),
                                       status=dw.status) == C.CORTEX_E_INVAL
    assert dw.status_code() == 0
