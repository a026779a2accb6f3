"""The ordering pre-pass and the work queue: results must not depend on the order items are processed in.

A call whose items all have a workgroup of their own uses neither an order nor a queue, so these problems hold at least twice as
many items as the launch has workgroups (the direct calls are compared with the oracle in test_gpu_dispatch.py)."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2509_16518_amd import fgattn as F
from paper_2509_16518_amd import workloads as W
from gpu_util import Problem, check_against_oracle, sample_items, say

pytestmark = pytest.mark.gpu


def skewed(M=64, N=8, d=128, L=6144, H=12, skew=0.8, seed=7, density=0.1):
    return dataclasses.replace(W.TINY, name="skew", H=H, L=L, d=d, M=M, N=N, kind=W.MASK_SKEW_LEN, skew=skew, density=density,
                               seed=seed, grid=(1, 1, 1))


def queued(prob):
    grid = F.fgattn_grid_size(prob.params())
    assert prob.w.items >= 2 * grid, (prob.w.items, grid)
    return prob


def control_words(ws):
    return ws[:256].view(torch.int32).cpu().numpy()


def read_order(prob, p, ws):
    n = prob.w.items
    return ws[256:256 + 4 * n].view(torch.int32).cpu().numpy()


def test_plan_orders_each_head_longest_first():
    prob = Problem(skewed())
    p = prob.params()
    ws = prob.workspace(p)
    ws.fill_(0xFF)
    F.fgattn_plan(prob.d_indptr, p, ws)
    torch.cuda.synchronize()
    order = read_order(prob, p, ws)
    w = prob.w
    assert sorted(order.tolist()) == list(range(w.items))            # a permutation: every item exactly once
    nnz = np.diff(prob.indptr)
    for s in range(w.B * w.H):
        seg = order[s * w.QB:(s + 1) * w.QB]
        assert ((seg >= s * w.QB) & (seg < (s + 1) * w.QB)).all()    # heads stay together, in order
        assert (np.diff(nnz[seg]) <= 0).all()                        # longest list first
    assert not control_words(ws).any()                  # the eight queues' counters among them


def test_plan_bucket_path_for_many_query_blocks():
    """More than 4096 query blocks per head takes the bucket-sort path: still a permutation, nearly sorted."""
    w = dataclasses.replace(skewed(M=16, N=64, d=64, L=70000, H=1, skew=0.9), name="manyblocks")
    prob = Problem(w)
    p = prob.params()
    ws = prob.workspace(p)
    F.fgattn_plan(prob.d_indptr, p, ws)
    torch.cuda.synchronize()
    order = read_order(prob, p, ws)
    assert w.QB > 4096 and sorted(order.tolist()) == list(range(w.items))
    nnz = np.diff(prob.indptr)[order]
    width = max(1, int(nnz.max()) // 2047 + 1)
    assert (np.diff(nnz) <= width).all()                             # descending up to one bucket width


def test_output_is_bitwise_independent_of_scheduling(oracle_mod):
    prob = queued(Problem(skewed()))
    base = prob.run()
    check_against_oracle(oracle_mod, prob, base, what="skewed lists", items=sample_items(prob.w, prob.indptr, 100))
    for flags in (F.FLAG_STATIC_ASSIGN, F.FLAG_FIFO_QUEUE):
        other = prob.run(flags=flags)
        assert np.array_equal(base[0], other[0]) and np.array_equal(base[1], other[1]), flags
    again = prob.run()
    assert np.array_equal(base[0], again[0]) and np.array_equal(base[1], again[1])   # run-to-run determinism


@pytest.mark.parametrize("M,N,d", [(16, 1, 128), (32, 8, 64), (64, 1, 128), (128, 1, 128), (128, 8, 64), (128, 1, 64)])
def test_repeated_runs_are_bitwise_identical_for_every_tiling(M, N, d):
    # every tile shape, ten runs under three schedules: a result that depended on timing (an instruction reading a
    # matrix-core result before it has landed, a slot read before its gather was waited for) would differ somewhere
    # (the 32-row tile runs up to nine workgroups per compute unit)
    prob = queued(Problem(skewed(M=M, N=N, d=d, L=18432 + 40 if M <= 32 else 8192 + 40, H=9 if M == 32 else 4 if M == 16 else 13 if M == 64 else 25,
                                 seed=31 + M, density=0.02)))
    first = prob.run()
    for i in range(9):
        other = prob.run(flags=(0, F.FLAG_STATIC_ASSIGN, F.FLAG_FIFO_QUEUE)[i % 3])
        assert np.array_equal(first[0], other[0]) and np.array_equal(first[1], other[1]), (i, M, N, d)


def test_reuse_plan_and_queue_rewind():
    """The stored order can be replayed without a pre-pass: a launch that reuses it has the queues' counters rewound."""
    prob = queued(Problem(skewed()))
    p = prob.params()
    ws = prob.workspace(p)
    F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, p, prob.out, prob.lse, ws)
    torch.cuda.synchronize()
    first = prob.out.clone(), prob.lse.clone()
    order = read_order(prob, p, ws)
    assert control_words(ws).any()   # items were popped
    pr = prob.params(flags=F.FLAG_REUSE_PLAN)
    for _ in range(3):
        prob.out.zero_()
        prob.lse.zero_()
        F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, pr, prob.out, prob.lse, ws)
        torch.cuda.synchronize()
        assert torch.equal(prob.out.view(torch.int16), first[0].view(torch.int16)) and torch.equal(prob.lse, first[1])
        assert control_words(ws).any() and np.array_equal(read_order(prob, p, ws), order)


def test_runs_on_a_side_stream():
    prob = queued(Problem(skewed()))
    base = prob.run()
    s = torch.cuda.Stream()
    p = prob.params()
    ws = prob.workspace(p)
    prob.out.zero_()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, p, prob.out, prob.lse, ws, stream=s)
    s.synchronize()
    from gpu_util import out_to_f64
    assert np.array_equal(out_to_f64(prob.out), base[0])
