"""Which variant and schedule a call takes depends on its sizes: the sizes on both sides of every line."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2509_16518_amd import fgattn as F
from paper_2509_16518_amd import workloads as W
from gpu_util import Problem, check_against_oracle

pytestmark = pytest.mark.gpu


def sparse_rows(items, M, N=1, d=64, H=1, keys=70, seed=50):
    """`items` query blocks over H heads, each with about `keys` active keys."""
    L = items // H * M
    return dataclasses.replace(W.TINY, name="dispatch", H=H, L=L, d=d, M=M, N=N, kind=W.MASK_RANDOM, density=min(1.0, keys / L),
                               grid=(1, 1, 1), seed=seed + items)


# 512 workgroups of the 64-row tile run at once (two per compute unit of 256): up to 512 items need no queue; the next
# ones are popped; fewer heads than queues, and heads that do not divide among them, leave queues empty or uneven
@pytest.mark.parametrize("items,H", [(1, 1), (7, 1), (9, 1), (511, 1), (512, 1), (513, 1), (520, 1), (1100, 11), (1536, 3)])
def test_direct_and_queued_assignment(oracle_mod, items, H):
    prob = Problem(sparse_rows(items, 64, d=128, H=H))
    first = prob.run()
    check_against_oracle(oracle_mod, prob, first, what="%d items" % items)
    # the stored order is replayed with the queues rewound (or not needed), with other work in between
    p, pr = prob.params(), prob.params(flags=F.FLAG_REUSE_PLAN)
    ws = prob.workspace(p)
    for params in (p, pr, pr):
        prob.out.zero_()
        F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, params, prob.out, prob.lse, ws)
        torch.cuda.synchronize()
        assert np.array_equal(W.bf16_bits_to_f64(prob.out.view(torch.int16).cpu().numpy().view(np.uint16)), first[0])


# A call whose items all have a workgroup of their own needs no order, but one on the same workspace may: at d = 64 the
# variants for lists run more workgroups than the dense ones.  (The workspace holds zeros at first: an order that nobody
# wrote would be item 0 over and over, in range.)
@pytest.mark.parametrize("M,items", [(128, 600), (128, 513), (32, 2100), (16, 2560), (64, 400), (128, 300)])
def test_direct_call_leaves_an_order(M, items):
    prob = Problem(sparse_rows(items, M))
    want = prob.run(dense=True)
    p, pr = prob.params(), prob.params(flags=F.FLAG_REUSE_PLAN)
    ws = prob.workspace(p)
    ws.zero_()
    order = ws[256:256 + 4 * items].view(torch.int32)
    F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, p, prob.out, prob.lse, ws)
    assert torch.equal(order.sort()[0], torch.arange(items, device="cuda", dtype=torch.int32))
    prob.out.view(torch.int16).fill_(0x7FC0)
    F.fgattn_dense_forward(prob.q, prob.k, prob.v, pr, prob.out, prob.lse, ws)
    assert np.array_equal(W.bf16_bits_to_f64(prob.out.view(torch.int16).cpu().numpy().view(np.uint16)), want[0])
    # an order that is there already stays
    F.fgattn_plan(prob.d_indptr, p, ws)
    planned = order.clone()
    F.fgattn_forward(prob.q, prob.k, prob.v, prob.d_indptr, prob.d_indices, pr, prob.out, prob.lse, ws)
    assert torch.equal(order, planned)


# A workgroup that is not resident keeps the item it begins with from the others, so a launch has no more of them than compute
# units hold: LDS is given out in pieces of 1280 bytes of 160 KiB (the 32-row tile takes 32768 bytes at d = 128, 16384 at 64)
@pytest.mark.parametrize("M", [16, 32])
@pytest.mark.parametrize("d,per_unit", [(128, 4), (64, 9)])
@pytest.mark.parametrize("N", [1, 8, 7])
def test_no_more_workgroups_than_are_resident(M, d, per_unit, N):
    q = torch.empty((1, 40, 4096, d), dtype=torch.bfloat16, device="cuda")
    grid = F.fgattn_grid_size(F.make_params(q, q, q, q, M, N, 0.1))
    assert 0 < grid <= per_unit * torch.cuda.get_device_properties(0).multi_processor_count


# keys per group on both sides of the tile sizes (32 and 64 keys), odd ones, more than a tile; the short last group stands
# first, in the middle or last in its list (shuffled), and lists end inside, at and just past a tile
@pytest.mark.parametrize("M", [16, 32, 64, 128])
@pytest.mark.parametrize("N,L", [(3, 1027), (31, 1000), (32, 1000), (33, 1024), (63, 2060), (64, 2050), (65, 2015), (200, 1999)])
def test_short_last_group_anywhere_in_the_list(oracle_mod, M, N, L):
    w = dataclasses.replace(W.TINY, name="short", H=2, L=L, d=64 if N % 2 else 128, M=M, N=N, kind=W.MASK_RANDOM, density=0.4,
                            grid=(1, 1, 1), seed=900 + M + N)
    rng = np.random.default_rng(M * 1000 + N)
    lists = []
    for i in range(w.items):
        ids = np.flatnonzero(rng.random(w.G) < 0.4)
        ids = np.union1d(ids, [w.G - 1]) if i % 3 else ids   # two items of three hold the last group
        lists.append(rng.permutation(ids if ids.size else np.array([0])).astype(np.int32))
    indptr = np.zeros(w.items + 1, dtype=np.int64)
    indptr[1:] = np.cumsum([x.size for x in lists])
    prob = Problem(w, mask=(indptr, np.concatenate(lists)))
    check_against_oracle(oracle_mod, prob, prob.run(), what="M=%d N=%d L=%d" % (M, N, L))


# The exponent base of a query follows the running maximum by steps of at least 2^8: scores that grow along the list by less
# than that and by more per tile (several moves), by far more than a float's exponent holds at one key (sums of +inf are formed
# and formed again), and that fall
@pytest.mark.parametrize("M,d", [(16, 64), (32, 128), (64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("shape", ["ramp", "jump", "fall"])
@pytest.mark.parametrize("N,L", [(1, 700), (8, 700)])
def test_exponent_base_moves(oracle_mod, M, d, shape, N, L):
    w = dataclasses.replace(W.TINY, name="base", H=2, L=L, d=d, M=M, N=N, kind=W.MASK_RANDOM, density=0.7, grid=(1, 1, 1),
                            seed=77 + M + d)
    q, k, v = W.make_qkv(w)
    gain = {"ramp": np.linspace(0.1, 40.0, L), "jump": np.where(np.arange(L) == L - 90, 400.0, 0.2),
            "fall": np.linspace(40.0, 0.1, L)}[shape]
    k = W.f32_to_bf16_bits((W.bf16_bits_to_f64(k) * gain[None, None, :, None]).astype(np.float32))
    prob = Problem(w, q, k, v)
    check_against_oracle(oracle_mod, prob, prob.run(), what="%s M=%d d=%d N=%d" % (shape, M, d, N))
    if N == 1:
        dense = Problem(dataclasses.replace(w, kind=W.MASK_ALL), q, k, v)
        check_against_oracle(oracle_mod, dense, dense.run(dense=True), what="dense " + shape)


# Dense calls on both sides of the line between items that all start at once (their own variant at 128 rows) and a queue
@pytest.mark.parametrize("M,d,items", [(128, 128, 511), (128, 128, 513), (128, 64, 512), (128, 64, 769), (64, 128, 512), (64, 64, 770)])
def test_dense_direct_and_queued(oracle_mod, M, d, items):
    heads = 16
    w = dataclasses.replace(W.TINY, name="dense", H=heads, L=(items // heads) * M + (M // 2 if items % heads else 0), d=d, M=M, N=1,
                            kind=W.MASK_ALL, grid=(1, 1, 1), seed=items)
    prob = Problem(w)
    check_against_oracle(oracle_mod, prob, prob.run(dense=True), what="%d items" % w.items, items=np.arange(0, w.items, 37))
