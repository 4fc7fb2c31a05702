"""Pins (no GPU) for partitions cut at layer granularity: cuts inside residual blocks, with the block's
shortcut value exchanged directly between the partition that holds the block's start and the one that
holds its end.

Citations: paper Section "Special Handling for Non-consecutive Models" (skip connections between
non-adjacent partitions, Forward / Backward lists, rank-sorted message order against deadlock);
"Implementing Distributed Back-Propagation" (Eq. 5-7: every partition back-propagates the partial errors
it receives); "Verifying the Correctness of HyPar-Flow" (the partitioned model computes what the
sequential one computes).
"""
from dataclasses import replace

import numpy as np
import pytest

from paper_1911_05146_amd import layer_cuts as LC
from paper_1911_05146_amd import workloads as W


def small_model():
    # bottleneck stage (projection at entry, identity after), stride-2 bottleneck entry, then basic blocks
    return (W.bottleneck_resnet_blocks([2, 2], (4, 8), (16, 32), 8) +
            [W.Block(W.BASIC, 32, 32, 32, 1), W.Block(W.BASIC, 32, 48, 48, 2)])


def build(cuts, b=2, m=2, seed=7, in_hw=8):
    return LC.split_at_layers("cutnet", small_model(), cuts, in_hw, 8, 5, b, m, seed)


CUT_SETS = {
    "every_layer": list(range(1, 16)),                 # one convolution per partition: every skip crosses partitions
    "middle_piece": [1, 2],                            # block 0 in three pieces: its skip jumps over partition 1
    "tail_and_head_in_one": [2, 4, 8, 13],             # partitions that end one block and start the next
    "block_boundaries_only": [3, 6, 9, 12, 14],        # no cut inside a block: plain chain
    "basic_blocks_cut": [13, 15],                      # cuts inside the basic blocks (identity and projection)
}


def chain_step(oracle, cm, inp, dtype, storage="none"):
    """The oracle's partitions chained through the messages of the cut model; returns loss and merged gradient."""
    parts = [oracle.OraclePartition(s, p, dtype, storage) for s, p in zip(cm.specs, cm.split_params(inp.params))]
    lists = LC.dependency_lists(cm)
    m = cm.whole.num_microbatches
    sent = [[{} for _ in range(m)] for _ in parts]
    for i in range(m):
        for p, part in enumerate(parts):
            got = {"act": inp.act_in[i] if p == 0 else None, "skip": None}
            for msg in lists[p].forward_recv:
                got[msg.tensor] = sent[msg.src][i][msg.tensor]
            o = part.forward(i, got["act"], inp.labels[i] if cm.specs[p].has_head else None, skip_in=got["skip"])
            sent[p][i] = {"act": o[0], "skip": o[1]} if isinstance(o, tuple) else {"act": o, "skip": None}
    loss = float(parts[-1].loss[0])
    back = [[{} for _ in range(m)] for _ in parts]
    for i in range(m):
        for p in reversed(range(len(parts))):
            got = {"act": None, "skip": None}
            for msg in lists[p].backward_recv:
                got[msg.tensor] = back[msg.dst][i][msg.tensor]
            e = parts[p].backward(i, got["act"], want_err_out=not cm.specs[p].has_stem, skip_err_in=got["skip"])
            back[p][i] = {"act": e[0], "skip": e[1]} if isinstance(e, tuple) else {"act": e, "skip": None}
    G = cm.merge([p.grad() for p in parts])
    for p in parts:
        p.close()
    return loss, G


@pytest.mark.parametrize("cuts", sorted(CUT_SETS))
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_layer_cut_chain_equals_unsplit_model(oracle, cuts, dtype):
    cm = build(CUT_SETS[cuts])
    inp = W.make_inputs(cm.whole, randomize_affine=True)
    ref = oracle.run_step(cm.whole, inp, dtype)
    loss, G = chain_step(oracle, cm, inp, dtype)
    assert loss == ref["loss"]
    assert np.array_equal(G, ref["grad"])                 # bitwise: same operations in the same order


def test_layer_cut_chain_keeps_the_premise_under_bf16_storage(oracle):
    cm = build(CUT_SETS["every_layer"])
    inp = W.make_inputs(cm.whole, randomize_affine=True)
    ref = oracle.run_step(cm.whole, inp, np.float32, storage="bf16")
    loss, G = chain_step(oracle, cm, inp, np.float32, storage="bf16")
    assert loss == ref["loss"] and np.array_equal(G, ref["grad"])   # tensors that cross a cut are stored tensors anyway


# ---------------------------------------------------------------------------------------------
# a cut partition on its own: gradients against finite differences of
#     sum_i <act_out_i, err_in_i> + <skip_out_i, skip_err_in_i>
# ---------------------------------------------------------------------------------------------
FD_SPECS = {
    # tail of a projection bottleneck (conv 2 + add, shortcut received) and head of the next block (convs 0, 1)
    "tail_then_head": dict(blocks=(W.Block(W.BOTTLENECK, 3, 2, 4, 2), W.Block(W.BOTTLENECK, 4, 2, 4, 1)), in_c=2, first_from=2, last_to=2),
    # middle piece: only the 3x3 convolution of a bottleneck
    "middle_piece": dict(blocks=(W.Block(W.BOTTLENECK, 4, 3, 4, 1),), in_c=3, first_from=1, last_to=2),
    # head piece of a projection block: bn1, conv0 and the projection; the shortcut value leaves
    "head_with_projection": dict(blocks=(W.Block(W.BOTTLENECK, 3, 2, 4, 2),), in_c=3, last_to=1),
    # head piece of an identity basic block: the shortcut value is the block input itself
    "head_identity_basic": dict(blocks=(W.Block(W.BASIC, 3, 3, 3, 1),), in_c=3, last_to=1),
    # tail piece of a basic block followed by a whole block
    "tail_basic_then_whole": dict(blocks=(W.Block(W.BASIC, 2, 3, 3, 2), W.Block(W.BASIC, 3, 3, 3, 1)), in_c=3, first_from=1),
}


def objective(oracle, spec, inp, params, act_in=None, skip_in=None):
    part = oracle.OraclePartition(spec, params, np.float64)
    tot = 0.0
    for i in range(spec.num_microbatches):
        o = part.forward(i, (act_in or inp.act_in)[i], None, skip_in=(skip_in or inp.skip_in)[i] if inp.skip_in else None)
        if isinstance(o, tuple):
            tot += float(np.sum(o[1] * inp.skip_err_in[i]))
            o = o[0]
        tot += float(np.sum(o * inp.err_in[i]))
    part.close()
    return tot


@pytest.mark.parametrize("case", sorted(FD_SPECS))
def test_cut_partition_gradients_match_finite_differences(oracle, case):
    kw = dict(FD_SPECS[case])
    spec = W.PartitionSpec(name=case, in_h=4, in_w=4, microbatch=2, num_microbatches=2, seed=23, **kw)
    inp = W.make_inputs(spec, randomize_affine=True)
    inp = replace(inp, params=inp.params.astype(np.float64), act_in=[a.astype(np.float64) for a in inp.act_in],
                  err_in=[e.astype(np.float64) for e in inp.err_in],
                  skip_in=[s.astype(np.float64) for s in inp.skip_in] if inp.skip_in else None,
                  skip_err_in=[s.astype(np.float64) for s in inp.skip_err_in] if inp.skip_err_in else None)
    assert (inp.skip_in is not None) == spec.has_skip_in and (inp.skip_err_in is not None) == spec.has_skip_out
    res = oracle.run_step(spec, inp, np.float64)
    G, h = res["grad"], 1e-6
    scale = max(np.abs(G).max(), 1.0)
    for i in range(inp.params.size):                               # every parameter
        e = np.zeros_like(inp.params)
        e[i] = h
        fd = (objective(oracle, spec, inp, inp.params + e) - objective(oracle, spec, inp, inp.params - e)) / (2 * h)
        assert abs(fd - G[i]) <= 1e-6 * scale, (i, fd, G[i])
    rs = np.random.default_rng(5)

    def check_input(field, grads):
        base = getattr(inp, field)
        sc = max(max(np.abs(g).max() for g in grads), 1.0)
        for _ in range(30):
            mb = rs.integers(spec.num_microbatches)
            idx = tuple(rs.integers(s) for s in base[0].shape)
            up = [a.copy() for a in base]
            dn = [a.copy() for a in base]
            up[mb][idx] += h
            dn[mb][idx] -= h
            fd = (objective(oracle, spec, inp, inp.params, **{field: up}) -
                  objective(oracle, spec, inp, inp.params, **{field: dn})) / (2 * h)
            assert abs(fd - grads[mb][idx]) <= 1e-6 * sc, (field, mb, idx, fd, grads[mb][idx])

    check_input("act_in", res["err_out"])
    if spec.has_skip_in:
        check_input("skip_in", res["skip_err_out"])


# ---------------------------------------------------------------------------------------------
# host logic: ownership, messages, Forward / Backward lists, message order
# ---------------------------------------------------------------------------------------------
def test_every_parameter_has_exactly_one_owner_and_shapes_chain():
    for cuts in CUT_SETS.values():
        cm = build(cuts)
        assert sum(W.n_params(s) for s in cm.specs) == W.n_params(cm.whole)
        v = np.arange(W.n_params(cm.whole), dtype=np.float64)
        assert np.array_equal(cm.merge(cm.split_params(v)), v)
        for a, b in zip(cm.specs, cm.specs[1:]):                   # the boundary tensor of neighbours
            assert a.out_shape() == (b.in_h, b.in_w, b.in_c)
        for msg in cm.messages:
            if msg.tensor == "skip":                               # the shortcut value keeps its shape on the way
                assert cm.specs[msg.src].skip_out_shape() == cm.specs[msg.dst].skip_in_shape()
                assert msg.dst > msg.src


def test_skip_of_a_block_in_three_pieces_bypasses_the_middle_partition():
    cm = build(CUT_SETS["middle_piece"])
    assert LC.Message("skip", 0, 2) in cm.messages
    assert not cm.specs[1].has_skip_in and not cm.specs[1].has_skip_out
    lists = LC.dependency_lists(cm)
    assert [(m.tensor, m.dst) for m in lists[0].forward_send] == [("act", 1), ("skip", 2)]   # next layer's partition first
    assert [(m.tensor, m.src) for m in lists[2].forward_recv] == [("skip", 0), ("act", 1)]
    assert [(m.tensor, m.dst) for m in lists[0].backward_recv] == [("skip", 2), ("act", 1)]
    assert [(m.tensor, m.src) for m in lists[2].backward_send] == [("act", 1), ("skip", 0)]


@pytest.mark.parametrize("cuts", sorted(CUT_SETS))
def test_rank_sorted_message_order_never_deadlocks_under_blocking_exchange(cuts):
    cm = build(CUT_SETS[cuts])
    lists = LC.dependency_lists(cm)
    assert LC.replay_blocking(lists, "forward") and LC.replay_blocking(lists, "backward")


def test_the_unsorted_order_of_the_papers_example_deadlocks():
    """Three partitions, a skip from the first to the third: if the first sends to the third before it sends to
    the second while the third waits for the second, every rank waits for another one."""
    cm = build(CUT_SETS["middle_piece"])
    bad = LC.dependency_lists(cm, sort_by_rank=False)
    assert [(m.tensor, m.dst) for m in bad[0].forward_send] == [("skip", 2), ("act", 1)]
    assert not LC.replay_blocking(bad, "forward")
    assert not LC.replay_blocking(bad, "backward")


def test_invalid_cut_descriptions_are_rejected(oracle):
    blk = (W.Block(W.BOTTLENECK, 4, 2, 4, 1),)
    good = W.PartitionSpec(name="x", in_h=4, in_w=4, in_c=2, blocks=blk, microbatch=1, num_microbatches=1, first_from=1)
    oracle.OraclePartition(good, np.zeros(W.n_params(good), np.float32)).close()
    for bad in (replace(good, first_from=3), replace(good, first_from=1, last_to=1), replace(good, last_to=3),
                replace(good, in_c=4)):
        with pytest.raises(ValueError):
            oracle.OraclePartition(bad, np.zeros(64, np.float32))


@pytest.mark.parametrize("set_to, queues", [(None, 4), ("2", 2), ("8", 8), ("", 4), ("all", 4), ("0", 1)])
def test_streams_of_a_pipeline_follow_as_many_used_ones_as_there_are_hardware_queues(monkeypatch, set_to, queues):
    """A stream gets the queue that the fewest hold when it is first used: every queue is held before the pipeline's own are made."""
    from contextlib import nullcontext
    from types import SimpleNamespace
    from paper_1911_05146_amd import pipeline
    made, used = [], []

    class Word:
        def zero_(self):
            used.append(current[-1])

    current = []

    def stream(s):
        current.append(s)
        return nullcontext()
    cuda = SimpleNamespace(Stream=lambda device: made.append(len(made)) or made[-1], stream=stream, synchronize=lambda device: None)
    if set_to is None:
        monkeypatch.delenv("GPU_MAX_HW_QUEUES", raising=False)
    else:
        monkeypatch.setenv("GPU_MAX_HW_QUEUES", set_to)
    got = pipeline._streams_apart(SimpleNamespace(cuda=cuda, empty=lambda n, device: Word()), "device", 3)
    assert got == [queues, queues + 1, queues + 2] and used == made == list(range(queues + 3))
