"""The weight-stationary expert FFN (bf16, d_h 128, d_ff 128, many slots per
expert) against the CPU oracle: experts whose slot counts sit at the edges of
its 32-slot blocks and 64-slot tiles, empty experts, several experts per
workgroup and one expert over many workgroups."""
import numpy as np
import pytest
import torch

import paper_2602_04870_amd as mh
import workloads
from tests.gpu_util import (DeviceWorkload, announce, check_rows, needs_gpu, to_device,
                            to_host_f64)

pytestmark = [pytest.mark.gpu, needs_gpu]

# first-choice slots of the experts 0, 1, ...; the rest of the tokens choose
# the expert after them, and every second choice is one of the last two
EDGE_COUNTS = [0, 1, 31, 32, 33, 63, 64, 65, 0, 96, 127, 129]


def _edge_routing(T, n_heads, seed):
    rng = np.random.default_rng(seed)
    Ne = len(EDGE_COUNTS) + 3
    idx = np.empty((T, n_heads, 2), np.int32)
    small = np.zeros(T, bool)
    for h in range(n_heads):
        first = np.full(T, len(EDGE_COUNTS), np.int32)
        order = rng.permutation(T)
        at = 0
        for e, c in enumerate(EDGE_COUNTS):
            first[order[at:at + c]] = e
            at += c
        small[order[:at]] = True
        idx[:, h, 0] = first
        idx[:, h, 1] = Ne - 2 + rng.integers(0, 2, T)
    gate = rng.random((T, n_heads, 2)) + 0.05
    gate /= gate.sum(-1, keepdims=True)
    return Ne, idx, gate.astype(np.float32), small


@pytest.mark.parametrize("expert", ["swiglu", "gelu"])
@pytest.mark.parametrize("T,n_heads", [(65537, 1), (11000, 9)])
def test_edge_counts(T, n_heads, expert, oracle_instance):
    Ne, idx, gate, small = _edge_routing(T, n_heads, seed=3)
    shape = workloads.Shape(T, n_heads, 128, Ne, 2, 128, "bf16", expert=expert)
    # the dispatch rule: at least 2^17 slots, 768 per expert on average
    assert shape.slots >= 1 << 17 and T * 2 >= 768 * Ne
    announce(f"stationary ffn {expert} T={T} heads={n_heads}")
    w = workloads.generate(shape, seed=5)
    d = DeviceWorkload(w)
    gi, gg = to_device(idx), to_device(gate)

    def run():
        if expert == "gelu":
            return mh.mhlmoe_experts_gelu(d.X, gi, gg, d.W1, d.W2)
        return mh.mhlmoe_experts(d.X, gi, gg, d.W1, d.W3, d.W2)

    Y, Y2 = run(), run()
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2), "not bitwise reproducible"
    # every token of a small expert, and a sample of the others
    rows = np.unique(np.concatenate([np.flatnonzero(small), workloads.sample_rows(T, 200)]))
    args = (w.exact("X", rows), idx[rows], gate[rows].astype(np.float64), w.exact("W1"))
    if expert == "gelu":
        want = oracle_instance.experts_gelu(*args, w.exact("W2"))
    else:
        want = oracle_instance.experts(*args, w.exact("W3"), w.exact("W2"))
    check_rows(to_host_f64(Y)[rows], want, "bf16", f"stationary ffn {expert}")


@pytest.mark.parametrize("T,n_heads,Ne,k", [(16400, 8, 8, 4), (8200, 8, 250, 8), (8200, 8, 260, 8)])
def test_either_side_of_the_rule(T, n_heads, Ne, k, oracle_instance):
    """Long runs, and a mean of 256 slots per expert from both sides (the
    last goes to the streaming kernel): the same outputs to bf16 rounding."""
    shape = workloads.Shape(T, n_heads, 128, Ne, k, 128, "bf16")
    announce(f"stationary ffn rule T={T} heads={n_heads} Ne={Ne} k={k}")
    w = workloads.generate(shape, seed=7)
    idx, gate = workloads.random_routing(T, n_heads, Ne, k, seed=9, skew=0.7)
    d = DeviceWorkload(w)
    Y = mh.mhlmoe_experts(d.X, to_device(idx), to_device(gate), d.W1, d.W3, d.W2)
    torch.cuda.synchronize()
    rows = workloads.sample_rows(T, 160)
    want = oracle_instance.experts(w.exact("X", rows), idx[rows], gate[rows].astype(np.float64),
                                   w.exact("W1"), w.exact("W3"), w.exact("W2"))
    check_rows(to_host_f64(Y)[rows], want, "bf16", f"stationary ffn Ne={Ne}")


@pytest.mark.parametrize("expert", ["swiglu", "gelu"])
@pytest.mark.parametrize("load", ["collapsed", "zipf"])
@pytest.mark.parametrize("T", [32768, 32767])
def test_uneven_loads(T, load, expert, oracle_instance):
    """Loads at which equal shares of the tiles are not equal work, from 2^19
    slots on (where the shares weigh an expert's weights) and just below: most
    experts of every head without a slot and a few with one to three, or a Zipf
    load; tokens of the rare experts are all compared."""
    n_heads, Ne, k = 8, 64, 2
    shape = workloads.Shape(T, n_heads, 128, Ne, k, 128, "bf16", expert=expert)
    announce(f"stationary ffn uneven {load} {expert} T={T}")
    w = workloads.generate(shape, seed=19)
    idx, gate = workloads.random_routing(T, n_heads, Ne, k, seed=21, skew=1.1)
    rows = workloads.sample_rows(T, 120)
    if load == "collapsed":
        rng = np.random.default_rng(23)
        for h in range(n_heads):
            used = rng.permutation(Ne)[:3 + h % 2]
            idx[:, h, 0] = used[0]
            idx[:, h, 1] = used[1 + rng.integers(0, 2, T)]
            rare = np.setdiff1d(np.arange(Ne), used)[:h]
            at = rng.permutation(T)[:2 * len(rare)]
            idx[at, h, 1] = np.repeat(rare, 2)
            rows = np.union1d(rows, at)
    else:
        for h in range(n_heads):
            c = np.bincount(idx[:, h].ravel(), minlength=Ne)
            rows = np.union1d(rows, np.flatnonzero((idx[:, h] == c.argmin()).any(-1))[:40])
    d = DeviceWorkload(w)
    gi, gg = to_device(idx), to_device(gate)
    Y = (mh.mhlmoe_experts_gelu(d.X, gi, gg, d.W1, d.W2) if expert == "gelu"
         else mh.mhlmoe_experts(d.X, gi, gg, d.W1, d.W3, d.W2))
    torch.cuda.synchronize()
    args = (w.exact("X", rows), idx[rows], gate[rows].astype(np.float64), w.exact("W1"))
    want = (oracle_instance.experts_gelu(*args, w.exact("W2")) if expert == "gelu"
            else oracle_instance.experts(*args, w.exact("W3"), w.exact("W2")))
    check_rows(to_host_f64(Y)[rows], want, "bf16", f"stationary ffn {load} {expert}")


@pytest.mark.parametrize("T,n_heads,Ne,k,expert", [
    (16390, 8, 16, 1, "swiglu"), (11000, 4, 20, 3, "swiglu"), (9001, 3, 40, 5, "gelu"),
    (5501, 2, 48, 12, "swiglu"), (2801, 2, 64, 24, "gelu"), (2200, 2, 64, 31, "swiglu"),
    (33001, 8, 64, 3, "gelu"), (33001, 8, 64, 3, "swiglu")])
def test_slot_division_and_long_runs(T, n_heads, Ne, k, expert, oracle_instance):
    """k = 1 and values that are no power of two (the kernel divides slot ids
    by a rounded magic number there), and 24 tiles per workgroup, three times
    round the ring of slot lists."""
    shape = workloads.Shape(T, n_heads, 128, Ne, k, 128, "bf16", expert=expert)
    # the dispatch rule: at least 2^17 slots, 768 per expert on average
    assert shape.slots >= 1 << 17 and T * k >= 768 * Ne
    announce(f"stationary ffn {expert} T={T} heads={n_heads} Ne={Ne} k={k}")
    w = workloads.generate(shape, seed=25)
    idx, gate = workloads.random_routing(T, n_heads, Ne, k, seed=27, skew=0.7)
    d = DeviceWorkload(w)
    gi, gg = to_device(idx), to_device(gate)
    Y = (mh.mhlmoe_experts_gelu(d.X, gi, gg, d.W1, d.W2) if expert == "gelu"
         else mh.mhlmoe_experts(d.X, gi, gg, d.W1, d.W3, d.W2))
    torch.cuda.synchronize()
    rows = workloads.sample_rows(T, 160)
    args = (w.exact("X", rows), idx[rows], gate[rows].astype(np.float64), w.exact("W1"))
    want = (oracle_instance.experts_gelu(*args, w.exact("W2")) if expert == "gelu"
            else oracle_instance.experts(*args, w.exact("W3"), w.exact("W2")))
    check_rows(to_host_f64(Y)[rows], want, "bf16", f"stationary ffn k={k} {expert}")
