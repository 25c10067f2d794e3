"""Layers at the widths where the prover's steps change: the p-phase's first
step and its later ones, the omega phases' table steps and tails, eq tables in
LDS or in memory, the line's register folds, and the level-0 steps' sums over
lanes or on the matrix cores (four entries a thread: forced on small layers by
the launch shape).  Transcripts equal the oracle's bit for bit."""
import numpy as np
import pytest

from gpu_util import say, device_tensor, oracle_threads
from oracle import oracle as O
import workloads as W
from workloads.circuits import Circuit

pytestmark = pytest.mark.gpu
P = (1 << 61) - 1


def G():
    import paper_1202_1350_amd as mod
    return mod


def circuit(sizes, kind, seed):
    """Layers of the given sizes, wires drawn over the gates of the layer below
    (its padding is never read, so the ranges end anywhere); kind 0 ADD, 1 MUL,
    None mixed."""
    rng = np.random.default_rng(seed)
    types, in1, in2 = [], [], []
    for s, below in zip(sizes, sizes[1:]):
        types.append(rng.integers(0, 2, s, np.uint8) if kind is None else np.full(s, kind, np.uint8))
        in1.append(rng.integers(0, below, s, np.uint32))
        in2.append(rng.integers(0, below, s, np.uint32))
    return Circuit(list(sizes), types, in1, in2, name=f"widths {sizes}")


def inputs(n, seed):
    x = W.splitmix64(seed, 1, n) % np.uint64(P)
    x[0], x[-1] = P - 1, P - 1
    return x


def check(sizes, kind, seed):
    c, x = circuit(sizes, kind, seed), inputs(sizes[-1], seed)
    say("widths", sizes, "kind", kind)
    O.set_threads(oracle_threads())
    want_m, want_c = O.prove(c, x, seed)
    got_m, got_c = G().gkr_prove(G().Circuit.from_workload(c), x, seed)
    assert np.array_equal(got_m, want_m) and np.array_equal(got_c, want_c)


@pytest.mark.parametrize("kind", [None, 0, 1])
@pytest.mark.parametrize("sizes", [
    [1024, 2048], [1025, 2049], [2047, 8192], [8193, 5000], [16384, 16385], [16385, 100003], [131071, 131073],
    [5, 70000, 1000], [5000, 16], [3, 300, 70001, 33]])
def test_widths(sizes, kind):
    check(sizes, kind, sum(sizes))


@pytest.mark.parametrize("sizes", [[9, 262145, 524289], [3, 1048577, 262143], [7, 70001, 1048577]])
def test_wide(sizes):
    check(sizes, None, sum(sizes))


@pytest.mark.parametrize("items", [4, 8])
@pytest.mark.parametrize("kind", [None, 0, 1])
@pytest.mark.parametrize("sizes", [[3000, 2048], [700, 2049], [5000, 6145], [40000, 40003]])
def test_level0_on_matrix_cores(sizes, kind, items):
    """Every grid step at `items` entries a thread."""
    g = G()
    g.gkr_tune_set(None)
    blob = bytearray(g.gkr_tune_get())
    shapes = 17 * 48  # step kinds by size classes, at the table's end
    blob[-shapes:] = bytes([{4: 2, 8: 3}[items]]) * shapes
    try:
        g.gkr_tune_set(bytes(blob))
        check(sizes, kind, items + sum(sizes))
    finally:
        g.gkr_tune_set(None)


@pytest.mark.parametrize("words", [2047, 2049, 5000])
def test_batch_of_long_and_short_transcripts(words):
    cs = [circuit(s, None, 5) for s in ([words, 300], [3, 5], [1, 2, 9])]
    xs = [inputs(c.sizes[-1], 3) for c in cs]
    say("batch transcript words", words)
    got = G().gkr_batch_prove([G().Circuit.from_workload(c) for c in cs], [device_tensor(x) for x in xs], [4, 5, 6])
    for c, x, seed, msgs in zip(cs, xs, [4, 5, 6], got):
        assert np.array_equal(msgs, O.prove(c, x, seed)[0])


@pytest.mark.parametrize("kind", [None, 0, 1])
@pytest.mark.parametrize("sizes", [[9000, 8192], [5000, 40960], [700, 40896]])
def test_four_entries_in_every_thread_or_not(sizes, kind):
    """At four entries a thread the matrix cores take a step whose wires are a
    multiple of 2048, over several workgroups; one that lacks the last 64 stays
    with the sums over lanes."""
    g = G()
    g.gkr_tune_set(None)
    blob = bytearray(g.gkr_tune_get())
    shapes = 17 * 48  # step kinds by size classes, at the table's end
    blob[-shapes:] = bytes([2]) * shapes
    try:
        g.gkr_tune_set(bytes(blob))
        check(sizes, kind, 4 + sum(sizes))
    finally:
        g.gkr_tune_set(None)
