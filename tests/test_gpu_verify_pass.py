"""The verifiers' one pass over device inputs: sizes at the edges of its
tiles, and inputs that do not start on a 16-byte boundary.  The verdicts are
exact: the honest transcript is accepted, one changed input is rejected."""
import numpy as np
import pytest

from gpu_util import say, device_tensor, oracle_threads
from oracle import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu
P = (1 << 61) - 1


def G():
    import paper_1202_1350_amd as mod
    return mod


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 3, 1023, 1025, 2047, 2049, 70001])
def test_circuit_inputs(n, offset):
    c = G().Circuit.from_workload(W.f2_circuit(n))
    x = W.splitmix64(n, 1, n) % np.uint64(P)
    x[-1] = P - 1
    # (out-of-range words around the values must not be read; offset 1 starts
    # them one word past a 16-byte boundary)
    bad = np.full(4, 2 ** 64 - 1, np.uint64)
    t = device_tensor(np.concatenate([bad[:2 + offset], x, bad]))[2 + offset:2 + offset + n]
    say("verify inputs n", n, "offset", offset)
    msgs, _ = G().gkr_prove(c, x, 5)
    assert G().gkr_verify(c, t, 5, msgs)[0]
    y = x.copy()
    y[n // 2] = (int(y[n // 2]) + 1) % P
    assert not G().gkr_verify(c, device_tensor(y), 5, msgs)[0]
    y[n // 2] = P
    with pytest.raises(G().GkrError) as e:
        G().gkr_verify(c, device_tensor(y), 5, msgs)
    assert e.value.code == G().GKR_ERR_RANGE


@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("logn", [0, 1, 10, 11, 12, 17])
def test_counts(logn, offset):
    n = 1 << logn
    a = (W.splitmix64(logn, 3, n) >> np.uint64(32)).astype(np.uint32)
    buf = device_tensor(np.concatenate([np.zeros(offset, np.uint32), a]))
    say("verify counts log n", logn, "offset", offset)
    msgs, _ = G().f2_sumcheck_prove(a, 6)
    assert G().f2_sumcheck_verify(buf[offset:], 6, msgs) == (True, -1, 0)
    b = a.copy()
    b[n // 3] ^= 1
    assert not G().f2_sumcheck_verify(device_tensor(b), 6, msgs)[0]


@pytest.mark.parametrize("n,h", [(64 * 512 * 9 - 1, 9), (64 * 512 * 9 + 10, 9), (2475 * 17, 2475)])
def test_rows(n, h):
    """Rows on both sides of the change of rows a workgroup takes at a time."""
    rng = np.random.default_rng(n)
    a = rng.integers(0, P, n).astype(np.uint64)
    say("verify rows n", n, "h", h)
    t = device_tensor(a)
    m = G().nif2_prove(t, h)
    f2 = sum(int(m[2 * j]) for j in range(h)) % P
    assert G().nif2_verify(t, h, 3, m) == (True, f2)
    a[n // 2] = (int(a[n // 2]) + 1) % P
    assert not G().nif2_verify(device_tensor(a), h, 3, m)[0]
    a[n - 1] = P
    with pytest.raises(G().GkrError) as e:
        G().nif2_verify(device_tensor(a), h, 3, m)
    assert e.value.code == G().GKR_ERR_RANGE


@pytest.mark.parametrize("sizes", [[5, 524288, 64], [5, 700001, 3, 1100003, 257], [2, 1048576, 1048577, 9]])
def test_layers_share_the_workgroups_of_one_pass(sizes):
    """Layers without a closed form whose gates want just the workgroups a pass
    has, or more (then shared by gates, one at least for the small ones): a
    changed v1 of each layer is found in that layer, as the oracle finds it."""
    rng = np.random.default_rng(sum(sizes))
    types, in1, in2 = [], [], []
    for s, below in zip(sizes, sizes[1:]):
        types.append(rng.integers(0, 2, s, np.uint8))
        in1.append(rng.integers(0, below, s, np.uint32))
        in2.append(rng.integers(0, below, s, np.uint32))
    circ = W.circuits.Circuit(list(sizes), types, in1, in2, name=f"shares {sizes}")
    x = W.splitmix64(3, 1, sizes[-1]) % np.uint64(P)
    say("verify shares", sizes)
    O.set_threads(oracle_threads())
    c, t = G().Circuit.from_workload(circ), device_tensor(x)
    msgs, _ = G().gkr_prove(c, t, 8)
    assert G().gkr_verify(c, t, 8, msgs) == (True, -1, -1, 0) == O.verify(circ, x, 8, msgs)
    at = sizes[0]
    for i, (s, below) in enumerate(zip(sizes, sizes[1:])):
        a, b = (s - 1).bit_length(), (below - 1).bit_length()
        v1 = at + 3 * (a + 2 * b)
        at = v1 + 2 + max(b - 1, 0)
        bad = msgs.copy()
        bad[v1] = (int(bad[v1]) + 1) % P
        got = G().gkr_verify(c, t, 8, bad)
        assert got == O.verify(circ, x, 8, bad) and got[:2] == (False, i)
    assert at == len(msgs)


@pytest.mark.parametrize("n,h", [(64 * 512 * 9 - 9, 9), (64 * 512 * 9, 9), (64 * 512 * 99 - 99, 99), (64 * 512 * 99 + 40, 99),
                                 (32833 * 65 - 7, 65)])
def test_rows_a_workgroup_takes(n, h):
    """Grids of 16, 512 and 64 rows a workgroup at the changes between them
    (32768 rows; rows of more than 64 values), the last group and the last
    column partly filled.  The verdicts are the oracle's; a changed value and one
    out of range are found in the last group and in the last column."""
    rng = np.random.default_rng(n)
    a = rng.integers(0, P, n).astype(np.uint64)
    a[0] = a[-1] = P - 1
    v = -(-n // h)
    say("verify rows a workgroup, n", n, "h", h, "rows", v)
    t = device_tensor(a)
    m = G().nif2_prove(t, h)
    f2 = sum(int(m[2 * j]) for j in range(h)) % P
    O.set_threads(oracle_threads())
    assert G().nif2_verify(t, h, 3, m) == (True, f2) == O.nif2_verify(a, h, 3, m)
    for k in (v - 1, n // 2, n - 1):
        b = a.copy()
        b[k] = (int(b[k]) + 1) % P
        assert G().nif2_verify(device_tensor(b), h, 3, m) == (False, f2) == O.nif2_verify(b, h, 3, m)
        b[k] = P
        with pytest.raises(G().GkrError) as e:
            G().nif2_verify(device_tensor(b), h, 3, m)
        assert e.value.code == G().GKR_ERR_RANGE


@pytest.mark.parametrize("h", [1001, 1287, 5005, 225225])
def test_long_proofs(h):
    """Proofs of one to 220 workgroups' words, the last one partly filled: every
    changed word is found, as the oracle finds it."""
    rng = np.random.default_rng(h)
    a = rng.integers(0, P, 3 * h + 1).astype(np.uint64)
    say("verify long proof h", h)
    t = device_tensor(a)
    m = G().nif2_prove(t, h)
    O.set_threads(oracle_threads())
    want = O.nif2_verify(a, h, 5, m)
    assert want[0] and G().nif2_verify(t, h, 5, m) == want
    for k in (0, 511, 2 * h // 2048 * 2048 - 1, 2 * h // 2048 * 2048, 2 * h - 1):
        if not 0 <= k < 2 * h:
            continue
        bad = m.copy()
        bad[k] = (int(bad[k]) + 1) % P
        assert not G().nif2_verify(t, h, 5, bad)[0], k
