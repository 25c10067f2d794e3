"""What the prover's and verifier's speed is measured on: calls a user of the
library makes through its Python entry points, at the sizes of the repository's
configurations, benchmark and tests.

A case names a call (`call`: "prove" or "verify") of one of the paths
  f2sc   the interactive F2 sum-check on a vector of n = 2^l counts,
  gkr    the GKR protocol on a circuit (`circuit`, `n`: inputs of F2 and F0,
         text length of PM and PM-F0, matrix side of MatMult and
         MatMult-check),
  batch  `count` uneven GKR proofs advancing together (sizes drawn from `mix`),
  nif2   the non-interactive F2 protocol on n values with rows of length h.
A verifier of f2sc or gkr receives two transcripts, an honest one and one with
a changed value, and returns both verdicts (the second names the check that
failed).  Inputs are device tensors unless `host` is true.  Circuits, servers' launch
plans and scratch are what a program keeps between calls.
"""
import numpy as np
import torch

import paper_1202_1350_amd as G
import workloads as W

P = (1 << 61) - 1
# admissible row lengths of the non-interactive protocol, short to long
ROWS = (9, 45, 63, 99, 225, 315, 585, 693, 1287, 2475, 5005)


def listed():
    return [
        # a vector of 2^10 counts: launches and one host copy, the latency of a proof
        {"name": "f2sc_prove_1k", "path": "f2sc", "call": "prove", "n": 1 << 10, "host": False},
        # the benchmark's sum-check, 2^26 counts: a stream over memory
        {"name": "f2sc_prove_64m", "path": "f2sc", "call": "prove", "n": 1 << 26, "host": False},
        # its verifier: the vector's multilinear extension at one point
        {"name": "f2sc_verify_64m", "path": "f2sc", "call": "verify", "n": 1 << 26, "host": False},
        # the smallest configuration, F2 on 2^10 inputs: nothing but dependent rounds
        {"name": "gkr_prove_f2_1k", "path": "gkr", "call": "prove", "circuit": "F2", "n": 1 << 10, "host": False},
        # the benchmark's proof, F2 on 2^22 inputs (12.6 million gates)
        {"name": "gkr_prove_f2_4m", "path": "gkr", "call": "prove", "circuit": "F2", "n": 1 << 22, "host": False},
        # matrix multiplication at N = 256: one very wide layer, many outputs, fan-out 256
        {"name": "gkr_prove_matmult_256", "path": "gkr", "call": "prove", "circuit": "MatMult", "n": 256,
         "host": False},
        # pattern matching on a text of no round length in host memory: mixed fan-out, ragged layers
        {"name": "gkr_prove_pm_100003", "path": "gkr", "call": "prove", "circuit": "PM", "n": 100003,
         "host": True},
        # distinct elements: 61 layers of the same ragged width (12 million gates, ~80 layers)
        {"name": "gkr_prove_f0_100003", "path": "gkr", "call": "prove", "circuit": "F0", "n": 100003,
         "host": False},
        # the verifier where the wiring has no closed form in most layers
        {"name": "gkr_verify_mmcheck_64", "path": "gkr", "call": "verify", "circuit": "MatMult-check", "n": 64,
         "host": False},
        # sixteen uneven proofs at once, as the batched configuration mixes them
        {"name": "batch_prove_16", "path": "batch", "call": "prove", "count": 16, "mix": 4},
        # Table 3's row near h = v / 4: 25 million values, proof of 4950 words
        {"name": "nif2_prove_25m_h2475", "path": "nif2", "call": "prove", "n": 25_000_000, "h": 2475, "host": False},
        # Table 3's other end for the verifier, which keeps one word a row
        {"name": "nif2_verify_25m_h585", "path": "nif2", "call": "verify", "n": 25_000_000, "h": 585, "host": False},
    ]


def _log(rng, lo, hi):
    """Whole number in [lo, hi], uniform in its logarithm."""
    return int(min(hi, max(lo, round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    path = rng.choice(("f2sc", "gkr", "gkr", "gkr", "gkr", "batch", "nif2", "nif2"))
    call = rng.choice(("prove", "prove", "prove", "verify"))
    host = rng.random() < 0.25
    if path == "f2sc":
        return {"path": path, "call": call, "n": 1 << rng.randint(11, 25), "host": host}
    if path == "batch":
        return {"path": path, "call": "prove", "count": rng.randint(3, 16), "mix": rng.randint(5, 10000)}
    if path == "nif2":
        return {"path": path, "call": call, "n": _log(rng, 50_000, 24_000_000), "h": rng.choice(ROWS), "host": host}
    circuit = rng.choice(("F2", "F2", "PM", "PM", "F0", "F0", "PM-F0", "PM-F0", "MatMult", "MatMult-check"))
    lo, hi = {"F2": (1 << 10, 1 << 21), "PM": (1 << 9, 1 << 18), "F0": (1 << 8, 1 << 16), "PM-F0": (1 << 8, 1 << 15),
              "MatMult": (4, 7), "MatMult-check": (2, 6)}[circuit]
    n = 1 << rng.randint(lo, hi) if circuit.startswith("MatMult") else _log(rng, lo, hi)
    return {"path": path, "call": call, "circuit": circuit, "n": n, "host": host}


_CIRCUITS = {"F2": W.f2_circuit, "PM": W.pm_circuit, "F0": W.f0_circuit, "PM-F0": W.pm_f0_circuit,
             "MatMult": W.matmult_circuit, "MatMult-check": W.matmult_check_circuit}


def _circuit_inputs(circuit, n, seed):
    if circuit == "F2":
        return W.f2_inputs(n, seed)
    if circuit == "F0":
        return W.f0_inputs(n, seed)
    if circuit == "MatMult":
        return W.matmult_inputs(n, seed)
    if circuit == "MatMult-check":
        return W.matmult_check_inputs(n, seed)[0]
    return W.pm_inputs(n, seed)[0]


def _place(x, host):
    """A vector as the call takes it: an array in host memory, or a device tensor."""
    if not host:
        return torch.from_numpy(x.view(np.int64)).cuda().view(torch.uint64)
    return x


def _counts(n, seed, dtype):
    """n counts uniform in [0, 2^16) on the device."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(0, 1 << 16, (n,), generator=g, device="cuda", dtype=dtype)


def _vector(case, seed):
    wide = case["path"] == "nif2"
    x = _counts(case["n"], seed, torch.int64 if wide else torch.int32)
    if case["host"]:
        return x.cpu().numpy().view(np.uint64 if wide else np.uint32)
    return x.view(torch.uint64 if wide else torch.uint32)


def prepare(case, seed):
    path = case["path"]
    state = {"path": path, "call": case["call"], "seed": seed, "h": case.get("h", 0)}
    if path == "batch":
        circs, inputs, seeds = [], [], []
        for k, (kind, circ, _, _) in enumerate(W.batch_mix(seed=case["mix"], count=case["count"])):
            size = circ.sizes[-1] - (8 if kind == "PM" else 0)
            circs.append(G.Circuit.from_workload(circ))
            inputs.append(_place(_circuit_inputs(kind, size, 64 * seed + k), False))
            seeds.append(64 * seed + k)
        state.update(circs=circs, inputs=inputs, seeds=seeds)
    elif path == "gkr":
        state["circ"] = G.Circuit.from_workload(_CIRCUITS[case["circuit"]](case["n"]))
        state["x"] = _place(_circuit_inputs(case["circuit"], case["n"], seed), case["host"])
    else:
        state["x"] = _vector(case, seed)
    torch.cuda.synchronize()  # the library reads inputs on a stream of its own
    if case["call"] == "verify":
        if path == "nif2":
            state["msgs"] = G.nif2_prove(state["x"], case["h"])
        else:
            msgs = (G.gkr_prove(state["circ"], state["x"], seed)[0] if path == "gkr"
                    else G.f2_sumcheck_prove(state["x"], seed)[0])
            state["msgs"], state["changed"] = msgs, _changed(msgs, seed)
    return state


def _changed(msgs, seed):
    """The transcript with one value, past the outputs, increased by one."""
    bad = msgs.copy()
    k = len(msgs) // 8 + 97 * seed % (len(msgs) - len(msgs) // 8)
    bad[k] = (int(bad[k]) + 1) % P
    return bad


def run(state):
    path, prove = state["path"], state["call"] == "prove"
    if path == "batch":
        return G.gkr_batch_prove(state["circs"], state["inputs"], state["seeds"])
    if path == "gkr":
        if prove:
            return G.gkr_prove(state["circ"], state["x"], state["seed"])
        return [G.gkr_verify(state["circ"], state["x"], state["seed"], m) for m in (state["msgs"], state["changed"])]
    if path == "f2sc":
        if prove:
            return G.f2_sumcheck_prove(state["x"], state["seed"])
        return [G.f2_sumcheck_verify(state["x"], state["seed"], m) for m in (state["msgs"], state["changed"])]
    if prove:
        return G.nif2_prove(state["x"], state["h"])
    return G.nif2_verify(state["x"], state["h"], state["seed"], state["msgs"])


def _log2up(n):
    return max(0, (int(n) - 1).bit_length())


def _circuit_work(circ, prove):
    """Bytes and field products (two operations each) of one circuit: inputs,
    both wires of every gate once and the transcript; a prover forms each
    gate's weight in three phases and halves three tables over each layer in
    two of them, a verifier reads the wires of the layers it has no formula for
    and extends the inputs."""
    S = [int(v) for v in circ.sizes]
    gates = sum(S[:-1])
    words = S[0] + sum(4 * (_log2up(a) + 2 * _log2up(b)) for a, b in zip(S, S[1:]))
    if not prove:
        return 8 * (S[-1] + words), 2 * S[-1]
    return 8 * (S[-1] + gates + words), 2 * sum(11 * a + 18 * b for a, b in zip(S, S[1:]))


def work(case):
    path, prove = case["path"], case["call"] == "prove"
    if path == "batch":
        w = [_circuit_work(c, True) for _, c, _, _ in W.batch_mix(seed=case["mix"], count=case["count"])]
        return {"bytes": sum(b for b, _ in w), "flops": sum(f for _, f in w)}
    if path == "gkr":
        b, f = _circuit_work(_CIRCUITS[case["circuit"]](case["n"]), prove)
        return {"bytes": b, "flops": f}
    n = case["n"]
    if path == "f2sc":
        return {"bytes": 4 * n + 32 * _log2up(n), "flops": 2 * (5 * n if prove else n)}
    h = case["h"]
    if prove:  # two transforms of every row and the squares of 2h columns
        f = sum({9: 9, 25: 10}.get(q, q) for q in _factors(h))
        return {"bytes": 8 * n + 16 * h, "flops": 2 * n * (2 * f + 3)}
    return {"bytes": 8 * n + 16 * h, "flops": 2 * n}


def _factors(h):
    """The coprime transform lengths whose product is h."""
    out = []
    for q in (25, 9, 13, 11, 7, 5, 3):
        if h % q == 0:
            out.append(q)
            h //= q
    return out


def _challenges(seed, purpose, count):
    """The verifier's coins: SplitMix64 outputs, their low 61 bits, redrawn on p."""
    out, z64 = [], (1 << 64) - 1
    state = (seed << 8 | purpose) & z64
    while len(out) < count:
        state = (state + 0x9E3779B97F4A7C15) & z64
        z = (state ^ state >> 30) * 0xBF58476D1CE4E5B9 & z64
        z = (z ^ z >> 27) * 0x94D049BB133111EB & z64
        z = (z ^ z >> 31) & P
        if z != P:
            out.append(z)
    return out


def exact(case, seed):
    """The sum-check's transcript by its definition in whole numbers (small
    vectors), and the verdict and F2 the non-interactive verifier returns."""
    if case["path"] == "nif2" and case["call"] == "verify":
        return True, int(_counts(case["n"], seed, torch.int64).square().sum()) % P
    if case["path"] != "f2sc" or case["call"] != "prove" or case["n"] > 1 << 16:
        return None
    a = _counts(case["n"], seed, torch.int32).cpu().numpy().astype(object)
    chals = _challenges(seed, 4, _log2up(case["n"]))
    msgs = [int((a * a).sum()) % P]
    for r in chals:
        lo, hi = a[0::2], a[1::2]
        two = 2 * hi - lo
        msgs += [int((v * v).sum()) % P for v in (lo, hi, two)]
        a = (lo + r * (hi - lo)) % P
    return np.array(msgs, np.uint64), np.array(chals, np.uint64)
