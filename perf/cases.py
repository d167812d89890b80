"""The work that is timed: amplitude batches of every kind that a program asks
this framework for, through the public entry points.

A case is a dict of plain values.  `kind` names the entry point:

  chain   Plan.amplitudes of a doped-Clifford CZ brickwork (n, d, k, batches;
          `storage` of the boundary tensor, `tiles` the plan options)
  bond4   Plan.amplitudes of a brickwork of generic two-qubit gates (k = 0)
  ring    RingPlan.amplitudes of a ring of CZ gates, by slicing
  serve   Server.submit / wait of a burst of mixed requests
  post    log-XEB, batched sampling and frugal rejection of amplitudes at hand

Gates are seeded uniform one-qubit Cliffords with T gates at a tenth of the
sites (Haar-random two- and one-qubit gates for bond4); output bitstrings are
uniform.
"""
import math

import numpy as np
import torch

from paper_2608_13110_amd import (STORE_BF16_BLOCKSCALE, STORE_C64, STORE_F16_BLOCKSCALE, Plan, RingPlan, Server,
                                  frugal_accept, logxeb, sample_batched)

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
STORAGE = {"c64": STORE_C64, "f16": STORE_F16_BLOCKSCALE, "bf16": STORE_BF16_BLOCKSCALE}
# Plan options: none (what Plan.from_circuit takes by itself) and the sets that
# the autotuner picks for wide boundary tensors.
TILES = {
    "default": None,
    "tile12": {"max_tile_bits": 12, "math": 2},
    "fused": {"reg_bits": 4, "math": 2},
    "fused13": {"max_tile_bits": 13, "low_bits": 5, "reg_bits": 4, "math": 2},
}


def _chain(name, n, d, k, batches, tiles="default", storage="c64"):
    return dict(name=name, kind="chain", n=n, d=d, k=k, batches=batches, tiles=tiles, storage=storage)


def listed():
    return [
        # every amplitude of a 12-qubit circuit: 512 batches of 8, launches and latency
        _chain("tiny all amplitudes", 12, 12, 3, 512),
        # one amplitude of a small circuit, the shortest call a program makes
        _chain("one amplitude w=10", 24, 20, 0, 1),
        # one mid-size request, odd depth (the top slot of the boundary comes and goes)
        _chain("one request w=17 odd", 41, 33, 5, 1),
        # a verification job: 64 prefixes of a 40-qubit circuit
        _chain("medium w=20 x64", 40, 40, 6, 64),
        # the widest request of the serving stream
        _chain("one request w=24", 56, 48, 8, 1),
        # the precision study (w = 28), with the options the autotuner picks there
        _chain("precision w=28", 70, 56, 8, 1, "fused"),
        # a production-size contraction, two binary orders below full width
        _chain("wide w=31", 70, 62, 8, 1, "fused13"),
        # block-scaled 16-bit storage of the boundary tensor
        _chain("f16 w=26", 70, 52, 8, 2, "fused", "f16"),
        # generic two-qubit gates, bond dimension four
        dict(name="bond4 w=25", kind="bond4", n=26, d=26, batches=1, tiles="fused13"),
        # a ring cut into 1024 open chains
        dict(name="ring n=20", kind="ring", n=20, d=20, k=4, batches=1),
        # a burst of requests of mixed shape into the serving loop
        dict(name="serve burst of 24", kind="serve", requests=24, n_low=24, n_high=56, d_low=20, d_high=48),
        # estimator and samplers over the amplitudes of 2051 measured prefixes
        dict(name="post 2051 x 256", kind="post", n=70, k=8, batches=2051),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    kind = rng.choice(["chain"] * 6 + ["bond4", "ring", "serve", "post"])
    if kind == "bond4":
        n = rng.randrange(8, 27, 2)
        return dict(kind=kind, n=n + rng.randrange(0, 3), d=n, batches=rng.randrange(1, 4),
                    tiles=rng.choice(["default", "fused13"]))
    if kind == "ring":
        n = rng.randrange(8, 21, 2)
        return dict(kind=kind, n=n, d=n, k=rng.randrange(0, 5), batches=rng.randrange(1, 4))
    if kind == "serve":
        return dict(kind=kind, requests=rng.randrange(6, 33), n_low=24, n_high=rng.randrange(30, 57), d_low=20,
                    d_high=rng.randrange(24, 49, 2))
    if kind == "post":
        return dict(kind=kind, n=rng.randrange(12, 71), k=rng.randrange(0, 11), batches=_log_uniform(rng, 1, 4096))
    d = rng.randrange(8, 61)
    w = (d + 1) // 2
    n = rng.randrange(max(8, w), 71)
    k = rng.randrange(0, min(8, d // 4) + 1)
    # together no larger than one batch of 2^30 entries
    batches = _log_uniform(rng, 1, max(1, min(1024, 1 << max(0, 30 - w - k // 2))))
    tiles = rng.choice(["default", "tile12", "fused", "fused13"])
    return dict(kind="chain", n=n, d=d, k=k, batches=batches, tiles=tiles,
                storage=rng.choice(["c64", "c64", "c64", "f16", "bf16"]))


# ---------------------------------------------------------------- inputs
class Circuit:
    """Gate lists as Plan.from_circuit and Server.submit take them."""

    def __init__(self, n, d, one_qubit, gates):
        self.n, self.d, self.one_qubit, self.gates = n, d, one_qubit, gates


def _cliffords():
    """The 24 one-qubit Cliffords, first nonzero entry real and positive."""
    gen = [np.array([[1, 1], [1, -1]]) / math.sqrt(2.0), np.array([[1, 0], [0, 1j]])]
    found = [np.eye(2, dtype=np.complex128)]
    for m in found:
        for g in gen:
            u = g @ m
            lead = u.flat[0] if abs(u.flat[0]) > 1e-9 else u.flat[1]
            u = u * (abs(lead) / lead)
            if not any(np.allclose(u, v) for v in found):
                found.append(u)
    return np.stack(found)


CLIFFORDS = _cliffords()
T_GATE = np.diag([1.0, np.exp(0.25j * math.pi)])


def _pairs(n, layer):
    return range(layer % 2, n - 1, 2)


def _haar(rng, shape, dim):
    z = rng.standard_normal(shape + (dim, dim)) + 1j * rng.standard_normal(shape + (dim, dim))
    q, r = np.linalg.qr(z)
    diag = np.diagonal(r, axis1=-2, axis2=-1)
    return q * (diag / np.abs(diag))[..., None, :]


def _circuit(rng, kind, n, d):
    if kind == "bond4":
        gates = [(layer, q, 1, _haar(rng, (), 4)) for layer in range(1, d + 1) for q in _pairs(n, layer)]
        return Circuit(n, d, _haar(rng, (d + 1, n), 2), gates)
    one = CLIFFORDS[rng.integers(0, 24, size=(d + 1, n))]
    doped = rng.random((d + 1, n)) < 0.1
    one[doped] = T_GATE @ one[doped]
    gates = []
    for layer in range(1, d + 1):
        gates += [(layer, q, 0, None) for q in _pairs(n, layer)]
        if kind == "ring" and layer % 2 == 1:
            gates.append((layer, n - 1, 0, None))
    return Circuit(n, d, one, gates)


def _inputs(case, seed):
    """The circuit and the bitstrings of a case, on the host."""
    rng = np.random.default_rng([seed, case["n"], case["d"]])
    circ = _circuit(rng, case["kind"], case["n"], case["d"])
    return circ, rng.integers(0, 2, size=(case["batches"], case["n"]), dtype=np.uint8)


def _requests(case, seed):
    # the shapes are the case's, the gates and bitstrings the seed's
    shapes = np.random.default_rng([case["requests"], case["n_high"], case["d_high"]])
    rng = np.random.default_rng([seed, case["requests"]])
    found = []
    for _ in range(case["requests"]):
        n = int(shapes.integers(case["n_low"], case["n_high"] + 1))
        d = int(shapes.integers(case["d_low"] // 2, case["d_high"] // 2 + 1)) * 2
        k = int(shapes.integers(0, min(8, d // 4) + 1))
        found.append((_circuit(rng, "chain", n, d), rng.integers(0, 2, size=(1, n), dtype=np.uint8), k))
    return found


def _post_inputs(case, seed):
    """Amplitudes with Porter-Thomas probabilities, uniforms, and a component per batch."""
    rng = np.random.default_rng([seed, case["batches"], case["k"]])
    shape = (case["batches"], 1 << case["k"])
    amps = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)) * 2.0 ** (-(case["n"] + 1) / 2)
    return (amps, rng.random(shape[0]), rng.random(shape),
            rng.integers(0, shape[1], size=shape[0], dtype=np.int32))


def prepare(case, seed):
    if case["kind"] == "post":
        amps, u_batch, u_all, select = (torch.from_numpy(x).to(DEVICE) for x in _post_inputs(case, seed))
        return dict(case=case, amps=amps, u_batch=u_batch, u_all=u_all, select=select)
    if case["kind"] == "serve":
        server = Server(arena_bytes=4 << 30)
        return dict(case=case, server=server, requests=_requests(case, seed))
    circ, bits = _inputs(case, seed)
    k, nb = case.get("k", 0), case["batches"]
    bits = torch.from_numpy(bits).to(DEVICE)
    out = torch.empty((nb, 1 << k), dtype=torch.complex128, device=DEVICE)
    if case["kind"] == "ring":
        plan = RingPlan.from_circuit(circ)
        size = plan.info(k, nb)["workspace_bytes"]
        call = {}
    else:
        plan = Plan.from_circuit(circ, TILES[case["tiles"]])
        plan.prepare(k)
        call = {"storage": STORAGE[case.get("storage", "c64")]}
        size = plan.workspace_bytes(k, nb, call["storage"])
    work = torch.empty(size, dtype=torch.uint8, device=DEVICE)
    return dict(case=case, plan=plan, bits=bits, k=k, call=dict(call, out=out, workspace=work))


def run(state):
    kind = state["case"]["kind"]
    if kind == "post":
        amps, n, k = state["amps"], state["case"]["n"], state["case"]["k"]
        xeb_all = logxeb(amps, k, n)
        xeb_drawn = logxeb(amps, k, n, select=state["select"])
        suffix, marginal = sample_batched(amps, state["u_batch"])
        accept, z = frugal_accept(amps, n, 10.0, state["u_all"])
        return [xeb_all, xeb_drawn, suffix, marginal, accept, z]
    if kind == "serve":
        server = state["server"]
        ids = [server.submit(circ, bits, k) for circ, bits, k in state["requests"]]
        return [server.wait(i)[0] for i in ids]
    return state["plan"].amplitudes(state["bits"], state["k"], **state["call"])


def work(case):
    kind = case["kind"]
    if kind == "post":
        count = case["batches"] << case["k"]
        # amplitudes and uniforms in, acceptance and z out; |a|^2, a logarithm, the sums
        return {"bytes": count * (16 + 8 + 1 + 8), "flops": count * 30}
    if kind == "serve":
        n, d, k, batches = (case["n_low"] + case["n_high"]) // 2, case["d_high"], 4, 1
        batches = max(1, case["requests"] // 6)  # a sixth of the depths is near the widest, which decides
        w = d // 2
    else:
        n, d, k, batches = case["n"], case["d"], case.get("k", 0), case["batches"]
        w = (d + 1) // 2
    rows = n - 2 if k == 0 else n - k - 1
    gates = (d + 1) * n * 4 * 16
    flops = 14.0 * rows * w * batches * 2.0 ** w + 8.0 * batches * 2.0 ** (w + k)
    if kind == "bond4":
        w = min(n, d - 1)
        flops = 30.0 * (n - 2) * (w // 2) * batches * 2.0 ** w
    if kind == "ring":
        flops *= 2.0 ** (d // 2)
    return {"bytes": gates + batches * (n + (16 << k)), "flops": flops}


# ---------------------------------------------------------------- in 64 bits
def _state_vector(circ, ring=False):
    """U|0^n>, qubit j on axis j."""
    n = circ.n
    psi = torch.zeros([2] * n, dtype=torch.complex128, device=DEVICE)
    psi[(0,) * n] = 1.0
    by_layer = {}
    for layer, q, kind, m in circ.gates:
        by_layer.setdefault(layer, []).append((q, kind, m))
    for layer in range(circ.d + 1):
        for q, kind, m in by_layer.get(layer, ()):
            lo, hi = sorted((q, (q + 1) % n))
            if kind == 0:
                psi.select(hi, 1).select(lo, 1).neg_()
            else:
                x = psi.reshape(1 << q, 4, -1).movedim(1, 0).reshape(4, -1)
                x = torch.from_numpy(np.ascontiguousarray(m)).to(DEVICE) @ x
                psi = x.reshape(4, 1 << q, -1).movedim(0, 1).reshape([2] * n)
        for q in range(n):
            g = circ.one_qubit[layer, q]
            x = psi.reshape(1 << q, 2, -1)
            a, b = x[:, 0], x[:, 1]
            y = torch.empty_like(x)
            for o in range(2):
                y[:, o] = complex(g[o, 0]) * a + complex(g[o, 1]) * b
            psi = y.reshape([2] * n)
    return psi.reshape(-1)


def _crossings(circ, cut):
    """Layers whose CZ joins qubits (cut, cut + 1), in order."""
    return sorted(layer for layer, q, _, _ in circ.gates if q == cut)


def _contract(circ, bits, k):
    """<a, b|U|0^n> of a CZ chain for one bitstring's prefix a, row by row: the
    tensor over the worldline values at a cut's crossings (layer order, first
    crossing slowest)."""
    n, d = circ.n, circ.d
    one = circ.one_qubit
    t = torch.ones((1, 1), dtype=torch.complex128, device=DEVICE)  # [made, to come]
    for q in range(n - max(k, 0)):
        up = set(_crossings(circ, q - 1)) if q else set()
        down = set(_crossings(circ, q))
        v = torch.zeros((2, 1, t.numel()), dtype=torch.complex128, device=DEVICE)  # [value, made, to come]
        v[0, 0] = t.reshape(-1)
        for layer in range(d + 1):
            if layer in up:
                x = v.reshape(2, v.shape[1], 2, -1)
                v = torch.stack([x[0, :, 0] + x[0, :, 1], x[1, :, 0] - x[1, :, 1]])
            if layer in down:
                x = torch.zeros((2, v.shape[1], 2, v.shape[2]), dtype=v.dtype, device=DEVICE)
                x[0, :, 0] = v[0]
                x[1, :, 1] = v[1]
                v = x.reshape(2, -1, v.shape[2])
            g = one[layer, q]
            v = torch.stack([complex(g[o, 0]) * v[0] + complex(g[o, 1]) * v[1] for o in range(2)])
        t = v[int(bits[q])].reshape(1, -1)
    if k == 0:
        return t.reshape(1)
    # the band: 2^k states, the crossings' values still to come on the last axis;
    # the last crossings in slices, so that a slice fits
    cut = _crossings(circ, n - k - 1)
    keep = max(0, len(cut) + k - 26)
    parts = t.reshape(-1, 1 << keep)
    ends = cut[len(cut) - keep:]
    done = []
    for i in range(1 << keep):
        done.append(_band(circ, k, parts[:, i].reshape(1, -1), cut[: len(cut) - keep],
                          {layer: (i >> (keep - 1 - j)) & 1 for j, layer in enumerate(ends)}))
    return sum(done)


def _band(circ, k, t, summed, fixed):
    n = circ.n
    s = torch.zeros((1 << k, t.numel()), dtype=torch.complex128, device=DEVICE)
    s[0] = t.reshape(-1)
    for layer in range(circ.d + 1):
        if layer in summed:
            x = s.reshape(2, (1 << k) // 2, 2, -1)
            s = torch.stack([x[0, :, 0] + x[0, :, 1], x[1, :, 0] - x[1, :, 1]]).reshape(1 << k, -1)
        elif fixed.get(layer):
            s[(1 << k) // 2:] *= -1.0
        for l2, q, _, _ in circ.gates:
            if l2 == layer and q >= n - k:
                s.reshape(1 << (q - n + k), 2, 2, -1)[:, 1, 1] *= -1.0
        for j in range(k):
            g = circ.one_qubit[layer, n - k + j]
            x = s.reshape(1 << j, 2, -1)
            s = torch.stack([complex(g[o, 0]) * x[:, 0] + complex(g[o, 1]) * x[:, 1] for o in range(2)], dim=1)
            s = s.reshape(1 << k, -1)
    return s.reshape(-1)


def _exact_amplitudes(kind, circ, bits, k):
    if kind != "chain" or circ.n <= 24:
        psi = _state_vector(circ)
        at = torch.from_numpy(bits.astype(np.int64) @ (1 << np.arange(circ.n - 1, -1, -1, dtype=np.int64))).to(DEVICE)
        return psi[((at >> k) << k)[:, None] + torch.arange(1 << k, device=DEVICE)[None]]
    return torch.stack([_contract(circ, b, k) for b in bits])


def exact(case, seed):
    kind = case["kind"]
    if kind == "post":
        amps, u_batch, u_all, select = _post_inputs(case, seed)
        p = amps.real ** 2 + amps.imag ** 2

        def xeb(x):
            lp = np.log(x.reshape(-1))
            mid = np.euler_gamma + case["n"] * math.log(2.0) + lp.mean()
            se = lp.std(ddof=1) / math.sqrt(lp.size) if lp.size > 1 else 0.0
            return np.array([mid, se, mid - 1.96 * se, mid + 1.96 * se, lp.size])

        return [xeb(p), xeb(p[np.arange(len(select)), select]), None, p.sum(axis=1), None, p * 2.0 ** case["n"]]
    if kind == "serve":
        return None  # a burst of two dozen circuits takes longer than a check may
    circ, bits = _inputs(case, seed)
    w = (case["d"] + 1) // 2
    if kind != "chain" and case["n"] > 26:
        return None
    if kind == "chain" and case["n"] > 24 and (w > 24 or case["n"] * w * w * case["batches"] * 2.0 ** max(0, w - 14) > 8e7):
        return None
    return _exact_amplitudes(kind, circ, bits, case.get("k", 0))
