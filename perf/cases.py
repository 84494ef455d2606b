"""The workloads whose speed is tracked: bootstrapped gates, circuits and
captured circuits at the library's evaluated parameter sets.

A case is a plain dict: `kind` says which entry point runs ("gates":
Context.bootstrap_gate, "noalloc": the same with the fixed scratch block,
"circuit": Context.eval_circuit, "graph": Context.circuit_graph and its
launch), `k` is the party count (Table 7 shape; k = 8 with the retuned key
noise) and the rest are the sizes.  Keys are generated and uploaded once per
party count, as a server keeps them; inputs are encryptions of seeded bits.
"""
import functools
import math

import numpy as np
import torch

import mk_inputs as mi
import paper_2205_05825_amd as mk

# Table 7 shape; gadget base 2^8 with 3 digits, key-switching base 2^2 with 8.
SHAPE = dict(n=560, N=1024, bk_ell=3, ks_t=8, lwe_noise_log2=15)
NOISE = {2: (30, 15), 4: (30, 15), 8: (31, 16)}
OPS = {"add": mk.OP_ADD, "sub": mk.OP_SUB, "mul": mk.OP_MUL}


def listed():
    return [
        # one gate of an interactive program: latency only
        dict(name="one_gate", kind="gates", k=2, count=1),
        # a level of the 16-bit divider on one or two pairs: narrow and ragged
        dict(name="narrow_level", kind="gates", k=2, count=33),
        # a level of a small circuit on some dozens of pairs
        dict(name="medium_level", kind="gates", k=2, count=201),
        # a serving loop that may not allocate device memory
        dict(name="serving_loop", kind="noalloc", k=2, count=500),
        # the headline batch: 1024 mixed gates, two parties
        dict(name="headline", kind="gates", k=2, count=1024),
        # a wide level (an operator's partial products over many pairs), ragged
        dict(name="wide_level", kind="gates", k=2, count=2600),
        # four parties (the 8-bit multiplier's setting), one level
        dict(name="four_parties", kind="gates", k=4, count=300),
        # eight parties (the largest party count of the regression runs)
        dict(name="eight_parties", kind="gates", k=8, count=64),
        # an operator evaluated level by level: 8-bit adder on 40 pairs
        dict(name="adder8", kind="circuit", k=2, op="add", bits=8, pairs=40),
        # a small operator replayed as a captured graph on new inputs
        dict(name="subtractor4_graph", kind="graph", k=2, op="sub", bits=4, pairs=12),
        # a four-party multiplier on a few pairs: few gates in most levels
        dict(name="multiplier4_four_parties", kind="circuit", k=4, op="mul", bits=4, pairs=5),
    ]


def _log_int(rng, lo, hi):
    return min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["gates", "gates", "gates", "gates", "noalloc", "circuit", "graph"])
    if kind == "gates":
        k = rng.choice([2, 2, 2, 4, 8])
        return dict(kind=kind, k=k, count=_log_int(rng, 1, {2: 2600, 4: 1000, 8: 300}[k]))
    if kind == "noalloc":
        return dict(kind=kind, k=2, count=_log_int(rng, 1, 990))
    k = rng.choice([2, 2, 4])
    op = rng.choice(["add", "sub", "mul"])
    bits = rng.randint(2, 4) if op == "mul" or k == 4 else rng.randint(2, 8)
    return dict(kind=kind, k=k, op=op, bits=bits, pairs=_log_int(rng, 1, 8 if op == "mul" or k == 4 else 40))


@functools.lru_cache(maxsize=None)
def _context(k):
    """The parties' keys, generated once and uploaded to the GPU."""
    bk_noise, ks_noise = NOISE[k]
    ctx = mk.Context(mk.Params(k=k, bk_noise_log2=bk_noise, ks_noise_log2=ks_noise, **SHAPE), 11)
    for party in range(k):
        ctx.keygen(party, 1000 + party)
    ctx.upload()
    return ctx


def _to_gpu(words):
    return torch.from_numpy(np.ascontiguousarray(words).view(np.int32)).to("cuda:0")


def prepare(case, seed):
    k = case["k"]
    ctx = _context(k)
    if case["kind"] in ("gates", "noalloc"):
        # mixed gate types and uniform bits, the operands from the first and the last party
        types, m1, m2 = mi.gate_batch(case["count"], seed=seed)
        a = _to_gpu(ctx.encrypt(0, m1, seed=2 * seed))
        b = _to_gpu(ctx.encrypt(k - 1, m2, seed=2 * seed + 1))
        return dict(kind=case["kind"], ctx=ctx, types=torch.from_numpy(types).to("cuda:0"), a=a, b=b,
                    out=torch.zeros_like(a))
    bits, pairs = case["bits"], case["pairs"]
    circuit = mk.build_operator(OPS[case["op"]], bits)
    x, y = mi.operand_pairs(pairs, bits, seed=seed)
    rows = [ctx.encrypt(0, col, seed=100 * seed + i) for i, col in enumerate(mi.to_bits(x, bits).T)]
    rows += [ctx.encrypt(k - 1, col, seed=100 * seed + 50 + i) for i, col in enumerate(mi.to_bits(y, bits).T)]
    inp = _to_gpu(np.stack(rows))
    out = torch.zeros((len(circuit.outputs), pairs, inp.shape[2]), dtype=torch.int32, device="cuda:0")
    state = dict(kind=case["kind"], ctx=ctx, circuit=circuit, inp=inp, out=out)
    if case["kind"] == "graph":
        state["graph"] = ctx.circuit_graph(circuit, inp, out)
    return state


def run(state):
    ctx = state["ctx"]
    if state["kind"] == "gates":
        ctx.bootstrap_gate(state["types"], state["a"], state["b"], state["out"])
    elif state["kind"] == "noalloc":
        ctx.bootstrap_gate(state["types"], state["a"], state["b"], state["out"], noalloc=True)
    elif state["kind"] == "circuit":
        ctx.eval_circuit(state["circuit"], state["inp"], state["out"])
    else:
        state["graph"].launch()
    return state["out"]


def work(case):
    """Bytes: the evaluation and key-switching keys once, inputs and outputs
    once.  Operations: per gate and CMux step of party i, with L = min(k+1,
    i+2) live accumulator polynomials, (L+1) ell forward and L+1 inverse real
    negacyclic transforms of N points (one complex transform of N/2 points
    each, 5 (N/2) log2(N/2) operations) and (2 L + 2) ell products of
    transforms (8 operations per complex point); per gate the key switch's
    row additions."""
    k, n, N, ell, t = case["k"], SHAPE["n"], SHAPE["N"], SHAPE["bk_ell"], SHAPE["ks_t"]
    h = N // 2
    transform, product = 5 * h * math.log2(h), 8 * h
    per_gate = 0
    for party in range(k):
        live = min(k + 1, party + 2)
        per_gate += n * (((live + 1) * ell + live + 1) * transform + (2 * live + 2) * ell * product)
    per_gate += k * N * t * 0.75 * (n + 1)
    row = 4 * (k * n + 1)
    if "op" in case:
        circuit = mk.build_operator(OPS[case["op"]], case["bits"])
        gates = mk.circuit_stats(circuit)[1] * case["pairs"]
        rows = (len(circuit.inputs) + len(circuit.outputs)) * case["pairs"]
    else:
        gates, rows = case["count"], 3 * case["count"]
    keys = 4 * ((k * n * 3 * ell + (k + 1) * ell) * N + k * N * t * 3 * (n + 1))
    return {"bytes": keys + rows * row, "flops": gates * per_gate}


def exact(case, seed):
    """The outputs are ciphertext words (whole numbers): no 64-bit value."""
    return None
