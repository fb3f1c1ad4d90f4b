"""The calls that a user of this framework makes, as timed cases.

Kinds of case:

  energy    qtn.Network.contract: one (gamma, beta) per call, as an outer
            optimiser that works point by point does
  angles    Network.contract_angles: many angle sets of one graph in one pass,
            the shape of a parameter scan and of the headline benchmark
  gradient  Network.energy_gradient: the energy and its derivatives
  batch     qtn_contract_batch: many graphs in one call, one angle set each
  bucket    Bucket.contract: one bucket of caller-given tensors
  train     CostModel.train: the learned kernel selector fitted to timings

A case names its graph (vertices, degree, depth, graph seed) or its index
sets, and the plan options; the seed of prepare() draws the angles, tensor
entries or timings.  Networks run by the planner's own rule: stored or
autotuned kernel choices exist for one graph only, and a new graph has none.

Complex64 and mixed networks hand their results over in single precision
(the accuracy they are computed to); the library returns them widened.
"""

from __future__ import annotations

import math

import numpy as np
import torch

import paper_2204_06045_amd as qtn
import qaoa_synth as qs

PRECISION = {"c128": qtn.QTN_C128, "c64": qtn.QTN_C64, "mixed": qtn.QTN_MIXED}
REAL = {"c128": np.float64, "c64": np.float32, "mixed": np.float32}


def listed():
    return [
        # the smallest call: a depth-1 energy of a 10-vertex graph, where
        # launches, copies and the wait are all there is
        dict(name="energy_n10_p1_c128", kind="energy", n=10, d=3, p=1, graph=0, precision="c128",
             trials=0, weight=0, slice=0),
        # an ordinary single evaluation: narrow buckets in workgroups and a
        # few dozen wide ones in launches of their own
        dict(name="energy_n20_p3_c128", kind="energy", n=20, d=3, p=3, graph=0, precision="c128",
             trials=0, weight=0, slice=0),
        # a quartic graph of 40 vertices at depth 3 in mixed precision, with
        # the plan options that its widths (26 and up) call for
        dict(name="energy_n40_d4_p3_mixed", kind="energy", n=40, d=4, p=3, graph=0,
             precision="mixed", trials=64, weight=4, slice=26),
        # the headline workload: 32 angle sets of a 30-vertex cubic graph at
        # depth 4, complex128; the largest case
        dict(name="angles_n30_p4_x32_c128", kind="angles", n=30, d=3, p=4, graph=0,
             precision="c128", trials=64, weight=4, slice=24, sets=32),
        # the same scan in complex64
        dict(name="angles_n30_p4_x32_c64", kind="angles", n=30, d=3, p=4, graph=0,
             precision="c64", trials=64, weight=4, slice=24, sets=32),
        # a scan of a shallower network: nearly every bucket is narrow, and
        # an odd number of sets
        dict(name="angles_n22_p3_x27_c128", kind="angles", n=22, d=3, p=3, graph=1,
             precision="c128", trials=0, weight=0, slice=0, sets=27),
        # one step of a gradient ascent: 4p + 1 = 17 evaluations
        dict(name="gradient_n16_p4_c128", kind="gradient", n=16, d=3, p=4, graph=1,
             precision="c128", trials=8, weight=4, slice=0),
        # a training set of graphs: cubic, 20 to 200 vertices, depths 2 to 4,
        # one persistent call (the batched benchmark's recipe, a quarter of
        # its graphs)
        dict(name="batch_16_cubic_c64", kind="batch", count=16, n_lo=20, n_hi=200, p_lo=2, p_hi=4,
             graph=2204, precision="c64", trials=8, weight=4, slice=0, hybrid=24),
        # single buckets: a matrix product on the matrix cores, the fixed
        # abcd,bcdf->acf contraction with every index of size 16, and a
        # merged bucket of the form that dominates the depth-4 networks
        # (8 summed indices, three large operands, the rest gates)
        dict(name="bucket_matmul_c128", kind="bucket", form="matmul", m=11, n=12, k=8, graph=0,
             precision="c128", variant=3),
        dict(name="bucket_fixed_n16_c64", kind="bucket", form="fixed", m=4, n=4, k=4, graph=0,
             precision="c64", variant=0),
        dict(name="bucket_merged_w23_c128", kind="bucket", form="merged", m=3, n=23, k=8, graph=5,
             precision="c128", variant=0),
        # the selector fitted to an autotuner's log
        dict(name="train_4000x60", kind="train", samples=4000, epochs=60),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["energy", "energy", "angles", "angles", "gradient", "batch", "bucket",
                       "bucket", "train"])
    graph = rng.randrange(1, 1000)
    precision = rng.choice(["c128", "c128", "c64", "mixed"])
    if kind in ("energy", "angles", "gradient"):
        d = rng.choice([3, 3, 3, 4])
        p = rng.randint(1, 4 if d == 3 else 2)
        n = 2 * rng.randint(5, 15 if p < 4 else (9 if kind == "gradient" else 11))
        if kind == "energy" and p <= 3 and d == 3 and rng.random() < 0.3:
            n = 2 * _log(rng, 16, 100)
        deep = p == 4
        case = dict(kind=kind, n=n, d=d, p=p, graph=graph, precision=precision,
                    trials=8 if deep else 0, weight=4 if deep else 0, slice=24 if deep else 0)
        if kind == "angles":
            case["sets"] = _log(rng, 2, 12 if deep else 48)
        return case
    if kind == "batch":
        return dict(kind=kind, count=_log(rng, 3, 24), n_lo=10, n_hi=2 * rng.randint(10, 60), p_lo=1,
                    p_hi=rng.randint(2, 3), graph=graph, precision=rng.choice(["c64", "c128"]),
                    trials=0, weight=0, slice=0, hybrid=24)
    if kind == "bucket":
        form = rng.choice(["matmul", "fixed", "merged", "pair"])
        precision = rng.choice(["c128", "c64"])
        case = dict(kind=kind, form=form, graph=graph, precision=precision, variant=0)
        if form == "matmul":
            return dict(case, m=rng.randint(5, 11), n=rng.randint(4, 11), k=rng.randint(3, 8), variant=3)
        if form == "fixed":
            return dict(case, m=rng.randint(3, 5), n=rng.randint(3, 5), k=rng.randint(2, 4))
        if form == "merged":
            return dict(case, m=rng.randint(2, 4), n=rng.randint(13, 23), k=rng.randint(3, 8))
        return dict(case, m=2, n=rng.randint(14, 24), k=rng.randint(1, 8))
    return dict(kind="train", samples=_log(rng, 100, 4000), epochs=rng.randint(5, 60))


# ------------------------------------------------------------------ inputs


def _graphs(case):
    """[(vertices, edges, depth)] of a network case."""
    if case["kind"] != "batch":
        inst = qs.instance(case["n"], case["d"], case["p"], case["graph"], 1)
        return [(inst["n"], inst["edges"], inst["p"])]
    insts = qs.batch_instances(case["graph"], case["count"], case["n_lo"], case["n_hi"],
                               tuple(range(case["p_lo"], case["p_hi"] + 1)), d=3)
    return [(it["n"], it["edges"], it["p"]) for it in insts]


def _angles(seed, graphs, sets):
    """gamma ~ U[0, pi), beta ~ U[0, pi/2): [graph][set] pairs."""
    rng = np.random.default_rng(seed)
    return [(rng.uniform(0, np.pi, (sets, p)), rng.uniform(0, np.pi / 2, (sets, p)))
            for _, _, p in graphs]


def _network(case, graph, gamma, beta):
    more = {} if case["kind"] != "batch" else {"executor": 5, "hybrid_width": case["hybrid"]}
    n, edges, _ = graph
    net = qtn.Network(n, edges, gamma, beta, order_trials=case["trials"],
                      order_weight=case["weight"], slice_width=case["slice"], **more)
    net.plan(PRECISION[case["precision"]])
    return net


def _labels(case):
    """Operand label lists (summed labels first) and output labels."""
    m, n, k = case["m"], case["n"], case["k"]
    if case["form"] == "matmul":  # A[k, m] B[k, n], binary labels
        s, a, b = list(range(k)), list(range(k, k + m)), list(range(k + m, k + m + n))
        return [s + a, s + b], a + b
    if case["form"] == "fixed":  # abcd,bcdf->acf: b, d of k labels each are summed
        sizes, at, lab = [("b", k), ("d", k), ("a", m), ("c", n), ("f", n)], 0, {}
        for name, size in sizes:
            lab[name] = list(range(at, at + size))
            at += size
        return ([lab["b"] + lab["d"] + lab["a"] + lab["c"], lab["b"] + lab["d"] + lab["c"] + lab["f"]],
                lab["a"] + lab["c"] + lab["f"])
    # m large operands over n labels of which the first k are summed
    rng = qs.Rng(case["graph"])
    summed, kept = list(range(k)), list(range(k, n))
    ops = [[] for _ in range(m)]
    if case["form"] == "pair":  # every summed label in both, a kept one in one or both
        for x in kept:
            side = rng.below(3)
            for i in range(2):
                if side != 1 - i:
                    ops[i].append(x)
        return [summed + o for o in ops], kept
    # merged buckets: the i-th operand enters after some labels are summed,
    # most kept labels are shared, and gates of one or two labels join in
    for i, o in enumerate(ops):
        o.extend(summed[min(k - 1, i * rng.below(3)):])
    for x in kept:
        out = rng.below(m + 1)  # the operand that lacks the label, m: none
        for i in range(m):
            if i != out or m == 1:
                ops[i].append(x)
    for _ in range(4):
        a, b = rng.below(n), rng.below(n)
        ops.append(sorted({a, b}))
    return ops, kept


def _dtype(case):
    return torch.complex128 if case["precision"] == "c128" else torch.complex64


def _entries(case, seed, ops, device="cuda"):
    """Normal complex entries of every operand, scaled to keep sums near one."""
    gen = torch.Generator(device=device)
    gen.manual_seed(seed)
    scale = 2.0 ** (-0.5 * case["k"] * (2 if case["form"] == "fixed" else 1) / len(ops))
    return [scale * torch.randn(1 << len(o), dtype=_dtype(case), device=device, generator=gen)
            for o in ops]


def _timings(case, seed):
    """Shape features and times of the kind an autotuner's log holds: widths,
    counts and log sizes; about one time in five is not measured."""
    rng = np.random.default_rng(seed)
    n = case["samples"]
    w = rng.integers(4, 28, n)
    x = np.empty((n, 16), np.float32)
    x[:, 0] = w
    x[:, 1] = rng.integers(1, 9, n)
    x[:, 2] = rng.integers(2, 20, n)
    x[:, 3:] = rng.normal(0.5, 0.3, (n, 13)) * w[:, None]
    ms = np.exp(0.4 * (w[:, None] - 18) + rng.normal(0, 0.5, (n, 4))) * 0.05
    ms[rng.random((n, 4)) < 0.2] = -1.0
    params = np.concatenate([
        rng.normal(0, 16 ** -0.5, 16 * 64), np.zeros(64), rng.normal(0, 0.125, 64 * 64),
        np.zeros(64), rng.normal(0, 0.125, 64 * 4), np.zeros(4)]).astype(np.float32)
    return x, ms, params


def prepare(case, seed):
    kind = case["kind"]
    state = {"case": case}
    if kind == "train":
        state["x"], state["ms"], state["params"] = _timings(case, seed)
        return state
    if kind == "bucket":
        ops, out = _labels(case)
        b = qtn.Bucket(ops, out, precision=PRECISION[case["precision"]], variant=case["variant"])
        data = torch.zeros(b.info()["data_bytes"], dtype=torch.uint8, device="cuda")
        for off, v in zip(b.offsets, _entries(case, seed, ops)):
            data[off:off + v.numel() * v.element_size()] = v.view(torch.uint8)
        size = _dtype(case).itemsize << len(out)
        state.update(bucket=b, data=data,
                     out=data[b.out_offset:b.out_offset + size].view(_dtype(case)))
        b.workspace()
        return state
    graphs = _graphs(case)
    angles = _angles(seed, graphs, case.get("sets", 1))
    nets = [_network(case, gr, g[0], b[0]) for gr, (g, b) in zip(graphs, angles)]
    state.update(nets=nets, angles=angles)
    if kind == "batch":
        handles = [net.h for net in nets]
        state.update(handles=handles, ws=qtn.workspace(qtn.qtn_batch_workspace(handles)))
    elif kind == "energy":
        state["ws"] = nets[0].workspace()
    elif kind == "angles":
        state["ws"] = qtn.workspace(nets[0].angles_workspace(case["sets"]))
    else:
        state["ws"] = qtn.workspace(qtn.qtn_gradient_workspace(nets[0].h))
    return state


# -------------------------------------------------------------------- calls

STEP = 1e-4  # central-difference step of the gradient cases
LR = 3e-3    # learning rate of the training cases


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "bucket":
        state["bucket"].contract(state["data"])
        return state["out"]
    if kind == "train":
        model = qtn.CostModel(state["params"])
        loss = model.train(state["x"], state["ms"], case["epochs"], LR)
        params = model.params()
        model.close()
        return {"loss": loss, "params": params}
    real = REAL[case["precision"]]
    nets, angles, ws = state["nets"], state["angles"], state["ws"]
    if kind == "batch":
        zz, energy = qtn.qtn_contract_batch(state["handles"], sum(net.m for net in nets), ws)
        zz, at = zz.astype(real), np.cumsum([0] + [net.m for net in nets])
        return {"zz": [zz[a:b] for a, b in zip(at, at[1:])], "energy": energy.astype(real)}
    gamma, beta = angles[0]
    if kind == "angles":
        zz, energy = nets[0].contract_angles(gamma, beta, ws)
        return {"zz": zz.astype(real), "energy": energy.astype(real)}
    if kind == "gradient":
        e, dg, db = nets[0].energy_gradient(gamma[0], beta[0], STEP, ws)
        return {"energy": real(e), "dgamma": dg.astype(real), "dbeta": db.astype(real)}
    nets[0].set_angles(gamma[0], beta[0])
    zz, zz_imag, energy = nets[0].contract(ws)
    return {"zz": zz.astype(real), "energy": real(energy)}


# --------------------------------------------------------------------- work


def work(case):
    """Inputs read and outputs written once, and the arithmetic: for a
    network the complex operations of its merged plan (its intermediates are
    not counted as bytes), for a bucket those of the merged sum."""
    if case["kind"] == "train":
        n, weights = case["samples"], 16 * 64 + 64 * 64 + 64 * 4
        return {"bytes": 4.0 * n * 24 + 8 * 5508, "flops": 6.0 * weights * n * case["epochs"]}
    if case["kind"] == "bucket":
        ops, out = _labels(case)
        b = qtn.Bucket(ops, out, precision=PRECISION[case["precision"]], variant=case["variant"])
        info = b.info()
        return {"bytes": info["bytes"], "flops": info["flops"]}
    graphs = _graphs(case)
    sets = {"angles": case.get("sets", 1), "gradient": 4 * case.get("p", 0) + 1}.get(case["kind"], 1)
    flops = nbytes = 0.0
    for n, edges, p in graphs:
        net = _network(case, (n, edges, p), [0.1] * p, [0.1] * p)
        flops += sets * net.stats()["flops"]
        nbytes += sets * 8.0 * (2 * p + 2 * len(edges) + 1)
        net.close()
    return {"bytes": nbytes, "flops": flops}


# -------------------------------------------------------------------- exact

DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
MOST_QUBITS = 24


def _statevector_zz(n, edges, gamma, beta, pairs):
    """<Z_j Z_k> of the given pairs from the 2^n amplitudes of the QAOA state."""
    x = torch.arange(1 << n, device=DEVICE)
    cut = torch.zeros(1 << n, dtype=torch.float64, device=DEVICE)
    for j, k in edges:
        cut += ((x >> j) ^ (x >> k)) & 1
    psi = torch.full((1 << n,), 2.0 ** (-0.5 * n), dtype=torch.complex128, device=DEVICE)
    for g, b in zip(gamma, beta):
        psi = psi * torch.polar(torch.ones_like(cut), -float(g) * cut)
        c, s = math.cos(float(b)), math.sin(float(b))
        for q in range(n):
            v = psi.view(-1, 2, 1 << q)
            psi = (c * v - 1j * s * v.flip(1)).reshape(-1)
    prob = psi.real ** 2 + psi.imag ** 2
    # <Z_j Z_k> = sum over the amplitudes of prob (1 - 2 (x_j xor x_k))
    return [float((prob * (1 - 2 * (((x >> j) ^ (x >> k)) & 1))).sum()) for j, k in pairs]


def _balls(n, edges, p):
    """Per edge, the vertices within distance p of it (None where they are
    more than a state vector holds)."""
    near = [set() for _ in range(n)]
    for j, k in edges:
        near[j].add(k)
        near[k].add(j)
    out = []
    for j, k in edges:
        ball = {j, k}
        for _ in range(p):
            ball |= set().union(*(near[v] for v in ball))
        if len(ball) > 16:
            return None
        out.append((j, k, sorted(ball)))
    return out


def _exact_zz(n, edges, gamma, beta):
    """Every <Z_j Z_k> of one graph, or None where no state vector fits: the
    whole graph, or per edge the part within distance p of it."""
    if n <= MOST_QUBITS:
        return np.array(_statevector_zz(n, edges, gamma, beta, edges))
    balls = _balls(n, edges, len(gamma))
    if balls is None:
        return None
    zz = []
    for j, k, ball in balls:
        at = {v: i for i, v in enumerate(ball)}
        inner = [(at[a], at[b]) for a, b in edges if a in at and b in at]
        zz += _statevector_zz(len(ball), inner, gamma, beta, [(at[j], at[k])])
    return np.array(zz)


def _energy(zz):
    return 0.5 * len(zz) - 0.5 * math.fsum(zz)


def _exact_network(case, seed):
    graphs = _graphs(case)
    sets = case.get("sets", 1)
    angles = _angles(seed, graphs, sets)
    if case["kind"] == "batch":
        zz = [_exact_zz(n, e, g[0], b[0]) for (n, e, _), (g, b) in zip(graphs, angles)]
        whole = all(z is not None for z in zz)
        return {"zz": zz, "energy": np.array([_energy(z) for z in zz]) if whole else None}
    (n, edges, p), (gamma, beta) = graphs[0], angles[0]
    if case["kind"] == "gradient":
        def energy(k, h):
            a = np.concatenate([gamma[0], beta[0]])
            if k >= 0:
                a[k] += h
            return _energy(_exact_zz(n, edges, a[:p], a[p:]))
        if n > MOST_QUBITS:
            return None
        diff = np.array([(energy(k, STEP) - energy(k, -STEP)) / (2 * STEP) for k in range(2 * p)])
        return {"energy": np.float64(energy(-1, 0.0)), "dgamma": diff[:p], "dbeta": diff[p:]}
    zz = []
    for g, b in zip(gamma, beta):
        z = _exact_zz(n, edges, g, b)
        if z is None:
            return None
        zz.append(z)
    if case["kind"] == "energy":
        return {"zz": zz[0], "energy": np.float64(_energy(zz[0]))}
    return {"zz": np.array(zz), "energy": np.array([_energy(z) for z in zz])}


def _exact_bucket(case, seed):
    ops, out = _labels(case)
    values = [v.to(torch.complex128) for v in _entries(case, seed, ops, DEVICE)]
    summed = sorted({x for o in ops for x in o} - set(out))
    place = {x: i for i, x in enumerate(summed + out)}
    w, nsum = len(place), len(summed)
    chunk = min(w, 24)
    got = []
    for c in range(1 << (w - chunk)):
        union = (c << chunk) + torch.arange(1 << chunk, device=DEVICE)
        term = torch.ones(1 << chunk, dtype=torch.complex128, device=DEVICE)
        for o, v in zip(ops, values):
            index = torch.zeros_like(union)
            for j, x in enumerate(o):
                index |= ((union >> place[x]) & 1) << j
            term *= v[index]
        got.append(term.view(-1, 1 << nsum).sum(1))
    return torch.cat(got)


def _exact_train(case, seed):
    x, ms, params = _timings(case, seed)
    x = x.astype(np.float64)
    mean, var = x.mean(0), x.var(0)
    x = torch.from_numpy((x - mean) / np.maximum(1e-3, np.sqrt(var))).to(DEVICE)
    mask = torch.from_numpy(ms > 0).to(DEVICE)
    target = torch.from_numpy(np.log(np.where(ms > 0, ms, 1.0))).to(DEVICE)
    flat = torch.from_numpy(params.astype(np.float64)).to(DEVICE)
    m1, m2 = torch.zeros_like(flat), torch.zeros_like(flat)
    sizes = [(16, 64), (64,), (64, 64), (64,), (64, 4), (4,)]
    loss = []
    for step in range(1, case["epochs"] + 1):
        flat.requires_grad_(True)
        w1, b1, w2, b2, w3, b3 = (t.view(s) for t, s in zip(
            flat.split([math.prod(s) for s in sizes]), sizes))
        y = torch.relu(torch.relu(x @ w1 + b1) @ w2 + b2) @ w3 + b3
        value = (((y - target) ** 2) * mask).sum() / mask.sum()
        (grad,) = torch.autograd.grad(value, flat)
        flat = flat.detach()
        loss.append(float(value))
        m1 = 0.9 * m1 + 0.1 * grad
        m2 = 0.999 * m2 + 0.001 * grad ** 2
        flat = flat - LR * (m1 / (1 - 0.9 ** step)) / (torch.sqrt(m2 / (1 - 0.999 ** step)) + 1e-8)
    return {"loss": np.array(loss), "params": flat.cpu().numpy()}


def exact(case, seed):
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "bucket":
        return _exact_bucket(case, seed)
    return _exact_network(case, seed)
