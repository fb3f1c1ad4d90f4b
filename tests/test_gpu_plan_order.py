"""Complex64 gradients and batches run in the plan's order of operations: their
results are the ones of the first kernels, bit for bit.

golden/plan_order_c64.json holds those results (hexadecimal floats) as the
library at commit 75c8b02 gave them, before any mapping reordered products or
sums.  Every other order of operations changes nearly all of them, since a
central difference with step 1e-4 multiplies roundings of 1e-7 by 5,000.
"""
import json
import os

import numpy as np
import pytest

import qaoa_synth as qs

pytestmark = pytest.mark.gpu

with open(os.path.join(os.path.dirname(__file__), "golden", "plan_order_c64.json")) as _f:
    GOLDEN = json.load(_f)


def _network(qtn, n, d, p, graph, **cfg):
    inst = qs.instance(n, d, p, graph, 1)
    g, b = (np.array(x) for x in inst["angles"][0])
    net = qtn.Network(n, inst["edges"], g, b, **cfg)
    net.plan(qtn.QTN_C64)
    return net, g, b


@pytest.mark.parametrize("row", GOLDEN, ids=[json.dumps(r["call"]) for r in GOLDEN])
def test_bits_of_the_plan_order(qtn, gpu, row):
    want = np.array([float.fromhex(x) for x in row["values"]])
    kind, *call = row["call"]
    print(row["call"], flush=True)
    if kind == "gradient":
        n, d, p, graph, cfg = call
        net, g, b = _network(qtn, n, d, p, graph, **cfg)
        e, dg, db = net.energy_gradient(g, b, 1e-4)
        got = np.concatenate([[e], dg, db])
        nets = [net]
    else:
        executor, cfg = call
        nets = [_network(qtn, n, d, p, graph, executor=executor, **cfg)[0]
                for n, d, p, graph in [(10, 3, 1, 0), (14, 3, 3, 1), (16, 3, 2, 2), (12, 3, 4, 0)]]
        handles = [net.h for net in nets]
        ws = qtn.workspace(qtn.qtn_batch_workspace(handles))
        zz, energy = qtn.qtn_contract_batch(handles, sum(net.m for net in nets), ws)
        got = np.concatenate([energy, zz])
    assert np.array_equal(got, want)
    for net in nets:
        net.close()
