"""C ABI without a GPU: exported symbols, planner, orders, widths, error paths.

Nothing here launches a kernel; qtn_contract is only called on paths that
fail before any HIP call.
"""
import ctypes
import os
import re

import numpy as np
import pytest

import qaoa_synth as qs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    with open(os.path.join(ROOT, "include", "qtn.h")) as f:
        text = f.read()
    names = set(re.findall(r"\b(qtn_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol(qtn):
    from paper_2204_06045_amd import _capi
    lib = _capi.lib()
    names = _declared()
    assert len(names) >= 12
    for name in names:
        assert hasattr(lib, name), name
    assert set(names) == set(_capi.EXPORTS)


def test_free_functions_accept_null(qtn):
    from paper_2204_06045_amd import _capi
    lib = _capi.lib()
    lib.qtn_network_free(None)
    lib.qtn_costmodel_free(None)
    lib.qtn_bucket_free(None)


def test_minfill_matches_oracle_rule(qtn, orc):
    for n, d, p, seed in [(10, 3, 1, 0), (16, 3, 3, 2), (30, 3, 4, 0), (40, 4, 3, 1)]:
        inst = qs.instance(n, d, p, seed)
        g, b = inst["angles"][0]
        net = qtn.Network(n, inst["edges"], g, b)
        for eid in range(0, len(inst["edges"]), 7):
            assert np.array_equal(net.order_minfill(eid),
                                  orc.edge_order(n, inst["edges"], eid, p))
        net.close()


def test_bucket_widths_match_oracle_recount(qtn, orc):
    inst = qs.instance(16, 3, 3, 4)
    g, b = inst["angles"][0]
    net = qtn.Network(16, inst["edges"], g, b, max_levels=1)
    net.plan(qtn.QTN_C128)
    for eid in range(0, len(inst["edges"]), 5):
        _, w_or = orc.edge_zz(16, inst["edges"], eid, g, b, return_widths=True)
        order = orc.edge_order(16, inst["edges"], eid, 3)
        w_q = net.bucket_widths(eid)
        # oracle widths are indexed by elimination position as well
        assert np.array_equal(np.asarray(w_or), w_q), eid
        nv, nt, wmax = net.info(eid)
        assert wmax == max(w_q) and nv == len(order)
        assert nt == orc.lightcone_size(16, inst["edges"], eid, 3)[1]
    net.close()


def test_plan_stats_consistency(qtn):
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]
    plain = qtn.Network(30, inst["edges"], g, b, max_levels=1)
    plain.plan(qtn.QTN_C128)
    merged = qtn.Network(30, inst["edges"], g, b)
    merged.plan(qtn.QTN_C128)
    sp, sm = plain.stats(), merged.stats()
    assert sp["n_buckets"] == sm["n_buckets"] == sum(sp["width_hist"])
    assert sp["n_groups"] == sp["n_buckets"]
    assert sm["n_groups"] < sm["n_buckets"]
    # merging never widens a bucket and removes intermediate traffic (Sec. II-C)
    assert sm["max_width"] == sp["max_width"]
    assert sm["bytes"] < sp["bytes"] / 5
    assert abs(sp["flops"] - sm["flops"]) / sp["flops"] < 1e-12
    assert sm["workspace"] < sp["workspace"]
    plain.close()
    merged.close()


def test_c64_plan_halves_bytes(qtn):
    inst = qs.instance(20, 3, 3, 1)
    g, b = inst["angles"][0]
    n1 = qtn.Network(20, inst["edges"], g, b)
    n1.plan(qtn.QTN_C128)
    n2 = qtn.Network(20, inst["edges"], g, b)
    n2.plan(qtn.QTN_C64)
    assert abs(n2.stats()["bytes"] * 2 - n1.stats()["bytes"]) < 1e-6 * n1.stats()["bytes"]


def test_mixed_plan_bytes_between_c64_and_c128(qtn):
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]
    st = {}
    for name, prec, mw in [("c128", 0, 0), ("c64", 1, 0), ("mixed", 2, 16), ("mixed32", 2, 32)]:
        net = qtn.Network(30, inst["edges"], g, b, mixed_width=mw)
        net.plan(prec)
        st[name] = net.stats()
        net.close()
    assert st["c64"]["bytes"] < st["mixed"]["bytes"] < st["c128"]["bytes"]
    # no group is 32 wide: mixed keeps every group in complex128
    assert abs(st["mixed32"]["bytes"] - st["c128"]["bytes"]) < 1e-6 * st["c128"]["bytes"]
    with pytest.raises(qtn.QtnError):
        qtn.Network(30, inst["edges"], g, b, mixed_width=33)
    net = qtn.Network(30, inst["edges"], g, b)
    with pytest.raises(qtn.QtnError):
        net.plan(3)
    net.close()


def test_matrix_form_scheduling(qtn):
    """The matrix form runs only when requested (or tuned), for groups that
    split into two sides with at least 4 n bits: own launches in every
    precision, inside workgroups and the persistent executors only in
    complex64 (complex128 tiles need more LDS than those kernels hold)."""
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]
    counts = {}
    for prec in (0, 1, 2):
        for variant in (0, 3):
            for executor in (0, 2):
                net = qtn.Network(30, inst["edges"], g, b, variant=variant, mixed_width=16,
                                  executor=executor)
                net.plan(prec)
                counts[prec, variant, executor] = net.stats()["n_matrix"]
                net.close()
    assert all(counts[p, 0, e] == 0 for p in (0, 1, 2) for e in (0, 2))
    assert counts[0, 3, 0] > 0 and counts[1, 3, 0] > 0 and counts[2, 3, 0] > 0
    # the persistent executor: complex64 groups only
    assert counts[0, 3, 2] == 0 and counts[1, 3, 2] > 0
    assert counts[1, 3, 0] >= counts[2, 3, 2]


def test_cell_mapping_scheduling_rules(qtn):
    """The cell mapping is the rule for own-launch groups it fits; never inside
    workgroups or the persistent executors, nor when another mapping is
    requested; more cell bits need wider groups."""
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]

    def cells(**cfg):
        net = qtn.Network(30, inst["edges"], g, b, **cfg)
        net.plan(0)
        st = net.stats()
        net.close()
        return st["n_cell"], st["n_wide"]

    n_cell, n_wide = cells()
    assert 0 < n_cell <= n_wide
    assert cells(variant=4) == (n_cell, n_wide)
    assert cells(variant=1)[0] == 0 and cells(variant=2)[0] == 0
    assert cells(executor=2)[0] == 0 and cells(executor=4)[0] == 0
    assert cells(variant=4, lane_sum_bits=4)[0] <= cells(variant=4, lane_sum_bits=2)[0]
    # a workgroup holds every group of width <= small_width
    assert cells(small_width=32)[0] == 0


def test_operands_over_4gib_take_the_generic_mapping(qtn):
    """The streaming and cell mappings address within an operand with 32-bit
    byte offsets, so a group holding an operand above 4 GiB must run the
    generic mapping (64-bit element indices) whatever mapping is requested.
    A 5-regular graph of 22 vertices at p=3 plans to width 32; in complex128
    a few of its groups hold rank-29 operands (8 GiB)."""
    inst = qs.instance(22, 5, 3, 0)
    g, b = inst["angles"][0]

    def stats(prec, **cfg):
        net = qtn.Network(22, inst["edges"], g, b, order_trials=8, **cfg)
        net.plan(prec)
        st = net.stats()
        net.close()
        return st

    for variant in (0, 2, 4):
        st = stats(0, variant=variant)
        assert st["max_width"] >= 30
        assert st["n_over4g"] > 0
        assert st["n_over4g_generic"] == st["n_over4g"], variant
        # the other groups keep the requested mapping
        assert st["n_cell"] + st["n_stream"] > 0
    st = stats(1, variant=4)
    assert st["n_over4g_generic"] == st["n_over4g"]
    # complex64 halves the operand bytes: no more groups cross the limit
    assert st["n_over4g"] <= stats(0, variant=4)["n_over4g"]


def test_tune_angles_workspace_query(qtn):
    """Workspace of autotuning on angle batches: grows with the set count, at
    least the angle-batch workspace; bad set counts and unplanned networks
    are refused."""
    inst = qs.instance(20, 3, 3, 6)
    g, b = inst["angles"][0]
    net = qtn.Network(20, inst["edges"], g, b)
    with pytest.raises(qtn.QtnError):
        qtn.qtn_tune_angles_workspace(net.h, 4)
    net.plan(0)
    one = qtn.qtn_tune_angles_workspace(net.h, 1)
    four = qtn.qtn_tune_angles_workspace(net.h, 4)
    assert four >= net.angles_workspace(4) > one > 0
    for bad in (0, 1025):
        with pytest.raises(qtn.QtnError):
            qtn.qtn_tune_angles_workspace(net.h, bad)
    net.close()


def test_gradient_workspace_and_validation(qtn):
    """The gradient's workspace is that of 4p + 1 angle sets; argument errors
    are reported before any device work."""
    inst = qs.instance(12, 3, 2, 1)
    g, b = inst["angles"][0]
    net = qtn.Network(12, inst["edges"], g, b)
    with pytest.raises(qtn.QtnError):
        qtn.qtn_gradient_workspace(net.h)  # not planned
    net.plan(0)
    assert qtn.qtn_gradient_workspace(net.h) == net.angles_workspace(4 * 2 + 1)
    with pytest.raises(ValueError):
        qtn.qtn_energy_gradient(net.h, 2, [0.1], [0.2, 0.3], None, 1e-4)
    net.close()


@pytest.mark.parametrize("edges,msg", [
    ([(0, 0)], "self-loop"),
    ([(0, 1), (1, 0)], "repeated"),
    ([(0, 5)], "out of range"),
])
def test_bad_graphs_rejected(qtn, edges, msg):
    with pytest.raises(qtn.QtnError) as ei:
        qtn.Network(3, edges, [0.1], [0.2])
    assert ei.value.code == -1 and msg in str(ei.value)


def test_bad_angles_and_depth(qtn):
    with pytest.raises(qtn.QtnError):
        qtn.Network(3, [(0, 1)], [float("nan")], [0.2])
    with pytest.raises(qtn.QtnError):
        qtn.Network(3, [(0, 1)], [], [])


def test_bad_order_and_width_cap(qtn):
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]
    net = qtn.Network(30, inst["edges"], g, b)
    nv = net.info(0)[0]
    bad = [None] * len(inst["edges"])
    bad[0] = np.zeros(nv, dtype=np.int32)  # not a permutation
    with pytest.raises(qtn.QtnError) as ei:
        net.plan(qtn.QTN_C128, orders=bad)
    assert ei.value.code == -1
    capped = qtn.Network(30, inst["edges"], g, b, max_width=12)
    with pytest.raises(qtn.QtnError) as ei:
        capped.plan(qtn.QTN_C128)
    assert ei.value.code == -2
    net.close()
    capped.close()


def test_contract_errors_leave_outputs_untouched(qtn):
    from paper_2204_06045_amd import _capi
    lib = _capi.lib()
    inst = qs.instance(10, 3, 1, 0)
    g, b = inst["angles"][0]
    net = qtn.Network(10, inst["edges"], g, b)
    zz = np.full(15, 7.0)
    en = ctypes.c_double(7.0)
    pd = ctypes.POINTER(ctypes.c_double)
    # before qtn_plan
    rc = lib.qtn_contract(net.h, ctypes.c_void_p(256), 1 << 20, None,
                          zz.ctypes.data_as(pd), None, ctypes.byref(en))
    assert rc == -5
    need = net.plan(qtn.QTN_C128)
    # workspace too small
    rc = lib.qtn_contract(net.h, ctypes.c_void_p(256), 1024, None,
                          zz.ctypes.data_as(pd), None, ctypes.byref(en))
    assert rc == -3 and "workspace" in qtn.qtn_last_error()
    # NULL workspace
    rc = lib.qtn_contract(net.h, None, need, None, zz.ctypes.data_as(pd), None,
                          ctypes.byref(en))
    assert rc == -1
    assert np.all(zz == 7.0) and en.value == 7.0
    # autotuning needs the workspace qtn_plan reported
    rc = lib.qtn_autotune(net.h, ctypes.c_void_p(256), need - 1, None, None)
    assert rc == -3 and "autotun" in qtn.qtn_last_error()
    net.close()


def test_set_angles_validation(qtn):
    net = qtn.Network(4, [(0, 1), (1, 2), (2, 3)], [0.1, 0.2], [0.3, 0.4])
    net.set_angles([0.5, 0.6], [0.7, 0.8])
    with pytest.raises(qtn.QtnError):
        net.set_angles([float("inf"), 0.0], [0.0, 0.0])
    net.close()


def test_lightcone_sizes_match_oracle(qtn, orc):
    inst = qs.instance(40, 4, 3, 2)
    g, b = inst["angles"][0]
    net = qtn.Network(40, inst["edges"], g, b)
    for eid in range(0, len(inst["edges"]), 9):
        nv, nt, _ = net.info(eid)
        assert (nv, nt) == orc.lightcone_size(40, inst["edges"], eid, 3)
    net.close()


def test_costmodel_host_side_checks(qtn):
    from paper_2204_06045_amd import _capi
    assert _capi.MLP_PARAMS == 16 * 64 + 64 + 64 * 64 + 64 + 64 * _capi.MLP_OUT + _capi.MLP_OUT
    p = np.linspace(-0.1, 0.1, qtn.CostModel.n_params).astype(np.float32)
    cm = qtn.CostModel(p)
    assert np.array_equal(cm.params(), p)
    # shapes are checked before any device work
    with pytest.raises(ValueError):
        cm.train(np.zeros((5, 16)), np.zeros((5, 3)), 1, 1e-3)
    with pytest.raises(ValueError):
        cm.predict(np.zeros(17))
    with pytest.raises(ValueError):
        cm.grad(np.zeros((2, 16)), np.zeros((2, 3)), np.ones((2, 3)))
    with pytest.raises(ValueError):
        qtn.CostModel(p[:-1])
    cm.close()


def test_tune_picks_round_trip_and_validation(qtn):
    inst = qs.instance(20, 3, 3, 1)
    g, b = inst["angles"][0]
    net = qtn.Network(20, inst["edges"], g, b)
    net.plan(qtn.QTN_C64)
    picks = net.tune_picks()
    assert len(picks) == net.stats()["n_groups"]
    assert all(p[2:5] == (-1, -1, -1) for p in picks)
    # generic kernel for every group: accepted, read back, and the plan's
    # matrix-form count stays zero
    chosen = [(e, gi, 1, 1, 2, sh) for (e, gi, _, _, _, sh) in picks]
    net.set_tune_picks(chosen)
    assert net.tune_picks() == chosen
    # a pick for a different group is refused and changes nothing
    bad = list(chosen)
    bad[0] = bad[0][:5] + ((bad[0][5] + 1) % (1 << 32),)
    with pytest.raises(qtn.QtnError) as ei:
        net.set_tune_picks(bad)
    assert ei.value.code == -1 and "different group" in str(ei.value)
    with pytest.raises(qtn.QtnError):
        net.set_tune_picks([(999, 0, 1, 1, 2, 0)])
    assert net.tune_picks() == chosen
    # matrix form requested through picks on complex64 groups that have one
    mf = [(e, gi, 1, 3, 2, sh) for (e, gi, _, _, _, sh) in picks]
    net.set_tune_picks(mf)
    assert net.stats()["n_matrix"] > 0
    net.close()


def test_angle_batch_workspace_and_validation(qtn):
    from paper_2204_06045_amd import _capi
    inst = qs.instance(16, 3, 3, 2)
    g, b = inst["angles"][0]
    net = qtn.Network(16, inst["edges"], g, b)
    net.plan(qtn.QTN_C128)
    w1, w4, w8 = (net.angles_workspace(k) for k in (1, 4, 8))
    # one data copy per set on top of fixed descriptors
    assert w1 <= net.ws_bytes and w1 < w4 < w8
    assert abs((w8 - w4) - (w4 - w1) * 4 / 3) < 4096 * 8
    for bad in (0, 1025):
        with pytest.raises(qtn.QtnError) as ei:
            net.angles_workspace(bad)
        assert ei.value.code == -1
    lib = _capi.lib()
    pd = ctypes.POINTER(ctypes.c_double)
    gs = np.array([[0.1, 0.2, float("nan")]])
    bs = np.zeros((1, 3))
    en = np.full(1, 7.0)
    rc = lib.qtn_contract_angles(net.h, ctypes.c_void_p(256), 1 << 30, None, 1,
                                 gs.ctypes.data_as(pd), bs.ctypes.data_as(pd), None,
                                 en.ctypes.data_as(pd), None)
    assert rc == -1 and "finite" in qtn.qtn_last_error() and en[0] == 7.0
    net.close()


def test_batch_autotune_validation(qtn):
    """The batched-call schedule search refuses, before any device work, a
    NULL list and networks whose batch runs per-group launches or the
    dataflow executor (no lockstep steps to order)."""
    from paper_2204_06045_amd import _capi
    lib = _capi.lib()
    rc = lib.qtn_autotune_batch(None, 0, ctypes.c_void_p(256), 1 << 20, None, None)
    assert rc == -1
    inst = qs.instance(12, 3, 2, 1)
    g, b = inst["angles"][0]
    for executor in (1, 3, 4):
        net = qtn.Network(12, inst["edges"], g, b, executor=executor)
        net.plan(qtn.QTN_C128)
        arr = (ctypes.c_void_p * 1)(net.h)
        rc = lib.qtn_autotune_batch(arr, 1, ctypes.c_void_p(256), 1 << 30, None, None)
        assert rc == -5 and "lockstep" in qtn.qtn_last_error(), executor
        net.close()


def test_bucket_plan_shapes_and_validation(qtn):
    """Single-bucket plans (no launch): union order, widths, algorithmic
    bytes and flops, mapping choice, and every rejected input."""
    # abcd,bcdf->acf with 2-bit indices: 4 summed labels (b, d), 6 kept
    a, b, c, d, f = ([2 * i, 2 * i + 1] for i in range(5))
    bk = qtn.Bucket([b + d + a + c, b + d + c + f], a + c + f)
    info = bk.info()
    assert (info["w"], info["L"], info["n_ops"]) == (10, 4, 2)
    assert info["bytes"] == 16 * (2 ** 8 + 2 ** 8 + 2 ** 6)
    # level 0: 2^10 products (6 flops) and 2^9 adds (2); levels 1..3: adds only
    assert info["flops"] == 2 ** 10 * 6 + sum(2 ** (10 - l - 1) * 2 for l in range(4))
    assert info["data_bytes"] == 2 * 4096 + 1024 and info["workspace_bytes"] % 256 == 0
    bk.close()
    # a wide bucket takes the cell mapping under the width rule; forcing the
    # generic mapping is honoured
    ops = [list(range(0, 20)), [0, 1] + list(range(20, 26))]
    assert qtn.Bucket(ops, list(range(2, 26))).info()["variant"] == 3
    assert qtn.Bucket(ops, list(range(2, 26)), variant=1).info()["variant"] == 0
    # the matrix form only in complex64
    mm = [[0, 1, 2, 3, 4, 5, 6, 7], [0, 1, 2, 8, 9, 10, 11]]
    for prec in (qtn.QTN_C64, qtn.QTN_C128):
        assert qtn.Bucket(mm, list(range(3, 12)), precision=prec, variant=3).info()["variant"] == 2
    # fewer than 4 kept labels private to the smaller side: no matrix form
    mm3 = [[0, 1, 2, 3, 4, 5], [0, 1, 2, 6, 7, 8]]
    assert qtn.Bucket(mm3, [3, 4, 5, 6, 7, 8], precision=qtn.QTN_C64, variant=3).info()["variant"] != 2
    bad = [
        (([[0, 1]], [0, 1]), "no summed"),            # nothing summed
        (([[0, 1, 2], [1, 2, 3]], [0, 3]), "union order"),
        (([[0, 0]], []), "union order"),              # repeated label
        (([[0, 1]], [2]), "no operand"),
        (([[0, 1]], [1, 1]), "repeated output"),
        (([list(range(9)) + [9]], [9]), "8 summed"),
        (([list(range(33))], list(range(1, 33))), "rank"),
    ]
    for (ops, out), msg in bad:
        with pytest.raises(qtn.QtnError) as ei:
            qtn.Bucket(ops, out)
        assert msg in str(ei.value), (ops, out, str(ei.value))
    with pytest.raises(qtn.QtnError, match="overlaps"):
        qtn.Bucket([[0, 1], [0, 2]], [1, 2], offsets=[0, 256], out_offset=256)
    with pytest.raises(qtn.QtnError, match="aligned"):
        qtn.Bucket([[0, 1], [0, 2]], [1, 2], offsets=[8, 512], out_offset=1024)
    with pytest.raises(qtn.QtnError, match="precision"):
        qtn.Bucket([[0, 1]], [1], precision=qtn.QTN_MIXED)


@pytest.mark.parametrize("cap,trials", [(24, 0), (22, 16), (10, 0)])
def test_slice_plan(qtn, cap, trials):
    """Index slicing: every light cone wider than the cap is planned with
    variables fixed; its widest bucket then fits the cap, the fixed
    variables are distinct and leave empty buckets, and the slice count and
    the per-evaluation bytes cover every slice."""
    n, p = (30, 4) if cap > 10 else (14, 3)
    inst = qs.instance(n, 3, p, 0)
    g, b = inst["angles"][0]
    plain = qtn.Network(n, inst["edges"], g, b, order_trials=trials)
    plain.plan(0)
    net = qtn.Network(n, inst["edges"], g, b, order_trials=trials, slice_width=cap)
    net.plan(0)
    st, st0 = net.stats(), plain.stats()
    assert st0["max_width"] > cap and st["max_width"] <= cap
    n_sliced, n_slices = 0, 0
    for e in range(len(inst["edges"])):
        sv = list(net.slice_vars(e))
        nv, _, _ = net.info(e)
        assert len(set(sv)) == len(sv) <= 10 and all(0 <= v < nv for v in sv)
        widths = net.bucket_widths(e)
        order = list(net.plan_order(e))
        for v in sv:
            assert widths[order.index(v)] == 0  # a fixed variable has no bucket
        if sv:
            n_sliced += 1
            assert max(plain.bucket_widths(e)) > cap or trials > 0
        n_slices += 1 << len(sv)
    assert st["n_sliced"] == n_sliced > 0 and st["n_slices"] == n_slices
    assert st["workspace"] < st0["workspace"]
    net.close()
    plain.close()


def test_slice_width_validation(qtn):
    # a cap below what fixing variables can reach is met as far as it can be
    inst = qs.instance(14, 3, 3, 0)
    net = qtn.Network(14, inst["edges"], *inst["angles"][0], slice_width=4)
    net.plan(0)
    st = net.stats()
    assert 4 < st["max_width"] and st["n_sliced"] > 0
    net.close()
    inst = qs.instance(10, 3, 1, 0)
    with pytest.raises(qtn.QtnError):
        qtn.Network(10, inst["edges"], *inst["angles"][0], slice_width=33)
    net = qtn.Network(10, inst["edges"], *inst["angles"][0], slice_width=30)
    net.plan(0)
    assert net.stats()["n_sliced"] == 0 and net.stats()["n_slices"] == len(inst["edges"])
    net.close()


@pytest.mark.parametrize("cap", [0, 24])
def test_order_search_by_plan_cost(qtn, cap):
    """Orders picked by the merged plan's flops + w * bytes: among the same
    candidate orders, the plan cost is never above that of the order with
    the smallest sum of 2^width (per light cone, so also in total)."""
    inst = qs.instance(30, 3, 4, 0)
    g, b = inst["angles"][0]
    st = {}
    for w in (0, 4):
        net = qtn.Network(30, inst["edges"], g, b, order_trials=16, slice_width=cap,
                          order_weight=w)
        net.plan(0)
        st[w] = net.stats()
        net.close()
    if cap == 0:
        assert st[4]["flops"] + 4 * st[4]["bytes"] <= st[0]["flops"] + 4 * st[0]["bytes"]
    assert st[4]["max_width"] <= max(st[0]["max_width"], cap or 32)
    with pytest.raises(qtn.QtnError):
        qtn.Network(30, inst["edges"], g, b, order_weight=-1)


@pytest.mark.parametrize("prec", [1, 2])
def test_gradient_schedule_in_plan_order_has_no_steps(qtn, prec):
    # step launches have no form in the plan's order, so that a gradient's
    # schedule in complex64 is the same with them (executor 0) and without (1)
    inst = qs.instance(20, 3, 3, 0)
    g, b = (np.array(a) for a in inst["angles"][0])
    need = []
    for executor in (0, 1):
        net = qtn.Network(20, inst["edges"], g, b, executor=executor, small_width=8, mixed_width=10)
        net.plan(prec)
        need.append(_gradient_bytes(qtn, net, g, b))
        net.close()
    assert need[0] == need[1]


def _bytes_needed(qtn, net, call, *args):
    """The bytes of a call, refused for its size before anything is queued."""
    assert call(net.h, ctypes.c_void_p(256), 1, None, *args) == -3
    return int(re.search(r"plan needs (\d+)", qtn.qtn_last_error())[1])


def _gradient_bytes(qtn, net, g, b):
    from paper_2204_06045_amd import _capi
    pd = ctypes.POINTER(ctypes.c_double)
    out = [np.zeros(net.p) for _ in range(3)]
    g, b, *out = [x.ctypes.data_as(pd) for x in (g, b, *out)]
    return _bytes_needed(qtn, net, _capi.lib().qtn_energy_gradient, g, b, 1e-4, *out)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n,d,p", [(24, 4, 2), (16, 3, 3), (10, 3, 1)])
def test_workspace_of_more_sets_serves_a_gradient(qtn, n, d, p, prec):
    """A workspace of as many angle sets as a gradient takes, or more, serves
    the gradient, and the gradient's serves as many sets."""
    from paper_2204_06045_amd import _capi
    inst = qs.instance(n, d, p, 0)
    g, b = (np.array(a) for a in inst["angles"][0])
    net = qtn.Network(n, inst["edges"], g, b, mixed_width=10)
    net.plan(prec)
    sets = 4 * p + 1
    enough = [net.angles_workspace(sets + k) for k in range(4)]
    gradient = qtn.qtn_gradient_workspace(net.h)
    need = _gradient_bytes(qtn, net, g, b)
    assert need <= gradient and need <= min(enough)
    pd = ctypes.POINTER(ctypes.c_double)
    zz, energy = np.zeros(sets * net.m), np.zeros(sets)
    arrays = [x.ctypes.data_as(pd) for x in (np.tile(g, (sets, 1)), np.tile(b, (sets, 1)), zz, energy)]
    assert gradient >= _bytes_needed(qtn, net, _capi.lib().qtn_contract_angles, sets, *arrays, None)
    net.close()


@pytest.mark.parametrize("prec", [0, 1])
def test_cell_pick_without_cells_is_generic(qtn, prec):
    # persistent executors have no cell kernels: up to 20 bits a pick of cells
    # runs the generic mapping there, and it is cells in launches of their own
    inst = qs.instance(16, 3, 4, 0)
    g, b = inst["angles"][0]
    for executor in (0, 2):
        net = qtn.Network(16, inst["edges"], g, b, executor=executor)
        net.plan(prec)
        before = net.stats()
        assert before["max_width"] <= 20
        net.set_tune_picks([(e, k, pl, 4, 3, sh) for e, k, pl, _, _, sh in net.tune_picks()])
        after = net.stats()
        if executor == 0:
            assert after["n_cell"] == before["n_cell"] > 0
        else:
            assert before["n_stream"] > 0 and after["n_stream"] == after["n_cell"] == 0
        net.close()
