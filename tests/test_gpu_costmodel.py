"""Learned cost model on the GPU: forward, gradient and Adam against the FP64
oracle; training; the trained selector against the width-rule fallback."""
import math

import numpy as np
import pytest

import qaoa_synth as qs

pytestmark = pytest.mark.gpu


def _rand_params(seed, scale=0.2):
    r = qs.Rng(seed)
    n = 5508
    # uniform in [-scale, scale) from the shared seeded generator
    return np.array([scale * (2 * r.uniform() - 1) for _ in range(n)], dtype=np.float32)


def test_forward_matches_oracle(qtn, orc, gpu):
    p = _rand_params(1)
    r = np.random.default_rng(2)
    x = r.standard_normal((300, 16)).astype(np.float32)
    cm = qtn.CostModel(p)
    y = cm.predict(x)
    ref = orc.mlp_forward(p.astype(np.float64), x.astype(np.float64))
    assert np.max(np.abs(y - ref)) <= 1e-4 * max(1.0, np.max(np.abs(ref)))
    cm.close()


def test_gradient_matches_oracle(qtn, orc, gpu):
    p = _rand_params(3)
    r = np.random.default_rng(4)
    x = r.standard_normal((257, 16)).astype(np.float32)
    t = r.standard_normal((257, 4)).astype(np.float32)
    m = (r.random((257, 4)) > 0.2).astype(np.float32)
    cm = qtn.CostModel(p)
    loss, g = cm.grad(x, t, m)
    rl, rg = orc.mlp_loss_grad(p.astype(np.float64), x.astype(np.float64),
                               t.astype(np.float64), m.astype(np.float64))
    assert abs(loss - rl) <= 1e-4 * max(1.0, rl)
    assert np.max(np.abs(g - rg)) <= 1e-4 * max(1.0, np.max(np.abs(rg)))
    cm.close()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 33, 4097])
def test_gradient_matches_oracle_at_chunk_edges(qtn, orc, gpu, n):
    # 16 samples per chunk; one partial gradient below 30 samples, a block per
    # chunk above, more chunks than blocks at 4,097.  Every sum has at most
    # 2^13 terms of FP32 rounding 6e-8: relative errors stay under 1e-4.
    p = _rand_params(11)
    r = np.random.default_rng(n)
    x = r.standard_normal((n, 16)).astype(np.float32)
    t = r.standard_normal((n, 4)).astype(np.float32)
    m = (r.random((n, 4)) > 0.2).astype(np.float32)
    cm = qtn.CostModel(p)
    loss, g = cm.grad(x, t, m)
    y = cm.predict(x)
    rl, rg = orc.mlp_loss_grad(p.astype(np.float64), x.astype(np.float64),
                               t.astype(np.float64), m.astype(np.float64))
    ry = orc.mlp_forward(p.astype(np.float64), x.astype(np.float64))
    assert abs(loss - rl) <= 1e-4 * max(1.0, rl)
    assert np.max(np.abs(g - rg)) <= 1e-4 * max(1.0, np.max(np.abs(rg)))
    assert np.max(np.abs(y - ry)) <= 1e-4 * max(1.0, np.max(np.abs(ry)))
    cm.close()


def test_training_follows_oracle_steps(qtn, orc, gpu):
    # 70 epochs (the loss slots wrap at 64) in two calls against FP64 steps
    p = _rand_params(12)
    r = np.random.default_rng(13)
    x = r.standard_normal((40, 16)).astype(np.float32)
    ms = np.exp(r.standard_normal((40, 4)))
    ms[::7, 1] = -1.0
    cm = qtn.CostModel(p)
    hist = np.concatenate([cm.train(x, ms, 66, 1e-3), cm.train(x, ms, 4, 1e-3)])
    mu, inv = cm.normalization()
    xs = (x.astype(np.float64) - mu) * inv
    t, m = np.log(np.where(ms > 0, ms, 1.0)), (ms > 0).astype(np.float64)
    q, m1, m2 = p.astype(np.float64), np.zeros(len(p)), np.zeros(len(p))
    for k in range(70):
        rl, g = orc.mlp_loss_grad(q, xs, t, m)
        assert abs(hist[k] - rl) <= 1e-3 * max(1.0, rl)
        q, m1, m2 = orc.mlp_adam(q, m1, m2, g, k + 1, 1e-3)
    cm.close()


def test_adam_step_matches_oracle(qtn, orc, gpu):
    p = _rand_params(5)
    g = _rand_params(6, scale=1.0)
    cm = qtn.CostModel(p)
    cm.adam_step(g, 0.01)
    cm.adam_step(g * 0.5, 0.01)
    q, m1, m2 = orc.mlp_adam(p.astype(np.float64), np.zeros(len(p)), np.zeros(len(p)),
                             g.astype(np.float64), 1, 0.01)
    q, m1, m2 = orc.mlp_adam(q, m1, m2, (g * 0.5).astype(np.float64), 2, 0.01)
    assert np.max(np.abs(cm.params() - q)) <= 1e-5
    cm.close()


def test_training_reduces_loss(qtn, gpu):
    r = np.random.default_rng(7)
    x = r.uniform(0, 30, (2000, 16)).astype(np.float32)
    # a smooth synthetic timing law: log ms grows with feature 0 and 10
    ms = np.stack([np.exp(0.2 * x[:, 0] - 4), np.exp(0.1 * x[:, 10] - 3),
                   np.exp(0.05 * (x[:, 0] + x[:, 10]) - 3), np.exp(0.15 * x[:, 3] - 5)], 1)
    ms[::5, 0] = -1.0  # unmeasured entries
    ms[::3, 3] = -1.0
    cm = qtn.CostModel(_rand_params(8, 0.1))
    hist = cm.train(x, ms, 400, 3e-3)
    assert hist[-1] < 0.05 * hist[0]
    pred = cm.predict(x[:10])
    assert np.all(np.isfinite(pred))
    cm.close()


def test_costmodel_selection_keeps_parity(qtn, orc, gpu):
    inst = qs.instance(18, 3, 3, 2)
    g, b = inst["angles"][0]
    ref, ref_en = orc.energy(18, inst["edges"], g, b, threads=8)
    net = qtn.Network(18, inst["edges"], g, b)
    net.plan(0)
    net.autotune()
    feats, ms = net.tune_log()
    cm = qtn.CostModel(_rand_params(9, 0.1))
    cm.train(feats, ms, 300, 3e-3)
    counts = qtn.qtn_apply_costmodel(net.h, cm)
    assert counts.sum() == net.stats()["n_groups"]
    zz, zi, en = net.contract()
    assert np.max(np.abs(zz - ref.real)) <= 1e-10
    assert abs(en - ref_en) / abs(ref_en) <= 1e-10
    net.close()
    cm.close()


def _time_contract(net, ws, reps):
    import torch
    import time
    net.contract(ws)
    torch.cuda.synchronize()
    ts = []
    for _ in range(reps):
        t0 = time.perf_counter()
        net.contract(ws)
        torch.cuda.synchronize()
        ts.append(time.perf_counter() - t0)
    return float(np.median(ts))


def test_trained_selector_gains_over_width_rule(qtn, gpu):
    """What the trained network gains: trained on autotuner timings of nine
    networks, it picks each group's kernel on six held-out graphs (N in
    [100, 300], degree 3 and 4, p=3), and the evaluation is timed (median of
    repeats, the two selections interleaved per graph) against the width-rule
    fallback on the same plan.  The summed time ratio is printed; the learned
    selection must be at least 3% faster (the bench row measures it on 32
    held-out graphs)."""
    feats, times = [], []
    for it in qs.batch_instances(2204, 64, 20, 200, (2, 3, 4), d=3)[:8]:
        net = qtn.Network(it["n"], it["edges"], *it["angles"][0], order_trials=8)
        net.plan(1)
        net.autotune()
        f, m = net.tune_log()
        feats.append(f)
        times.append(m)
        net.close()
    it = qs.instance(30, 3, 4, 0)
    net = qtn.Network(30, it["edges"], *it["angles"][0], order_trials=16)
    net.plan(1)
    net.autotune()
    f, m = net.tune_log()
    feats.append(f)
    times.append(m)
    net.close()
    cm = qtn.CostModel(_rand_params(4242, 0.15))
    hist = cm.train(np.concatenate(feats), np.concatenate(times), 600, 3e-3)
    assert hist[-1] < hist[0]
    rr = qs.Rng(5100)
    fb_total = ln_total = 0.0
    gains = []
    for i in range(6):
        d = 3 if i % 2 == 0 else 4
        sizes = [n for n in range(100, 301) if (n * d) % 2 == 0]
        n = sizes[rr.below(len(sizes))]
        inst = qs.instance(n, d, 3, 7100 + i)
        fb = qtn.Network(n, inst["edges"], *inst["angles"][0], order_trials=4)
        fb.plan(1)
        ln = qtn.Network(n, inst["edges"], *inst["angles"][0], order_trials=4)
        ln.plan(1)
        qtn.qtn_apply_costmodel(ln.h, cm)
        wf, wl = fb.workspace(), ln.workspace()
        tf = tl = 0.0
        for _ in range(3):
            tf += _time_contract(fb, wf, 5)
            tl += _time_contract(ln, wl, 5)
        fb_total += tf
        ln_total += tl
        gains.append(tf / tl)
        fb.close()
        ln.close()
    cm.close()
    gain = fb_total / ln_total
    print(f"trained selector vs width rule on 6 held-out graphs: {gain:.3f}x "
          f"(per graph {', '.join(f'{g:.2f}' for g in gains)})", flush=True)
    assert gain >= 1.03
