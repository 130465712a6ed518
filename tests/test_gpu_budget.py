"""The adaptive budget on the GPU (dt_plan_set_adaptive_budget; CaDDTree's
stopping rule, section 2.5, in the conditional pop loop, section 3.4) against
the oracle's, through the C ABI.

Each case takes C_d = 1 and a convex C_v(n) = c n^2, c chosen on the oracle so
that the first tree stops inside the budget and every stop decision of every
tree is decisive (relative theta margins above 1e-4): the GPU tree must then
stop at the same node and match the oracle's as the fixed-budget trees do.
"""
import numpy as np
import pytest

import oracle
from gpu_util import DeviceWorkload, compare_tree, to_dev
from helpers import run_oracle
from paper_2607_08642_amd import binding, synth

pytestmark = pytest.mark.gpu
TOL = 1e-4


def first_stop(pis, c):
    """Stop of the greedy rule on a pop sequence of probabilities, C_d = 1, C_v = c n^2."""
    phi, theta = 0.0, 1.0
    for i, p in enumerate(pis):
        th = (1.0 + phi + p) / (1.0 + c * (i + 1) ** 2)
        if th <= theta:
            return i
        phi, theta = phi + p, th
    return len(pis)


def pick_costs(wl, kw, trees=None):
    """(C_d, C_v) with C_v(n) = c n^2: the first tree stops near the middle of the
    budget and every tree's stop decisions are decisive."""
    trees = range(wl.batch) if trees is None else trees
    full = run_oracle(wl, 0, **kw)
    n_full = full["n_nodes"]
    pis = np.exp(full["scores"][:n_full])
    grid = [c for c in np.geomspace(1e-5, 1.0, 80) if 0 < first_stop(pis, c) < n_full]
    grid.sort(key=lambda c: abs(first_stop(pis, c) - n_full / 2))
    for c in grid:
        costs = (1.0, [float(c) * n * n for n in range(wl.B + 1)])
        refs = [run_oracle(wl, t, budget_costs=costs, **kw) for t in trees]
        if all(min((v for k, v in r["gaps"] if k == "budget"), default=1.0) > 1e-4 for r in refs):
            return costs, refs
    raise AssertionError("no decisive cost model found")


def run_budget(wl, name, trees=None, tol=None, **kw):
    okw = {k: v for k, v in kw.items()}
    costs, refs = pick_costs(wl, okw, trees)
    print(f"[budget] {name} batch={wl.batch} B={wl.B} c={costs[1][1]:.3g} "
          f"stops={[r['n_nodes'] for r in refs]}", flush=True)
    dw = DeviceWorkload(wl, **kw)
    try:
        dw.plan.set_adaptive_budget(*costs)
        got = dw.run()
    finally:
        dw.close()
    out = []
    for t in (range(wl.batch) if trees is None else trees):
        out.append(compare_tree(wl, t, got, dict(dw.kw, budget_costs=costs), tol=tol,
                                name=f"budget-{name}"))
    assert int(got["n_nodes"][0]) < wl.B
    return out


CASES = [
    # (seed, batch, L, V, M, B, T, d_e, d_h, dtype, kw, extra)
    (2, 3, 6, 500, 16, 24, 0.7, 64, 64, synth.DT_F32, {}, dict(h0=True)),
    (5, 4, 8, 700, 32, 16, 0.0, 96, 64, synth.DT_BF16, dict(norm_mode=1), {}),
    (9, 3, 10, 2000, 64, 48, 0.8, 64, 64, synth.DT_BF16, dict(max_children=8), dict(h0=True)),
]


@pytest.mark.parametrize("scorer", [0, 1, 2], ids=["cond", "marg", "static"])
@pytest.mark.parametrize("case", CASES, ids=[f"s{c[0]}" for c in CASES])
def test_adaptive_budget_small(case, scorer):
    seed, batch, L, V, M, B, T, d_e, d_h, dt, kw, extra = case
    wl = synth.random_small(seed, batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=d_e, d_h=d_h,
                            dtype=dt, **extra)
    run_budget(wl, f"s{seed}-arm{scorer}", scorer=scorer, **kw)


def test_adaptive_budget_deep_qwen_shape():
    # one tree per call: the register-list expansion, one workgroup per CU
    run_budget(synth.deep(), "deep", tol=TOL)


def test_adaptive_budget_deep_concurrent_sampled():
    # 32 trees per call: the register-list expansion, two workgroups per CU
    run_budget(synth.deep_concurrent(), "deep_concurrent", trees=[0, 3, 11, 20, 31], tol=TOL)


def test_adaptive_budget_domino_head():
    wl = synth.random_small(32, batch=3, L=6, V=500, M=16, B=24, T=0.7, d_e=64, d_h=64, h0=True)
    wl.head = synth.domino_head(32, wl.weights.V, 96, wl.weights.d_h, 64, wl.weights.dtype)
    wl.H = synth.hidden_states(32, wl.batch, wl.L, 96, wl.weights.dtype)
    run_budget(wl, "head", scorer=oracle.SCORER_HEAD)


def test_adaptive_budget_off_again_and_errors():
    wl = synth.random_small(3, batch=2, L=5, V=1000, M=64, B=16, T=1.0, d_e=128, d_h=64,
                            dtype=synth.DT_BF16)
    dw = DeviceWorkload(wl)
    try:
        fixed = dw.run()
        dw.plan.set_adaptive_budget(1.0, [0.0] + [50.0] * wl.B)   # stops at 0 nodes
        empty = dw.run()
        assert (empty["n_nodes"] == 0).all() and (empty["tokens"] == -1).all()
        assert (empty["mask"] == 0).all()
        dw.plan.set_adaptive_budget(None)
        again = dw.run()
        for k in fixed:
            np.testing.assert_array_equal(fixed[k], again[k], err_msg=k)
        with pytest.raises(binding.DTError) as e:
            dw.plan.set_adaptive_budget(1.0, [0.0] * wl.B)          # B entries, B + 1 needed
        assert e.value.status == -2
        with pytest.raises(binding.DTError) as e:
            dw.plan.set_adaptive_budget(1.0, [0.0] * 5 + [-2.0] * (wl.B - 4))
        assert e.value.status == -2
    finally:
        dw.close()
