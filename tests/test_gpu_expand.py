"""The general expansion kernel (menus or budgets over 64, wider states, more than 16 segment lists per
row) under every children function and option, against the oracle: the register-list expansion takes the
smaller shapes, so these sizes are the ones that reach it."""
import numpy as np
import pytest

from gpu_util import DeviceWorkload, compare_tree
from paper_2607_08642_amd import binding, synth
from test_gpu_budget import run_budget
from test_gpu_grow import check_siblings

pytestmark = pytest.mark.gpu
F, H = synth.DT_F32, synth.DT_BF16

# name, batch, L, V, M, B, T, d_h, weights, k, h0, norm
CASES = [
    ("budget_65", 3, 5, 900, 16, 65, 0.7, 64, F, 0, True, 0),
    ("budget_256", 2, 6, 700, 64, 256, 1.0, 64, H, 8, True, 0),
    ("menu_65", 2, 4, 800, 65, 16, 1.3, 96, F, 5, False, 1),
    ("menu_200", 2, 3, 23000, 200, 65, 1.0, 256, H, 0, True, 0),
    ("wide_state", 1, 4, 500, 32, 24, 0.7, 544, H, 0, True, 0),
    ("wide_state_f32", 2, 4, 500, 32, 24, 0.7, 288, F, 0, True, 1),
    ("many_lists", 1, 4, 200000, 32, 16, 1.0, 64, F, 0, True, 0),
    ("trees_over_cus", 300, 3, 300, 8, 66, 0.8, 32, F, 2, True, 0),
]


@pytest.mark.parametrize("scorer", [0, 1, 2], ids=["cond", "marg", "static"])
@pytest.mark.parametrize("c", CASES, ids=[c[0] for c in CASES])
def test_shapes(c, scorer):
    name, batch, L, V, M, B, T, d_h, dt, k, h0, norm = c
    print(f"[expand] {name} scorer {scorer}", flush=True)
    wl = synth.random_small(len(name) + B, batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=48, d_h=d_h, dtype=dt,
                            h0=h0, w_scale=1.0 / np.sqrt(d_h))
    dw = DeviceWorkload(wl, max_children=k, norm_mode=norm, scorer=scorer)
    got = dw.run()
    again = dw.run()
    for f in got:
        np.testing.assert_array_equal(got[f], again[f], err_msg=f)
    for t in sorted({0, batch // 2, batch - 1}):
        compare_tree(wl, t, got, dw.kw, name=name)
    dw.close()


@pytest.mark.parametrize("k", [0, 8])
def test_deep_tree_16_members(k):
    # d_h = 512, M = 64, L = 16, bf16, one tree per call
    wl = synth.deep()
    wl.B = 80
    dw = DeviceWorkload(wl, max_children=k)
    got = dw.run()
    compare_tree(wl, 0, got, dw.kw, tol=1e-4, name=f"deep B=80 k={k}")
    assert int(got["depth"].max()) >= 9
    dw.close()


def test_deep_trees_8_members():
    # ... 32 trees per call
    wl = synth.deep_concurrent()
    wl.B = 72
    dw = DeviceWorkload(wl)
    got = dw.run()
    for t in (0, 5, 18, 31):
        compare_tree(wl, t, got, dw.kw, tol=1e-4, name="deep_concurrent B=72")
    dw.close()


@pytest.mark.parametrize("scorer", [0, 1, 2], ids=["cond", "marg", "static"])
@pytest.mark.parametrize("M,B", [(16, 96), (96, 32)])
def test_adaptive_budget(M, B, scorer):
    wl = synth.random_small(2, batch=3, L=6, V=500, M=M, B=B, T=0.7, d_e=64, d_h=64, h0=True)
    run_budget(wl, f"general M={M} B={B} arm{scorer}", scorer=scorer)


@pytest.mark.parametrize("name", ["deep", "deep_concurrent"])
def test_spin_limit(name):
    # one poll: the members of a tree give up almost at once, and say so
    wl = getattr(synth, name)()
    wl.B = 80
    print(f"[timeout] {name} B=80 spin limit 1", flush=True)
    dw = DeviceWorkload(wl, debug_spin_limit=1)
    got = dw.run()
    dw.close()
    out = (got["status"] & binding.DT_TREE_TIMEOUT) != 0
    assert out.any()
    assert (got["n_nodes"][out] == 0).all() and (got["tokens"][out] == -1).all() and (got["mask"][out] == 0).all()
    dw = DeviceWorkload(wl)
    again = dw.run()
    dw.close()
    assert not again["status"].any()
    compare_tree(wl, 0, again, {}, tol=1e-4, name=f"after-timeout-{name}")


@pytest.mark.parametrize("scorer", [0, 2], ids=["cond", "static"])
@pytest.mark.parametrize("c", [(16, 80, 2, 0, True), (70, 100, 2, 0, False)], ids=["budget", "menu"])
def test_siblings_of_one_score(c, scorer):
    check_siblings(c, scorer)
