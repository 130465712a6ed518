"""The register-list expansion (menus and budgets of at most 64) at the edges of what it takes,
against the oracle: sizes around its constants (64 slots, 64 entries, 16 nodes per chunk, 32 units
per workgroup), more trees than resident groups, and exact score ties."""
import numpy as np
import pytest

from gpu_util import DeviceWorkload, compare_tree
from helpers import run_oracle
from paper_2607_08642_amd import synth

pytestmark = pytest.mark.gpu
F, H = synth.DT_F32, synth.DT_BF16

# name, batch, L, V, M, B, T, d_h, weights, k, h0, norm, logit scale and spikes
CASES = [
    ("one_member", 3, 4, 301, 8, 8, 1.0, 32, F, 0, True, 0, 2.0),
    ("one_slot", 2, 6, 300, 1, 16, 0.7, 64, F, 0, False, 0, 2.0),
    ("budget_one", 2, 3, 300, 64, 1, 1.0, 64, H, 0, True, 1, 2.0),
    ("full_list", 2, 5, 900, 64, 64, 0.0, 128, F, 0, True, 0, 0.3),
    ("full_list_bf16", 1, 4, 2000, 64, 64, 0.0, 256, H, 0, False, 1, 0.3),
    ("odd_members", 2, 4, 500, 33, 33, 0.7, 96, H, 5, True, 0, 1.0),
    ("odd_members_f32", 2, 4, 500, 63, 17, 1.3, 160, F, 0, True, 1, 1.0),
    ("cut_menus", 2, 4, 700, 64, 48, 1.0, 256, F, 3, True, 0, 0.3),
    ("uneven_members_bf16", 1, 4, 400, 40, 20, 1.0, 416, H, 0, True, 0, 1.0),
    ("deepest", 1, 64, 200, 8, 64, 1.0, 64, F, 2, False, 0, 6.0),
    ("trees_in_turn", 37, 3, 400, 16, 12, 0.7, 512, H, 0, True, 0, 1.0),
    ("trees_in_turn_one_per_cu", 20, 3, 400, 16, 64, 0.7, 512, H, 0, False, 0, 0.5),
]


@pytest.mark.parametrize("c", CASES, ids=[c[0] for c in CASES])
def test_edges(c):
    name, batch, L, V, M, B, T, d_h, dt, k, h0, norm, scale = c
    print(f"[grow] {name}", flush=True)
    wl = synth.random_small(len(name) + B, batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=48, d_h=d_h, dtype=dt,
                            h0=h0, logit_scale=scale, spikes=3, spike=3.0 * scale, w_scale=1.0 / np.sqrt(d_h))
    dw = DeviceWorkload(wl, max_children=k, norm_mode=norm)
    got = dw.run()
    again = dw.run()
    for f in got:
        np.testing.assert_array_equal(got[f], again[f], err_msg=f)
    for t in sorted({0, batch // 2, batch - 1}):
        compare_tree(wl, t, got, dw.kw, name=name)
    dw.close()


@pytest.mark.parametrize("B", [16, 64])
def test_plateau_order(B):
    """Certain tokens: a child's log-prob rounds to 0, so whole chains share one score, beside twins
    that tie exactly.  The heap works such a plateau first in, first out."""
    wl = synth.twin_tokens(synth.random_small(5, batch=2, L=8, V=257, M=32, B=B, T=1.0, d_e=32, d_h=64, dtype=F,
                                              emb_std=0.05, logit_scale=1.0, spikes=1, spike=0.0))
    x = wl.logits
    top = x.max(axis=-1, keepdims=True)
    x[:, ::2] = np.where(x[:, ::2] == top[:, ::2], x[:, ::2] + 40.0, x[:, ::2])  # twins share every second row
    dw = DeviceWorkload(wl)
    got = dw.run()
    for t in range(wl.batch):
        n = int(got["n_nodes"][t])
        s, p = got["scores"][t][:n], got["parents"][t][:n]
        assert n == B and (np.diff(s) <= 0).all() and (p < np.arange(n)).all()
        # first in, first out: within one score, nodes are ordered by (level, parent's place)
        level = np.array([0] * n)
        for i in range(n):
            level[i] = level[p[i]] + 1 if p[i] >= 0 and s[p[i]] == s[i] else 0
        key = list(zip(-s.astype(np.float64), level, p))
        assert key == sorted(key), key
        compare_tree(wl, t, got, dw.kw, name="plateau")
    dw.close()


ARM_CASES = [c for c in CASES if c[0] not in ("budget_one", "cut_menus")] + [
    ("budget_one_chain", 2, 3, 300, 64, 1, 1.0, 64, H, 0, True, 1, 2.0),
    ("cut_menus_chain", 2, 4, 700, 64, 48, 1.0, 256, F, 3, True, 0, 0.3),
    ("chains_in_rounds", 600, 3, 90, 8, 6, 1.0, 64, F, 0, True, 0, 1.0),
    ("one_level", 3, 1, 300, 16, 16, 1.0, 128, H, 0, True, 0, 1.0),
]


@pytest.mark.parametrize("scorer", [1, 2], ids=["marg", "static"])
@pytest.mark.parametrize("c", ARM_CASES, ids=[c[0] for c in ARM_CASES])
def test_arms(c, scorer):
    """The path-independent children functions: a marginal tree per workgroup, and the greedy chain
    (its own exchange) with the trees built from its menus by the group's members."""
    name, batch, L, V, M, B, T, d_h, dt, k, h0, norm, scale = c
    print(f"[grow] {name} scorer {scorer}", flush=True)
    wl = synth.random_small(len(name) + B, batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=48, d_h=d_h, dtype=dt,
                            h0=h0, logit_scale=scale, spikes=3, spike=3.0 * scale, w_scale=1.0 / np.sqrt(d_h))
    x = wl.logits.copy()
    bad = batch // 3 if batch > 2 else None  # a tree that cannot be built, beside ones that can
    if bad is not None:
        x[bad, 0, 3] = np.nan if dt == F else 0x7FC0
    wl.logits = x
    dw = DeviceWorkload(wl, max_children=k, norm_mode=norm, scorer=scorer)
    got = dw.run()
    again = dw.run()
    for f in got:
        np.testing.assert_array_equal(got[f], again[f], err_msg=f)
    for t in sorted({0, batch // 2, batch - 1} - {bad}):
        compare_tree(wl, t, got, dw.kw, name=name)
    if bad is not None:
        assert got["status"][bad] != 0 and got["n_nodes"][bad] == 0
    dw.close()


@pytest.mark.parametrize("scorer", [1, 2], ids=["marg", "static"])
def test_arm_copies_agree(scorer):
    """Two trees of many short steps (a child count and a few children read and written anew in each),
    768 copies of each side by side: every copy is the same tree, and the oracle's."""
    wl = synth.random_small(21, batch=2, L=24, V=150, M=8, B=64, T=1.0, d_e=32, d_h=64, dtype=F, h0=True,
                            logit_scale=1.0, spikes=2, spike=9.0, w_scale=0.125)
    n = 768
    wl.logits, wl.h0, wl.batch = np.tile(wl.logits, (n, 1, 1)), np.tile(wl.h0, (n, 1)), 2 * n
    print(f"[grow] copies scorer {scorer}", flush=True)
    dw = DeviceWorkload(wl, max_children=2, scorer=scorer)
    for _ in range(4):
        got = dw.run()
        for f in got:
            pair = got[f].reshape(n, 2, -1)
            np.testing.assert_array_equal(pair, np.broadcast_to(pair[:1], pair.shape), err_msg=f)
    for t in (0, 1):
        compare_tree(wl, t, got, dw.kw, name="copies")
    dw.close()


# M, B, L, k, path-dependent correction: a step's list of at most 64 entries and of more, cut within a
# family of siblings or not, ties below the root's children and one depth further
SIBLINGS = [(4, 20, 2, 0, False), (4, 10, 2, 0, True), (4, 12, 2, 3, False), (16, 64, 2, 0, False),
            (16, 41, 2, 0, True), (16, 64, 3, 0, True), (32, 64, 2, 0, False), (5, 64, 3, 0, True)]


@pytest.mark.parametrize("scorer", [0, 2], ids=["cond", "static"])
@pytest.mark.parametrize("c", SIBLINGS, ids=["-".join(map(str, c)) for c in SIBLINGS])
def test_siblings_of_one_score(c, scorer):
    check_siblings(c, scorer)


@pytest.mark.parametrize("d_h,dt,batch", [(32, F, 3), (64, F, 3), (96, F, 3), (160, F, 3), (256, H, 3), (416, H, 3),
                                          (512, H, 3), (512, H, 20)])
def test_siblings_by_their_path(d_h, dt, batch):
    """... where the path state decides their order: its parts from 1 to 16 workgroups, one and (the last)
    two to a CU."""
    check_siblings((16, 60 if batch < 20 else 30, 3, 0, "state"), 0, d_h, dt, batch)


def check_siblings(c, scorer, d_h=64, dt=F, batch=3):
    """Siblings whose log-probs differ by 2^-20 below parents that score about -200 (an ulp of 2^-16):
    their scores round together, and they leave in the order of their log-probs, which the correction
    made another order than the slots'.  The oracle's (64-bit) scores are all apart: the same trees,
    node for node."""
    M, B, L, k, path = c
    V = 4 * M
    wl = synth.random_small(M, batch=batch, L=L, V=V, M=M, B=B, T=1.0, d_e=32, d_h=d_h, dtype=dt, logits_dtype=F,
                            h0=bool(path), w_scale=4.0 / np.sqrt(d_h))
    w, r = wl.weights, np.random.default_rng(B)
    e = 2.0 ** -20
    slot = np.arange(M)
    store = synth.f32_to_bf16_bits if dt == H else (lambda a: a)
    emb, w_c, b_c = np.zeros((V, 32), np.float32), np.zeros((32, d_h), np.float32), np.zeros(32, np.float32)
    b_c[0] = 0.0 if path == "state" else 1.0
    if path == "state":   # (values, not log-probs, order siblings: they need not be ulps of a log-prob apart)
        w_c[0] = 2.0 ** -2 * np.sign(r.standard_normal(d_h))
    elif path:   # (|w S| <= 64 2^-12 max |S|: slots' corrections of at most 32 2^-20 move by less than 2^-21,
        # so log-probs stay two ulps apart or more: a chain's menus hold them rounded)
        w_c[0] = 2.0 ** -12 * np.sign(r.standard_normal(d_h))
    # the last depth's tokens: slots 2^-20 apart, the correction shuffles them
    emb[V - M:, 0] = (slot + r.permutation(M)) * e
    w.emb, w.w_c, w.b_c = store(emb), store(w_c), store(b_c)
    wl.logits[:] = -1000.0
    for t in range(wl.batch):
        for d in range(L - 1):   # well apart: one certain token, the others far below
            wl.logits[t, d, d * M:(d + 1) * M] = np.where(slot == 0, 0.0, -200.0 - (1.0 + 6.1 * d) * slot - 0.01 * t)
        wl.logits[t, L - 1, V - M:] = -slot * e
    print(f"[grow] siblings {c} scorer {scorer}", flush=True)
    dw = DeviceWorkload(wl, max_children=k, scorer=scorer)
    got = dw.run()
    dw.close()
    turned = 0
    for t in range(wl.batch):
        ref = run_oracle(wl, t, **dw.kw)
        n = ref["n_nodes"]
        assert int(got["n_nodes"][t]) == n
        gap = np.abs(np.diff(ref["scores"][:n]))   # (all but siblings well apart, or a certain child's: 0)
        assert ((gap > 1e-3) | (gap == 0) | (np.diff(ref["parents"][:n]) == 0)).all()
        for f in ("tokens", "parents", "depth", "mask"):
            np.testing.assert_array_equal(got[f][t], ref[f], err_msg=f"tree {t} {f}")
        s, p, tok = got["scores"][t], got["parents"][t], got["tokens"][t]
        turned += int(np.sum((s[1:n] == s[:n - 1]) & (p[1:n] == p[:n - 1]) & (tok[1:n] < tok[:n - 1])))
    assert turned >= 1   # (tokens ascend with the slot)
