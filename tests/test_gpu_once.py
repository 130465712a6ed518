"""One-shot calls (binding.build_tree): trees from raw weights, on both of their routes (the candidates'
rows folded, or a plan of the whole vocabulary), against the oracle; and the fold kernels' edges."""
import numpy as np
import pytest
import torch

from gpu_util import compare_tree, to_dev
from paper_2607_08642_amd import binding, synth

pytestmark = pytest.mark.gpu
F, H = synth.DT_F32, synth.DT_BF16

# name, batch, L, V, M, B, d_e, d_h, weights, bias, h0, options
CASES = [
    ("rows", 2, 4, 3001, 33, 16, 72, 64, F, True, True, {}),
    ("rows_bf16", 2, 4, 3001, 33, 16, 72, 64, H, True, True, {}),
    ("ragged_width", 1, 5, 2000, 16, 8, 37, 96, H, False, False, {}),       # d_e % 8 != 0
    ("ragged_width_f32", 1, 5, 2000, 16, 8, 33, 32, F, False, True, {}),
    ("many_rows", 3, 8, 20011, 64, 16, 96, 512, H, False, True, dict(max_children=8)),  # 1,536 rows
    ("slice_offset", 1, 3, 999, 64, 64, 40, 128, F, True, False, dict(norm_mode=1, pos_offset=7)),
    ("dead_slots", 2, 3, 500, 40, 16, 64, 64, F, False, False, {}),
    ("vocabulary", 4, 4, 300, 32, 16, 64, 64, F, True, True, {}),           # batch L M >= V: a plan
    ("wide", 1, 3, 4000, 96, 16, 64, 64, H, False, False, {}),              # M > 64: a plan
    ("marg", 1, 3, 4000, 16, 16, 64, 64, F, False, False, dict(scorer=1)),  # another arm: a plan
    ("marg_bias", 1, 3, 4000, 16, 16, 64, 64, F, True, True, dict(scorer=1)),  # (no E b_c in marginal menus)
    ("static_bias", 2, 3, 4000, 16, 16, 64, 64, F, True, True, dict(scorer=2)),
]


@pytest.mark.parametrize("c", CASES, ids=[c[0] for c in CASES])
def test_once(c):
    name, batch, L, V, M, B, d_e, d_h, dt, bias, h0, opts = c
    print(f"[once] {name}", flush=True)
    wl = synth.random_small(len(name), batch=batch, L=L, V=V, M=M, B=B, T=0.7, d_e=d_e, d_h=d_h, dtype=dt,
                            gru_bias=bias, head_bias=bias or dt == H, h0=h0, w_scale=1.0 / np.sqrt(d_h),
                            emb_std=2.0 / np.sqrt(d_e))
    if name == "dead_slots":   # fewer finite logits than slots
        wl.logits[:, 1, 25:] = -np.inf
    w = wl.weights
    x = {k: to_dev(getattr(w, k), dt) for k in ("emb", "w_ih", "w_hh", "b_ih", "b_hh", "w_c", "b_c")}
    t = binding.build_tree(to_dev(wl.logits, wl.logits_dtype), x["emb"],
                           (x["w_ih"], x["w_hh"], x["b_ih"], x["b_hh"]), (x["w_c"], x["b_c"]), L, M, B, wl.T,
                           h0=None if wl.h0 is None else torch.from_numpy(wl.h0).cuda(), **opts)
    got = {k: getattr(t, k).cpu().numpy() for k in
           ("tokens", "parents", "depth", "position_ids", "mask", "scores", "n_nodes", "status")}
    for i in range(batch):
        compare_tree(wl, i, got, dict(opts), name=name)


def test_once_on_a_side_stream():
    """Weights written on the default stream, the call on another."""
    wl = synth.random_small(3, batch=1, L=4, V=3000, M=32, B=16, T=1.0, d_e=64, d_h=64)
    w = wl.weights
    side = torch.cuda.Stream()
    with torch.cuda.stream(torch.cuda.default_stream()):
        x = {k: to_dev(getattr(w, k), F) * 1.0 for k in ("emb", "w_ih", "w_hh", "b_ih", "b_hh", "w_c", "b_c")}
        logits = to_dev(wl.logits, F) * 1.0
    with torch.cuda.stream(side):
        t = binding.build_tree(logits, x["emb"], (x["w_ih"], x["w_hh"], x["b_ih"], x["b_hh"]),
                               (x["w_c"], x["b_c"]), 4, 32, 16, 1.0)
    got = {k: getattr(t, k).cpu().numpy() for k in
           ("tokens", "parents", "depth", "position_ids", "mask", "scores", "n_nodes", "status")}
    compare_tree(wl, 0, got, {}, name="side")


@pytest.mark.parametrize("dt,d_e,d_h", [(H, 72, 64), (H, 37, 96), (F, 33, 32)])
def test_weights_at_any_element_address(dt, d_e, d_h):
    """Weights one element past a 16-byte boundary: the same trees, bit for bit, on both routes."""
    wl = synth.random_small(7, batch=2, L=4, V=3001, M=24, B=16, T=0.7, d_e=d_e, d_h=d_h, dtype=dt,
                            gru_bias=True, head_bias=True)
    w = {k: to_dev(getattr(wl.weights, k), dt) for k in ("emb", "w_ih", "w_hh", "b_ih", "b_hh", "w_c", "b_c")}

    def shifted(t):
        s = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)[1:].view(t.shape)
        return s.copy_(t)

    off = {k: t if k == "emb" else shifted(t) for k, t in w.items()}
    logits = to_dev(wl.logits, wl.logits_dtype)
    trees = []
    for x in (w, off):
        gru, head = (x["w_ih"], x["w_hh"], x["b_ih"], x["b_hh"]), (x["w_c"], x["b_c"])
        trees.append(binding.build_tree(logits, x["emb"], gru, head, 4, 24, 16, wl.T))
        plan = binding.Plan(x["emb"], *gru, *head, L=4, M=24, B=16, logits_dtype=wl.logits_dtype, max_batch=2)
        trees.append(plan.build_tree(logits, wl.T))
        torch.cuda.synchronize()
        plan.close()
    for a, b in ((0, 2), (1, 3)):
        for f in ("tokens", "parents", "mask", "scores", "n_nodes", "status"):
            assert torch.equal(getattr(trees[a], f), getattr(trees[b], f)), f
    got = {k: getattr(trees[2], k).cpu().numpy() for k in
           ("tokens", "parents", "depth", "position_ids", "mask", "scores", "n_nodes", "status")}
    for i in range(2):
        compare_tree(wl, i, got, {}, name="shifted")
