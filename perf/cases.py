"""Performance cases of the draft-tree builder: what its callers run, end to end.

Every case goes through the Python binding as a serving program does: a plan
(or a one-shot call), resident logits, preallocated output trees, no
synchronisation.  Four families:

* ``tree``    -- ``Plan.build_tree``: the three scorers, the frontier builder,
                 the adaptive budget, with and without root states;
* ``head``    -- ``Plan.build_tree_head``: Domino's own rank-r SiLU head;
* ``scan``    -- ``scan_topm``: the top-M scan alone, as a sampler or a
                 candidate filter calls it;
* ``oneshot`` -- ``binding.build_tree``: logits, embedding table and weights in,
                 trees out, nothing kept between calls (scripts, tests,
                 evaluation of checkpoints).

Logits are 2 N(0, 1) with planted spikes per row, as the benchmark draws them:
``peaked`` (1-4 of +U(6, 12): shallow, wide trees), ``flat`` (4-16 of +U(3, 6))
and ``deep`` (2-4 of +U(13, 17): the spikes dominate the row, so a tree grows
long paths and the expansion runs a long chain of dependent steps).
"""
import heapq
import math

import torch

from paper_2607_08642_amd import binding

DEV = "cuda"
QWEN3_VOCAB = 151936
SPIKES = {"peaked": (1, 4, 6.0, 12.0), "flat": (4, 16, 3.0, 6.0), "deep": (2, 4, 13.0, 17.0)}
SCORERS = {"cond": binding.DT_SCORER_COND, "marg": binding.DT_SCORER_MARG,
           "static": binding.DT_SCORER_STATIC}
FIELDS = ("tokens", "parents", "depth", "position_ids", "mask", "scores", "n_nodes", "status")
LOGIT_BYTES = 32 * 16 * QWEN3_VOCAB * 2   # of a drawn call at most: 32 trees of the Qwen3 shape


def _tree(name=None, family="tree", batch=1, L=16, V=QWEN3_VOCAB, M=64, B=16, T=1.0, d_e=4096, d_h=512,
          wdtype="bf16", ldtype="bf16", logits="peaked", h0=False, bias=False, k=0, scorer="cond",
          norm="tail", frontier=0, adaptive=False, rank=0, d_H=0):
    c = dict(family=family, batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=d_e, d_h=d_h, wdtype=wdtype,
             ldtype=ldtype, logits=logits, h0=h0, bias=bias, k=k, scorer=scorer, norm=norm,
             frontier=frontier, adaptive=adaptive, rank=rank, d_H=d_H)
    return c if name is None else dict(c, name=name)


def _scan(name=None, rows=16, V=QWEN3_VOCAB, M=64, T=1.0, ldtype="bf16", logits="peaked"):
    c = dict(family="scan", rows=rows, V=V, M=M, T=T, ldtype=ldtype, logits=logits)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # the smallest call: a toy drafter in fp32, all latency
        _tree("tiny_fp32", L=4, V=1024, M=8, B=8, T=0.0, d_e=64, d_h=64, wdtype="f32", ldtype="f32",
              bias=True),
        # the headline: one decoding round of one Qwen3-8B-shaped stream
        _tree("single_8b"),
        # the same stream on easy text, with the paper's branching factor 8: long paths
        _tree("single_deep_k8", logits="deep", k=8),
        # a large verification budget on uncertain text, greedy, Qwen3-4B shape
        _tree("budget64_4b", B=64, T=0.0, d_e=2560, logits="flat"),
        # a serving batch: 32 requests, sampled, each continuing from its own path state
        _tree("serving_32", batch=32, T=0.7, h0=True),
        # a large serving batch on easy text (more trees than the chip takes side by side in groups)
        _tree("serving_100_deep", batch=100, T=0.7, logits="deep", h0=True),
        # the drafter's own trained head (rank 256) for a few concurrent streams
        _tree("head_b8", family="head", batch=8, T=0.7, h0=True, rank=256, d_H=4096),
        # the paper's Cond-static arm: a greedy chain, then a tree from its menus
        _tree("static_8b", scorer="static"),
        # the serving (frontier) builder on a small fp32 drafter with an odd vocabulary
        _tree("frontier_fp32", batch=4, L=8, V=32003, M=32, B=32, T=0.7, d_e=1024, d_h=256, wdtype="f32",
              ldtype="f32", bias=True, norm="slice", frontier=8),
        # the scan alone at the size of a serving batch
        _scan("scan_512", rows=512, T=0.7),
        # the scan alone on rows of an odd vocabulary, wide menus
        _scan("scan_odd_m128", rows=128, V=151937, M=128),
        # one tree from raw weights, Qwen3-4B shape
        _tree("oneshot_4b", family="oneshot", d_e=2560),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng):
    v = _logint(rng, 1000, 151937)
    return rng.choice([v, v | 1, v // 8 * 8, QWEN3_VOCAB])


def draw(rng):
    family = rng.choice(["tree"] * 5 + ["scan"] * 3 + ["head", "oneshot"])
    V = _vocab(rng)
    T = rng.choice([0.0, 0.7, 1.0, round(rng.uniform(0.3, 1.5), 2)])
    logits = rng.choice(["peaked", "flat", "deep"])
    ldtype = rng.choice(["bf16", "bf16", "f32"])
    size = 2 if ldtype == "bf16" else 4
    most = max(1, LOGIT_BYTES // (V * size))   # rows
    if family == "scan":
        return _scan(rows=_logint(rng, 1, min(512, most)), V=V, M=_logint(rng, 8, 128), T=T,
                     ldtype=ldtype, logits=logits)
    L = rng.choice([4, 8, 16, rng.randint(3, 16)])
    wdtype = rng.choice(["bf16", "bf16", "f32"])
    d_h = rng.choice([64, 128, 256, 512, 512, 768])
    d_e = rng.choice([1024, 2048, 2560])
    if wdtype == "f32":   # (small fp32 drafters)
        d_h, d_e, V = min(d_h, 256), 512, min(V, 32003)
    M = rng.choice([16, 32, 64, 64, rng.randint(8, 128)])
    B = rng.choice([8, 16, 16, 32, 64, rng.randint(8, 64)])
    batch = _logint(rng, 1, max(1, min(100, most // L)))
    c = dict(batch=batch, L=L, V=V, M=M, B=B, T=T, d_e=d_e, d_h=d_h, wdtype=wdtype, ldtype=ldtype,
             logits=logits, h0=rng.random() < 0.5, bias=rng.random() < 0.5, k=rng.choice([0, 0, 8]),
             norm=rng.choice(["tail", "tail", "slice"]))
    if family == "oneshot":
        return _tree(family="oneshot", **dict(c, batch=min(batch, 4), d_h=min(d_h, 512),
                                              V=V if wdtype == "bf16" else min(V, 4001)))
    if family == "head":
        c.update(M=min(M, 64), B=min(B, 32), k=8)
        return _tree(family="head", rank=rng.choice([128, 256, 256]), d_H=d_e, **c)
    option = rng.choice(["", "", "", "adaptive", "frontier", "static", "marg"])
    if option == "marg":   # (bf16 marginals tie exactly: any order of tied nodes is right)
        c["ldtype"] = "f32"
        c["batch"] = max(1, batch // 2)
    return _tree(adaptive=option == "adaptive", frontier=8 if option == "frontier" else 0,
                 scorer=option if option in ("static", "marg") else "cond", **c)


# ---- inputs ---------------------------------------------------------------------

def _dt(name):
    return torch.bfloat16 if name == "bf16" else torch.float32


def _logits(g, shape, kind, dtype):
    """2 N(0, 1) plus n ~ U{lo..hi} spikes of +U(a, b) per row."""
    lo, hi, a, b = SPIKES[kind]
    V = shape[-1]
    x = torch.randn(shape, generator=g, device=DEV).mul_(2.0).reshape(-1, V)
    rows = x.shape[0]
    n = torch.randint(lo, hi + 1, (rows, 1), generator=g, device=DEV)
    at = torch.randint(0, V, (rows, hi), generator=g, device=DEV)
    up = torch.rand((rows, hi), generator=g, device=DEV) * (b - a) + a
    up = torch.where(torch.arange(hi, device=DEV) < n, up, torch.zeros_like(up))
    for j in range(hi):   # (one spike a row at a time: no two writers of one element)
        x.scatter_add_(1, at[:, j:j + 1], up[:, j:j + 1])
    return x.to(dtype).reshape(shape)


def _inputs(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    if case["family"] == "scan":
        return dict(logits=_logits(g, (case["rows"], case["V"]), case["logits"], _dt(case["ldtype"])))
    wd, V, d_e, d_h, b, L = (_dt(case["wdtype"]), case["V"], case["d_e"], case["d_h"], case["batch"],
                             case["L"])

    def uniform(*shape, scale=1.0 / math.sqrt(d_h)):
        return ((torch.rand(shape, generator=g, device=DEV) * 2 - 1) * scale).to(wd)

    x = dict(logits=_logits(g, (b, L, V), case["logits"], _dt(case["ldtype"])))
    x["emb"] = torch.empty((V, d_e), device=DEV, dtype=wd).normal_(0.0, 0.02, generator=g)
    x["w_ih"], x["w_hh"], x["w_c"] = uniform(3 * d_h, d_e), uniform(3 * d_h, d_h), uniform(d_e, d_h)
    x["b_ih"] = uniform(3 * d_h) if case["bias"] else None
    x["b_hh"] = uniform(3 * d_h) if case["bias"] else None
    x["b_c"] = uniform(d_e)
    x["h0"] = torch.randn((b, d_h), generator=g, device=DEV) * 0.1 if case["h0"] else None
    if case["family"] == "head":
        r, d_H = case["rank"], case["d_H"]
        x["H"] = torch.randn((b, L, d_H), generator=g, device=DEV).to(wd)
        x["w1"] = uniform(r, d_H + d_h, scale=1.0 / math.sqrt(d_H + d_h))
        x["w2"] = uniform(V, r, scale=1.0 / math.sqrt(r))
    return x


def _costs(case):
    """C_d and a convex C_v(0..B): the verifier's cost rises once the batch fills its matrix tiles."""
    return 3.0, [20.0 + 0.02 * n + 0.01 * max(0, n - 6) ** 2 for n in range(case["B"] + 1)]


def _norm(case):
    return binding.DT_NORM_TAIL if case["norm"] == "tail" else binding.DT_NORM_SLICE


def prepare(case, seed):
    x = _inputs(case, seed)
    s = dict(case=case, logits=x["logits"])
    if case["family"] == "scan":
        return s
    if case["family"] == "oneshot":
        return dict(s, **x)
    plan = binding.Plan(x["emb"], x["w_ih"], x["w_hh"], x["b_ih"], x["b_hh"], x["w_c"], x["b_c"],
                        L=case["L"], M=case["M"], B=case["B"],
                        logits_dtype=binding.DT_BF16 if case["ldtype"] == "bf16" else binding.DT_F32,
                        max_batch=case["batch"], max_children=case["k"], norm_mode=_norm(case),
                        scorer=SCORERS[case["scorer"]], frontier_width=case["frontier"])
    if case["adaptive"]:
        plan.set_adaptive_budget(*_costs(case))
    s.update(plan=plan, h0=x["h0"], out=binding.Tree.empty(case["batch"], case["B"], DEV))
    if case["family"] == "head":
        s.update(H=x["H"], w1=x["w1"], w2=x["w2"])
    return s


def run(state):
    c = state["case"]
    if c["family"] == "scan":
        ids, vals, tail, flags = binding.scan_topm(state["logits"], c["M"], c["T"])
        return dict(ids=ids, vals=vals, tail=tail, flags=flags)
    if c["family"] == "oneshot":
        s = state
        t = binding.build_tree(s["logits"], s["emb"], (s["w_ih"], s["w_hh"], s["b_ih"], s["b_hh"]),
                               (s["w_c"], s["b_c"]), c["L"], c["M"], c["B"], c["T"], h0=s["h0"],
                               max_children=c["k"], norm_mode=_norm(c))
    elif c["family"] == "head":
        t = state["plan"].build_tree_head(state["logits"], state["H"], state["w1"], state["w2"], c["T"],
                                          h0=state["h0"], out=state["out"])
    else:
        t = state["plan"].build_tree(state["logits"], c["T"], h0=state["h0"], out=state["out"])
    return {f: getattr(t, f) for f in FIELDS}


def work(case):
    size = 2 if case["ldtype"] == "bf16" else 4
    if case["family"] == "scan":
        rows, V, M = case["rows"], case["V"], case["M"]
        # the logits in, the menus out; an exponential and a sum for each logit
        return dict(bytes=rows * (V * size + M * 8 + 8), flops=2.0 * rows * V)
    b, L, V, M, B, d_e, d_h = (case[k] for k in ("batch", "L", "V", "M", "B", "d_e", "d_h"))
    ws = 2 if case["wdtype"] == "bf16" else 4
    nodes = b * (B + 1)   # the root and every emitted node expanded once
    nbytes = b * L * V * size + b * B * (24 + B)
    flops = 2.0 * b * L * V
    if case["scorer"] == "marg":
        return dict(bytes=nbytes, flops=flops)
    # W_hh once, the input projections of the emitted tokens, the correction
    # rows of the root's and one more depth's menu
    nbytes += 3 * d_h * d_h * ws + b * B * 3 * d_h * 4 + b * 2 * M * d_h * 4
    flops += nodes * 2.0 * (3 * d_h * d_h + M * d_h)
    if case["family"] == "head":
        r, d_H = case["rank"], case["d_H"]
        nbytes += r * (d_H + d_h) * ws + b * L * d_H * ws + b * 2 * M * r * ws
        flops += 2.0 * b * L * r * d_H + nodes * 2.0 * r * (d_h + M)
    if case["family"] == "oneshot":
        # the embedding rows of the candidates, W_ih and W_c; their projections
        nbytes += 4 * d_h * d_e * ws + b * L * M * d_e * ws
        flops += 2.0 * b * L * M * d_e * 4 * d_h
    return dict(bytes=nbytes, flops=flops)


def tolerance(case):
    # Scores and log-sum-exps are fp32 with fp32 sums: against exact() the
    # scores' error was 0.3-2.6e-7 and the log-sum-exps' 2-5e-8 over these cases
    # and drawn ones.  Tokens and topology are whole numbers, equal unless two
    # scores lie within rounding of each other; menus are exact.
    if case["family"] == "scan":
        return dict(rel=3e-7, max=3e-6, differ=0.0)
    return dict(rel=1e-6, max=1e-5, differ=0.01)


# ---- the same in 64 bits, in plain torch ------------------------------------------

def _menus(x, M, tau):
    """Top-M ids (value desc, id asc), their logits and the tail's log-sum-exp of [rows, V] logits."""
    ids, vals, tail = [], [], []
    for r in x:
        v, i = torch.sort(r.float(), descending=True, stable=True)
        ids.append(i[:M])
        vals.append(v[:M].double())
        rest = v[M:].double() / tau
        tail.append(torch.logsumexp(rest, 0) if rest.numel() else torch.tensor(-math.inf, device=DEV).double())
    return torch.stack(ids), torch.stack(vals), torch.stack(tail)


class _Exact:
    """One tree's children function in 64 bits."""

    def __init__(self, case, w, ids, vals, tail, tau, H):
        self.c, self.w, self.ids, self.vals, self.tail, self.tau, self.H = case, w, ids, vals, tail, tau, H
        c = case
        self.k = min(c["k"] or min(c["M"], c["B"]), c["M"], c["B"])
        self.table = None

    def gru(self, tok, S):
        w = self.w
        gi = w["w_ih"] @ w["emb"][tok].double() + w["b_ih"]
        gh = w["w_hh"] @ S + w["b_hh"]
        (ir, iz, i_n), (hr, hz, hn) = gi.chunk(3), gh.chunk(3)
        z = torch.sigmoid(iz + hz)
        return (1 - z) * torch.tanh(i_n + torch.sigmoid(ir + hr) * hn) + z * S

    def menu(self, d, S):
        """Normalised log-probs of depth d's slots (d = 0: the root's children)."""
        if self.table is not None:
            return self.table[d]
        w, x = self.w, self.vals[d]
        if S is not None:
            if self.H is not None:
                y = w["w1"] @ torch.cat([self.H[d].double(), S])
                x = x + w["w2"][self.ids[d]].double() @ (y * torch.sigmoid(y))
            else:
                x = x + w["emb"][self.ids[d]].double() @ (w["w_c"] @ S + w["b_c"])
        z = x / self.tau
        both = torch.cat([z, self.tail[d:d + 1]]) if self.c["norm"] == "tail" else z
        return z - torch.logsumexp(both, 0)

    def children(self, d, S):
        v, s = torch.sort(self.menu(d, S), descending=True, stable=True)
        tok = self.ids[d][s[:self.k]]
        return list(zip(v[:self.k].tolist(), tok.tolist()))

    def static_table(self, S):
        rows = []
        for d in range(self.c["L"]):
            m = self.menu(d, S)
            rows.append(m)
            S = self.gru(self.ids[d][torch.argmax(m)], S)
        self.table = rows

    def scores(self, S0):
        """Emitted scores in order (the heap of the paper's algorithm, or its frontier builder)."""
        c, cond = self.c, self.c["scorer"] == "cond"
        if c["scorer"] == "static":
            self.static_table(S0)
        root = None if c["scorer"] == "marg" else S0
        if c["frontier"]:
            ledger, lanes = [], [(0.0, None, S0)]
            for d in range(c["L"]):
                row = []
                for g, tok, S in lanes:
                    if tok is not None and cond:
                        S = self.gru(tok, S)
                    row += [(g + lp, t, S) for lp, t in self.children(d, S if d or cond else root)]
                ledger += [g for g, _, _ in row]
                lanes = sorted(row, key=lambda r: -r[0])[:c["frontier"]]
            return sorted(ledger, reverse=True)[:c["B"]]
        heap, n, out = [], 0, []
        for lp, tok in self.children(0, root):
            heapq.heappush(heap, (-lp, n, 1, tok, S0))
            n += 1
        cd, cv = _costs(c)
        phi, theta = 0.0, 1.0 / (cd + cv[0])
        while heap and len(out) < c["B"]:
            g, _, d, tok, S = heapq.heappop(heap)
            if c["adaptive"]:
                th = (1 + phi + math.exp(-g)) / (cd + cv[len(out) + 1])
                if th <= theta:
                    break
                phi, theta = phi + math.exp(-g), th
            out.append(-g)
            if d < c["L"] and len(out) < c["B"]:
                S1 = self.gru(tok, S) if cond else root
                for lp, t in self.children(d, S1):
                    heapq.heappush(heap, (g - lp, n, d + 1, t, S1))
                    n += 1
        return out


def exact(case, seed):
    x = _inputs(case, seed)
    tau = case["T"] if case["T"] > 0 else 1.0
    if case["family"] == "scan":
        ids, vals, tail = _menus(x["logits"], case["M"], tau)
        return dict(ids=None, vals=vals, tail=tail, flags=None)
    d_h, L, b = case["d_h"], case["L"], case["batch"]
    w = {k: x[k].double() for k in ("w_ih", "w_hh", "w_c", "b_c")}
    for k in ("b_ih", "b_hh"):
        w[k] = torch.zeros(3 * d_h, dtype=torch.float64, device=DEV) if x[k] is None else x[k].double()
    w["emb"] = x["emb"]
    if case["family"] == "head":
        w["w1"], w["w2"] = x["w1"].double(), x["w2"]
    scores = torch.full((b, case["B"]), -math.inf, dtype=torch.float64)
    for t in range(b):
        e = _Exact(case, w, *_menus(x["logits"][t], case["M"], tau), tau,
                   x["H"][t] if case["family"] == "head" else None)
        S0 = torch.zeros(d_h, dtype=torch.float64, device=DEV) if x["h0"] is None else x["h0"][t].double()
        got = e.scores(S0)
        scores[t, :len(got)] = torch.tensor(got, dtype=torch.float64)
    out = dict.fromkeys(FIELDS)
    out["scores"] = scores
    return out
