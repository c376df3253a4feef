"""Workloads that the compression pass and decode attention are timed on.

A case is a packed batch of GUI trajectories (screens of rows x cols patches,
each followed by a run of text) and one thing that a serving loop or an
ablation study does with it:

* ``pass``    -- the whole compression pass, ``compress()``;
* ``decode``  -- one decode step's attention over the full or the compacted cache;
* ``select``  -- the top-B selection and the compaction on given priors;
* ``css``     -- the saliency over a wider neighbourhood (the ablation entry point);
* ``concat``  -- the procedure over the concatenated key space, ``compress_concat()``.

Screens, their redundancy, the query targets and the key statistics follow
``paper_2603_00188_amd.workload``: the patch embeddings come from its
``make_scene``; keys, values and queries are drawn on the GPU by the same recipe.
"""
import random

import numpy as np
import torch

from paper_2603_00188_amd import stlite as S
from paper_2603_00188_amd import workload as W

D = 128
DEV = "cuda"

# The benchmark's models: 28 query heads over 4 kv heads.
BASE = dict(kind="pass", layers=28, q_heads=28, kv_heads=4, window=64, beta_num=1, beta_den=5, layout=0,
            seqs=1, frames_min=1, frames_max=1, rows=36, cols=80, text_min=256, text_max=256,
            change_lo=0.05, change_hi=0.15, dup=0.0, element_h=3, element_w=4)


def listed():
    return [
        # one layer of three small screens: nothing but launches and latency
        dict(BASE, name="tiny_pass", layers=1, window=32, frames_min=3, frames_max=3, rows=16, cols=16,
             text_min=48, text_max=48, element_h=2, element_w=2),
        # an agent's first step: one screenshot and the instruction, no history
        dict(BASE, name="step_pass", window=32, text_min=512, text_max=512, element_h=2, element_w=2),
        # an early step of a trajectory that is compressed anew at each step
        dict(BASE, name="early_pass", frames_min=5, frames_max=5),
        # a fifty-step trajectory with a third of its screens repeated (bench.py's default)
        dict(BASE, name="trajectory_pass", frames_min=48, frames_max=48, change_hi=0.2, dup=0.3),
        # a batch of trajectories of different lengths, packed
        dict(BASE, name="ragged_pass", window=32, beta_den=10, layout=4, seqs=8, frames_min=6, frames_max=24,
             text_min=128, text_max=512),
        # odd grids, another GQA group, and screens that share nothing with each other
        dict(BASE, name="odd_fresh_pass", layers=12, q_heads=16, kv_heads=2, window=32, beta_num=3, beta_den=10,
             layout=7, seqs=3, frames_min=4, frames_max=11, rows=27, cols=49, text_min=17, text_max=301,
             change_lo=1.0, change_hi=1.0),
        # the decode step after step_pass: a short compacted cache
        dict(BASE, name="decode_step", kind="decode", cache="compact", window=32, text_min=512, text_max=512),
        # the decode step after trajectory_pass
        dict(BASE, name="decode_compact", kind="decode", cache="compact", frames_min=48, frames_max=48),
        # decode without compression over a twenty-screen context, what the method is compared with
        dict(BASE, name="decode_full", kind="decode", cache="full", frames_min=20, frames_max=20),
        # ranking and gathering alone, as a caller with a prior, saliency or gate of its own uses them
        dict(BASE, name="select_compact", kind="select", frames_min=20, frames_max=20),
        # the neighbourhood-size ablation
        dict(BASE, name="css_5x5", kind="css", nbhd=5, frames_min=20, frames_max=20),
        # one kept set per layer (concatenated heads)
        dict(BASE, name="concat_pass", kind="concat", frames_min=20, frames_max=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(2.0 ** rng.uniform(np.log2(lo), np.log2(hi))))


def draw(rng):
    """Another case of the ranges above: any shape, redundancy from repeated to
    wholly fresh screens, no dearer than the trajectory."""
    while True:
        q_heads, kv_heads = rng.choice([(28, 4), (28, 4), (16, 2), (32, 8), (24, 4), (8, 8)])
        c = dict(BASE, kind=rng.choice(["pass", "pass", "pass", "decode", "decode", "select", "css", "concat"]),
                 layers=_log_int(rng, 1, 28), q_heads=q_heads, kv_heads=kv_heads,
                 window=rng.choice([1, 8, 16, 32, 32, 37, 64, 64]), beta_num=rng.choice([1, 1, 2, 3]),
                 beta_den=rng.choice([5, 7, 10]), layout=rng.randrange(1 << 16), seqs=_log_int(rng, 1, 8),
                 rows=rng.randint(9, 45), cols=rng.randint(11, 97), text_min=rng.randint(70, 200))
        c["frames_min"] = _log_int(rng, 1, 40)
        c["frames_max"] = c["frames_min"] + rng.choice([0, 0, 3, 9])
        c["text_max"] = c["text_min"] + rng.choice([0, 13, 300])
        c["change_lo"], c["change_hi"] = rng.choice([(0.05, 0.15), (0.05, 0.2), (0.2, 0.5), (1.0, 1.0)])
        c["dup"] = rng.choice([0.0, 0.0, 0.3])
        if c["kind"] == "decode":
            c["cache"] = rng.choice(["compact", "compact", "full"])
        if c["kind"] == "css":
            c["nbhd"] = rng.choice([3, 5, 7, 9])
        if c["kind"] == "concat" and kv_heads not in (2, 4):
            continue
        top = _shape(dict(BASE, frames_min=48, frames_max=48))
        s = _shape(c)
        if s["tokens"] * s["units"] <= top["tokens"] * top["units"] and s["pairs"] * s["units"] <= top["pairs"] * top["units"]:
            return c


def _workload(case, seed):
    """The batch as workload.Workload: the layout comes from the case, the content from the seed."""
    r = random.Random(case["layout"])
    seqs = []
    for _ in range(case["seqs"]):
        segs = []
        for _ in range(r.randint(case["frames_min"], case["frames_max"])):
            segs += [(W.FRAME, case["rows"], case["cols"]), (W.TEXT, r.randint(case["text_min"], case["text_max"]))]
        seqs.append(tuple(segs))
    fresh = case["change_lo"] >= 1.0
    red = W.Redundancy(rects=((case["rows"], case["cols"]),) if fresh else None,
                       frac=(case["change_lo"], case["change_hi"]), dup_frac=case["dup"])
    return W.Workload("case", case["layers"], case["q_heads"], case["kv_heads"], case["window"],
                      (case["beta_num"], case["beta_den"]), tuple(seqs), red,
                      ((1, case["element_h"]), (1, case["element_w"])), seed=seed)


def _shape(case):
    """Token counts of a case (all sequences) and its (historical, current) token pairs."""
    w = _workload(case, 0)
    patches = case["rows"] * case["cols"]
    frames = [sum(1 for s in segs if s[0] == W.FRAME) for segs in w.seqs]
    lens = w.seq_lengths()
    return dict(units=w.n_layers * w.n_kv_heads, tokens=sum(lens), frames=sum(frames), patches=patches,
                budget=sum(n * w.beta[0] // w.beta[1] for n in lens), hist=sum(f - 1 for f in frames) * patches,
                pairs=sum(f - 1 for f in frames) * patches * patches, group=w.group)


def _keys(w, scene, gen):
    """Keys [layers * kv heads, tokens, d] bf16 and window queries [layers, seqs, q heads, window, d] bf16 by
    workload's recipe."""
    lay, hk, G = scene.layout, w.n_kv_heads, w.group
    inv = D ** -0.5
    emb = torch.from_numpy(np.concatenate(scene.frame_emb)).to(DEV)
    spots = np.concatenate([np.arange(o, o + r * c) for o, r, c in lay.frame_meta])
    vis = torch.from_numpy(spots).to(DEV)
    k = torch.empty((w.n_layers, hk, lay.total_tokens, D), dtype=torch.bfloat16, device=DEV)
    q = torch.empty((w.n_layers, lay.n_seqs, w.n_q_heads, w.window, D), dtype=torch.bfloat16, device=DEV)
    cells = []
    for s in range(lay.n_seqs):
        off, _, cols = (int(x) for x in lay.seq_frames(s)[-1])
        u0, v0, h, ww = scene.element[s]
        cells.append(torch.tensor([off + (u0 + a) * cols + v0 + b for a in range(h) for b in range(ww)], device=DEV))
    for layer in range(w.n_layers):
        for h in range(hk):
            proj = torch.randn((D, D), generator=gen, device=DEV) * inv
            x = torch.randn((lay.total_tokens, D), generator=gen, device=DEV) * inv
            x[vis] = emb @ proj.T
            k[layer, h] = x
            for s in range(lay.n_seqs):
                noise = torch.randn((G, w.window, D), generator=gen, device=DEV) * 0.1
                q[layer, s, h * G:(h + 1) * G] = x[cells[s]].sum(0) + noise
    return k.view(w.n_layers * hk, -1, D), q


def prepare(case, seed):
    w = _workload(case, seed)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    lay = W.make_layout(w)
    p = S.Problem(w.n_layers, w.n_q_heads, w.n_kv_heads, w.window, lay.cu_seqlens, lay.cu_frames, lay.frame_meta,
                  S.budgets(lay.cu_seqlens, *w.beta), device=DEV)
    st = dict(kind=case["kind"], case=case, p=p, w=w, lay=lay)
    U, L, B = p.units, p.total_tokens, max(p.total_budget, 1)
    if case["kind"] == "decode":
        # keys and values of whatever rows the cache holds; queries near the sum of a few of them
        n = L if case["cache"] == "full" else B
        st["cache"] = S.CACHE_FULL if case["cache"] == "full" else S.CACHE_COMPACT
        st["k"] = torch.empty((U, n, D), dtype=torch.bfloat16, device=DEV)
        for u in range(U):
            st["k"][u] = torch.randn((n, D), generator=gen, device=DEV) * D ** -0.5
        st["v"] = torch.randn((U, n, D), generator=gen, device=DEV, dtype=torch.bfloat16)
        aim = st["k"][:, :4].float().sum(1).view(p.n_layers, 1, p.n_kv_heads, 1, D)
        noise = torch.randn((p.n_layers, p.n_seqs, p.n_kv_heads, w.group, D), generator=gen, device=DEV)
        st["q"] = (aim + 0.1 * noise).to(torch.bfloat16).view(p.n_layers, p.n_seqs, p.n_q_heads, D).contiguous()
        call = S.CALL_DECODE_FULL if case["cache"] == "full" else S.CALL_DECODE_COMPACT
        st["out"] = torch.empty((p.n_layers, p.n_seqs, p.n_q_heads, D), device=DEV)
        st["ws"] = torch.empty(max(p.workspace_size(call), 256), dtype=torch.uint8, device=DEV)
        return st
    if case["kind"] == "select":
        # a prior like the window score's, saliencies around 1, a gate that admits some of the history
        st["a"] = torch.exp(torch.randn((U, L), generator=gen, device=DEV)) * (w.window / L)
        st["phi"] = 1.0 + 0.03 * torch.randn((U, L), generator=gen, device=DEV)
        st["gate"] = (torch.rand((U, L), generator=gen, device=DEV) < 0.25).to(torch.uint8)
        for s in range(lay.n_seqs):
            fm = lay.seq_frames(s)
            hist = torch.zeros(L, dtype=torch.bool, device=DEV)
            for o, r, c in fm[:-1]:
                hist[o:o + r * c] = True
            a, b = int(lay.cu_seqlens[s]), int(lay.cu_seqlens[s + 1])
            st["gate"][:, a:b][:, ~hist[a:b]] = 1
        text = torch.from_numpy(W.text_positions(lay)).to(DEV)
        st["phi"][:, text] = 0.0
        st["k"] = torch.randn((U, L, D), generator=gen, device=DEV, dtype=torch.bfloat16)
        st["v"] = torch.randn((U, L, D), generator=gen, device=DEV, dtype=torch.bfloat16)
        st["kept"] = torch.empty((U, B), dtype=torch.int32, device=DEV)
        st["k_out"] = torch.empty((U, B, D), dtype=torch.int16, device=DEV)
        st["v_out"] = torch.empty((U, B, D), dtype=torch.int16, device=DEV)
        st["ws"] = torch.empty(max(p.workspace_size(S.CALL_SELECT_TOPK), 256), dtype=torch.uint8, device=DEV)
        return st
    st["k"], st["q"] = _keys(w, W.make_scene(w), gen)
    if case["kind"] == "css":
        st["phi"] = torch.empty((U, L), device=DEV)
        return st
    st["v"] = torch.randn((U, L, D), generator=gen, device=DEV, dtype=torch.bfloat16)
    if case["kind"] == "concat":
        st["pl"] = S.layer_problem(p)
    else:
        st["out"] = S.Buffers(p, device=DEV)
    return st


def run(st):
    p = st["p"]
    if st["kind"] == "pass":
        o = S.compress(p, st["q"], st["k"], st["v"], st["out"], alpha=st["w"].alpha)
        # The kept list, K' and V' follow from comparing scores: an ulp in one
        # score swaps two tokens and shifts every entry between them (and an ulp
        # of rho at the threshold gates a token in or out of phi and the
        # scores), so they say nothing about precision here; "select" returns
        # the list and the gathered rows for given scores, exactly.
        got = {"a_base": o.a_base, "rho": o.rho, "tau": o.tau, "gate": o.gate}
        if st["case"]["frames_max"] == 1:  # no history: nothing is gated
            got.update(phi=o.phi, score=o.score)
        return got
    if st["kind"] == "decode":
        return S.decode(p, st["q"], st["k"], st["v"], st["cache"], st["out"], st["ws"])
    if st["kind"] == "select":
        S.stlite_select_topk(p, st["a"], st["phi"], st["gate"], st["w"].alpha, st["kept"], None, st["ws"])
        S.stlite_compact_kv(p, st["k"], st["v"], st["kept"], st["k_out"], st["v_out"])
        return {"kept": st["kept"], "k_out": st["k_out"], "v_out": st["v_out"]}
    if st["kind"] == "css":
        S.stlite_css_saliency_nbhd(p, st["case"]["nbhd"], st["k"], st["phi"])
        return st["phi"]
    r = S.compress_concat(p, st["pl"], st["q"], st["k"], st["v"], alpha=st["w"].alpha)
    return {"a_layer": r["a_layer"], "rho": r["rho"], "tau": r["tau"], "gate": r["gate"]}


def work(case):
    s = _shape(case)
    U, L, B, layers = s["units"], s["tokens"], s["budget"], case["layers"]
    row = 2 * D
    q = layers * case["seqs"] * case["q_heads"] * D * 2
    if case["kind"] == "decode":
        n = L if case["cache"] == "full" else B
        return {"bytes": U * n * 2 * row + 3 * q, "flops": 4 * U * s["group"] * n * D}
    if case["kind"] == "select":
        return {"bytes": U * (L * 9 + B * 4 + 4 * B * row), "flops": 2 * U * L}
    if case["kind"] == "css":
        vis, cells = s["frames"] * s["patches"], case["nbhd"] ** 2
        return {"bytes": U * (vis * row + 4 * L), "flops": 2 * D * U * vis * ((cells - 1) // 2 + 1)}
    score = 2 * U * s["group"] * case["window"] * L * D
    rho = 2 * U * s["pairs"] * D
    css = 2 * D * U * s["frames"] * s["patches"] * 5
    # keys once, the kept rows of V once, both caches out; priors, similarity, gate, saliency, scores and lists out
    per = 1 if case["kind"] == "pass" else case["kv_heads"]
    out = U * L * 4 + U // per * (L * (4 + 1 + 4) + B * 4) + (U * L * 4 if case["kind"] == "pass" else U // per * L * 4)
    return {"bytes": U * (L * row + 3 * B * row) + q * case["window"] + out, "flops": score + rho + css}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    # four times the error against 64 bits (priors 5e-7, similarities 1e-7, decode 5e-7); a gate differs where
    # rho is within an ulp of its threshold
    return {"rel": 2e-6, "max": 1e-4, "differ": 1e-4}


def _f64_a_base(w, lay, q, k):
    a = torch.empty((k.shape[0], lay.total_tokens), dtype=torch.float64, device=DEV)
    for u in range(k.shape[0]):
        layer, kv = divmod(u, w.n_kv_heads)
        for s in range(lay.n_seqs):
            b, e = int(lay.cu_seqlens[s]), int(lay.cu_seqlens[s + 1])
            rows = q[layer, s, kv * w.group:(kv + 1) * w.group].double().reshape(-1, D)
            x = rows @ k[u, b:e].double().T * D ** -0.5
            x = x.view(w.group, w.window, e - b)
            for i in range(w.window):  # the window query i sees the keys up to its own position
                x[:, i, e - b - w.window + i + 1:] = -torch.inf
            a[u, b:e] = torch.softmax(x, -1).sum((0, 1)) / w.group
    return a


def _unit(x):
    n = x.norm(dim=-1, keepdim=True)
    return torch.where(n > 0, x / n, torch.zeros_like(x))


def _f64_rho(lay, k):
    """k [units, tokens, dims]: rho, and its m-th smallest value per sequence for budgets B."""
    rho = torch.zeros(k.shape[:2], dtype=torch.float64, device=DEV)
    for u in range(k.shape[0]):
        for s in range(lay.n_seqs):
            fm = lay.seq_frames(s)
            o, r, c = (int(x) for x in fm[-1])
            cur = _unit(k[u, o:o + r * c].double()).T.contiguous()
            for o, r, c in fm[:-1]:
                x = (_unit(k[u, o:o + r * c].double()) @ cur).amax(-1).clamp(-1, 1)
                rho[u, o:o + r * c] = torch.where(x >= 1 - 1e-4, torch.ones_like(x), x)
    return rho


def _f64_tau(p, lay, rho):
    tau = torch.full((rho.shape[0], p.n_seqs), torch.nan, dtype=torch.float64, device=DEV)
    B = np.diff(p.h["cu_budget"])
    for s in range(p.n_seqs):
        fm = lay.seq_frames(s)
        hist = torch.from_numpy(np.concatenate([np.arange(o, o + r * c) for o, r, c in fm[:-1]] or [np.empty(0, int)])).to(DEV)
        m = min(int(B[s]), len(hist))
        if m:
            tau[:, s] = rho[:, hist].sort(-1).values[:, m - 1]
    return tau


def _f64_phi(lay, k, nbhd):
    phi = torch.zeros(k.shape[:2], dtype=torch.float64, device=DEV)
    rad = nbhd // 2
    for u in range(k.shape[0]):
        for o, r, c in lay.frame_meta:
            x = _unit(k[u, o:o + r * c].double()).view(r, c, D)
            total = torch.zeros((r, c), dtype=torch.float64, device=DEV)
            count = torch.zeros((r, c), dtype=torch.float64, device=DEV)
            for i in range(-rad, rad + 1):
                for j in range(-rad, rad + 1):
                    if (i or j) and abs(i) < r and abs(j) < c:
                        a = (slice(max(0, i), r + min(0, i)), slice(max(0, j), c + min(0, j)))
                        b = (slice(max(0, -i), r + min(0, -i)), slice(max(0, -j), c + min(0, -j)))
                        total[b] += (x[a] * x[b]).sum(-1)
                        count[b] += 1
            y = 1 - total / count.clamp(min=1)
            phi[u, o:o + r * c] = torch.where(count > 0, y, torch.zeros_like(y)).reshape(-1)
    return phi


def exact(case, seed):
    st = prepare(case, seed)
    p, w, lay, k = st["p"], st["w"], st["lay"], st.get("k")
    if case["kind"] == "select":
        return None
    if case["kind"] == "css":
        return _f64_phi(lay, k, case["nbhd"]) if case["nbhd"] <= 5 else None
    if case["kind"] == "decode":
        cu = p.h["cu_seqlens" if case["cache"] == "full" else "cu_budget"]
        out = torch.zeros((p.n_layers, p.n_seqs, p.n_q_heads, D), dtype=torch.float64, device=DEV)
        for u in range(p.units):
            layer, kv = divmod(u, p.n_kv_heads)
            heads = slice(kv * w.group, (kv + 1) * w.group)
            for s in range(p.n_seqs):
                b, e = int(cu[s]), int(cu[s + 1])
                if e > b:
                    x = st["q"][layer, s, heads].double() @ k[u, b:e].double().T * D ** -0.5
                    out[layer, s, heads] = torch.softmax(x, -1) @ st["v"][u, b:e].double()
        return out
    a = _f64_a_base(w, lay, st["q"], k)
    if case["kind"] == "concat":
        k = k.view(p.n_layers, p.n_kv_heads, -1, D).permute(0, 2, 1, 3).reshape(p.n_layers, -1, p.n_kv_heads * D)
        rho = _f64_rho(lay, k)
        return {"a_layer": a.view(p.n_layers, p.n_kv_heads, -1).mean(1), "rho": rho,
                "tau": _f64_tau(p, lay, rho), "gate": None}
    rho = _f64_rho(lay, k)
    got = {"a_base": a, "rho": rho, "tau": _f64_tau(p, lay, rho), "gate": None}
    if case["frames_max"] == 1:
        phi = _f64_phi(lay, k, 3)
        vis = torch.ones(lay.total_tokens, dtype=torch.float64, device=DEV)
        vis[torch.from_numpy(W.text_positions(lay)).to(DEV)] = 0
        got.update(phi=phi, score=a + w.alpha * phi * vis)
    return got
