"""The calls whose time counts: what a program that uses this package has it do, and the values it gets.

Three kinds of case, all through the package's public calls:

  self    hierarchical self-attention of one encoder layer: (layout build,) forward (, backward)
  cross   decoder cross-attention over a level subset of the encoder's positions
  front   the positional encoding in front of the encoder: parents from levels, index vectors, the add

The listed sizes are the benchmark's five configurations and the sizes of the tests; `draw` spreads over the
same ranges.  Documents are drawn from the seed with the benchmark's recipes (sections of 3-30 sentences, of 5-60
or 10-80 tokens each; pseudo-sections of 32 sentences; ListOps-shaped trees), Q, K, V and dO are iid N(0, 1).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2407_08330_amd as hdt
from paper_2407_08330_amd import inputs

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _self(name, batch, heads, head_dim, n_pos, doc, *, sent_lo=10, sent_hi=80, dtype="bf16", tile="128x64", edges=7,
          build=True, deferred=True, backward=True):
    case = dict(kind="self", batch=batch, heads=heads, head_dim=head_dim, n_pos=n_pos, doc=doc, sent_lo=sent_lo,
                sent_hi=sent_hi, dtype=dtype, tile=tile, edges=edges, build=build, deferred=deferred, backward=backward)
    return dict(case, name=name) if name else case


def _cross(name, batch, heads, head_dim, n_enc, n_dec, level_mask, *, build, backward=True):
    case = dict(kind="cross", batch=batch, heads=heads, head_dim=head_dim, n_enc=n_enc, n_dec=n_dec,
                level_mask=level_mask, build=build, backward=backward, sent_lo=10, sent_hi=80)
    return dict(case, name=name) if name else case


def _front(name, batch, n_pos, d_model, dtype, table_rows=1024):
    case = dict(kind="front", batch=batch, n_pos=n_pos, d_model=d_model, dtype=dtype, table_rows=table_rows, sent_lo=10,
                sent_hi=80)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest configuration: one document of 512 positions, one head, in the fp32 path (the run that checks
        # a model's numbers), the mask's own gradient included
        _self("check-f32-512", 1, 1, 64, 512, "sections", sent_lo=5, sent_hi=60, dtype="f32", deferred=False),
        # one ragged document through one encoder layer, forward only: a request that is served, where latency and
        # launches count; the plain build that waits
        _self("serve-1000", 1, 12, 64, 1000, "sections", sent_lo=5, sent_hi=60, deferred=False, backward=False),
        # an encoder-sized batch, forward, with the batch's layout
        _self("encoder-4096", 8, 12, 64, 4096, "sections", sent_lo=5, sent_hi=60, backward=False),
        # an inner layer of a long-document encoder, forward: the batch's layout is there already
        _self("longdoc-layer-8192", 4, 12, 64, 8192, "sections", build=False, backward=False),
        # the training step the benchmark's metric is quoted on: build, forward, backward
        _self("train-8192", 4, 12, 64, 8192, "sections", tile="64x32"),
        # the same on one very long document at head size 128
        _self("train-32768-d128", 1, 16, 128, 32768, "sections", sent_lo=5, sent_hi=60, tile="64x32"),
        # an inner layer's forward and backward on flat text in pseudo-sections, an odd length, the default tiles
        _self("pseudo-layer-2047", 3, 12, 64, 2047, "pseudo", build=False),
        # a training step under a thinned (directed) mask on ListOps-shaped trees: small trees, two schedules
        _self("listops-1536", 16, 4, 64, 1536, "tree", edges=6, tile="64x32"),
        # decoder layer of a summarisation model that sees the [SEC] and [SENT] anchors: build, forward, backward
        _cross("cross-anchors", 4, 12, 64, 8192, 512, 6, build=True),
        # an inner decoder layer that sees the regular tokens as well; the layout is there already
        _cross("cross-tokens-layer", 4, 12, 64, 8192, 512, 14, build=False),
        # the encoder's front end on a batch of embeddings
        _front("front-8192", 4, 8192, 768, "bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["self", "self", "self", "self", "check", "tree", "cross", "cross", "front"])
    if what == "check":
        return _self(None, 1, rng.randint(1, 4), rng.choice([64, 128]), _log_int(rng, 100, 1000), "sections", sent_lo=5,
                     sent_hi=60, dtype="f32", deferred=False, backward=rng.random() < 0.5)
    if what == "tree":
        n = _log_int(rng, 256, 2048)
        return _self(None, rng.randint(1, max(1, 24576 // n)), rng.choice([2, 4, 8]), 64, n, "tree",
                     edges=rng.choice([6, 4, 7]), tile=rng.choice(["64x32", "128x64"]))
    if what == "cross":
        mask = rng.choice([2, 6, 14])
        n_enc, n_dec = _log_int(rng, 512, 8192), _log_int(rng, 64, 512)
        return _cross(None, rng.randint(1, 4), rng.choice([4, 8, 12]), 64 if mask == 14 else rng.choice([64, 128]), n_enc,
                      n_dec, mask, build=rng.random() < 0.5, backward=rng.random() < 0.7)
    if what == "front":
        n = _log_int(rng, 512, 32768)
        return _front(None, rng.randint(1, max(1, 32768 // n)), n, rng.choice([512, 768, 1024]),
                      rng.choice(["bf16", "bf16", "f32"]))
    d, heads, n = rng.choice([64, 64, 128]), rng.choice([4, 8, 12, 16]), _log_int(rng, 256, 32768)
    most = max(1, 50_000_000 // (d * heads * n))
    lo, hi = rng.choice([(5, 60), (10, 80)])
    return _self(None, rng.randint(1, min(8, most)), heads, d, n, rng.choice(["sections", "sections", "pseudo"]), sent_lo=lo,
                 sent_hi=hi, tile=rng.choice(["64x32", "128x64"]), build=rng.random() < 0.6, deferred=rng.random() < 0.6,
                 backward=rng.random() < 0.6)


# ---- inputs ---------------------------------------------------------------------------------------------------
def _sections(rng, n_pos, lo, hi):
    """Sections of 3-30 sentences of lo-hi tokens until the next sentence does not fit; the tail is pad."""
    sections, used, full = [], 1, False
    while not full:
        section = []
        for _ in range(int(rng.integers(3, 31))):
            length = int(rng.integers(lo, hi + 1))
            cost = 1 + length + (0 if section else 1)
            full = used + cost > n_pos
            if full:
                break
            used += cost
            section.append(length)
        if section:
            sections.append(section)
    return sections


def _documents(case, seed, n_pos):
    """level, parent: int32 [batch][n_pos] on the host."""
    levels, parents = [], []
    for b in range(case["batch"]):
        rng = np.random.default_rng([seed, b, n_pos])
        doc = case.get("doc", "sections")
        if doc == "tree":
            lv, pr = inputs.listops_like_tree(rng, n_pos)
        elif doc == "pseudo":
            lv, pr, _ = inputs.pseudo_section_document(rng, n_pos, (case["sent_lo"], case["sent_hi"]))
        else:
            lv, pr = inputs.document_from_sections(_sections(rng, n_pos, case["sent_lo"], case["sent_hi"]), n_pos)
        levels.append(lv)
        parents.append(pr)
    return np.stack(levels), np.stack(parents)


def _tile(case):
    m, n = case["tile"].split("x")
    return dict(tile_m=int(m), tile_n=int(n))


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    state = dict(case=case)
    if case["kind"] == "front":
        level, _ = _documents(case, seed, case["n_pos"])
        state["level"] = torch.from_numpy(level).cuda()
        state["x"] = _normal(gen, (case["batch"], case["n_pos"], case["d_model"]), DTYPES[case["dtype"]])
        state["table"] = hdt.hdt_hpe_table(case["table_rows"], case["d_model"])
        return state
    B, H, D = case["batch"], case["heads"], case["head_dim"]
    state["scale"] = 1.0 / math.sqrt(D)
    if case["kind"] == "self":
        level, parent = _documents(case, seed, case["n_pos"])
        state["level"], state["parent"] = torch.from_numpy(level).cuda(), torch.from_numpy(parent).cuda()
        n_q = n_kv = case["n_pos"]
        dtype = DTYPES[case["dtype"]]
        if not case["build"]:
            state["layout"] = hdt.hdt_build_layout(state["level"], state["parent"], edges=case["edges"], **_tile(case))
    else:
        level, _ = _documents(case, seed, case["n_enc"])
        state["level"] = torch.from_numpy(level).cuda()
        n_q, n_kv, dtype = case["n_dec"], case["n_enc"], torch.bfloat16
        kept = hdt.hdt_build_cross_layout(state["level"], n_q, case["level_mask"])
        # the forward's workspace for long key lists: a program keeps one for all its layers
        need = hdt.hdt_attn_fwd_workspace_bytes(kept, H, D, 0)
        state["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda") if need else None
        if not case["build"]:
            state["layout"] = kept
    state["q"] = _normal(gen, (B, H, n_q, D), dtype)
    state["k"] = _normal(gen, (B, H, n_kv, D), dtype)
    state["v"] = _normal(gen, (B, H, n_kv, D), dtype)
    if case["backward"]:
        state["d_o"] = _normal(gen, (B, H, n_q, D), dtype)
    return state


# ---- one pass -------------------------------------------------------------------------------------------------
def run(state):
    case = state["case"]
    if case["kind"] == "front":
        parent = hdt.hdt_parents_from_levels(state["level"])
        p = hdt.hdt_index_vectors(state["level"], parent, 3)
        return dict(parent=parent, p=p, x=hdt.hdt_hpe_add(p, state["table"], state["x"]))
    layout = state.get("layout")
    if layout is None:
        if case["kind"] == "self":
            layout = hdt.hdt_build_layout(state["level"], state["parent"], edges=case["edges"],
                                          deferred=case["deferred"], **_tile(case))
        else:
            layout = hdt.hdt_build_cross_layout(state["level"], case["n_dec"], case["level_mask"])
    q, k, v, scale = state["q"], state["k"], state["v"], state["scale"]
    o, lse = hdt.hdt_attn_fwd(layout, q, k, v, scale, workspace=state.get("workspace"))
    out = dict(o=o, lse=lse)
    if case["backward"]:
        out["dq"], out["dk"], out["dv"] = hdt.hdt_attn_bwd(layout, q, k, v, o, lse, state["d_o"], scale)
    if "layout" not in state:
        layout.destroy()
    return out


# ---- what a pass cannot do without ----------------------------------------------------------------------------
def _pairs(case):
    """Allowed (query, key) pairs of one head over the batch, on documents of this case."""
    if case["kind"] == "cross":
        level, _ = _documents(case, 0, case["n_enc"])
        return case["n_dec"] * int(sum(((level == l).sum() for l in range(4) if case["level_mask"] >> l & 1)))
    level, parent = _documents(case, 0, case["n_pos"])
    real, child = int((level >= 0).sum()), int((parent >= 0).sum())
    pairs = real  # every position and itself
    for row in parent:
        c = np.bincount(row[row >= 0]).astype(np.int64)
        pairs += int((c * c - c).sum()) if case["edges"] & 2 else 0
    return pairs + child * ((case["edges"] & 1) + (case["edges"] >> 2 & 1))


def work(case):
    if case["kind"] == "front":
        positions = case["batch"] * case["n_pos"]
        x = positions * case["d_model"]
        return {"bytes": positions * (4 + 4 + 12) + 2 * x * (2 if case["dtype"] == "bf16" else 4), "flops": 3 * x}
    bh, D = case["batch"] * case["heads"], case["head_dim"]
    size = 4 if case.get("dtype") == "f32" else 2
    n_q = case["n_pos"] if case["kind"] == "self" else case["n_dec"]
    n_kv = case["n_pos"] if case["kind"] == "self" else case["n_enc"]
    pairs = _pairs(case)
    # K and V: the rows that the mask makes visible
    seen = bh * n_kv if case["kind"] == "self" else case["heads"] * pairs // n_q
    rows = 2 * bh * n_q + 2 * seen                                        # q, o; k, v
    rows += 2 * bh * n_q + 2 * bh * n_kv if case["backward"] else 0       # d_o, dq; dk, dv
    ids = (8 if case["kind"] == "self" else 4) * case["batch"] * n_kv if case["build"] else 0
    return {"bytes": rows * D * size + 4 * bh * n_q + ids, "flops": (14 if case["backward"] else 4) * pairs * case["heads"] * D}


def tolerance(case):
    # fp32: sums of up to a few hundred products in another order.  bf16: inputs are exact, probabilities and results
    # are rounded to 8 bits.  front: the ids are whole numbers; x is one rounding of an fp32 sum.
    if case["kind"] == "front":
        return {"rel": 1e-3 if case["dtype"] == "bf16" else 1e-6, "max": 0.01 if case["dtype"] == "bf16" else 1e-5, "differ": 0.0}
    if case.get("dtype") == "f32":
        return {"rel": 5e-6, "max": 2e-4}
    return {"rel": 0.012, "max": 0.2}


# ---- the same in 64 bits --------------------------------------------------------------------------------------
def _allowed(level, parent, r0, r1, edges):
    """Rows r0..r1 of one sample's mask, from the definition (parent, siblings, children, itself; no pads)."""
    pos = torch.arange(level.numel(), device=level.device)
    i, pi, pj = pos[r0:r1, None], parent[r0:r1, None], parent[None, :]
    m = i == pos[None, :]
    if edges & 1:
        m |= pi == pos[None, :]
    if edges & 2:
        m |= (pi == pj) & (pi >= 0)
    if edges & 4:
        m |= pj == i
    return m & (level >= 0)[None, :] & (level >= 0)[r0:r1, None]


def _exact_attention(state, case):
    q, k, v, d_o, scale = state["q"], state["k"], state["v"], state.get("d_o"), state["scale"]
    B, H, n_q, _ = q.shape
    out = dict(o=torch.zeros(q.shape, dtype=torch.float64, device="cuda"),
               lse=torch.full((B, H, n_q), -math.inf, dtype=torch.float64, device="cuda"))
    if case["backward"]:
        for name, like in (("dq", q), ("dk", k), ("dv", k)):
            out[name] = torch.zeros(like.shape, dtype=torch.float64, device="cuda")
    step = 4096
    for b in range(B):
        level = state["level"][b]
        for r0 in range(0, n_q, step):
            r1 = min(n_q, r0 + step)
            if case["kind"] == "self":
                mask = _allowed(level, state["parent"][b], r0, r1, case["edges"])
            else:
                seen = torch.zeros_like(level, dtype=torch.bool)
                for l in range(4):
                    if case["level_mask"] >> l & 1:
                        seen |= level == l
                mask = seen[None, :].expand(r1 - r0, -1)
            dead = ~mask.any(dim=1)
            for h in range(H):
                qd, kd, vd = q[b, h, r0:r1].double(), k[b, h].double(), v[b, h].double()
                s = (qd @ kd.T).mul_(scale).masked_fill_(~mask, -math.inf)
                lse = torch.logsumexp(s, dim=1)
                p = s.sub_(lse.masked_fill(dead, 0.0)[:, None]).exp_()
                o = p @ vd
                out["lse"][b, h, r0:r1], out["o"][b, h, r0:r1] = lse, o
                if case["backward"]:
                    do = d_o[b, h, r0:r1].double()
                    out["dv"][b, h] += p.T @ do
                    ds = (do @ vd.T).sub_((do * o).sum(dim=1, keepdim=True)).mul_(p).mul_(scale)
                    out["dq"][b, h, r0:r1] = ds @ kd
                    out["dk"][b, h] += ds.T @ qd
    return out


def _exact_front(state, case):
    level = state["level"].cpu().numpy()
    B, N, d = case["batch"], case["n_pos"], case["d_model"]
    p = np.zeros((B, N, 3), np.int64)
    for b in range(B):
        last, count = [-1] * 4, [0] * 4     # last position and ordinal of every level on the path to the root
        for i, l in enumerate(level[b]):
            if l < 0:
                continue
            count[l] += 1
            count[l + 1:] = [0] * (3 - l)
            last[l] = i
            p[b, i, :l] = count[1:l + 1]
    w = 10000.0 ** (-2.0 * (torch.arange(d, device="cuda", dtype=torch.float64) // 2) / d)
    x = state["x"].double()
    for l in range(3):
        a = torch.from_numpy(p[:, :, l]).cuda().double()[:, :, None] * w
        x += torch.where(torch.arange(d, device="cuda") % 2 == 0, a.sin(), a.cos())
    return dict(parent=None, p=None, x=x)


def exact(case, seed):
    state = prepare(case, seed)
    return _exact_front(state, case) if case["kind"] == "front" else _exact_attention(state, case)
