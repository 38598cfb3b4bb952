"""Performance cases: the calls a serving program makes through `paper_2609_34060_amd.kvc`, over their real range.

Every case is one call (or the calls that always go together) on data that is already on the GPU: correcting a
segment (`apply`), fitting an agent edge's state (`fit`, per KV head or per layer), composing two states (`chain`) and
one transfer estimated from an anchor pool (`anchored`: gate distances, token-wise weights, anchored apply).  Shapes
are the package's own workloads (synth.WORKLOADS and the shapes bench.py times).

Inputs: source rows are N(0, 1); a deviation has a decaying spectrum, one decade over the first `rank` directions,
that goes on for as many directions again below the truncation, RMS 0.25, plus N(0, 1e-2) noise.  The pool of a layer
holds the source sequences' blocks and then the destination sequences' blocks, each shuffled through its block tables.
"""
import math

import numpy as np
import torch

from paper_2609_34060_amd import kvc, synth

DEV = "cuda"
ROPE_THETA = 5e5
NOISE = 1e-2


def _case(name, op, **kw):
    c = {"name": name, "op": op, "layers": 32, "heads": 8, "dim": 128, "tokens": 4096, "requests": 1, "rank": 16,
         "rank2": 0, "anchors": 0, "dtype": "bf16", "block": 16, "paged": True, "rope": 0, "offset": 0, "shift": 0,
         "uncovered": 0, "grouping": "head"}
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: float32, contiguous rows, two layers (the "tiny" workload): latency only.
        _case("apply_tiny_f32", "apply", layers=2, heads=4, dim=64, tokens=256, rank=8, dtype="f32", paged=False),
        # The smallest fit: the same float32 edge, where the eigensolver and the launches are everything.
        _case("fit_tiny_f32", "fit", layers=2, heads=4, dim=64, tokens=256, rank=8, dtype="f32", paged=False),
        # An ordinary transfer of an 8B model: 4K shared tokens at rank 16.
        _case("apply_8b_4k", "apply"),
        # The longest single context: 32K shared tokens at rank 32.
        _case("apply_8b_32k", "apply", tokens=32768, rank=32),
        # A vision-language context with rotary keys that moves to another position, on a slot that no block starts
        # at; its last 77 rows are past the state's coverage (Appendix A.3).
        _case("apply_vlm_rope", "apply", layers=28, heads=4, tokens=3328, rank=32, rope=1, offset=5, shift=731,
              uncovered=77),
        # One layer of a serving batch: 64 requests of 1K-16K tokens in one launch at rank 64.
        _case("apply_serving", "apply", layers=1, tokens=16384, requests=64, rank=64),
        # The state of an ordinary edge after its dense prefill.
        _case("fit_8b_4k", "fit"),
        # The state of the longest edge.
        _case("fit_8b_32k", "fit", tokens=32768, rank=32),
        # One layer's states of the serving batch.
        _case("fit_serving", "fit", layers=1, tokens=16384, requests=64, rank=64),
        # The per-layer factorisation (all heads of a layer together, D = 1024) of the longest edge.
        _case("fit_layer_8b_32k", "fit", tokens=32768, rank=32, grouping="layer"),
        # Composing two edges of the longest context, 32 + 32 -> 32.
        _case("chain_8b_32k", "chain", tokens=32768, rank=32, rank2=32),
        # A transfer estimated from the default pool of ten anchors of rank 32 on a 4K segment.
        _case("anchored_8b_4k", "anchored", rank=32, anchors=10),
    ]


def draw(rng):
    def log_int(lo, hi):
        return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))

    op = rng.choices(["apply", "fit", "layer", "chain", "anchored"], [35, 25, 8, 12, 20])[0]
    heads, dim = rng.choice([(8, 128), (8, 128), (4, 128), (2, 128), (4, 64), (8, 64)])
    c = _case("", "fit" if op == "layer" else op, heads=heads, dim=dim)
    del c["name"]
    c["layers"] = log_int(1, 32)
    c["tokens"] = log_int(64, 32768)
    c["rank"] = rng.choice([8, 16, 16, 24, 32, 32, 48, 64]) if rng.random() < 0.85 else rng.randrange(3, 64)
    c["dtype"] = "f32" if rng.random() < 0.15 else "bf16"
    c["block"] = rng.choice([16, 16, 16, 8, 32, 64])
    c["paged"] = rng.random() < 0.9
    c["offset"] = rng.choice([0, rng.randrange(0, 4 * c["block"])])
    if op == "chain":
        c["rank2"] = rng.choice([c["rank"], 8, 16, 32])
        c["rank"] = min(c["rank"], dim - c["rank2"])
        c["tokens"] = max(c["tokens"], 8 * max(c["rank"], c["rank2"]))
    elif rng.random() < 0.3:
        c["rope"] = rng.choice([1, 1, 2])
        c["shift"] = rng.randrange(0, 5000)
    if op in ("apply", "fit") and rng.random() < 0.3:
        c["requests"] = log_int(2, 64)
        c["layers"] = min(c["layers"], 4)
    if op == "apply" and rng.random() < 0.15:
        c["grouping"] = "layer"
    if op in ("apply", "anchored") and rng.random() < 0.4:
        c["uncovered"] = rng.randrange(0, 1 + c["tokens"] // 8)
    if op == "layer":
        c["grouping"] = "layer"
        c["heads"], c["dim"] = rng.choice([(8, 128), (4, 128), (8, 64), (2, 128)])
        c["rank"] = min(c["rank"], 48)
        if c["dtype"] == "f32":
            c["rank"] = min(c["rank"], 32)
    if op == "anchored":
        c["anchors"] = rng.randrange(2, 17)
        c["rank"] = min(c["rank"], 32) if c["anchors"] > 8 else c["rank"]
    if c["op"] == "fit":
        c["rank"] = min(c["rank"], 48 if c["dim"] == 64 and op != "layer" else 64)
        # every request keeps at least eight rows for each direction of its state
        c["tokens"] = min(32768, max(c["tokens"], 8 * c["rank"] * (16 if c["requests"] > 1 else 1)))
    # no drawn case costs more than the largest listed one: the VALU kernels of float32 caches, the anchor sets and
    # the per-layer factorisation have tighter limits
    limit = 4e9 if c["dtype"] == "bf16" else 4e8
    limit /= {"anchored": 2, "layer": 2}.get(op, 1)
    while work(c)["bytes"] > limit:
        if c["layers"] > 1:
            c["layers"] = (c["layers"] + 1) // 2
        elif c["requests"] > 1:
            c["requests"] = (c["requests"] + 1) // 2
        else:
            c["tokens"] = c["tokens"] * 3 // 4
    c["uncovered"] = min(c["uncovered"], c["tokens"] // 8)
    return c


# ---- sizes -----------------------------------------------------------------------------------------------------

def _lengths(c):
    if c["requests"] == 1:
        return [c["tokens"]]
    rng = np.random.Generator(np.random.PCG64([1005, c["requests"], c["tokens"]]))
    return [int(x) for x in rng.integers(max(1, c["tokens"] // 16), c["tokens"] + 1, size=c["requests"])]


def _covered(c):
    return [max(0, t - c["uncovered"]) for t in _lengths(c)]


def _es(c):
    return 2 if c["dtype"] == "bf16" else 4


def work(case):
    c = case
    units, d, r, es = c["layers"] * 2 * c["heads"], c["dim"], c["rank"], _es(c)
    rows, cov = sum(_lengths(c)), sum(_covered(c))
    groups = c["layers"] * 2 if c["grouping"] == "layer" else units
    D = d * c["heads"] if c["grouping"] == "layer" else d
    basis = groups * len(_lengths(c)) * r * D * 4
    if c["op"] == "apply":
        return {"bytes": units * rows * 2 * d * es + groups * cov * r * es + basis, "flops": 2 * units * cov * d * r}
    if c["op"] == "fit":
        # rows of both sides read once, coefficients and bases written; Z^T Z (one triangle) and Z R
        return {"bytes": units * rows * 2 * d * es + groups * rows * r * es + basis,
                "flops": groups * rows * (D * (D + 1) + 2 * D * r)}
    if c["op"] == "chain":
        m, ro = r + c["rank2"], max(r, c["rank2"])
        return {"bytes": units * (rows * (m + ro) * es + (m + ro) * d * 4),
                "flops": units * rows * (m * (m + 1) + 2 * m * ro)}
    V, per = c["anchors"], d * es  # anchored
    gate = units // 2 * (cov * (per + V * r * es) + V * r * d * 4)
    weights = units * (cov * (per + V * r * es) + V * r * d * 4) + c["layers"] * 2 * cov * V * 4
    apply = units * (rows * 2 * per + cov * V * r * es + V * r * d * 4) + c["layers"] * 2 * cov * V * 4
    return {"bytes": gate + weights + apply, "flops": units * cov * V * r * d * 2 * 2.5}


def tolerance(case):
    return {"rel": 2e-5} if case["dtype"] == "f32" else {"rel": 8e-3}


# ---- inputs ----------------------------------------------------------------------------------------------------

def _dt(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _gen(c, seed, *keys):
    g = torch.Generator(device=DEV)
    g.manual_seed(synth.derive_seed(seed, c["tokens"], c["rank"], *keys))
    return g


def _spectrum(g, units, n, rank, D):
    """Decaying singular values [units, n] (one decade per `rank`) of rows of D features with RMS 0.25."""
    i = torch.arange(n, device=DEV, dtype=torch.float32) + 0.5 * torch.rand(units, n, generator=g, device=DEV)
    s = torch.pow(10.0, -i / rank)
    return s * (0.25 * math.sqrt(D) / s.square().sum(-1, keepdim=True).sqrt())


def _orthonormal(g, units, D, n):
    """Orthonormal directions [units, D, n], each with one outlier channel of its own (as K/V features have), so that
    the canonical sign of a singular vector does not hang on a tie of two entries."""
    v = torch.randn(units, D, n, generator=g, device=DEV)
    at = torch.rand(units, D, generator=g, device=DEV).argsort(dim=1)[:, :n].unsqueeze(1)
    return synth.orthonormal_columns(v.scatter_add_(1, at, torch.full_like(v[:, :1], 8.0)))


def _inv_freq(c):
    return [ROPE_THETA ** (-2.0 * i / c["dim"]) for i in range(c["dim"] // 2)]


def _rotate(x, c, pos):
    """R(pos) of rows x [..., dim] in x's own precision (angles in float64)."""
    if c["rope"] == 0 or pos == 0:
        return x
    th = torch.tensor(_inv_freq(c), dtype=torch.float64, device=x.device) * pos
    co, si = torch.cos(th).to(x.dtype), torch.sin(th).to(x.dtype)
    h = c["dim"] // 2
    if c["rope"] == 1:
        a, b = x[..., :h], x[..., h:]
        return torch.cat([a * co - b * si, a * si + b * co], dim=-1)
    a, b = x[..., 0::2], x[..., 1::2]
    return torch.stack([a * co - b * si, a * si + b * co], dim=-1).flatten(-2)


class _Layout:
    """Blocks of the source and the destination sequences of a case."""

    def __init__(self, c):
        bs, off = c["block"], c["offset"]
        self.lengths = _lengths(c)
        need = [-(-(off + t) // bs) for t in self.lengths]
        self.n_side = sum(need)
        self.max_blocks = max(need)
        self.starts = np.concatenate([[0], np.cumsum(need)]).astype(np.int64)
        rng = np.random.Generator(np.random.PCG64([31, c["tokens"], self.n_side]))
        self.tables = []  # logical block -> physical block, per side and request
        for side in range(2):
            ids = rng.permutation(self.n_side) if c["paged"] else np.arange(self.n_side)
            self.tables.append([side * self.n_side + ids[self.starts[q]:self.starts[q + 1]]
                                for q in range(len(need))])

    def rows(self, c, side, q):
        """(block, slot) index tensors of request q's rows on a side."""
        p = np.arange(self.lengths[q]) + c["offset"]
        return (torch.from_numpy(self.tables[side][q][p // c["block"]].astype(np.int64)).to(DEV),
                torch.from_numpy(p % c["block"]).to(DEV))

    def table(self, side):
        t = np.full((len(self.lengths), self.max_blocks), -1, dtype=np.int32)
        for q, ids in enumerate(self.tables[side]):
            t[q, :len(ids)] = ids
        return torch.from_numpy(t).to(DEV)

    def offsets(self, c, side):
        if c["paged"]:
            return [c["offset"]] * len(self.lengths)
        return [int(side * self.n_side + s) * c["block"] + c["offset"] for s in self.starts[:-1]]


def _positions(c):
    return (c["shift"] // 2, c["shift"]) if c["rope"] else (0, 0)


def _random_factors(c, g, units, D, rank, T):
    """Coefficients [units, T, rank] (storage dtype) and orthonormal basis rows [units, rank, D]."""
    s = _spectrum(g, units, rank, rank, D)
    coef = torch.empty(units, T, rank, dtype=_dt(c), device=DEV)
    for u in range(units):
        coef[u] = torch.randn(T, rank, generator=g, device=DEV) * s[u]
    return coef, _orthonormal(g, units, D, rank).transpose(-2, -1).contiguous()


def _states(c, g, fill, ranks=None, tokens=None):
    """States of a case's requests, their arrays cut from one slab each: (states, slabs)."""
    L, H, d, r = c["layers"], c["heads"], c["dim"], c["rank"]
    layerwise = c["grouping"] == "layer"
    units, D = (L * 2, H * d) if layerwise else (L * 2 * H, d)
    cov = tokens if tokens is not None else _covered(c)
    starts = np.concatenate([[0], np.cumsum([-(-units * t * r // 64) * 64 for t in cov])])
    coef = torch.zeros(int(starts[-1]), dtype=_dt(c), device=DEV)
    basis = torch.zeros(len(cov), units * r * D, dtype=torch.float32, device=DEV)
    sigma = torch.zeros(len(cov), units * r, dtype=torch.float32, device=DEV)
    states = []
    for q, t in enumerate(cov):
        cq = coef[int(starts[q]):int(starts[q]) + units * t * r]
        if fill:
            a, b = _random_factors(c, g, units, D, r, t)
            cq.copy_(a.flatten())
            basis[q].copy_(b.flatten())
            sigma[q].copy_(a.float().norm(dim=1).flatten())
        if layerwise:
            states.append(kvc.State(cq.view(L, 2, t, r), basis[q].view(L, 2, r, H, d), sigma[q].view(L, 2, r)))
        else:
            states.append(kvc.State(cq.view(L, 2, H, t, r), basis[q].view(L, 2, H, r, d),
                                    sigma[q].view(L, 2, H, r)))
    return states, {"coef": coef, "basis": basis, "sigma": sigma}


def _cache(c, slab):
    L = c["layers"]
    return kvc.Cache([slab[l, 0] for l in range(L)], [slab[l, 1] for l in range(L)], rope_style=c["rope"],
                     rope_inv_freq=_inv_freq(c) if c["rope"] else None)


def _batch(c, lay, states):
    n = len(lay.lengths)
    ps, pd = _positions(c)
    return kvc.Batch(lay.lengths, lay.offsets(c, 0), lay.offsets(c, 1), states,
                     lay.table(0) if c["paged"] else None, lay.table(1) if c["paged"] else None, device=DEV,
                     src_positions=[ps] * n, dst_positions=[pd] * n)


def _slab(c, lay, g):
    """Pools [layers, K/V, blocks, block, heads, dim]: source rows N(0, 1), destination rows zero."""
    slab = torch.zeros(c["layers"], 2, 2 * lay.n_side, c["block"], c["heads"], c["dim"], dtype=_dt(c), device=DEV)
    for l in range(c["layers"]):
        for kv in range(2):
            slab[l, kv, :lay.n_side] = torch.randn(lay.n_side, c["block"], c["heads"], c["dim"], generator=g,
                                                   device=DEV).to(_dt(c))
    return slab


def _fill_destination(c, lay, slab, g):
    """Destination rows: the source agent's row plus a deviation of decaying spectrum, each rounded once; the keys of
    a rotary cache are rotated to the positions of their side."""
    H, d, r = c["heads"], c["dim"], c["rank"]
    layerwise = c["grouping"] == "layer"
    D, per = (H * d, 1) if layerwise else (d, H)
    n = min(2 * r, 3 * D // 4)
    ps, pd = _positions(c)
    reqs, L = len(lay.lengths), c["layers"]
    v = _orthonormal(g, L * 2 * reqs * per, D, n).view(L, 2, reqs, per, D, n)
    s = _spectrum(g, L * 2 * reqs * per, n, r, D).view(L, 2, reqs, per, 1, n)
    index = [[lay.rows(c, side, q) for side in range(2)] for q in range(reqs)]
    for l in range(L):
        for kv in range(2):
            basis = (v[l, kv] * s[l, kv]).transpose(-2, -1).contiguous()  # [reqs, per, n, D]
            for q, T in enumerate(lay.lengths):
                x = torch.randn(T, H, d, generator=g, device=DEV)
                w = math.sqrt(T) * synth.orthonormal_columns(torch.randn(per, T, n, generator=g, device=DEV))
                dev = torch.matmul(w, basis[q]) + NOISE * torch.randn(per, T, D, generator=g, device=DEV)
                dev = dev.transpose(0, 1).reshape(T, H, d)
                for side, (rows, pos) in enumerate(((x, ps), (x + dev, pd))):
                    b, sl = index[q][side]
                    slab[l, kv][b, sl] = (_rotate(rows, c, pos) if kv == 0 else rows).to(_dt(c))


def prepare(case, seed):
    c = case
    g = _gen(c, seed, 1)
    if c["op"] == "chain":
        st = {"c": c}
        for name, r, t in (("first", c["rank"], c["tokens"]), ("second", c["rank2"], c["tokens"])):
            st[name] = _states(dict(c, rank=r), g, True, tokens=[t])[0][0]
        out_c = dict(c, rank=max(c["rank"], c["rank2"]))
        (st["out"],), st["slabs"] = _states(out_c, g, False, tokens=[c["tokens"]])
        need = kvc.kvc_chain_workspace_bytes(st["first"], st["second"], st["out"])
        st["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
        return st
    lay = _Layout(c)
    slab = _slab(c, lay, g)
    cache = _cache(c, slab)
    st = {"c": c, "lay": lay, "slab": slab, "cache": cache, "dst": slab[:, :, lay.n_side:]}
    if c["op"] == "apply":
        states, _ = _states(c, g, True)
        st["batch"] = _batch(c, lay, states)
    elif c["op"] == "fit":
        _fill_destination(c, lay, slab, g)
        states, st["slabs"] = _states(c, g, False)
        st["batch"] = _batch(c, lay, states)
        need = kvc.kvc_fit_workspace_bytes(cache, st["batch"])
        st["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
    else:
        _prepare_anchors(c, lay, slab, g, st)
    return st


def _prepare_anchors(c, lay, slab, g, st):
    """The pool's anchors share a base of rank `rank` with the segment: the source rows are that base plus noise, and
    anchor v's coefficients differ from it by a share that grows over the anchors (near and far contexts)."""
    L, H, d, r, V = c["layers"], c["heads"], c["dim"], c["rank"], c["anchors"]
    T, (Ts,) = lay.lengths[0], _covered(c)
    units = L * 2 * H
    ps, _ = _positions(c)
    base = _orthonormal(g, units, d, r).transpose(-2, -1).contiguous().view(L, 2, H, r, d)
    s = (4 * _spectrum(g, units, r, r, d)).view(L, 2, H, 1, r)
    coefs = [torch.empty(L, 2, H, Ts, r, dtype=_dt(c), device=DEV) for _ in range(V)]
    b, sl = lay.rows(c, 0, 0)
    for l in range(L):
        for kv in range(2):
            a0 = torch.randn(H, T, r, generator=g, device=DEV) * s[l, kv]
            rows = torch.matmul(a0, base[l, kv]) + 0.3 * torch.randn(H, T, d, generator=g, device=DEV)
            rows = _rotate(rows, c, ps) if kv == 0 else rows
            slab[l, kv][b, sl] = rows.transpose(0, 1).to(_dt(c))
            for v in range(V):
                off = (0.05 + 0.9 * v / V) * torch.randn(H, Ts, r, generator=g, device=DEV) * s[l, kv]
                coefs[v][l, kv] = (a0[:, :Ts] + off).to(_dt(c))
    bases = [kvc.State(a, base.clone()) for a in coefs]
    deltas = []
    for _ in range(V):
        a, bb = _random_factors(c, g, units, d, r, Ts)
        deltas.append(kvc.State(a.view(L, 2, H, Ts, r), bb.view(L, 2, H, r, d)))
    empty = kvc.State(torch.zeros(L, 2, H, 0, 0, dtype=_dt(c), device=DEV),
                      torch.zeros(L, 2, H, 0, d, dtype=torch.float32, device=DEV))
    st["bases"] = kvc.Anchors(bases, Ts, L)
    st["deltas"] = st["bases"].with_states(deltas)
    st["batch"] = _batch(c, lay, [empty])
    st["prefix"] = max(1, Ts)
    st["distances"] = torch.zeros(V, dtype=torch.float32, device=DEV)
    need = kvc.kvc_gate_workspace_bytes(st["cache"], st["bases"], st["prefix"])
    st["workspace"] = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)


# ---- one pass ----------------------------------------------------------------------------------------------------

def run(state):
    st = state
    op = st["c"]["op"]
    if op == "apply":
        kvc.kvc_apply(st["cache"], st["batch"])
        return st["dst"]
    if op == "fit":
        kvc.kvc_fit_state(st["cache"], st["batch"], workspace=st["workspace"])
        return st["slabs"]
    if op == "chain":
        kvc.kvc_chain(st["first"], st["second"], st["out"], workspace=st["workspace"])
        return st["slabs"]
    # a transfer: the three launches are queued together; the program reads the distances when it needs its decision
    kvc.kvc_gate_distances(st["cache"], st["batch"], st["bases"], st["prefix"], distances=st["distances"],
                           workspace=st["workspace"])
    kvc.kvc_anchor_weights(st["cache"], st["batch"], st["bases"])
    kvc.kvc_apply_anchored(st["cache"], st["batch"], st["deltas"])
    return {"distances": st["distances"], "weights": st["bases"].weights, "dst": st["dst"]}


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

def _f64_rows(c, lay, slab, l, kv, side, q):
    b, s = lay.rows(c, side, q)
    return slab[l, kv][b, s].to(torch.float64)  # [T, H, d]


def _top(gram, r):
    """Top-r eigenvectors (columns, canonical sign: the first entry within 2^-20 of the largest magnitude positive)
    and singular values of Gram matrices [n, D, D]."""
    lam, vec = torch.linalg.eigh(gram.cpu())
    lam, vec = lam[:, -r:].flip(-1), vec[:, :, -r:].flip(-1)
    mag = vec.abs()
    first = (mag >= mag.amax(dim=1, keepdim=True) * (1 - 2.0 ** -20)).to(torch.uint8).argmax(dim=1, keepdim=True)
    vec = vec * torch.sign(vec.gather(1, first))
    return vec.to(gram.device), lam.clamp_min(0).sqrt().to(gram.device)


def _pack(c, per_request, rank):
    """Per request (coef [units, T, r], basis [units, r, D], sigma [units, r]) into the slabs of _states."""
    coefs = []
    for coef, _, _ in per_request:
        n = coef.numel()
        coefs.append(torch.cat([coef.flatten(), torch.zeros(-n % 64, dtype=torch.float64, device=DEV)]))
    return {"coef": torch.cat(coefs), "basis": torch.stack([x[1].flatten() for x in per_request]),
            "sigma": torch.stack([x[2].flatten() for x in per_request])}


def _exact_apply(c, st):
    lay, slab, H, d, r = st["lay"], st["slab"], c["heads"], c["dim"], c["rank"]
    ps, pd = _positions(c)
    out = torch.zeros(st["dst"].shape, dtype=torch.float64, device=DEV)
    for q, cov in enumerate(_covered(c)):
        state = st["batch"].states[q]
        b, s = lay.rows(c, 1, q)
        for l in range(c["layers"]):
            for kv in range(2):
                x = _f64_rows(c, lay, slab, l, kv, 0, q)
                x = _rotate(x, c, -ps) if kv == 0 else x
                a, bb = state.coef[l, kv].double(), state.basis[l, kv].double()
                if c["grouping"] == "layer":
                    x[:cov] += torch.matmul(a, bb.reshape(r, H * d)).view(cov, H, d)
                else:
                    x[:cov] += torch.matmul(a, bb).transpose(0, 1)
                out[l, kv][b - lay.n_side, s] = _rotate(x, c, pd) if kv == 0 else x
    return out


def _exact_fit(c, st):
    lay, slab, H, d, r = st["lay"], st["slab"], c["heads"], c["dim"], c["rank"]
    ps, pd = _positions(c)
    layerwise = c["grouping"] == "layer"

    def deviation(l, kv, q):
        x, y = (_f64_rows(c, lay, slab, l, kv, side, q) for side in range(2))
        z = y - x if kv == 1 else _rotate(y, c, -pd) - _rotate(x, c, -ps)
        return z.reshape(1, -1, H * d) if layerwise else z.transpose(0, 1).contiguous()

    found = []
    for q in range(len(lay.lengths)):
        pairs = [(l, kv) for l in range(c["layers"]) for kv in range(2)]
        grams = []
        for l, kv in pairs:
            z = deviation(l, kv, q)
            grams.append(torch.matmul(z.transpose(-2, -1).contiguous(), z))
        vec, sigma = _top(torch.cat(grams), r)
        per = vec.shape[0] // len(pairs)
        coef = torch.cat([torch.matmul(deviation(l, kv, q), vec[i * per:(i + 1) * per].contiguous())
                          for i, (l, kv) in enumerate(pairs)])
        found.append((coef, vec.transpose(-2, -1).contiguous(), sigma))
    return _pack(c, found, r)


def _exact_chain(c, st):
    out = st["out"]
    r, units, d = out.rank, c["layers"] * 2 * c["heads"], c["dim"]
    parts = [(s.coef.reshape(units, -1, s.rank), s.basis.reshape(units, s.rank, d))
             for s in (st["first"], st["second"])]

    def total(u):
        return sum(torch.matmul(a[u].double(), b[u].double()) for a, b in parts)

    grams = []
    for u in range(units):
        z = total(u)
        grams.append(torch.matmul(z.t().contiguous(), z))
    vec, sigma = _top(torch.stack(grams), r)
    coef = torch.stack([torch.matmul(total(u), vec[u].contiguous()) for u in range(units)])
    return _pack(c, [(coef, vec.transpose(-2, -1).contiguous(), sigma)], r)


def _exact_anchored(c, st):
    lay, slab, V = st["lay"], st["slab"], c["anchors"]
    (Ts,), ps, pd = _covered(c), *_positions(c)
    square = torch.zeros(V, dtype=torch.float64, device=DEV)
    weights = torch.zeros(c["layers"], 2, Ts, V, dtype=torch.float64, device=DEV)
    out = torch.zeros(st["dst"].shape, dtype=torch.float64, device=DEV)
    b, s = lay.rows(c, 1, 0)
    for l in range(c["layers"]):
        for kv in range(2):
            x = _f64_rows(c, lay, slab, l, kv, 0, 0)
            x = _rotate(x, c, -ps) if kv == 0 else x
            top, dist = x[:Ts].transpose(0, 1), []
            for v, a in enumerate(st["bases"].states):
                off = top - torch.matmul(a.coef[l, kv].double(), a.basis[l, kv].double())
                dist.append(off.abs().mean(dim=(0, 2)))
                if kv == 1:
                    square[v] += off[:, :st["prefix"]].square().sum()
            w = torch.softmax(-torch.stack(dist, dim=-1), dim=-1)
            weights[l, kv] = w
            for v, a in enumerate(st["deltas"].states):
                corr = torch.matmul(a.coef[l, kv].double(), a.basis[l, kv].double()).transpose(0, 1)
                x[:Ts] += w[:, v, None, None] * corr
            out[l, kv][b - lay.n_side, s] = _rotate(x, c, pd) if kv == 0 else x
    return {"distances": square.sqrt(), "weights": weights, "dst": out}


def exact(case, seed):
    st = prepare(case, seed)
    return {"apply": _exact_apply, "fit": _exact_fit, "chain": _exact_chain, "anchored": _exact_anchored}[
        case["op"]](case, st)
