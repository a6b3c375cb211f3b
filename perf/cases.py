"""The workloads by which the speed of this framework is measured.

One speculative-decoding round has three parts on the GPU, and each has its
cases here, called through the Python binding as a serving program calls it:

* building the round's draft tree (``TreeBuilder.run``; ``chain_decode`` for the
  plain greedy chain), from one small float32 request to a batch of eight
  requests at the 14B drafter's shape;
* one tree-masked attention layer of the verification forward
  (``TreeAttention``);
* the bookkeeping after it (``build_retrieve``, ``accept_greedy``, ``compact_kv``).

``listed()`` holds the named cases, ``draw(rng)`` one more of the same ranges.
Inputs are synthetic with the distributions of ``synth.py`` (base logits with a
few peaks at Zipf-distributed tokens, small Gaussian head weights), made on the
GPU from a seed.  ``exact`` evaluates the same definitions in float64 with
plain torch.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_02123_amd import pctree as P

_DT = {"f32": (torch.float32, P.F32), "bf16": (torch.bfloat16, P.BF16)}
_MODES = {"parent": P.MODE_PARENT, "shared": P.MODE_SHARED, "independent": P.MODE_INDEPENDENT}


def _round(name, V, B, N, k, r, R, dtype="bf16", peak="decay", mode="parent"):
    return {"name": name, "op": "round", "V": V, "B": B, "N": N, "k": k, "r": r, "R": R,
            "dtype": dtype, "peak": peak, "mode": mode}


def _attn(name, R, N, Hq, Hkv, D, pmin, pmax):
    return {"name": name, "op": "attn", "R": R, "N": N, "Hq": Hq, "Hkv": Hkv, "D": D,
            "pmin": pmin, "pmax": pmax}


def listed():
    return [
        # the smallest round: a float32 drafter with a small vocabulary; launches
        # and the latency of the stages are all there is
        _round("tiny_f32", 1024, 4, 16, 4, 32, 1, "f32", "const8"),
        # one interactive user, short blocks, the 4B and the 8B drafter's shapes
        _round("qwen4b_b7", 151936, 7, 32, 8, 256, 1, peak="const8"),
        _round("qwen8b_b7", 151936, 7, 48, 8, 384, 1, peak="uniform"),
        # the headline round: one user, long blocks
        _round("qwen4b_b16", 151936, 16, 64, 8, 256, 1),
        # one user of the largest drafter: 16 frontier rows, the widest rank
        _round("qwen14b_b16_r1", 151936, 16, 128, 16, 512, 1),
        # a serving batch of the largest drafter: 128 frontier rows, the largest case
        _round("qwen14b_b16_r8", 151936, 16, 128, 16, 512, 8),
        # ragged: three requests, a vocabulary that is no multiple of anything,
        # branching factor and budget that are no powers of two
        _round("ragged_r3", 50021, 9, 45, 6, 96, 3),
        # a float32 drafter at its largest rank, two requests
        _round("f32_r2", 32000, 8, 48, 4, 128, 2, "f32"),
        # the greedy chain (no tree) of the headline shape: decoding without branching
        {"name": "chain_4b_b16", "op": "chain", "V": 151936, "B": 16, "r": 256, "R": 1,
         "dtype": "bf16", "peak": "decay"},
        # one verification attention layer: one user, and a batch of eight
        _attn("attn_4b_r1", 1, 64, 32, 8, 128, 64, 1024),
        _attn("attn_14b_r8", 8, 128, 40, 8, 128, 64, 1024),
        # after the verification forward of a batch: retrieve rows, greedy
        # acceptance, compaction of the cache (36 layers, K and V)
        {"name": "verify_r8", "op": "verify", "R": 8, "N": 128, "B": 16, "V": 151936,
         "groups": 72, "slot": 1024, "pmax": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["round"] * 5 + ["chain"] + ["attn"] * 2 + ["verify"])
    if op in ("round", "chain"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        # vocabularies: any size, or (as real ones are) a multiple of 64
        V = _log_int(rng, 1000, 151936)
        if rng.random() < 0.5:
            V = max(1024, V // 64 * 64)
        r = 32 * rng.randint(1, 16) if dtype == "bf16" else 16 * rng.randint(1, 8)
        B = rng.randint(4, 16)
        if op == "chain":
            return {"op": "chain", "V": V, "B": B, "r": r, "R": rng.choice([1, 1, 2, 4, 8]),
                    "dtype": dtype, "peak": rng.choice(["const8", "uniform", "decay"])}
        c = _round("", V, B, _log_int(rng, 8, 128), rng.choice([2, 3, 4, 5, 6, 8, 8, 8, 12, 16]), r,
                   rng.choice([1, 1, 1, 2, 2, 3, 4, 5, 8]), dtype,
                   rng.choice(["const8", "uniform", "decay"]),
                   rng.choice(["parent"] * 4 + ["shared", "independent"]))
        del c["name"]
        return c
    if op == "attn":
        Hq, Hkv = rng.choice([(32, 8), (32, 8), (40, 8), (40, 8), (16, 16), (28, 4)])
        pmax = _log_int(rng, 64, 1024)
        c = _attn("", rng.choice([1, 1, 2, 3, 4, 8]), rng.choice([16, 32, 45, 48, 64, 96, 128]),
                  Hq, Hkv, rng.choice([64, 128, 128]), min(64, pmax), pmax)
        del c["name"]
        return c
    return {"op": "verify", "R": rng.choice([1, 2, 3, 4, 8]), "N": _log_int(rng, 8, 128),
            "B": rng.randint(4, 16), "V": 151936, "groups": rng.choice([56, 64, 72]),
            "slot": rng.choice([256, 512, 1024]), "pmax": _log_int(rng, 64, 1024)}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _round_inputs(c, seed):
    """A drafter's head (E, W) and one round's L, h, root and prefix lengths."""
    g, rng = _gen(seed), np.random.default_rng(seed)
    dt = _DT[c["dtype"]][0]
    R, B, V, r = c["R"], c["B"], c["V"], c["r"]
    L = torch.randn(R, B, V, generator=g, device="cuda") * 3.0
    # peaks at three distinct tokens per depth, Zipf(1.1) over the vocabulary
    cdf = np.cumsum(np.arange(1, V + 1, dtype=np.float64) ** -1.1)
    cdf /= cdf[-1]
    tok = np.zeros((R, B, 3), dtype=np.int64)
    height = np.zeros((R, B, 1), dtype=np.float32)
    for q in range(R):
        for d in range(B):
            seen = []
            while len(seen) < 3:
                t = min(int(np.searchsorted(cdf, rng.random(), side="right")), V - 1)
                if t not in seen:
                    seen.append(t)
            tok[q, d] = seen
            height[q, d] = {"const8": 8.0, "uniform": rng.uniform(4.0, 12.0),
                            "decay": 12.0 - 9.0 * d / max(B - 1, 1)}[c["peak"]]
    L.scatter_add_(2, torch.from_numpy(tok).cuda(),
                   torch.from_numpy(np.repeat(height, 3, axis=2)).cuda())
    return {
        "L": L.to(dt),
        "E": (torch.randn(V, r, generator=g, device="cuda") * 0.02).to(dt),
        "Wt": (torch.randn(V, r, generator=g, device="cuda") * 0.05).to(dt),
        "h": torch.randn(R, B, r, generator=g, device="cuda"),
        "root": torch.from_numpy(rng.integers(0, V, R).astype(np.int32)).cuda(),
        "prefix_len": torch.from_numpy(rng.integers(1, 1025, R).astype(np.int32)).cuda(),
    }


def _random_trees(rng, R, N, max_depth, V):
    """Trees in the builder's layout (parents before children): token, parent [R][N].

    Nodes hang below earlier ones, recent ones preferred, so that the depths
    are those of a drafted tree."""
    token = rng.integers(0, V, (R, N)).astype(np.int32)
    parent = np.full((R, N), -1, dtype=np.int32)
    for q in range(R):
        depth = np.zeros(N, dtype=np.int64)
        for i in range(1, N):
            p = int(i - 1 - min(rng.geometric(0.15) - 1, i - 1))
            while depth[p] >= max_depth:
                p = int(parent[q, p])
            parent[q, i], depth[i] = p, depth[p] + 1
    return token, parent


def prepare(case, seed):
    c = case
    if c["op"] == "round":
        inp = _round_inputs(c, seed)
        b = P.TreeBuilder(c["V"], c["B"], c["N"], c["k"], c["r"], c["R"], _DT[c["dtype"]][1],
                          mask=True, mode=_MODES[c["mode"]])
        return {"op": "round", "builder": b, "inp": inp}
    if c["op"] == "chain":
        inp = _round_inputs(c, seed)
        return {"op": "chain", "inp": inp}
    rng = np.random.default_rng(seed)
    R, N = c["R"], c["N"]
    if c["op"] == "attn":
        g = _gen(seed)
        Hq, Hkv, D = c["Hq"], c["Hkv"], c["D"]
        _, parent = _random_trees(rng, R, N, 16, 1 << 17)
        parent = torch.from_numpy(parent).cuda()
        count = torch.full((R,), N, dtype=torch.int32, device="cuda")
        prefix = rng.integers(c["pmin"], c["pmax"] + 1, R).astype(np.int32)
        C = c["pmax"] + N  # the cache is sized for the longest request

        def bf(*shape):
            return torch.randn(*shape, generator=g, device="cuda").to(torch.bfloat16)

        return {"op": "attn", "layer": P.TreeAttention(R, N, Hq, Hkv, D, C, D ** -0.5),
                "q": bf(R, N, Hq, D), "k": bf(R, Hkv, C, D), "v": bf(R, Hkv, C, D),
                "mask": P.build_mask(parent, count), "count": count,
                "prefix": torch.from_numpy(prefix).cuda()}
    # verify
    token, parent = _random_trees(rng, R, N, c["B"], c["V"])
    target = rng.integers(0, c["V"], (R, N)).astype(np.int32)
    for q in range(R):  # at most nodes the target continues with one of the children
        kids = {}
        for i in range(1, N):
            kids.setdefault(int(parent[q, i]), []).append(i)
        for p, ch in kids.items():
            if rng.random() < 0.8:
                target[q, p] = token[q, ch[int(rng.integers(0, len(ch)))]]
    cap = c["pmax"] + N
    g = _gen(seed)
    cache = torch.empty(R, c["groups"], cap, c["slot"], dtype=torch.bfloat16, device="cuda")
    cache.normal_(generator=g)

    def up(a):
        return torch.from_numpy(a).cuda()

    return {"op": "verify", "token": up(token), "parent": up(parent), "target": up(target),
            "count": torch.full((R,), N, dtype=torch.int32, device="cuda"), "cache": cache,
            "prefix": up(rng.integers(1, c["pmax"] + 1, R).astype(np.int32)), "B": c["B"], "N": N}


def run(state):
    s = state
    if s["op"] == "round":
        return s["builder"].run(**s["inp"])
    if s["op"] == "chain":
        return P.chain_decode(**s["inp"])
    if s["op"] == "attn":
        return s["layer"](s["q"], s["k"], s["v"], s["mask"], s["count"], s["prefix"])
    rows, nrows = P.build_retrieve(s["parent"], s["count"], s["B"])
    acc = P.accept_greedy(s["token"], rows, nrows, s["target"])
    P.compact_kv(s["cache"], s["prefix"], acc["accept_node"], acc["accept_len"], s["N"])
    return {"rows": rows, "nrows": nrows, **acc, "cache": s["cache"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    c = case
    if c["op"] in ("round", "chain"):
        es = 4 if c["dtype"] == "f32" else 2
        k = c.get("k", 1)
        N = c.get("N", c["B"] + 1)
        mode = c.get("mode", "parent")
        rows = c["R"] * (1 + (c["B"] - 1) * (k if mode == "parent" else 1))
        head = mode != "independent"
        nbytes = (c["R"] * c["B"] * c["V"] * es                       # base logits
                  + (c["V"] * c["r"] * es + rows * c["r"] * es        # W once, parents' E rows
                     + c["R"] * c["B"] * c["r"] * 4 if head else 0)   # depth features
                  + c["R"] * N * (5 * 4 + 4 * ((N + 31) // 32)))      # the tree and its mask
        return {"bytes": nbytes, "flops": 2 * rows * c["r"] * c["V"] if head else 0}
    if c["op"] == "attn":
        mean = (c["pmin"] + c["pmax"]) / 2  # prefix lengths are uniform
        slots = c["R"] * (mean + c["N"])
        q = 2 * c["R"] * c["N"] * c["Hq"] * c["D"] * 2
        return {"bytes": 2 * slots * c["Hkv"] * c["D"] * 2 + q,
                "flops": 4 * c["R"] * c["N"] * (mean + 8) * c["Hq"] * c["D"]}
    # verify: the indices, and about four accepted slots moved in every group
    return {"bytes": c["R"] * c["N"] * 4 * (4 + 2 * (c["B"] + 1))
            + 2 * 4 * c["R"] * c["groups"] * c["slot"] * 2, "flops": 0}


def tolerance(case):
    if case["op"] == "verify":
        return "exact"  # indices and moved bytes
    if case["op"] == "attn":
        return {"rel": 9e-3, "max": 0.1}  # bf16 weights and outputs (2.2e-3 off float64)
    # path scores are sums of float32 log-probabilities (1e-7 to 2e-7 off float64
    # as measured); tokens may change places only where two scores tie in float32
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same definitions in float64
# ---------------------------------------------------------------------------

def _head_input(E, h, tokens, dtype):
    x = E[tokens].double() + h.double()
    u = (x / (1.0 + torch.exp(-x))).float()  # rounded to the drafter's precision
    return (u.to(torch.bfloat16) if dtype == "bf16" else u).double()


def _best(logp, k):
    """The k best of each row, ties to the lowest token."""
    v, i = torch.sort(logp, dim=-1, descending=True, stable=True)
    return v[..., :k], i[..., :k]


def _exact_tree(c, inp, W64, q):
    B, V, k, N, mode = c["B"], c["V"], min(c["k"], c["V"]), c["N"], c["mode"]
    nodes = [(0.0, 0, int(inp["root"][q]), -1, 0)]  # score, depth, token, parent, slot
    front, chain = [0], int(inp["root"][q])
    for d in range(B):
        L = inp["L"][q, d].double()
        toks = [nodes[i][2] for i in front] if mode == "parent" else [chain]
        z = L[None].expand(len(toks), V)
        if mode != "independent":
            u = _head_input(inp["E"], inp["h"][q, d], torch.tensor(toks, device="cuda"), c["dtype"])
            z = z + u @ W64.T
        v, t = _best(torch.log_softmax(z, -1), k)
        v, t = v.cpu().numpy(), t.cpu().numpy()
        chain = int(t[0, 0])
        layer = []
        for s, p in enumerate(front):
            row = s if mode == "parent" else 0
            for j in range(k):
                layer.append(len(nodes))
                nodes.append((nodes[p][0] + float(v[row, j]), d + 1, int(t[row, j]), p, s))
        front = sorted(layer, key=lambda i: (-nodes[i][0], nodes[i][2], nodes[i][4]))[:k]
    chosen = sorted(range(len(nodes)), key=lambda i: (-nodes[i][0],) + nodes[i][1:3]
                    + (nodes[i][4],))[:N]
    place, order = {}, []
    for lev in range(B + 1):
        for i in sorted((i for i in chosen if nodes[i][1] == lev),
                        key=lambda i: (place.get(nodes[i][3], -1), nodes[i][2])):
            place[i] = len(order)
            order.append(i)
    n = len(order)
    out = {"token": np.full(N, -1, np.int32), "parent": np.full(N, -1, np.int32),
           "depth": np.full(N, -1, np.int32), "position": np.full(N, -1, np.int32),
           "logprob": np.full(N, -np.inf), "count": n,
           "mask": np.zeros((N, (N + 31) // 32), np.uint32)}
    for e, i in enumerate(order):
        score, depth, tok, p, _ = nodes[i]
        out["token"][e], out["depth"][e], out["logprob"][e] = tok, depth, score
        out["position"][e] = int(inp["prefix_len"][q]) + depth
        if p >= 0:
            out["parent"][e] = place[p]
            out["mask"][e] = out["mask"][place[p]]
        out["mask"][e, e // 32] |= np.uint32(1 << (e % 32))
    return out


def exact(case, seed):
    c = case
    if c["op"] == "round":
        inp = _round_inputs(c, seed)
        W64 = inp["Wt"].double()
        trees = [_exact_tree(c, inp, W64, q) for q in range(c["R"])]
        out = {n: np.stack([np.asarray(t[n]) for t in trees]) for n in trees[0]}
        out["mask"] = out["mask"].view(np.int32)
        out["count"] = out["count"].astype(np.int32)
        return out
    if c["op"] == "chain":
        inp = _round_inputs(c, seed)
        W64 = inp["Wt"].double()
        tok, cum = inp["root"].long(), torch.zeros(c["R"], dtype=torch.float64, device="cuda")
        toks, cums = [tok], [cum]
        for d in range(c["B"]):
            u = _head_input(inp["E"], inp["h"][:, d], tok, c["dtype"])
            v, t = _best(torch.log_softmax(inp["L"][:, d].double() + u @ W64.T, -1), 1)
            tok, cum = t[:, 0], cum + v[:, 0]
            toks.append(tok)
            cums.append(cum)
        return torch.stack(toks, 1).int(), torch.stack(cums, 1)
    if c["op"] == "attn":
        s = prepare(c, seed)
        R, N, Hq, Hkv = c["R"], c["N"], c["Hq"], c["Hkv"]
        bits = torch.arange(32, device="cuda", dtype=torch.int32)
        tree = ((s["mask"][..., None] >> bits) & 1).bool().reshape(R, N, -1)[..., :N]
        out = []
        for q in range(R):
            n = int(s["prefix"][q])
            adm = torch.cat([torch.ones(N, n, dtype=torch.bool, device="cuda"), tree[q]], 1)
            k = s["k"][q, :, :n + N].double().repeat_interleave(Hq // Hkv, 0)
            v = s["v"][q, :, :n + N].double().repeat_interleave(Hq // Hkv, 0)
            z = torch.matmul(s["q"][q].double().transpose(0, 1).contiguous(),
                             k.transpose(1, 2).contiguous()) * c["D"] ** -0.5
            w = torch.softmax(z.masked_fill(~adm[None], -math.inf), -1)
            out.append(torch.matmul(w, v).transpose(0, 1))
        return torch.stack(out)
    return None  # the verify steps move bytes and indices: nothing is computed in floats
