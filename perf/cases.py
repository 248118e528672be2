"""Workloads on which the framework's speed is measured.

A speculative decoding server calls the framework once per decoding cycle: the
LM heads produce the logits of every tree node (target) and of every node with
children (draft), the sampler draws the draft trees' tokens, the verifier
accepts a chain of every tree, and the commit step lays that chain out. Each
case below is one such call (or the verification and commit that follow each
other), at batch sizes from a single tree (latency) to 256 trees.

Logits follow N(0, 3^2) with +6 on about 1% of the ids (a peaked next-token
distribution), the draft adds N(0, 1.5^2); tokens are drawn from the parent's
tempered draft distribution (Gumbel maxima, so no code of the framework makes
its own inputs); uniforms are multiples of 2^-24.
"""

import math

import numpy as np
import torch

import paper_2505_12398_amd as tv

WITHOUT = tv.TV_SIBLINGS_WITHOUT_REPLACEMENT
WITH = tv.TV_SIBLINGS_WITH_REPLACEMENT


def _verify(name, batch, shape, nodes, depth, vocab, dtype="bf16", temperature=1.0,
            replacement=False, theta=False, stats=False, tokenlevel=False, commit=False):
    return {"name": name, "kind": "verify", "batch": batch, "shape": shape, "nodes": nodes,
            "depth": depth, "vocab": vocab, "dtype": dtype, "temperature": temperature,
            "replacement": replacement, "theta": theta, "stats": stats, "tokenlevel": tokenlevel,
            "commit": commit}


def _sample(name, batch, nodes, depth, vocab, dtype="bf16", temperature=1.0, replacement=False):
    return {"name": name, "kind": "sample", "batch": batch, "shape": "irregular", "nodes": nodes,
            "depth": depth, "vocab": vocab, "dtype": dtype, "temperature": temperature,
            "replacement": replacement}


def _lmhead(name, rows, hidden, vocab, temperature=1.0):
    return {"name": name, "kind": "lmhead", "rows": rows, "hidden": hidden, "vocab": vocab,
            "temperature": temperature}


def listed():
    return [
        # a full server batch: 256 irregular trees of 64 draft nodes, Llama-3 vocabulary
        _verify("verify-256", 256, "irregular", 64, 7, 128256),
        # one user: a single tree and the commit that follows, where latency counts
        _verify("verify-commit-1", 1, "irregular", 64, 7, 128256, commit=True),
        # a small batch at the Qwen2 vocabulary, acceptance probabilities logged
        _verify("verify-theta-16", 16, "irregular", 60, 6, 151936, theta=True),
        # single-chain drafting with fp32 logits, Llama-2 vocabulary
        _verify("verify-chain-f32-64", 64, "chain", 5, 5, 32000, dtype="f32", theta=True,
                commit=True),
        # Sequoia-scale trees: hundreds of nodes, depth about 30, few per launch
        _verify("verify-deep-8", 8, "windowed", 767, 0, 128256),
        # a full server batch whose LM heads already gave the row statistics
        _verify("verify-stats-256", 256, "irregular", 64, 7, 128256, stats=True),
        # the token-level baseline on complete binary trees with i.i.d. children
        _verify("tokenlevel-binary-32", 32, "binary", 30, 4, 128256, temperature=0.7,
                replacement=True, theta=True, tokenlevel=True),
        # drafting for a full server batch
        _sample("sample-256", 256, 64, 7, 128256),
        # drafting for two users, an odd vocabulary (rows off the 16-byte grid)
        _sample("sample-2", 2, 64, 7, 32003),
        # the target model's LM head: all nodes of a full batch, of 16 trees, of one tree
        _lmhead("lmhead-16640", 16640, 4096, 128256),
        _lmhead("lmhead-1040", 1040, 4096, 128256),
        _lmhead("lmhead-65", 65, 4096, 128256),
    ]


VOCABS = (32000, 32003, 50257, 128256, 151936)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("verify", "verify", "verify", "sample", "lmhead", "lmhead"))
    vocab = rng.choice(VOCABS)
    temperature = rng.choice((1.0, 1.0, 0.7, 1.3))
    if kind == "lmhead":
        rows = _log_int(rng, 1, 4096)
        hidden = 8 * _log_int(rng, 128, 512)
        return {k: v for k, v in _lmhead("", rows, hidden, vocab, temperature).items()
                if k != "name"}
    dtype = rng.choice(("bf16", "bf16", "f32"))
    nodes = rng.randint(24, 90)
    depth = rng.randint(6, 8)
    # at most the logits of 256 trees of 64 nodes at 128256 bf16
    size = 2 if dtype == "bf16" else 4
    most = 256 * 65 * 128256 * 2
    if kind == "sample":
        batch = _log_int(rng, 2, max(2, min(256, most // ((nodes + 1) * vocab * size))))
        c = _sample("", batch, nodes, depth, vocab, dtype, temperature, rng.random() < 0.4)
    else:
        shape = rng.choice(("irregular", "irregular", "chain", "binary", "windowed"))
        top = 256
        if shape == "chain":
            nodes = depth = rng.randint(3, 8)
        elif shape == "binary":
            depth = rng.randint(3, 5)
            nodes = 2 ** (depth + 1) - 2
        elif shape == "windowed":
            nodes, depth, top = rng.randint(200, 1000), 0, 8
        batch = _log_int(rng, 1, max(1, min(top, most // ((nodes + 1) * vocab * size))))
        extra = rng.choice(("", "", "theta", "stats", "tokenlevel"))
        c = _verify("", batch, shape, nodes, depth, vocab, dtype, temperature,
                    rng.random() < 0.3, extra in ("theta", "tokenlevel"), extra == "stats",
                    extra == "tokenlevel", rng.random() < 0.5)
    return {k: v for k, v in c.items() if k != "name"}


# --- inputs ------------------------------------------------------------------


def _irregular(rng, nodes, depth):
    """Breadth-first tree of exactly ``nodes`` draft nodes no deeper than
    ``depth``: branching factors 1..4 with probability proportional to 2^-k,
    redrawn when the depth limit leaves nodes over."""
    p = 2.0 ** -np.arange(1, 5)
    for attempt in range(2000):
        # a budget that the depth cannot hold at the usual branching takes wider draws
        w = p if attempt < 1000 else np.ones(4)
        ks = rng.choice((1, 2, 3, 4), size=nodes + 1, p=w / w.sum()).tolist()
        par, dep, head = [-1], [0], 0
        while head < len(par) and len(par) <= nodes:
            if dep[head] < depth:
                n = min(ks[head], nodes + 1 - len(par))
                par += [head] * n
                dep += [dep[head] + 1] * n
            head += 1
        if len(par) == nodes + 1:
            return np.array(par)
    raise ValueError("no tree of %d nodes within depth %d" % (nodes, depth))


def _parents(case, seed):
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 1])
    n, shape = case["nodes"], case["shape"]
    if shape == "chain":
        one = [np.arange(-1, n)] * case["batch"]
    elif shape == "binary":
        t = (np.arange(n + 1) - 1) // 2
        t[0] = -1
        one = [t] * case["batch"]
    elif shape == "windowed":
        i = np.arange(1, n + 1)
        one = [np.concatenate([[-1], rng.integers(np.maximum(0, i - 64), i)])
               for _ in range(case["batch"])]
    else:
        one = [_irregular(rng, n, case["depth"]) for _ in range(case["batch"])]
    return np.stack(one).astype(np.int32)


def _sibling_rank(parents):
    rank = np.zeros_like(parents)
    for b in range(parents.shape[0]):
        seen = {}
        for i, p in enumerate(parents[b].tolist()):
            rank[b, i] = seen.get(p, 0)
            seen[p] = rank[b, i] + 1
    return rank


def _chunks(batch, per_tree):
    step = max(1, (1 << 28) // per_tree)
    return [(b, min(batch, b + step)) for b in range(0, batch, step)]


def _trees(case, seed, target=True, tokens=True):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    parents = _parents(case, seed)
    B, n1 = parents.shape
    V, T = case["vocab"], float(np.float32(case["temperature"]))
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    s = {"case": case, "parents": torch.as_tensor(parents, device=dev),
         "temperature": case["temperature"],
         "mode": WITH if case["replacement"] else WITHOUT}
    s["draft"] = torch.empty((B, n1, V), dtype=dtype, device=dev)
    if target:
        s["target"] = torch.empty((B, n1, V), dtype=dtype, device=dev)
    tok = torch.zeros((B, n1), dtype=torch.int32, device=dev)
    rank = torch.as_tensor(_sibling_rank(parents), device=dev, dtype=torch.int64)
    par = torch.as_tensor(np.maximum(parents, 0), device=dev, dtype=torch.int64)
    kmax = int(rank[:, 1:].max()) + 1 if n1 > 1 else 0
    for b0, b1 in _chunks(B, n1 * V):
        z = torch.randn((b1 - b0, n1, V), generator=g, device=dev).mul_(3.0)
        z += 6.0 * (torch.rand(z.shape, generator=g, device=dev) < 0.01)
        if target:
            s["target"][b0:b1] = z
        z += 1.5 * torch.randn(z.shape, generator=g, device=dev)
        s["draft"][b0:b1] = z
        if tokens:
            # Gumbel maxima of the values the framework reads; without replacement
            # each winner leaves before the next sibling's draw
            z = s["draft"][b0:b1].to(torch.float32) * (1.0 / T)
            e = torch.empty_like(z).exponential_(generator=g).log_()
            z -= e
            pick = []
            for _ in range(kmax):
                y = z.argmax(dim=-1)
                pick.append(y)
                if case["replacement"]:
                    z += e
                    e.exponential_(generator=g).log_()
                    z -= e
                else:
                    z.scatter_(-1, y.unsqueeze(-1), -math.inf)
            pick = torch.stack(pick, dim=-1)                        # [b, n1, kmax]
            mine = pick.gather(1, par[b0:b1].unsqueeze(-1).expand(-1, -1, kmax))
            tok[b0:b1] = mine.gather(2, rank[b0:b1].unsqueeze(-1)).squeeze(-1).to(torch.int32)
            del e
        del z
    if tokens:
        tok[:, 0] = 0
        s["tokens"] = tok
    u = torch.randint(0, 1 << 24, (B, n1), generator=g, device=dev)
    s["uniforms"] = u.to(torch.float32) * 2.0 ** -24
    return s


def _row_stats(z, T):
    """Maximum and sum of exp((z - max) / T) of every row, in 64 bits."""
    m, t = [], []
    for b0, b1 in _chunks(z.shape[0], z[0].numel()):
        x = z[b0:b1].to(torch.float64)
        top = x.amax(dim=-1)
        m.append(top.to(torch.float32))
        t.append(((x - top.unsqueeze(-1)) / T).exp().sum(dim=-1))
    return torch.cat(m), torch.cat(t)


def _lm_inputs(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    M, K, N = case["rows"], case["hidden"], case["vocab"]
    x = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * (3.0 / math.sqrt(K))).to(torch.bfloat16)
    return x, w


def prepare(case, seed):
    if case["kind"] == "lmhead":
        x, w = _lm_inputs(case, seed)
        return {"case": case, "hidden": x, "weight": w, "temperature": case["temperature"]}
    if case["kind"] == "sample":
        return _trees(case, seed, target=False, tokens=False)
    s = _trees(case, seed)
    if case["stats"]:
        T = float(np.float32(case["temperature"]))
        s["stats"] = _row_stats(s["target"], T) + _row_stats(s["draft"], T)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "lmhead":
        logits, row_max, row_sum = tv.lmhead_stats(s["hidden"], s["weight"], s["temperature"])
        return {"logits": logits, "row_max": row_max, "row_sum": row_sum}
    if c["kind"] == "sample":
        tokens, status = tv.draft_tokens(s["parents"], s["draft"], s["temperature"],
                                         s["uniforms"], s["mode"])
        return {"tokens": tokens, "status": status}
    out = tv.verify_batch(s["parents"], s["tokens"], s["target"], s["draft"], s["temperature"],
                          s["uniforms"], s["mode"], tokenlevel=c["tokenlevel"],
                          want_theta=c["theta"], stats=s.get("stats"))
    r = {"accept_len": out.accept_len, "accepted_node": out.accepted_node,
         "bonus_token": out.bonus_token, "status": out.status, "node_state": out.node_state,
         "counters": out.counters}
    if c["theta"]:
        r["theta"] = out.node_theta
    if c["commit"]:
        r["path_nodes"], r["path_tokens"], r["path_len"] = tv.commit_paths(
            s["parents"], s["tokens"], out, max_len=16)
    return r


# --- work and tolerances -----------------------------------------------------

def _tree_work(case):
    """Means per tree on these inputs, from the framework's own work counters
    (temperature and vocabulary change them little): nodes whose two rows the
    traversal consults, residual passes over a node's two rows (fewer where no
    acceptance probabilities are asked for: some updates then decide nothing),
    accepted leaves (one target row more)."""
    n, d, full = case["nodes"], case["depth"], case["theta"]
    if case["tokenlevel"]:
        return 2.2, {"chain": 0.95, "windowed": 3.5}.get(case["shape"], 2.0), 0.1
    if case["shape"] == "chain":
        return float(n), 0.8 * n if full else 1.1, 0.1
    if case["shape"] == "binary":
        return 1.5 * d - 1.2, 2.7 * d - 4.2 if full else 1.5 * d - 1.7, 0.2
    if case["shape"] == "windowed":
        return 7.5, 15.0 if full else 10.7, 0.1
    return d + 0.1, 1.37 * d if full else 0.8 * d, 0.1


def work(case):
    if case["kind"] == "lmhead":
        M, K, N = case["rows"], case["hidden"], case["vocab"]
        return {"bytes": 2.0 * (M * K + N * K + M * N) + 12.0 * M, "flops": 2.0 * M * N * K}
    row = case["vocab"] * (2 if case["dtype"] == "bf16" else 4)
    small = case["batch"] * (case["nodes"] + 1) * 16.0
    if case["kind"] == "sample":
        # the draft row of every node with children: about 56% of these trees' nodes
        return {"bytes": case["batch"] * (case["nodes"] + 1) * 0.56 * row + small, "flops": 0.0}
    # a consulted node's rows are read once for their normalisers, unless those
    # are given, and once for every residual pass
    rows, passes, leaf = _tree_work(case)
    reads = 2.0 * passes + leaf + (0.0 if case["stats"] else 2.0 * rows)
    return {"bytes": case["batch"] * reads * row + small, "flops": 0.0}


def tolerance(case):
    if case["kind"] == "lmhead":
        # bf16 logits: 1.7e-3 from 64 bits, one unit in the last place at most
        return {"rel": 7e-3, "max": 0.016}
    # probabilities: fp32 terms summed in fp64, up to 7e-7 off in 64 bits' terms;
    # decisions and tokens are the same but where a uniform meets a boundary
    # within the sums' rounding
    return {"rel": 4e-6, "max": 4e-5, "differ": 0.01}


# --- results in 64 bits ------------------------------------------------------


def _verify_tree(parents, tokens, zb, zs, T, u, replacement, tokenlevel):
    """Algorithm 3 of the paper (or its token-level baseline) on one tree with
    explicit probability vectors in 64 bits: the probability every node was
    tested with (0 for pruned nodes, -1 for untested ones)."""
    n1 = len(parents)
    kids = [[] for _ in range(n1)]
    for i in range(1, n1):
        kids[parents[i]].append(i)
    theta = [-1.0] * n1

    def law(z, j):
        return torch.softmax(z[j].to(torch.float64) / T, dim=-1)

    def rejected(p, b, s, x):
        r = (p * b - s).clamp_(min=0.0)
        mass = float(r.sum())
        if not replacement:
            s = s.clone()
            s[x] = 0.0
            s /= s.sum()
        return mass, (r / mass if mass > 0.0 else r), s

    if tokenlevel:
        j = 0
        while kids[j]:
            b, s = law(zb, j), law(zs, j)
            for c in kids[j]:
                x = tokens[c]
                theta[c] = min(float(b[x] / s[x]), 1.0)
                if u[c] < theta[c]:
                    break
                _, b, s = rejected(1.0, b, s, x)
            else:
                return theta
            j = c
        return theta

    # one frame per node on the path: [node, rate, b, s, next child]
    def frame(j, p):
        return [j, p, law(zb, j), law(zs, j), 0] if kids[j] and p > 0.0 else [j, p, None, None, 0]

    def prune(j):
        for c in kids[j]:
            theta[c] = 0.0
            prune(c)

    path = [frame(0, 1.0)]
    while True:
        j, p, b, s, k = path[-1]
        if k < len(kids[j]) and p > 0.0:
            c = kids[j][k]
            x = tokens[c]
            path.append(frame(c, min(p * float(b[x] / s[x]), 1.0)))
            continue
        if k < len(kids[j]):
            for c in kids[j][k:]:
                theta[c] = 0.0
                prune(c)
        if j == 0:
            return theta
        theta[j] = p
        if u[j] < p:
            return theta
        path.pop()
        up = path[-1]
        mass, up[2], up[3] = rejected(up[1], up[2], up[3], tokens[j])
        up[1] = mass / (mass + (1.0 - up[1])) if mass > 0.0 else 0.0
        up[4] += 1


def exact(case, seed):
    if case["kind"] == "lmhead":
        x, w = _lm_inputs(case, seed)
        T = float(np.float32(case["temperature"]))
        logits = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float64, device=x.device)
        wd = w.to(torch.float64)
        for i in range(0, x.shape[0], 2048):
            torch.matmul(x[i:i + 2048].to(torch.float64), wd.T, out=logits[i:i + 2048])
        # the statistics are those of the logits as they are handed out, in bf16
        z = logits.to(torch.bfloat16).unsqueeze(1)
        row_max, row_sum = _row_stats(z, T)
        return {"logits": logits, "row_max": row_max[:, 0], "row_sum": row_sum[:, 0]}
    if case["kind"] != "verify" or not case["theta"] or case["batch"] * case["vocab"] > 1 << 23:
        return None
    s = _trees(case, seed)
    T = float(np.float32(case["temperature"]))
    par, tok = s["parents"].tolist(), s["tokens"].tolist()
    u = s["uniforms"].to(torch.float64).tolist()
    theta = [_verify_tree(par[b], tok[b], s["target"][b], s["draft"][b], T, u[b],
                          case["replacement"], case["tokenlevel"]) for b in range(case["batch"])]
    return {"theta": torch.tensor(theta, dtype=torch.float64)}
