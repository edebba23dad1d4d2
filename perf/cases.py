"""What the speed of this library is measured on: verify calls as a serving loop makes them.

A case is one call of one entry point of `paper_2502_20704_amd` on logits that are already on the GPU.
The listed cases are the library's own configurations (`synth.CONFIGS`: one sequence, a batch of 64, a
batch of 256, a batch of token trees) and the sizes between and beside them that the same program
meets: a few sequences, a vocabulary with added tokens (rows that are not 16-byte aligned), the
strict baseline, reducible FSD, and a draw with the usual sampling-method warpers.  `draw` gives more
calls of these ranges.

The random numbers of a call (seed, offset) are part of its inputs, so a case has one right answer:
lengths, paths and token ids are whole numbers that agree except where a divergence lies within
rounding of the threshold or two scores of a draw are equal to rounding.
"""
from __future__ import annotations

import math

import torch

import paper_2502_20704_amd as fsd

DIVS = {"kl": fsd.DIV_KL, "js": fsd.DIV_JS, "tv": fsd.DIV_TV}
MODES = {"sample": fsd.SAMPLE, "greedy": fsd.GREEDY}
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
OUTPUTS = {
    "chain": ("accept_len", "out_tokens", "divergences", "row_status"),
    "tree": ("path_len", "path_nodes", "out_tokens", "divergences", "row_status"),
    "sd": ("accept_len", "out_tokens", "log_ratio", "row_status"),
    "sd_tree": ("path_len", "path_nodes", "out_tokens", "log_ratio", "row_status"),
    "rfsd": ("accept_len", "out_tokens", "divergences", "log_ratio", "row_status"),
}
DEPTH = 6        # layers of a token tree
BRANCH = 4       # contexts a layer expands, and tokens a context proposes


def _case(name, call, B, rows, V, dtype, logits, sigma, **more):
    """sigma: the draft's noise; one number, or the two ends of a range for [sigma, sigma_hi] per sequence."""
    c = dict(name=name, call=call, B=B, rows=rows, V=V, dtype=dtype, logits=logits, sigma=sigma, sigma_hi=sigma,
             masked=0, div="js", T=0.1, mode="sample", temperature=1.0, top_k=0, top_p=1.0)
    c.update(more)
    return c


def listed():
    return [
        # one user, a small vocabulary, binary32 logits: the smallest call, its latency
        _case("single_f32", "chain", 1, 4, 32000, "f32", "flat", 0.5, T=0.05),
        # one user of a model with a large vocabulary
        _case("single_bf16", "chain", 1, 8, 128256, "bf16", "peaked", 1.0),
        # a few users, the total-variation rule, greedy correction
        _case("few_f32_tv", "chain", 8, 5, 32000, "f32", "flat", 0.5, div="tv", mode="greedy", T=0.2),
        # a moderate batch of a model whose vocabulary was extended by three tokens: no row is 16-byte aligned
        _case("ragged", "chain", 16, 5, 128259, "bf16", "peaked", 0.25, sigma_hi=4.0),
        # the serving batch of the benchmark
        _case("batch", "chain", 64, 8, 128256, "bf16", "peaked", 0.25, sigma_hi=4.0),
        # the largest batch, binary32 logits
        _case("large_f32", "chain", 256, 16, 151936, "f32", "zipf", 1.0, T=0.3),
        # a batch of token trees
        _case("tree", "tree", 32, 60, 128256, "bf16", "peaked", 1.0, T=0.15),
        # the strict baseline on the serving batch and on the trees
        _case("strict", "sd", 64, 8, 128256, "bf16", "peaked", 0.25, sigma_hi=4.0),
        _case("strict_tree", "sd_tree", 32, 60, 128256, "bf16", "peaked", 1.0),
        # reducible FSD, long candidates, the largest vocabulary of the configurations
        _case("reducible", "rfsd", 32, 10, 256000, "bf16", "peaked", 0.25, sigma_hi=4.0),
        # the serving batch with temperature, top-k and top-p where the token is drawn
        _case("warped", "chain", 64, 8, 128256, "bf16", "peaked", 0.25, sigma_hi=4.0, temperature=0.7, top_k=50, top_p=0.9),
        # a few token trees with a nucleus alone
        _case("warped_tree", "tree", 8, 60, 128256, "bf16", "peaked", 1.0, T=0.15, top_p=0.95),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["chain", "chain", "chain", "tree", "sd", "sd_tree", "rfsd", "warped", "warped_tree"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    V = _log_uniform(rng, 32000, 256000)
    ragged = rng.random() < 0.25
    V = V | 1 if ragged else V // 64 * 64
    is_tree = call in ("tree", "sd_tree", "warped_tree")
    rows = rng.randint(8, 64) if is_tree else rng.randint(1, 16)
    # bytes of the logits a drawn call reads: at most a third of the largest listed case's
    most = 3.0e8 if ragged else 1.6e9
    B = max(1, min(_log_uniform(rng, 1, 256), int(most / (2 * rows * V * (2 if dtype == "bf16" else 4)))))
    warp = {}
    if call.startswith("warped"):
        call = "tree" if is_tree else "chain"
        B = min(B, 64)
        warp = rng.choice([dict(temperature=0.8), dict(top_k=rng.randint(2, 200)), dict(top_p=round(rng.uniform(0.5, 0.99), 2)),
                           dict(temperature=round(rng.uniform(0.3, 1.5), 2), top_k=rng.randint(10, 100), top_p=0.95)])
    lo = round(rng.uniform(0.25, 1.5), 2)
    c = _case(None, call, B, rows, V, dtype, rng.choice(["flat", "peaked", "zipf"]), lo,
              sigma_hi=round(lo * rng.choice([1.0, 1.0, 2.5]), 2), masked=rng.choice([0, 0, 0, rng.randint(1, 200)]),
              div=rng.choice(["js", "js", "js", "tv", "kl"]), T=rng.choice([0.05, 0.1, 0.2, 0.3]),
              mode=rng.choice(["sample", "sample", "sample", "greedy"]), **warp)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------- inputs


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _target_rows(g, n, V, kind):
    z = torch.randn((n, V), generator=g, device="cuda")
    if kind == "flat":        # N(0, 2^2)
        return z.mul_(2.0)
    if kind == "peaked":      # N(0, 3^2) and 20 entries of a row 8 above the rest
        z.mul_(3.0)
        at = torch.randint(0, V, (n, 20), generator=g, device="cuda")
        return z.scatter_add_(1, at, torch.full((n, 20), 8.0, device="cuda"))
    # -1.1 ln(rank) + N(0, 1), the rank of an entry uniform in 1 .. V
    rank = torch.rand((n, V), generator=g, device="cuda").mul_(V).floor_().add_(1.0)
    return z.add_(rank.log_(), alpha=-1.1)


def _shape_of_tree(rng_seed, B, N):
    """parent and rank among its siblings of every node: trees of DEPTH layers in which a layer expands its
    BRANCH best contexts into BRANCH tokens each; the N best proposals are kept, numbered layer by layer."""
    import random

    rng = random.Random(rng_seed)
    parents, ranks = [], []
    for _ in range(B):
        props, frontier = [], [(-1, 0.0, 0)]        # (parent proposal, rank, score, layer)
        for layer in range(1, DEPTH + 1):
            new = []
            for pid, score, _l in frontier:
                for r in range(BRANCH):
                    s = score - 0.4 * (r + 1) * (0.5 + rng.random())
                    props.append((pid, r, s, layer))
                    new.append((len(props) - 1, s, layer))
            frontier = sorted(new, key=lambda x: -x[1])[:BRANCH]
        keep = sorted(range(len(props)), key=lambda i: -props[i][2])[:N]
        order = sorted(keep, key=lambda i: (props[i][3], i))
        number = {i: k for k, i in enumerate(order)}
        parents.append([number.get(props[i][0], -1) for i in order])
        ranks.append([props[i][1] for i in order])
    return parents, ranks


def prepare(case, seed):
    B, rows, V, dtype = case["B"], case["rows"], case["V"], DTYPES[case["dtype"]]
    is_tree = case["call"] in ("tree", "sd_tree")
    g = _generator(seed)
    sigma = torch.rand(B, generator=g, device="cuda") * (case["sigma_hi"] - case["sigma"]) + case["sigma"]
    target = torch.empty((B, rows + 1, V), dtype=dtype, device="cuda")
    draft = torch.empty((B, rows, V), dtype=dtype, device="cuda")
    tokens = torch.empty((B, rows), dtype=torch.int32, device="cuda")
    s = dict(call=case["call"], case=case, seed=seed)
    if is_tree:
        parents, ranks = _shape_of_tree(seed, B, rows)
        s["parent"] = torch.tensor(parents, dtype=torch.int32, device="cuda")
        rank = torch.tensor(ranks, dtype=torch.int64, device="cuda")
    for b in range(B):
        t = _target_rows(g, rows + 1, V, case["logits"])
        if case["masked"]:       # the padded end of the vocabulary has no mass in either model
            t[:, V - case["masked"]:] = -math.inf
        noise = torch.randn((rows, V), generator=g, device="cuda").mul_(sigma[b])
        context = t[s["parent"][b].long() + 1] if is_tree else t[:rows]
        d = context.add(noise)
        target[b] = t
        draft[b] = d
        if is_tree:              # a context proposes its draft's most probable tokens
            top = draft[b].float().topk(BRANCH, dim=1).indices
            tokens[b] = top.gather(1, rank[b][:, None])[:, 0].int()
        else:                    # a candidate is drawn from its draft row
            e = torch.empty((rows, V), device="cuda").exponential_(generator=g)
            tokens[b] = (draft[b].float() - e.log_()).argmax(1).int()
    code = fsd.BF16 if case["dtype"] == "bf16" else fsd.F32
    s.update(target=target, draft=draft, tokens=tokens, out=None,
             workspace=torch.empty(fsd.fsd_workspace_bytes(B, rows, V, code) + 256, dtype=torch.uint8, device="cuda"))
    return s


# ---------------------------------------------------------------------------------------------------- one call


def run(s):
    """One verify call on the output tensors and the workspace the loop keeps."""
    c, call = s["case"], s["call"]
    mode, div = MODES[c["mode"]], DIVS[c["div"]]
    keep = dict(out=s["out"], workspace=s["workspace"])
    rnd = dict(seed=s["seed"] + 1, offset=3)
    warp = dict(temperature=c["temperature"], top_k=c["top_k"], top_p=c["top_p"])
    warped = c["temperature"] != 1.0 or c["top_k"] > 0 or c["top_p"] < 1.0
    if call == "chain" and warped:
        out = fsd.fsd_verify_chain_warped(s["target"], s["draft"], s["tokens"], c["T"], div, mode, **rnd, **warp, **keep)
    elif call == "chain":
        out = fsd.fsd_verify_chain(s["target"], s["draft"], s["tokens"], c["T"], div, mode, **rnd, **keep)
    elif call == "tree" and warped:
        out = fsd.fsd_verify_tree_warped(s["target"], s["draft"], s["tokens"], s["parent"], DEPTH, c["T"], div, mode,
                                         **rnd, **warp, **keep)
    elif call == "tree":
        out = fsd.fsd_verify_tree(s["target"], s["draft"], s["tokens"], s["parent"], DEPTH, c["T"], div, mode, **rnd, **keep)
    elif call == "sd":
        out = fsd.sd_verify_chain(s["target"], s["draft"], s["tokens"], mode, **rnd, **keep)
    elif call == "sd_tree":
        out = fsd.sd_verify_tree(s["target"], s["draft"], s["tokens"], s["parent"], DEPTH, mode, **rnd, **keep)
    else:
        out = fsd.rfsd_verify_chain(s["target"], s["draft"], s["tokens"], c["T"], div, mode, **rnd, **keep)
    s["out"] = out
    return {k: out[k] for k in OUTPUTS[call]}


def work(case):
    """Every draft row and every target row a position refers to, once.  (The row after the last candidate is
    read only when everything is accepted, any other row a token is drawn from has been read already.)
    Arithmetic per entry: the exponential's argument, the exponential, the sum, and the divergence's terms."""
    B, rows, V = case["B"], case["rows"], case["V"]
    contexts = B * rows
    if case["call"] in ("tree", "sd_tree"):   # the children of a node share a target row
        contexts = sum(len(set(p)) for p in _shape_of_tree(0, B, rows)[0])
    entries = (B * rows + contexts) * V
    size = 2 if case["dtype"] == "bf16" else 4
    return {"bytes": entries * size + B * (3 * rows + 4) * 4, "flops": entries * (4 if case["call"].startswith("sd") else 7)}


def tolerance(case):
    """Both logit types are evaluated in binary32.  A divergence sums V terms of separately rounded exponentials
    (relative 1.2e-7 each); what is left of it after the terms cancel is at most 4e-6 of the result over these
    ranges (nearly equal rows, measured against 64 bits).  `differ`: a position whose divergence is the threshold to rounding, or a draw
    whose two best scores are equal to rounding, may go either way."""
    return {"rel": 2e-5, "max": 2e-4, "differ": 0.005}


# ---------------------------------------------------------------------------------------------------- in 64 bits


def _divergence(lp, lq, kind):
    p, q = lp.exp(), lq.exp()
    if kind == "tv":
        return 0.5 * (p - q).abs().sum(-1)
    if kind == "kl":
        return torch.where(p > 0, p * (lp - lq), torch.zeros_like(p)).sum(-1)
    lm = (0.5 * (p + q)).log()
    zero = torch.zeros_like(p)
    return 0.5 * (torch.where(p > 0, p * (lp - lm), zero) + torch.where(q > 0, q * (lq - lm), zero)).sum(-1)


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 (Salmon et al., SC'11)"""
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c0, 0xCD9E8D57 * c2
        c0, c1, c2, c3 = (p1 >> 32) ^ c1 ^ k0, p1 & 0xFFFFFFFF, (p0 >> 32) ^ c3 ^ k1, p0 & 0xFFFFFFFF
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c0, c1, c2, c3


def _uniform(seed, offset, b, index):
    word = _philox((index >> 2) | (1 << 30), b, offset & 0xFFFFFFFF, offset >> 32, seed & 0xFFFFFFFF, seed >> 32)[index & 3]
    return (2 * (word >> 9) + 1) * 2.0 ** -24


def _walk(s, b, N):
    """Strict SD over tree b: (path, log-ratio of every node tried), children in index order, the residual
    after every rejection."""
    parent, tokens = s["parent"][b].tolist(), s["tokens"][b].tolist()
    ratio, path, cur = [math.nan] * N, [], -1
    while True:
        p = torch.softmax(s["target"][b, cur + 1].double(), 0)
        taken = None
        for j in (j for j in range(N) if parent[j] == cur):
            lq = torch.log_softmax(s["draft"][b, j].double(), 0)
            ratio[j] = (p[tokens[j]].log() - lq[tokens[j]]).item()
            if min(0.0, ratio[j]) - math.log(_uniform(s["seed"] + 1, 3, b, j)) > 0.0:
                taken = j
                break
            left = (p - lq.exp()).clamp_(min=0.0)
            total = left.sum()
            p = left / total if total > 0 else p
        if taken is None:
            return path, ratio
        path.append(taken)
        cur = taken


def exact(case, seed):
    s = prepare(case, seed)
    B, rows, call = case["B"], case["rows"], case["call"]
    dev = s["target"].device
    if call == "sd_tree":
        walks = [_walk(s, b, rows) for b in range(B)]
        nodes = torch.full((B, DEPTH), -1, dtype=torch.int32, device=dev)
        for b, (path, _) in enumerate(walks):
            nodes[b, :len(path)] = torch.tensor(path, dtype=torch.int32, device=dev)
        return dict(path_len=torch.tensor([len(p) for p, _ in walks], dtype=torch.int32, device=dev), path_nodes=nodes,
                    out_tokens=None, log_ratio=torch.tensor([r for _, r in walks], dtype=torch.float64, device=dev),
                    row_status=torch.zeros(B, dtype=torch.int32, device=dev))
    div, ratio = [], []
    for b in range(B):
        at = s["parent"][b].long() + 1 if call == "tree" else slice(0, rows)
        lp = torch.log_softmax(s["target"][b][at].double(), -1)
        lq = torch.log_softmax(s["draft"][b].double(), -1)
        x = s["tokens"][b].long()[:, None]
        ratio.append((lp.gather(1, x) - lq.gather(1, x))[:, 0])
        if call != "sd":
            div.append(_divergence(lp, lq, case["div"]))
    values = dict(divergences=torch.stack(div) if div else None, log_ratio=torch.stack(ratio))
    # the random draws (and with them strict SD's lengths) are the library's own sequence of numbers
    if call == "chain":
        values["accept_len"] = (values["divergences"] <= case["T"]).int().cumprod(1).sum(1).int()
    values["row_status"] = torch.zeros(B, dtype=torch.int32, device=dev)
    return {k: values.get(k) for k in OUTPUTS[call]}
