"""What a user of libpcg has it do, as cases that can be timed and compared: one speculative step
per call (`verify`) from a single sequence on a small vocabulary to a full batch on the paper's
65 536-entry one, the same step by thinning, the draft's proposals, group probabilities of whole
rows, and the construction of the groups.  Inputs are made on the GPU from the seed; memberships
are nearest-neighbour sets of random embeddings, as in the recipes of `workloads/`.

A case is a dict:
  call      "verify" | "thinning" | "propose" | "group_probs" | "asg"
  V         vocabulary; every token's group is a set of its nearest neighbours
  groups    "knn": `size` members each; "ragged": 1 .. `size` members (half of them `size`, a
            quarter at most a third of it), neighbours in clusters whose sizes follow Zipf's law
  B, K      sequences and draft positions (group_probs: B (K + 1) rows)
  dtype, temperature, logits ("normal", "zipf" or "peaked": every second draft row four times
            as sharp)
  layout    "prepared" (made once per membership) or "csr" (the arrays as they are)
  weighted  general weights per entry instead of the equal split
  scratch   "kept" (outputs and workspace of the caller, as in a serving loop), "static" (the
            library's own scratch array) or "default" (neither is given)
"""
import functools
import math

import numpy as np
import torch

import paper_2511_13732_amd as pcg

_BASE = dict(call="verify", V=65536, groups="knn", size=32, B=64, K=8, dtype="bf16",
             temperature=1.0, logits="normal", layout="prepared", weighted=False, scratch="kept")
_ASG_THETA_SIGMAS = 3.36      # threshold in standard deviations of a random cosine: about 26 members at V = 65 536


def listed():
    return [
        # the smallest step: one sequence, four drafted tokens, a vocabulary of a thousand
        dict(_BASE, name="verify_b1_v1024_f32", V=1024, size=8, B=1, K=4, dtype="f32"),
        # one sequence on the full codec vocabulary: interactive decoding, latency counts
        dict(_BASE, name="verify_b1_v65536", B=1),
        # a small batch on a small codebook, by the call that needs no workspace
        dict(_BASE, name="verify_b8_v4096_static", V=4096, size=16, B=8, scratch="static"),
        # sizes that fit nothing: odd vocabulary (rows not 16-byte aligned), odd batch, plain call
        dict(_BASE, name="verify_b5_v20011_odd", V=20011, size=21, B=5, K=7, scratch="default"),
        # the throughput workload: a full serving batch on the full vocabulary
        dict(_BASE, name="verify_b64_v65536"),
        # the largest batch: fp32 logits, groups of 1 to 128, low temperature, sharp draft rows
        dict(_BASE, name="verify_b128_v32768_f32", V=32768, groups="ragged", size=128, B=128, K=6,
             dtype="f32", temperature=0.7, logits="peaked"),
        # the throughput workload with learned (general) weights
        dict(_BASE, name="verify_b64_v65536_weights", weighted=True),
        # a membership fresh from its construction, used as it is: no prepared layout
        dict(_BASE, name="verify_b32_v16384_csr", V=16384, B=32, logits="zipf", layout="csr"),
        # the step with the paper's own residual sampler
        dict(_BASE, name="thinning_b64_v65536", call="thinning"),
        # the draft's side: one token for every sequence after each of its forward passes
        dict(_BASE, name="propose_b64_v65536", call="propose", K=1),
        # scoring: group distributions of every target row of a step
        dict(_BASE, name="group_probs_576x65536", call="group_probs"),
        # building the groups of a codebook from its embeddings
        dict(name="asg_v65536_d1024", call="asg", V=65536, d=1024),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(["verify"] * 7 + ["thinning", "propose", "group_probs", "group_probs", "asg"])
    if call == "asg":
        return dict(call="asg", V=_log_uniform(rng, 2048, 65536), d=64 * rng.randint(2, 16))
    V = _log_uniform(rng, 1000, 65536)
    V += -V % rng.choice([1, 1, 8, 64])
    c = dict(_BASE, call=call, V=min(V, 65536), B=_log_uniform(rng, 1, 128), K=rng.randint(1, 8),
             size=_log_uniform(rng, 4, 140), dtype=rng.choice(["bf16", "bf16", "f32"]),
             temperature=rng.choice([1.0, 1.0, 0.7, 1.3]), groups=rng.choice(["knn", "knn", "ragged"]),
             logits=rng.choice(["normal", "normal", "zipf", "peaked"]),
             layout=rng.choice(["prepared"] * 4 + ["csr"]),
             weighted=rng.random() < 0.2, scratch=rng.choice(["kept", "default"]))
    # no more logits than the largest batch above, no more entries to sum than it has
    while c["B"] > 1 and (_logit_bytes(c) > 180e6 or c["B"] * _nnz(c) > 250e6 or
                          (c["call"] == "group_probs" and c["B"] * (c["K"] + 1) * _nnz(c) > 1.2e9)):
        c["B"] -= max(1, c["B"] // 8)
    return c


# ------------------------------------------------------------------------------------- inputs

def _generator(seed, purpose):
    return torch.Generator(device="cuda").manual_seed(1_000_003 * (seed + 1) + purpose)


def _sizes(c):
    """Members of every group, in the order of a fixed permutation of the tokens."""
    if c["groups"] == "knn":
        return np.full(c["V"], c["size"], np.int64)
    u = (np.random.default_rng(7).permutation(c["V"]) + 0.5) / c["V"]
    return np.maximum(1, np.rint(c["size"] * np.minimum(1.0, (2.0 * u) ** 1.7))).astype(np.int64)


def _membership(c, seed):
    """CSR (row_ptr, members) on the host: token t and its nearest neighbours, members ascending."""
    V, width, g = c["V"], c["size"], _generator(seed, 1)
    if c["groups"] == "ragged":
        n = min(512, max(1, V // 8))
        w = torch.arange(1, n + 1, device="cuda", dtype=torch.float64) ** -1.2
        which = torch.multinomial(w, V, replacement=True, generator=g)
        E = torch.randn((n, 64), device="cuda", generator=g)[which]
        E += 0.5 * torch.randn((V, 64), device="cuda", generator=g)
    else:
        E = torch.randn((V, 64), device="cuda", generator=g)
    E /= E.norm(dim=1, keepdim=True)
    near = torch.empty((V, width), dtype=torch.int32, device="cuda")
    for lo in range(0, V, 8192):
        hi = min(V, lo + 8192)
        sim = E[lo:hi] @ E.T
        sim[torch.arange(hi - lo, device="cuda"), torch.arange(lo, hi, device="cuda")] = 2.0
        near[lo:hi] = torch.topk(sim, width, dim=1).indices.to(torch.int32)    # nearest first, itself ahead
    sizes = torch.from_numpy(_sizes(c)).cuda()
    inside = torch.arange(width, device="cuda")[None, :] < sizes[:, None]
    near = torch.where(inside, near, V).sort(dim=1).values
    row_ptr = torch.zeros(V + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = sizes.cumsum(0)
    return row_ptr.cpu().numpy(), near[near < V].cpu().numpy()


def _weights(V, members, seed):
    raw = np.random.default_rng([seed, 77]).gamma(0.7, size=len(members)) + 1e-12
    return (raw / np.bincount(members, raw, minlength=V)[members]).astype(np.float32)


def _rows(c, n, k, g):
    """[n, k, V] float32 logits."""
    shape = (n, k, c["V"])
    if c["logits"] == "zipf":
        rank = torch.rand(shape, device="cuda", generator=g).argsort(dim=2).float()
        return -1.1 * (rank + 1).log_() + 0.5 * torch.randn(shape, device="cuda", generator=g)
    return 4.0 * torch.randn(shape, device="cuda", generator=g)


def _target_rows(c, seed):
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    return _rows(c, c["B"], c["K"] + 1, _generator(seed, 2)).to(dt)


def prepare(case, seed):
    c = case
    V = c["V"]
    if c["call"] == "asg":
        # one codebook per size; the seed orders its tokens and turns its axes round, so that the
        # groups have other members but their number and total size stay
        emb = torch.randn((V, c["d"]), device="cuda", generator=_generator(2511, 0))
        g = _generator(seed, 0)
        emb = emb[torch.randperm(V, device="cuda", generator=g)]
        emb *= torch.randint(0, 2, (c["d"],), device="cuda", generator=g) * 2.0 - 1.0
        return dict(call="asg", emb=emb, theta=_ASG_THETA_SIGMAS / math.sqrt(c["d"]))
    B, K = c["B"], c["K"]
    rows = B * (K + 1) if c["call"] == "group_probs" else B
    row_ptr, members = _membership(c, seed)
    groups = pcg.Groups.from_csr(V, row_ptr, members, "cuda", prepare=c["layout"] == "prepared",
                                 chunk_groups=pcg.suggest_chunk_groups(len(row_ptr) - 1, rows),
                                 reverse=True, weights=_weights(V, members, seed) if c["weighted"] else None)
    target = _target_rows(c, seed)
    s = dict(call=c["call"], groups=groups, temperature=c["temperature"], seed=seed, offset=5 + seed % 1000)
    kept = c["scratch"] == "kept"
    new = functools.partial(torch.empty, device="cuda")
    scratch = lambda n: new(n, dtype=torch.uint8)  # noqa: E731
    if c["call"] == "group_probs":
        s["logits"] = target.view(rows, V)
        s["out"] = new((rows, groups.G), dtype=torch.float32) if kept else None
        s["workspace"] = scratch(pcg.group_probs_workspace_bytes(V, rows)) if kept else None
        return s
    g = _generator(seed, 3)
    draft = target[:, :K].float() + torch.randn((B, K, V), device="cuda", generator=g)
    if c["logits"] == "peaked":
        sharp = (torch.arange(B, device="cuda")[:, None] + torch.arange(K, device="cuda")[None]) % 2 == 1
        draft *= torch.where(sharp, 4.0, 1.0)[:, :, None]
    s["draft"] = draft.to(target.dtype)
    # what the draft proposes: a token by the Gumbel-max trick, one of the groups that hold it
    noise = torch.empty_like(draft).exponential_(generator=g).log_()
    token = (s["draft"].float() / c["temperature"] - noise).argmax(dim=2)
    first, many = groups.tok_ptr[token].long(), groups.mult[token].long()
    entry = (torch.rand((B, K), device="cuda", generator=g) * many).long().clamp_(max=many - 1)
    s["prop_tokens"], s["prop_groups"] = token.int(), groups.tok_groups[first + entry]
    if c["call"] == "propose":
        s["pos0"] = min(3, 64 - K)
        s["out"] = (new((B, K), dtype=torch.int32), new((B, K), dtype=torch.int32)) if kept else (None, None)
        s["workspace"] = scratch(pcg.propose_workspace_bytes(V, B, K)) if kept else None
        return s
    s["target"] = target
    s["static"] = c["scratch"] == "static"
    s["out"] = s["trials"] = s["workspace"] = None
    if kept or s["static"]:
        s["out"] = pcg.VerifyOutput(new(B, dtype=torch.int32), new((B, K + 1), dtype=torch.int32),
                                    new((B, K + 1), dtype=torch.int32))
        s["trials"] = new(B, dtype=torch.int32)
    if kept:
        s["workspace"] = scratch(pcg.verify_workspace_bytes(V, groups.G, B, K) if c["call"] == "verify"
                                 else pcg.verify_thinning_workspace_bytes(V, B, K))
    return s


def run(state):
    s = state
    if s["call"] == "asg":
        a = pcg.asg_build_exact(s["emb"], s["theta"])
        return dict(row_ptr=a.row_ptr, members=a.members, mult=a.mult, seed_of=a.seed_of,
                    sizes=[a.G, a.nnz, a.max_size])
    if s["call"] == "group_probs":
        return pcg.group_probs(s["groups"], s["logits"], s["temperature"], out=s["out"], workspace=s["workspace"])
    if s["call"] == "propose":
        return pcg.propose(s["groups"], s["draft"], temperature=s["temperature"], seed=s["seed"],
                           offset=s["offset"], pos0=s["pos0"], prop_tokens=s["out"][0],
                           prop_groups=s["out"][1], workspace=s["workspace"])
    if s["call"] == "thinning":
        o, trials = pcg.verify_thinning(s["groups"], s["target"], s["draft"], s["prop_tokens"], s["prop_groups"],
                                        temperature=s["temperature"], seed=s["seed"], offset=s["offset"],
                                        out=s["out"], trials=s["trials"], workspace=s["workspace"])
        return dict(accept_len=o.accept_len, tokens=o.out_tokens, groups=o.out_groups, trials=trials)
    o = pcg.verify(s["groups"], s["target"], s["draft"], s["prop_tokens"], s["prop_groups"],
                   temperature=s["temperature"], seed=s["seed"], offset=s["offset"], out=s["out"],
                   workspace=s["workspace"], static_scratch=s["static"])
    return dict(accept_len=o.accept_len, tokens=o.out_tokens, groups=o.out_groups)


# ------------------------------------------------------------------------------ work, tolerance

def _nnz(c):
    return int(_sizes(c).sum())


def _logit_rows(c):
    return {"verify": c["B"] * (2 * c["K"] + 1), "thinning": c["B"] * (2 * c["K"] + 1),
            "propose": c["B"] * c["K"], "group_probs": c["B"] * (c["K"] + 1)}[c["call"]]


def _logit_bytes(c):
    return _logit_rows(c) * c["V"] * (2 if c["dtype"] == "bf16" else 4)


def work(case):
    """Every logit once (one exponential and two additions each); the membership once where all
    groups are summed, and one addition per entry and summed row."""
    c = case
    V = c["V"]
    if c["call"] == "asg":
        # one product per distinct pair of tokens; the embeddings once, about 26 members a group
        return {"bytes": 4 * V * c["d"] + 4 * 30 * V, "flops": float(c["d"]) * V * (V + 1)}
    rows = _logit_rows(c)
    nbytes, flops = _logit_bytes(c), 3.0 * rows * V
    if c["call"] in ("verify", "group_probs"):
        nnz = _nnz(c)
        summed = rows if c["call"] == "group_probs" else c["B"]
        nbytes += 4 * (nnz * (2 if c["weighted"] else 1) + 2 * V + 1)
        flops += float(summed) * nnz * (2 if c["weighted"] else 1)
    if c["call"] == "group_probs":
        nbytes += 4 * rows * V
    else:
        nbytes += 16 * c["B"] * (c["K"] + 1)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    c = case
    if c["call"] == "asg":
        return "exact"           # memberships are decided by cosines in double
    if c["call"] == "group_probs":
        # fp32 terms (exponential, weight) and fp32 sums of up to 140 of them: 8e-8 to 2.1e-7 from
        # the same in double
        return {"rel": 1e-6, "max": 1e-5}
    # Whole values, each decided by comparing a uniform with a sum of fp32 terms: against the same
    # step in double 1 of 109 800 sequences drew the neighbouring group.  Room for one such draw.
    return {"rel": 0.0, "differ": min(0.01, 1.5 / (c["B"] * (c["K"] + 1)))}


def exact(case, seed):
    """Group probabilities in double; the other calls return decisions, not computed numbers."""
    c = case
    if c["call"] != "group_probs":
        return None
    V = c["V"]
    row_ptr, members = _membership(c, seed)
    sizes = np.diff(row_ptr)
    mem = torch.from_numpy(members).cuda().long()
    group = torch.repeat_interleave(torch.arange(V, device="cuda"), torch.from_numpy(sizes).cuda())
    if c["weighted"]:
        w = torch.from_numpy(_weights(V, members, seed)).cuda().double()
    else:
        w = 1.0 / torch.bincount(mem, minlength=V).double()[mem]
    logits = _target_rows(c, seed).view(-1, V)
    out = torch.zeros((len(logits), V), dtype=torch.float64, device="cuda")
    for lo in range(0, len(logits), 32):
        p = torch.softmax(logits[lo:lo + 32].double() / float(np.float32(c["temperature"])), dim=1)
        out[lo:lo + 32].index_add_(1, group, p[:, mem] * w)
    return out
