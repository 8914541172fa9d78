"""What a program does with this library, as cases that can be timed and compared.

Two kinds.  "gemm": one product through poss_gemm_static, the entry for callers that cannot allocate (weights come
row-major, the call packs them).  "decode": a context with its weights loaded, on which a pass is one step of a
generation: with `fresh` a new request (reset, prefill) and its first round, otherwise one round of a request that is
under way, which is replaced by the next prompt once `new` tokens have been committed.  A round drafts (`draft`) and
verifies a tree of `rows` rows; rows == 1 is plain decoding, the root alone.  The tree that is verified is the
program's own (random tokens, so that its shape and its rows do not hang on near-ties of the drafter), except with
`drawn`, where children are drawn at temperature 1 and the drafted tree is tested by the rejection rule.

Weights are random, but shaped like a trained model's where that decides what the kernels meet: residual projections
scaled with the depth, and a Head that is confident about one successor of every token.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2506_03566_amd as P

F32, BF16, F16 = 0, 1, 2
TORCH = {F32: torch.float32, BF16: torch.bfloat16, F16: torch.float16}

# Layer shapes of the repository's configurations.
L8B = dict(d=4096, hq=32, hkv=8, dh=128, ffn=14336, theta=500000.0, dtype=BF16)
L13B = dict(d=5120, hq=40, hkv=40, dh=128, ffn=13824, theta=10000.0, dtype=F16)
MID_BF16 = dict(d=512, hq=8, hkv=2, dh=64, ffn=1408, theta=500000.0, dtype=BF16)
MID_F16 = dict(d=640, hq=5, hkv=5, dh=128, ffn=1728, theta=10000.0, dtype=F16)
TINY_F32 = dict(d=256, hq=4, hkv=4, dh=64, ffn=688, theta=10000.0, dtype=F32)


def decode(layer, **kw):
    c = dict(kind="decode", **layer)
    c.update(layers=4, vocab=32000, S=3, n=2, k=10, depth=6, total=60, batch=1, prompt=512, new=256, rows=61,
             draft=False, fresh=False, drawn=False)
    c.update(kw)
    return c


def listed():
    return [
        # one activation row through a small projection: launches and latency are all there is
        dict(name="gemm_small", kind="gemm", dtype=BF16, M=1, N=512, K=512),
        # a tree's rows through a projection with odd sizes, the most the static scratch holds
        dict(name="gemm_tree", kind="gemm", dtype=F16, M=61, N=1720, K=5000),
        # the float32 reference shape: a whole short request, prompt and first round
        dict(decode(TINY_F32, layers=2, vocab=4096, k=4, total=24, prompt=64, rows=25, draft=True, fresh=True), name="request_f32"),
        # plain decoding of a half-precision target, one row at a time
        dict(decode(L13B, prompt=1024, rows=1), name="decode_row_f16"),
        # verification of a whole tree: the layers that carry the round
        dict(decode(L8B), name="verify_tree_bf16"),
        # the same against a long context, where the cache counts as much as the weights
        dict(decode(L8B, prompt=8192, new=512, depth=7, total=80, rows=81), name="verify_long_bf16"),
        # several sequences in one weight stream
        dict(decode(L8B, batch=4), name="verify_batch4_bf16"),
        # a request of ragged length: prompt, then the first draft and verification
        dict(decode(L13B, prompt=1001, draft=True, fresh=True), name="request_ragged_f16"),
        # a request with a long prompt, up to its first round
        dict(decode(L8B, prompt=8192, draft=True, fresh=True), name="request_long_bf16"),
        # drafting alone counts here (one specialist per position, full vocabulary, a target of one layer)
        dict(decode(L8B, layers=1, vocab=128256, S=6, n=1, rows=1, draft=True), name="draft_bf16"),
        # drawn children and the rejection rule at temperature 1 over the full vocabulary
        dict(decode(L8B, layers=1, vocab=128256, draft=True, drawn=True), name="drawn_round_bf16"),
        # the whole round of the benchmark's model
        dict(decode(L8B, layers=32, vocab=128256, draft=True), name="round_8b_bf16"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["gemm", "gemm", "f32", "row", "tree", "tree", "long", "batch", "request", "prompt", "draft", "drawn"])
    if what == "gemm":
        dt = rng.choice([F32, BF16, BF16, F16])
        return dict(kind="gemm", dtype=dt, M=_log_int(rng, 1, 128), N=_log_int(rng, 64, 1700),
                    K=8 * _log_int(rng, 8, 300 if dt == F32 else 625))
    if what == "f32":
        k, depth = rng.randint(2, 6), rng.randint(2, 6)
        total = rng.randint(2, min(40, k + (depth - 1) * k * k))
        return decode(TINY_F32, layers=rng.randint(1, 2), vocab=rng.randint(1000, 4096), k=k, depth=depth, total=total,
                      prompt=_log_int(rng, 2, 300), rows=rng.randint(1, total + 1), draft=True, fresh=True,
                      hkv=rng.choice([2, 4]))
    layer = rng.choice([L8B, L8B, L13B, MID_BF16, MID_F16])
    layers = rng.randint(1, 4)
    total = rng.randint(16, 100)
    if what == "row":
        return decode(layer, layers=layers, prompt=_log_int(rng, 8, 2048), rows=1)
    if what == "tree":
        return decode(layer, layers=layers, prompt=_log_int(rng, 8, 2048), total=total, rows=rng.randint(2, total + 1))
    if what == "long":
        return decode(layer, layers=layers, prompt=rng.randint(2049, 8192), new=512, total=total, rows=rng.randint(1, total + 1))
    if what == "batch":
        batch = rng.randint(2, 8)
        return decode(layer, layers=layers, batch=batch, prompt=_log_int(rng, 16, 512), total=total, rows=rng.randint(1, total + 1))
    if what == "request":
        return decode(layer, layers=layers, prompt=_log_int(rng, 8, 2048), total=total, rows=rng.randint(1, total + 1),
                      draft=True, fresh=True)
    if what == "prompt":
        return decode(layer, layers=layers, prompt=_log_int(rng, 100, 8192), rows=rng.choice([1, 16]), fresh=True)
    vocab = rng.choice([8192, 32000, 128256])
    prompt = _log_int(rng, 16, 512)
    if what == "draft":
        S = rng.randint(1, 6)
        depth = rng.randint(3, 7)
        return decode(layer, layers=1, vocab=vocab, S=S, n=max(1, depth // S), depth=depth, prompt=prompt, rows=1, draft=True)
    return decode(layer, layers=1, vocab=vocab, prompt=prompt, draft=True, drawn=True)


# ---------------------------------------------------------------- what the program has in hand
def _config(c):
    need = c["prompt"] + c["new"] + 2 * c["depth"] + 4
    return SimpleNamespace(
        n_layers=c["layers"], d_model=c["d"], n_q_heads=c["hq"], n_kv_heads=c["hkv"], head_dim=c["dh"], d_ffn=c["ffn"],
        vocab=c["vocab"], rms_eps=1e-5, rope_theta=c["theta"], dtype=c["dtype"], n_specialists=c["S"],
        positions_per_specialist=c["n"], fc_bias=1, top_k=c["k"], depth=c["depth"], total_tokens=c["total"],
        max_seq=(need + 63) // 64 * 64, kv_page_tokens=64, kv_page_order=0, batch=c["batch"])


def _weights(c, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = TORCH[c["dtype"]]

    def normal(*shape, std=0.02):
        return torch.empty(*shape, dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    d, qd, kd, ffn, vocab = c["d"], c["hq"] * c["dh"], c["hkv"] * c["dh"], c["ffn"], c["vocab"]
    out_std = 0.02 / math.sqrt(2 * max(c["layers"], 2))
    w = {"embed": normal(vocab, d, std=1.0), "final_norm": 1 + normal(d, std=0.1)}
    w["lm_head"] = normal(vocab, d)
    successor = torch.randperm(vocab, generator=g, device="cuda")
    w["lm_head"][successor] += w["embed"] * (0.4 / math.sqrt(d))

    def layer(pre):
        w[pre + "attn_norm"], w[pre + "mlp_norm"] = 1 + normal(d, std=0.1), 1 + normal(d, std=0.1)
        w[pre + "wq"], w[pre + "wk"], w[pre + "wv"] = normal(qd, d), normal(kd, d), normal(kd, d)
        w[pre + "wo"] = normal(d, qd, std=out_std)
        w[pre + "w_gate"], w[pre + "w_up"] = normal(ffn, d), normal(ffn, d)
        w[pre + "w_down"] = normal(d, ffn, std=out_std)

    for i in range(c["layers"]):
        layer("layer%d." % i)
    for s in range(c["S"]):
        fc = normal(d, 2 * d, std=0.005)
        fc[:, :d] += torch.eye(d, dtype=dt, device="cuda")
        w["spec%d.fc_w" % s], w["spec%d.fc_b" % s] = fc, normal(d)
        layer("spec%d." % s)
    return w


def _tree(c, rs):
    """A tree like the drafter's: parents drawn among the earlier nodes that are not too deep, siblings different."""
    token, parent, depth, kids = [0], [-1], [0], [set()]
    while len(token) < c["rows"]:
        low = max(0, len(token) - 3 * c["k"]) if rs.rand() < 0.8 else 0
        p = int(rs.randint(low, len(token)))
        t = int(rs.randint(0, c["vocab"]))
        if depth[p] == c["depth"] or t in kids[p]:
            continue
        token.append(t), parent.append(p), depth.append(depth[p] + 1), kids.append(set())
        kids[p].add(t)
    return token, parent


def _inputs(c, seed):
    rs = np.random.RandomState(seed)
    prompts = [rs.randint(0, c["vocab"], c["prompt"]).astype(np.int32) for _ in range(c["batch"])]
    return prompts, [_tree(c, rs) for _ in range(c["batch"])], rs


def prepare(case, seed):
    c = case
    if c["kind"] == "gemm":
        g = torch.Generator(device="cuda").manual_seed(seed)
        dt = TORCH[c["dtype"]]
        x = torch.empty(c["M"], c["K"], dtype=dt, device="cuda").normal_(generator=g)
        w = torch.empty(c["N"], c["K"], dtype=dt, device="cuda").normal_(0.0, 0.02, generator=g)
        return dict(case=c, x=x, w=w, y=torch.empty(c["M"], c["N"], dtype=torch.float32, device="cuda"))
    weights = _weights(c, seed)
    ctx = P.Poss(_config(c), weights)
    del weights                                    # the library keeps its own copy
    prompts, trees, rs = _inputs(c, seed)
    s = dict(case=c, ctx=ctx, prompts=prompts, trees=[P.TreeArrays.from_lists(*t) for t in trees], left=0)
    rows = c["total"] + 1 if c["drawn"] else c["rows"]
    s["logits"] = torch.empty(rows, c["vocab"], dtype=torch.float32, device="cuda")
    s["feats"] = torch.empty(rows, c["d"], dtype=torch.float32, device="cuda")
    if c["drawn"]:
        k, depth = c["k"], c["depth"]
        s["numbers"] = [(rs.random_sample(depth + 1).astype(np.float32) * np.float32(0.999),
                         rs.random_sample((depth, k, k)).astype(np.float32) * np.float32(0.999),
                         rs.random_sample((depth + 1, k + 1)).astype(np.float32) * np.float32(0.999)) for _ in range(16)]
        s["round"] = 0
    if not c["fresh"]:
        _start(s)
    return s


def _start(s):
    """The next request: every sequence gets its prompt."""
    ctx, c = s["ctx"], s["case"]
    ctx.reset()
    if c["drawn"]:
        ctx.set_sampling(0.0)
    for b, p in enumerate(s["prompts"]):
        ctx.prefill(p, seq=b)
    s["left"] = c["new"]


def run(state):
    s = state
    c = s["case"]
    if c["kind"] == "gemm":
        P.gemm_static(c["dtype"], s["x"], s["w"], s["y"])
        return s["y"]
    ctx, out = s["ctx"], {}
    if c["fresh"] or s["left"] <= 0:
        _start(s)
    if c["drawn"]:
        u, u_draft, u_accept = s["numbers"][s["round"] % 16]
        s["round"] += 1
        ctx.set_sampling(1.0, u)
        ctx.set_draft_sampling(u_draft, u_accept)
    if c["draft"]:
        trees = [ctx.draft_tree()] + [ctx.get_tree(b) for b in range(1, c["batch"])]
        # Which of two near-tied children a 16-bit drafter keeps hangs on its rounding, their scores do not: its tokens come
        # back where the verified rows hang on them anyway.
        out["draft"] = [t.score[:t.n] for t in trees]
        if c["drawn"] or c["dtype"] == F32:
            out["tokens"] = [t.token[:t.n] for t in trees] + [t.parent[:t.n] for t in trees]
    ctx.verify_tree(None if c["drawn"] else s["trees"], logits_out=s["logits"], feat_out=s["feats"])
    _, _, tokens = ctx.accept_and_commit()
    s["left"] -= len(tokens)
    out["logits"], out["feats"], out["token"] = s["logits"], s["feats"], tokens[-1]
    return out


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    c = case
    es = 4 if c["dtype"] == F32 else 2
    if c["kind"] == "gemm":
        return {"bytes": (c["M"] + c["N"]) * c["K"] * es + c["M"] * c["N"] * 4, "flops": 2 * c["M"] * c["N"] * c["K"]}
    d, qd, kd, ffn, vocab = c["d"], c["hq"] * c["dh"], c["hkv"] * c["dh"], c["ffn"], c["vocab"]
    layer = d * (2 * qd + 2 * kd + 3 * ffn)
    kv = 2 * kd * es                               # bytes of one token's keys and values in one layer
    rows = (c["total"] + 1 if c["drawn"] else c["rows"]) * c["batch"]
    nbytes = flops = 0
    if c["fresh"]:                                 # the prompt through every layer, the specialists' keys and values
        n = c["prompt"] * c["batch"]
        nbytes += c["layers"] * (layer * es + n * kv) + c["S"] * ((2 * d * d + 2 * d * kd) * es + n * kv) + vocab * d * es
        flops += 2 * n * c["layers"] * layer + 2 * n * c["layers"] * c["prompt"] * qd
        flops += 2 * n * c["S"] * (2 * d * d + 2 * d * kd) + 2 * c["batch"] * vocab * d
    if c["draft"]:                                 # each level: its specialist and the Head, k rows (the first: one)
        draft_rows = (1 + (c["depth"] - 1) * c["k"]) * c["batch"]
        nbytes += c["depth"] * ((layer + 2 * d * d + vocab * d) * es + c["batch"] * c["prompt"] * kv)
        flops += 2 * draft_rows * (layer + 2 * d * d + vocab * d + 2 * c["prompt"] * qd)
    nbytes += c["layers"] * (layer * es + c["batch"] * c["prompt"] * kv) + vocab * d * es
    nbytes += rows // c["batch"] * (vocab + d) * 4
    flops += 2 * rows * (c["layers"] * (layer + 2 * c["prompt"] * qd) + vocab * d)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what another order of the sums changes (other K splits, other attention splits), or the distance
    to 64 bits where that is larger.  Drawn children are held to the same figures, although other sums can draw other
    children altogether."""
    c = case
    if c["kind"] == "gemm":
        return {"rel": 3e-6}
    if c["dtype"] == F32:
        return {"rel": 5e-6}
    return {"rel": 2.6e-2 if c["dtype"] == BF16 or c["draft"] else 4e-3}


# ---------------------------------------------------------------- the same in 64 bits
def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * gain.double()


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device="cuda") * 2 / x.shape[-1])
    ang = pos.double()[:, None, None] * inv
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _forward(c, w, tokens, pos, allowed):
    """Features of every row; allowed(r0, r1): which rows the rows [r0, r1) attend to."""
    n, hq, hkv, dh = len(tokens), c["hq"], c["hkv"], c["dh"]
    h = w["embed"][tokens].double()
    for i in range(c["layers"]):
        p = "layer%d." % i
        u = _norm(h, w[p + "attn_norm"])
        q = _rope((u @ w[p + "wq"].double().T).view(n, hq, dh), pos, c["theta"]).transpose(0, 1).contiguous()
        k = _rope((u @ w[p + "wk"].double().T).view(n, hkv, dh), pos, c["theta"]).permute(1, 2, 0).contiguous()
        v = (u @ w[p + "wv"].double().T).view(n, hkv, dh).transpose(0, 1).contiguous()
        att = torch.empty(n, hq, dh, dtype=torch.float64, device="cuda")
        for r0 in range(0, n, 1024):
            r1 = min(n, r0 + 1024)
            see = allowed(r0, r1)
            for x in range(hq):
                sc = (q[x, r0:r1] @ k[x * hkv // hq]) / math.sqrt(dh)
                att[r0:r1, x] = torch.softmax(sc.masked_fill(~see, -math.inf), -1) @ v[x * hkv // hq]
        h = h + att.view(n, hq * dh) @ w[p + "wo"].double().T
        u = _norm(h, w[p + "mlp_norm"])
        gate = u @ w[p + "w_gate"].double().T
        h = h + (gate * torch.sigmoid(gate) * (u @ w[p + "w_up"].double().T)) @ w[p + "w_down"].double().T
    return h


def exact(case, seed):
    c = case
    if c["kind"] == "gemm":
        s = prepare(c, seed)
        return s["x"].double() @ s["w"].double().T
    if c["drawn"]:
        return None                                # which tree is drawn hangs on the drafter's own rounding
    w = _weights(c, seed)
    prompts, trees, _ = _inputs(c, seed)
    prompt, (token, parent) = prompts[0], trees[0]
    n, m = len(prompt), len(token)

    def head(f):
        x, out = _norm(f, w["final_norm"]), []
        for v0 in range(0, c["vocab"], 16384):
            out.append(x @ w["lm_head"][v0:v0 + 16384].double().T)
        return torch.cat(out, -1)

    ids = torch.from_numpy(prompt).long().cuda()
    at = torch.arange(n + m, device="cuda")
    first = int(head(_forward(c, w, ids, at[:n], lambda a, b: at[:n] <= at[a:b, None])[-1:]).argmax())
    depth, mask = [0] * m, torch.zeros(m, m, dtype=torch.bool)
    for i in range(m):
        mask[i, i] = True
        if i:
            depth[i] = depth[parent[i]] + 1
            mask[i] |= mask[parent[i]]
    mask = mask.cuda()
    rows = torch.tensor([first] + token[1:], device="cuda")
    pos = torch.cat([at[:n], n + torch.tensor(depth, device="cuda")])

    def allowed(a, b):
        see = at <= at[a:b, None]
        if b > n:
            see[max(n - a, 0):, n:] = mask[max(a - n, 0):b - n]
        return see

    feats = _forward(c, w, torch.cat([ids, rows]), pos, allowed)[n:]
    out = dict(logits=head(feats), feats=feats, token=None)
    if c["draft"]:
        out["draft"] = [None] * c["batch"]
    return out
