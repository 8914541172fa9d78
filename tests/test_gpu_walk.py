"""Attention over long walks (attn_walk_kernel: splits of 32 blocks of 32 keys and more) against the kernel of shorter splits, and the
prompts' kernel at query-head groups that leave its workgroups partly empty against the oracle."""
import numpy as np
import pytest

from gpu_util import have_gpu, Pair
from test_gpu_prefill import test_long_prompt_leaves_the_oracles_caches as check_prompt

pytestmark = pytest.mark.gpu

if have_gpu():
    import torch
    import paper_2506_03566_amd as P
    from synth import get_config, make_weights
    from synth.gen import to_float64, to_storage


def _tree(rows, vocab, seed):
    rng = np.random.default_rng(seed)
    parent, depth = [-1], [0]
    while len(parent) < rows:
        p = int(rng.integers(max(0, len(parent) - 20), len(parent)))
        p = p if depth[p] < 6 else 0
        parent.append(p)
        depth.append(depth[p] + 1)
    return P.TreeArrays.from_lists([0] + [int(t) for t in rng.permutation(vocab)[:rows - 1]], parent)


# Rows around the edges of a wave's 32 query rows x heads and a workgroup's 128; keys around the edges of blocks, key-way pairs and
# splits (1024 keys: the last split of 4097 + rows has one block or two, 4000 + rows ends inside a block); groups of 1, 2, 3 and 4 query
# heads, both head widths, every page size; two sequences of different length in one launch.
# One layer without an MLP (down projection 0), queries and keys scaled so that a row's probabilities sit on a few keys: a feature is
# the embedding plus the projected attention outputs.  Both paths see the same keys, values and queries; their sums differ by far less
# than an output's rounding, so at the most every output is rounded the other way: a unit in the last place, at
# most 2^-7 of it, and a random projection keeps that ratio.
@pytest.mark.parametrize("name,prompts,rows,over", [
    ("t_mid_bf16", (4000,), 1, {}),
    ("t_mid_bf16", (4000,), 8, dict(kv_page_tokens=32, kv_page_order=1)),
    ("t_mid_bf16", (4097,), 9, dict(kv_page_tokens=128)),
    ("t_mid_bf16", (4095,), 33, dict(n_q_heads=6, n_kv_heads=2)),
    ("t_mid_bf16", (4001, 4130), 65, dict(n_q_heads=4, n_kv_heads=2, head_dim=128)),
    ("t_mid_bf16", (4097,), 100, dict(n_q_heads=2, n_kv_heads=2, head_dim=128)),
    ("t_mid_bf16", (4064, 4000), 31, dict(n_q_heads=4, n_kv_heads=1, head_dim=64)),
    ("t_mid_bf16", (3000,), 101, {}),
])
def test_long_walk_is_the_short_one(name, prompts, rows, over):
    print(f"walk {name} prompts={prompts} rows={rows} {over}", flush=True)
    over = dict(dict(n_layers=1, max_seq=4480, n_specialists=1, positions_per_specialist=6, total_tokens=100), **over)
    cfg = get_config(name, **over)
    storage = make_weights(cfg)
    storage["layer0.w_down"] = np.zeros_like(storage["layer0.w_down"])
    for w in ("layer0.wq", "layer0.wk"):
        storage[w] = to_storage(8 * to_float64(storage[w], cfg.dtype), cfg.dtype)
    pair = Pair(name, storage=storage, lib_over=dict(batch=len(prompts)), **over)
    trees = [_tree(rows, cfg.vocab, b) for b in range(len(prompts))]
    base = to_float64(storage["embed"], cfg.dtype)[[t for tr in trees for t in tr.token[:rows]]]
    out = {}
    for keys in (512, 1024):
        pair.ctx.reset()
        for b, n in enumerate(prompts):
            pair.ctx.prefill(np.random.default_rng(b).integers(0, cfg.vocab, n).astype(np.int32), seq=b)
            base[b * rows] = to_float64(storage["embed"], cfg.dtype)[pair.ctx.tokens(b)[-1]]
        pair.ctx.set_tuning(0, keys)
        feats = torch.zeros(rows * len(prompts), cfg.d_model, dtype=torch.float32, device="cuda")
        pair.ctx.verify_tree(trees if len(trees) > 1 else trees[0], feat_out=feats)
        out[keys] = feats.cpu().numpy().astype(np.float64) - base
    pair.close()
    assert np.isfinite(out[1024]).all()
    size = np.linalg.norm(out[512], axis=1)
    err = np.linalg.norm(out[1024] - out[512], axis=1) / size
    print(f"  outputs of norm {size.min():.3f} .. {size.max():.3f}, largest relative difference of a row {err.max():.2e}", flush=True)
    assert err.max() <= 2.0 ** -7


# 3 heads per KV head, 2 and 4 of width 128, one; a last range of one row, of two, of all; pages of every size
@pytest.mark.parametrize("name,n_prompt,over", [
    ("t_mid_bf16", 700, dict(n_q_heads=6, n_kv_heads=2)),
    ("t_mid_bf16", 645, dict(n_q_heads=4, n_kv_heads=2, head_dim=128, kv_page_tokens=32)),
    ("t_mid_f16", 900, dict(n_q_heads=4, n_kv_heads=1)),
    ("t_mid_f16", 1025, {}),
    ("t_mid_f16", 770, dict(kv_page_tokens=32, kv_page_order=1)),
])
def test_prompts_of_other_head_groups(name, n_prompt, over):
    check_prompt(name, n_prompt, over)


def test_splits_of_a_very_long_context_stay_within_what_a_wave_can_address():
    """271000 tokens in splits of 1056 keys would be 257 splits: they become splits of 2048 keys (64 blocks, a page-table entry per lane),
    not of 2112.  The same bits as 2048 keys asked for; one KV head, reversed pages."""
    over = dict(n_layers=1, n_q_heads=2, n_kv_heads=1, d_model=128, d_ffn=64, vocab=300, max_seq=271360, kv_page_order=1, n_specialists=1,
                positions_per_specialist=6)
    print("walk over 271000 tokens", flush=True)
    pair = Pair("t_mid_bf16", **over)
    tree = _tree(9, 300, 0)
    out = []
    for keys in (2048, 1056):
        pair.ctx.reset()
        pair.ctx.prefill(np.random.default_rng(3).integers(0, 300, 271000).astype(np.int32))
        pair.ctx.set_tuning(0, keys)
        feats = torch.zeros(9, 128, dtype=torch.float32, device="cuda")
        pair.ctx.verify_tree(tree, feat_out=feats)
        out.append(feats.cpu().numpy())
    pair.close()
    assert np.isfinite(out[0]).all() and np.array_equal(out[0], out[1])


def _round(x, cfg):
    return to_float64(to_storage(x, cfg.dtype), cfg.dtype)


def _attention_scales(q, k, seen, s, cfg):
    """Rows (q: [rows, heads, dh]) over keys k [keys, KV heads, dh] that they see, values s[key] c[dim]: the float64 output as a multiple of c per
    row and head, and that multiple as it is read from rounded outputs (the mean over the dims) when the probabilities enter P V as hi + lo,
    as hi alone, and as hi + the low halves of the keys 8 further."""
    dh, group = cfg.head_dim, cfg.n_q_heads // cfg.n_kv_heads
    c = (128 + np.arange(dh) * (128 // dh)) / 128
    score = np.stack([q[:, h] @ k[:, h // group].T for h in range(cfg.n_q_heads)], 1) / np.sqrt(dh)
    score = np.where(seen[:, None], score, -np.inf)
    p = np.exp(score - score.max(-1, keepdims=True))
    hi = _round(p, cfg)
    lo = _round(p - hi, cfg)
    z = p.sum(-1)
    return p @ s / z, [(_round((x @ s / z)[..., None] * c, cfg) / c).mean(-1) for x in (hi + lo, hi, hi + np.roll(lo, 8, -1))]


# Both head widths (8 and 16 fragments of keys in a step), rows that leave a workgroup's last wave partly empty, a last split of one block;
# splits of 2048 keys use all 64 page-table entries that a wave holds
@pytest.mark.parametrize("n_prompt,rows,over", [(4000, 61, dict(kv_page_tokens=32, kv_page_order=1)), (4064, 100, dict(n_q_heads=4, n_kv_heads=2, head_dim=128))])
def test_low_halves_of_the_probabilities_count(n_prompt, rows, over):
    """bf16 probabilities enter P V as the sum of two bf16 numbers, in walks and prompts.  One layer without an MLP whose values are s c[dim] with s
    1 or 2 per token (exact), output projection the identity: an output is a multiple of c, rounded, and the mean over the dims reads the multiple
    to 4e-5 to 7e-5, where one bf16 number per probability is off by 2e-4.  The median error over rows and heads against float64
    (keys from the cache; queries formed here, whose rounding a float32 sum flips in a few rows) is held to what the float64 model
    of hi + lo shows, output rounding included, and a quarter; models without the low halves, or with another key's, are off by more."""
    over = dict(dict(n_layers=1, max_seq=4480, n_specialists=1, positions_per_specialist=6, total_tokens=100, norm_gain_jitter=0.0), **over)
    cfg = get_config("t_mid_bf16", **over)
    print(f"low halves prompt={n_prompt} rows={rows} {over}", flush=True)
    rng, d, dh = np.random.default_rng(5), cfg.d_model, cfg.head_dim
    qd, kd = cfg.n_q_heads * dh, cfg.n_kv_heads * dh
    assert qd == d
    c = (128 + np.arange(dh) * (128 // dh)) / 128
    embed = rng.choice([-1.0, 1.0], (cfg.vocab, d))        # RMSNorm leaves them as they are
    embed[:, :2] = 1
    wq, wk = rng.normal(0, 2 / np.sqrt(d), (qd, d)), rng.normal(0, 2 / np.sqrt(d), (kd, d))     # scores of standard deviation 4
    wv = np.zeros((kd, d))
    wv[:, 0], wv[:, 1], wv[:, 2] = np.tile(c, cfg.n_kv_heads), np.tile(c / 2, cfg.n_kv_heads), np.tile(c / 2, cfg.n_kv_heads)
    storage = make_weights(cfg)
    for name, w in (("embed", embed), ("layer0.wq", wq), ("layer0.wk", wk), ("layer0.wv", wv), ("layer0.wo", np.eye(d)),
                    ("layer0.w_down", np.zeros((d, cfg.d_ffn)))):
        storage[name] = to_storage(w, cfg.dtype)
    pair = Pair("t_mid_bf16", storage=storage, **over)
    wq = _round(wq, cfg)

    def queries(ids, pos):
        x = (embed[ids] @ wq.T).reshape(-1, cfg.n_q_heads, dh)
        ang = np.asarray(pos)[:, None, None] * cfg.rope_theta ** (-2.0 * np.arange(dh // 2) / dh)
        a, b = x[..., :dh // 2], x[..., dh // 2:]
        return _round(np.concatenate([a * np.cos(ang) - b * np.sin(ang), b * np.cos(ang) + a * np.sin(ang)], -1), cfg)

    def check(what, out, ids, pos, k, seen, s):
        want, (both, one, other) = _attention_scales(queries(ids, pos), k, seen, s, cfg)
        got = (out.reshape(-1, cfg.n_q_heads, dh) / c).mean(-1)
        err, both, one, other = [float(np.median(np.abs(x / want - 1))) for x in (got, both, one, other)]
        print(f"  {what}: {err:.2e}; model {both:.2e}, high halves alone {one:.2e}, other low halves {other:.2e}", flush=True)
        assert 1.25 * both < min(one, other)
        assert err <= 1.25 * both, what

    prompt = rng.integers(0, cfg.vocab, n_prompt).astype(np.int32)
    last = (n_prompt - 1) % 256 + 1
    taps = torch.zeros(2, last, d, dtype=torch.float32, device="cuda")
    tree = _tree(rows, cfg.vocab, 1)
    for keys in (0, 512, 1024, 2048):
        pair.ctx.reset()
        pair.ctx.set_tuning(0, keys)
        pair.ctx.debug_set_taps(taps if keys == 0 else None)
        pair.ctx.prefill(prompt)
        pair.ctx.debug_set_taps(None)
        ids = np.array([pair.ctx.tokens()[-1]] + [int(t) for t in tree.token[1:rows]])
        s = 1.5 + 0.5 * embed[np.concatenate([prompt, ids]), 2]
        if keys == 0:
            pos = np.arange(n_prompt - last, n_prompt)
            k = pair.ctx.debug_read_kv(-1, 0, 0, n_prompt)[0].astype(np.float64)
            seen = np.arange(n_prompt)[None] <= pos[:, None]
            check("prompt", (taps[1] - taps[0]).cpu().numpy().astype(np.float64), prompt[pos], pos, k, seen, s[:n_prompt])
        feats = torch.zeros(rows, d, dtype=torch.float32, device="cuda")
        pair.ctx.verify_tree(tree, feat_out=feats)
        k, v = pair.ctx.debug_read_kv(-1, 0, 0, n_prompt + rows)
        assert np.array_equal(v[:, 0], (s[:, None] * c).astype(np.float32))
        seen, depth = np.zeros((rows, n_prompt + rows), bool), np.zeros(rows, int)
        seen[:, :n_prompt] = True
        for i in range(rows):
            p = int(tree.parent[i])
            if p >= 0:
                seen[i] |= seen[p]
                depth[i] = depth[p] + 1
            seen[i, n_prompt + i] = True
        check(f"{keys or 'usual'} keys a split", feats.cpu().numpy().astype(np.float64) - embed[ids], ids, n_prompt + depth, k.astype(np.float64), seen, s)
    pair.close()
