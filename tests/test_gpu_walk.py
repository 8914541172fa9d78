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
