"""Prompts of more than 512 tokens go through the many-row kernels (gemm_block_kernel and what
surrounds it).  The caches they leave, the target's and every specialist's, against the oracle's, at prompt lengths around the
edges of tiles and chunks and at widths that select each tile shape.  Tolerances: those of the other cache comparisons, 2e-2
for 16-bit storage (rounding points are the oracle's; float32 against float64 sums flip a few of them)."""
import numpy as np
import pytest

from gpu_util import have_gpu, Pair, tol_for

pytestmark = pytest.mark.gpu

if have_gpu():
    import torch
    from oracle.model import specialist_kv
    from synth import make_prompt


# (shape, prompt, layers, overrides): tiles of 128 x 128 (few columns), 256 x 256 (gate/up of 14336 units), 256 x 128 (gate/up of
# 3072 units, 1001 rows); K not a multiple of 32 in the down projection (1416, 1736) and odd k-step counts; a specialist's catch-up of 512
# rows (the weight-streaming kernels) and of more
@pytest.mark.parametrize("name,n_prompt,over", [
    ("t_mid_bf16", 513, {}),
    ("t_mid_bf16", 514, dict(d_ffn=1416, kv_page_tokens=32, kv_page_order=1)),
    ("t_mid_f16", 641, dict(d_ffn=1736)),
    ("t_mid_f16", 769, dict(kv_page_tokens=128)),
    ("t_mid_bf16", 600, dict(d_ffn=14336)),
    ("t_mid_bf16", 1001, dict(d_ffn=3072)),
    ("t_mid_f16", 1100, dict(fc_bias=0)),
    ("t_mid_f16", 2305, dict(max_seq=2560)),                                         # a walk of more than 64 key blocks
    ("t_mid_bf16", 4400, dict(max_seq=4480, d_model=128, n_q_heads=2, n_kv_heads=1)),   # two passes; more than 128 blocks
])
def test_long_prompt_leaves_the_oracles_caches(name, n_prompt, over):
    print(f"prefill {name} prompt={n_prompt} {over}", flush=True)
    pair = Pair(name, **dict(dict(n_layers=2, max_seq=1280, n_specialists=2, positions_per_specialist=3), **over))
    cfg, tol = pair.cfg, tol_for(pair.cfg)
    prompt = make_prompt(cfg, n=n_prompt)
    o = pair.oracle()
    o.prefill(prompt)
    first = pair.ctx.prefill(prompt)
    for layer in range(cfg.n_layers):
        k, v = pair.ctx.debug_read_kv(-1, layer, 0, n_prompt)
        err = max(np.abs(k - o.kv[layer][0]).max(), np.abs(v - o.kv[layer][1]).max())
        print(f"  layer {layer}: {err:.2e}", flush=True)
        assert err <= tol
    for s in range(cfg.n_specialists):
        wk, wv = specialist_kv(pair.W, cfg, s, prompt[1:], np.stack(o.feats[:n_prompt - 1]), np.arange(n_prompt - 1), pair.act)
        k, v = pair.ctx.debug_read_kv(s, 0, 0, n_prompt - 1)
        err = max(np.abs(k - wk).max(), np.abs(v - wv).max())
        print(f"  specialist {s}: {err:.2e}", flush=True)
        assert err <= tol
    o.tokens[-1] = first                                   # (a near-tie may go either way; the round below has its own checks)
    assert pair.ctx.draft_tree().n == cfg.total_tokens + 1
    pair.ctx.verify_tree()
    assert len(pair.ctx.accept_and_commit()[2]) >= 1
    pair.close()


# down projections of few columns and a long K: their planes are summed by the residual + norm epilogue.  Three splits of 64 pairs of
# k-steps, four of 79 with an odd last k-step, five of 86; both types; the last layer's features go to the stash through it
@pytest.mark.parametrize("name,n_prompt,ffn", [("t_mid_f16", 513, 4088), ("t_mid_f16", 600, 5000), ("t_mid_bf16", 700, 5480)])
def test_split_products_leave_the_oracles_caches(name, n_prompt, ffn):
    test_long_prompt_leaves_the_oracles_caches(name, n_prompt, dict(d_ffn=ffn))


@pytest.mark.parametrize("name", ["t_mid_bf16", "t_mid_f16"])
def test_unsplit_products_are_the_streaming_kernels_bit_for_bit(name):
    """d_model of 512 and 640: the streaming kernels do not split the K of the QKV projection either, so the first layer's keys
    and values of a long prompt are those of its first 500 tokens alone."""
    pair = Pair(name, n_layers=1, max_seq=1280, n_specialists=1, positions_per_specialist=6)
    prompt = make_prompt(pair.cfg, n=700)
    pair.ctx.prefill(prompt[:500])
    want = pair.ctx.debug_read_kv(-1, 0, 0, 500)
    pair.ctx.reset()
    pair.ctx.prefill(prompt)
    got = pair.ctx.debug_read_kv(-1, 0, 0, 500)
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
    pair.close()


@pytest.mark.parametrize("name", ["t_mid_bf16", "t_mid_f16"])
def test_first_rows_of_a_long_prompt_round_as_the_streaming_kernels_do(name):
    """Products that neither path splits (K of at most 704) and rows that see at most 120 keys: every layer's keys and values of a
    long prompt's first 120 tokens are those of these tokens alone, through norms, rotary embedding, SiLU and residual - in fp16
    too, where a conversion can round a product once or twice."""
    pair = Pair(name, n_layers=3, d_ffn=704, max_seq=1280, n_specialists=1, positions_per_specialist=6)
    for seed in range(3):
        prompt = np.random.default_rng(seed).integers(0, pair.cfg.vocab, 700).astype(np.int32)
        got = []
        for n in (120, 700):
            pair.ctx.reset()
            pair.ctx.prefill(prompt[:n])
            got.append([pair.ctx.debug_read_kv(-1, layer, 0, 120) for layer in range(3)])
        for layer in range(3):
            assert all(np.array_equal(a, b) for a, b in zip(got[0][layer], got[1][layer])), (seed, layer)
    pair.close()


@pytest.mark.parametrize("name,over", [("t_mid_bf16", dict(d_ffn=5480)), ("t_mid_f16", {})])
def test_a_long_prompts_sums_do_not_hang_on_batch_or_capacity(name, over):
    got = []
    for max_seq, batch in ((768, 1), (8192, 1), (1280, 3)):
        pair = Pair(name, lib_over=dict(batch=batch), n_layers=2, n_specialists=1, positions_per_specialist=6, max_seq=max_seq, **over)
        pair.ctx.prefill(make_prompt(pair.cfg, n=700))
        got.append(caches(pair, 700))
        pair.close()
    for other in got[1:]:
        for (k, v), (wk, wv) in zip(other, got[0]):
            assert np.array_equal(k, wk) and np.array_equal(v, wv)


def caches(pair, n):
    cfg, ctx = pair.cfg, pair.ctx
    return ([ctx.debug_read_kv(-1, layer, 0, n) for layer in range(cfg.n_layers)] +
            [ctx.debug_read_kv(s, 0, 0, n - 1) for s in range(cfg.n_specialists)])


@pytest.mark.parametrize("name,n_prompt", [("t_mid_bf16", 600), ("t_mid_f16", 768), ("t_mid_f16", 1025)])
def test_taps_show_the_pass_that_runs_without_them(name, n_prompt):
    """The caches are bit for bit those of the same prompt without taps; the taps hold the rows of the prompt's last 256-row
    chunk (88, 256 and 1 of them): the embeddings first, the oracle's features last, nothing behind them."""
    print(f"taps {name} prompt={n_prompt}", flush=True)
    pair = Pair(name, n_layers=2, max_seq=1280, n_specialists=2, positions_per_specialist=3)
    cfg, ctx = pair.cfg, pair.ctx
    prompt = make_prompt(cfg, n=n_prompt)
    ctx.prefill(prompt)
    want = caches(pair, n_prompt)
    rows = (n_prompt - 1) % 256 + 1
    buf = torch.full(((cfg.n_layers + 1) * rows * cfg.d_model + 64,), -7.0, device="cuda")
    ctx.reset()
    ctx.debug_set_taps(buf)
    ctx.prefill(prompt)
    ctx.debug_set_taps(None)
    for (k, v), (wk, wv) in zip(caches(pair, n_prompt), want):
        assert np.array_equal(k, wk) and np.array_equal(v, wv)
    assert (buf[-64:] == -7).all()
    taps = buf[:-64].view(cfg.n_layers + 1, rows, cfg.d_model)
    ids = torch.as_tensor(np.asarray(prompt[-rows:]), device="cuda").long()
    assert torch.equal(taps[0], pair.dev_weights["embed"][ids].float())
    o = pair.oracle()
    o.prefill(prompt)
    feats = np.stack(o.feats[n_prompt - rows:n_prompt])
    assert np.abs(taps[-1].cpu().numpy() - feats).max() <= tol_for(cfg) * max(1.0, np.abs(feats).max())
    pair.close()


def test_profile_counts_the_products_of_a_long_prompt():
    """Every product of the prompt's pass and of the specialists' catch-up, its weights once."""
    pair = Pair("t_mid_bf16", n_layers=2, max_seq=1280, n_specialists=2, positions_per_specialist=3)
    cfg, ctx = pair.cfg, pair.ctx
    ctx.profile_gemm(True)
    ctx.gemm_profile()
    ctx.prefill(make_prompt(cfg, n=600))
    launches, ms, nbytes = ctx.gemm_profile()
    ctx.profile_gemm(False)
    d, qd, kd, ffn = cfg.d_model, cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim, cfg.d_ffn
    assert launches == 4 * cfg.n_layers + 1 + 2 * cfg.n_specialists
    assert nbytes == 2 * (cfg.n_layers * d * (2 * qd + 2 * kd + 3 * ffn) + cfg.vocab * d + cfg.n_specialists * d * (2 * d + 2 * kd))
    assert 0 < ms < 100
    pair.close()


# 4096 rows: 16 row tiles, 18 or 17 column tiles of 256 - one round of the larger tiles, then 64 or 32 of the smaller.  QKV (the rest: values), gate and
# up, the residual projections (whose sums must not be split over K: K below 2048 or few columns)
@pytest.mark.parametrize("name,over", [("t_mid_bf16", dict(n_layers=1, d_model=128, n_q_heads=28, n_kv_heads=4, d_ffn=512)),
                                       ("t_mid_f16", dict(n_layers=2, d_model=128, n_q_heads=2, n_kv_heads=2, d_ffn=2176)),
                                       ("t_mid_f16", dict(n_layers=2, d_model=4344, n_q_heads=2, n_kv_heads=2, d_ffn=520))])
def test_two_tile_shapes_in_one_launch_give_the_bits_of_one(name, over):
    """Keys and values of a prompt's first 600 rows: 4096 rows take both tile shapes in one launch, 600 rows one; the same bits."""
    print(f"mixed tiles {name} {over}", flush=True)
    pair = Pair(name, head_dim=128, vocab=300, n_specialists=1, positions_per_specialist=6, max_seq=4224, **over)
    prompt = np.random.default_rng(7).integers(0, 300, 4096).astype(np.int32)
    got = []
    for n in (600, 4096):
        pair.ctx.reset()
        pair.ctx.prefill(prompt[:n])
        got.append([pair.ctx.debug_read_kv(-1, layer, 0, 600) for layer in range(pair.cfg.n_layers)])
    for few, many in zip(*got):
        assert np.abs(few[0]).max() > 0 and np.array_equal(few[0], many[0]) and np.array_equal(few[1], many[1])
    pair.close()
