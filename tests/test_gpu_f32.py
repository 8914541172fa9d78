"""float32 storage: the matrix-core product at sizes where its tiles, its k-steps of 16 and its 16-byte loads end inside the
matrix, against float64 products (bound: float32 sums of exact products), and the attention kernel at both head sizes that
the layer runs with (four and two groups over the keys), over fewer and more keys than it has threads, against the oracle."""
import numpy as np
import pytest

from gpu_util import have_gpu, Pair, tol_for

pytestmark = pytest.mark.gpu

if have_gpu():
    import torch
    import paper_2506_03566_amd as P
    from oracle.tree import Tree
    from synth import get_config, make_prompt, make_weights
    from synth.gpu import to_device


# 16 x 16 tiles (few outputs), 32 x 32 tiles (64 K outputs and more); K below a k-step, odd (scalar loads), ragged
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (3, 70, 7), (16, 17, 16), (17, 130, 68), (33, 33, 1030), (64, 1024, 260), (65, 1025, 332),
                                   (128, 1700, 2400), (61, 2000, 131)])
def test_f32_gemm_at_the_edges_of_its_tiles(M, N, K):
    print(f"f32 gemm {M} {N} {K}", flush=True)
    rng = np.random.default_rng(M + N + K)
    x, w = rng.normal(size=(M, K)).astype(np.float32), (rng.normal(size=(N, K)) * 0.02).astype(np.float32)
    y, _ = P.debug_gemm(0, to_device(x, 0), to_device(w, 0))
    err = np.abs(y.cpu().numpy().astype(np.float64) - x.astype(np.float64) @ w.astype(np.float64).T).max()
    assert err < 2e-5 * np.sqrt(max(K, 256) / 256.0), err


@pytest.mark.parametrize("head_dim,n_prompt", [(64, 300), (64, 3), (128, 257), (128, 17)])
def test_f32_attention_head_sizes_and_key_counts(head_dim, n_prompt):
    print(f"f32 attention dh={head_dim} prompt={n_prompt}", flush=True)
    pair = Pair("c0_tiny_f32", head_dim=head_dim, n_kv_heads=2)
    cfg = pair.cfg
    prompt = make_prompt(cfg, n=n_prompt)
    o = pair.oracle()
    o.prefill(prompt)
    assert pair.ctx.prefill(prompt) == o.tokens[-1]
    from oracle.tree import Tree
    tree = ([o.tokens[-1], 5, 6, 7], [-1, 0, 0, 1])
    logits = torch.zeros(4, cfg.vocab, device="cuda")
    pair.ctx.verify_tree(P.TreeArrays.from_lists(*tree), logits_out=logits)
    _, want, _ = o.verify_tree(Tree(*tree))
    assert np.abs(logits.cpu().numpy() - want).max() <= tol_for(cfg)
    pair.close()


# rows around a row tile and the change to two tiles by two (64 K sums); d_ffn that ends inside a group of 16 units, odd (scalar loads
# in the down projection); both head widths, K above and below what four waves keep in flight
@pytest.mark.parametrize("over", [dict(d_model=256, n_kv_heads=2, d_ffn=333), dict(d_model=72, n_q_heads=3, n_kv_heads=1, head_dim=128, d_ffn=17),
                                  dict(d_model=600, n_q_heads=6, n_kv_heads=3, d_ffn=1030)])
def test_f32_rows_do_not_hang_on_the_rows_around_them(over):
    """SiLU, rotary embedding and cache writes inside the products: the first layer's keys and values of a prompt's first rows are the
    same bits for any number of rows in the launch (later layers follow the attention, whose threads share out all the keys of the
    launch), the logits behind the last layer the oracle's."""
    print(f"f32 layers {over}", flush=True)
    pair = Pair("c0_tiny_f32", **over)
    cfg, prompt = pair.cfg, make_prompt(pair.cfg, n=120)
    pair.ctx.prefill(prompt)
    want = pair.ctx.debug_read_kv(-1, 0, 0, 120)
    from oracle.tree import Tree
    for n in (1, 2, 15, 16, 17, 33, 64, 65, 100):
        pair.ctx.reset()
        o = pair.oracle()
        o.prefill(prompt[:n])
        assert pair.ctx.prefill(prompt[:n]) == o.tokens[-1]
        for got, whole in zip(pair.ctx.debug_read_kv(-1, 0, 0, n), want):
            assert np.array_equal(got, whole[:n]), n
        tree = ([o.tokens[-1], 5, 6, 7], [-1, 0, 0, 1])
        logits = torch.zeros(4, cfg.vocab, device="cuda")
        pair.ctx.verify_tree(P.TreeArrays.from_lists(*tree), logits_out=logits)
        assert np.abs(logits.cpu().numpy() - o.verify_tree(Tree(*tree))[1]).max() <= tol_for(cfg), n
    pair.close()


# fewer ids than threads, around them, the last count of one launch and the first of two; 5 children: the third pair of equals is cut
@pytest.mark.parametrize("vocab,k", [(17, 16), (200, 5), (255, 5), (257, 16), (4095, 5), (4096, 16), (4097, 5)])
def test_f32_children_with_equal_logits(vocab, k):
    """Every even id's row of the head matrix is also the next odd id's: the k best of pairs of equal logits, lower ids first."""
    print(f"f32 children vocab={vocab} k={k}", flush=True)
    over = dict(vocab=vocab, top_k=k, depth=1, total_tokens=k, n_layers=1, n_specialists=1, positions_per_specialist=1, d_model=64,
                n_q_heads=1, n_kv_heads=1, d_ffn=64)
    st = make_weights(get_config("c0_tiny_f32", **over))
    st["lm_head"][1::2] = st["lm_head"][:vocab - 1:2][:len(st["lm_head"][1::2])]
    pair = Pair("c0_tiny_f32", storage=st, **over)
    prompt = make_prompt(pair.cfg, n=20)
    o = pair.oracle()
    o.prefill(prompt)
    pair.ctx.prefill(prompt)
    o.tokens[-1] = int(pair.ctx.tokens()[-1])
    got, want = pair.ctx.draft_tree().as_dict(), o.draft_tree()
    assert got["token"] == want.token and got["parent"] == want.parent
    assert np.abs(np.array(got["score"]) - np.array(want.score)).max() <= 1e-4
    pair.close()


# one id beyond the first half of a row, in between, and the most that one launch takes
@pytest.mark.parametrize("vocab", [2049, 3000, 4096])
def test_f32_scores_are_those_of_the_two_launches(vocab):
    """Children's scores are bit for bit what they are with ids that have no mass behind the vocabulary: 4200 ids take two launches, which
    sum 2048 ids each and merge the sums.  Feature 0 is about 8 in every row; ids without mass have logits of about -1600."""
    print(f"f32 scores vocab={vocab}", flush=True)
    over = dict(top_k=16, depth=1, total_tokens=16, n_layers=1, n_specialists=1, positions_per_specialist=1, d_model=64, n_q_heads=1,
                n_kv_heads=1, d_ffn=64)
    st = make_weights(get_config("c0_tiny_f32", vocab=4200, **over))
    st["embed"][:, 0] = 1
    st["spec0.fc_w"][0, 0] = 1
    st["lm_head"] *= 100
    st["lm_head"][:, 0] = -1.2                             # (log-sum-exp near 0, where its unit in the last place is small)
    st["lm_head"][vocab:] = 0
    st["lm_head"][vocab:, 0] = -200
    got = []
    for v in (vocab, 4200):
        pair = Pair("c0_tiny_f32", storage=dict(st, embed=st["embed"][:v].copy(), lm_head=st["lm_head"][:v].copy()), vocab=v, **over)
        out = []
        for seed in range(64):
            pair.ctx.reset()
            pair.ctx.prefill(np.random.default_rng(seed).integers(0, vocab, 20).astype(np.int32))
            d = pair.ctx.draft_tree().as_dict()
            out.append((d["token"], d["score"]))
        got.append(out)
        pair.close()
    differ = [seed for seed, (a, b) in enumerate(zip(*got)) if a[0] != b[0] or not np.array_equal(a[1], b[1])]
    print(f"  scores {got[0][0][1][1]:.3f} .. {got[0][0][1][-1]:.3f}, {len(differ)} of 64 prompts differ", flush=True)
    assert max(max(t) for t, _ in got[1]) < vocab and not differ


# half a head in one group of 16 pairs, an odd number of groups (and of 16-byte pieces a thread group), the widest; K of 72 and heads that
# share keys
@pytest.mark.parametrize("head_dim,n_prompt,over", [(32, 100, {}), (96, 17, dict(d_model=72)), (160, 70, dict(n_kv_heads=1)), (256, 33, {})])
def test_f32_head_sizes_other_than_the_16_bit_types(head_dim, n_prompt, over):
    """A whole round: prompt, draft (the keys and values of the specialists), verification against the oracle."""
    print(f"f32 head_dim={head_dim} prompt={n_prompt} {over}", flush=True)
    pair = Pair("c0_tiny_f32", head_dim=head_dim, **dict(dict(n_kv_heads=2), **over))
    cfg, prompt = pair.cfg, make_prompt(pair.cfg, n=n_prompt)
    o = pair.oracle()
    o.prefill(prompt)
    assert pair.ctx.prefill(prompt) == o.tokens[-1]
    for layer in range(cfg.n_layers):
        for got, want in zip(pair.ctx.debug_read_kv(-1, layer, 0, n_prompt), o.kv[layer]):
            assert np.abs(got - want).max() <= tol_for(cfg)
    tr = pair.ctx.draft_tree()
    from oracle.tree import Tree
    d, want = tr.as_dict(), o.draft_tree()
    assert np.abs(np.sort(np.array(d["score"])) - np.sort(np.array(want.score))).max() <= tol_for(cfg)
    logits = torch.zeros(tr.n, cfg.vocab, device="cuda")
    pair.ctx.verify_tree(logits_out=logits)
    assert np.abs(logits.cpu().numpy() - o.verify_tree(Tree(d["token"], d["parent"]))[1]).max() <= tol_for(cfg)
    assert len(pair.ctx.accept_and_commit()[2]) >= 1
    pair.close()


@pytest.mark.parametrize("d,ffn,vocab,rows", [(256, 688, 4096, 25), (70, 90, 4096, 17), (96, 250, 4097, 1), (1100, 1030, 100, 33), (32, 64, 8200, 16)])
def test_norms_inside_the_products(d, ffn, vocab, rows):
    """Float32 layers whose products norm their own operands: widths that are and are not multiples of 4 and of a k-step, more k-steps
    than a wave keeps in flight, row counts around a tile; greedy choices of one and of two segments.  Against the oracle in float64:
    sums of at most 1100 products of size 1, five layers and norms deep, 1e-4 as everywhere in float32; the chosen token is the largest logit,
    logits in the caller's array are those the choice was made from."""
    pair = Pair("c0_tiny_f32", d_model=d, d_ffn=ffn, vocab=vocab, n_q_heads=2, n_kv_heads=2, head_dim=32, depth=6, total_tokens=40)
    ctx, o = pair.ctx, pair.oracle()
    prompt = make_prompt(pair.cfg, n=20)
    ctx.prefill(prompt)
    o.prefill(prompt)
    o.tokens[-1] = ctx.tokens()[-1]
    tree = [int(o.tokens[-1])] + [(7 * i) % vocab for i in range(1, rows)]
    parent = [-1] + [(i - 1) // 2 for i in range(1, rows)]
    logits, feats = torch.zeros(rows, vocab, device="cuda"), torch.zeros(rows, d, device="cuda")
    g = ctx.verify_tree(P.TreeArrays.from_lists(tree, parent), logits_out=logits, feat_out=feats)[:rows]
    _, want, want_f = o.verify_tree(Tree(tree, parent))
    assert np.abs(logits.cpu().numpy() - want).max() < 1e-4
    assert np.abs(feats.cpu().numpy() - want_f).max() < 1e-4
    assert g.tolist() == logits.argmax(1).tolist()
    pair.close()
