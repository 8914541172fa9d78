"""Dispatch branches at the sizes where they can go wrong: draws from vocabularies around a block of 256 ids and beyond 1024 blocks,
attention merged from 2 to 16 splits, and outputs that the kernels write straight into the caller's arrays."""
import numpy as np
import pytest

from gpu_util import have_gpu, Pair, tol_for

pytestmark = pytest.mark.gpu

if have_gpu():
    import torch
    import paper_2506_03566_amd as P
    from oracle.sampling import softmax_t
    from oracle.tree import Tree
    from synth import get_config, make_prompt
    from synth.gpu import make_weights_on_device


# a block and one id less and more; segments of 4096; 1025 blocks: two blocks per share of the scan
@pytest.mark.parametrize("vocab", [255, 256, 257, 4096, 4100, 262401])
def test_drawn_children_lie_in_their_cdf_intervals(vocab):
    """The children of the root and of one frontier node against the float64 inverse CDF of the library's own drafter logits
    (float32 prefix sums of up to 262401 masses: within 3e-5 of the interval, the bound of the full-vocabulary test), and a whole
    round of drafting, rejection walk and commit."""
    print(f"draws from {vocab} ids", flush=True)
    pair = Pair("c0_tiny_f32", vocab=vocab, d_model=64, n_q_heads=1, n_kv_heads=1, d_ffn=64, n_layers=1, n_specialists=1,
                positions_per_specialist=6)
    cfg, ctx, k = pair.cfg, pair.ctx, pair.cfg.top_k
    ctx.prefill(make_prompt(cfg, n=12))
    ctx.set_sampling(0.8, np.zeros(cfg.depth + 1, np.float32))
    for seed in range(3):
        rng = np.random.default_rng(seed)
        UD = (rng.random((cfg.depth, k, k)) * 0.999).astype(np.float32)
        UD[0, 0, 0], UD[0, 0, 1] = (0.0, 0.9999999) if seed == 0 else UD[0, 0, :2]       # the first and the last id with mass
        ctx.set_draft_sampling(UD, (rng.random((cfg.depth + 1, k + 1)) * 0.999).astype(np.float32))
        d = ctx.draft_tree().as_dict()
        root = [i for i in range(1, d["n"]) if d["parent"][i] == 0]
        q = softmax_t(ctx.debug_draft_logits(0, 1)[0].cpu().numpy().astype(np.float64), 0.8)
        left = q.copy()
        for j, node in enumerate(root):
            c = d["token"][node]
            cdf = np.cumsum(left) / left.sum()
            lo, hi = (cdf[c - 1] if c else 0.0), cdf[c]
            assert 0 <= c < vocab and lo - 3e-5 <= float(UD[0, 0, j]) < hi + 3e-5, (seed, j, c, lo, hi)
            assert abs(d["score"][node] - np.log(q[c])) <= 1e-4
            left[c] = 0.0
        assert len({d["token"][i] for i in root}) == len(root) == k
        ctx.verify_tree()
        path, m, toks = ctx.accept_and_commit()
        assert len(toks) == m + 1 and all(0 <= t < vocab for t in toks)
    pair.close()


# keys per split -> splits of the prefix and the tree's rows: 2, 4 (registers), 7, 12 (registers), 13 and 16 (the loop)
@pytest.mark.parametrize("name", ["t_mid_bf16", "t_mid_f16"])
@pytest.mark.parametrize("n_prompt,keys", [(60, 64), (240, 64), (430, 64), (750, 64), (800, 64), (1000, 64)])
def test_attention_merged_from_any_number_of_splits(name, n_prompt, keys):
    print(f"merge {name} prompt={n_prompt} keys per split={keys}", flush=True)
    pair = Pair(name, n_layers=1, max_seq=1152, n_specialists=1)
    cfg = pair.cfg
    prompt = make_prompt(cfg, n=n_prompt)
    o = pair.oracle()
    o.prefill(prompt)
    pair.ctx.prefill(prompt)
    pair.ctx.set_tuning(0, keys)
    tree = ([pair.ctx.tokens()[-1], 5, 6, 7, 8], [-1, 0, 0, 1, 3])
    logits = torch.zeros(5, cfg.vocab, device="cuda")
    pair.ctx.verify_tree(P.TreeArrays.from_lists(*tree), logits_out=logits)
    o.tokens[-1] = tree[0][0]                              # (a near-tie may choose either first token)
    _, want, _ = o.verify_tree(Tree(*tree))
    assert np.abs(logits.cpu().numpy() - want).max() <= tol_for(cfg)
    pair.close()


@pytest.mark.parametrize("name,over", [("t_mid_f16", dict(vocab=5003)), ("t_mid_bf16", dict(vocab=4097)), ("c0_tiny_f32", dict(vocab=1001))])
def test_outputs_end_where_the_callers_arrays_end(name, over):
    """Logits and features written by the kernels themselves: an odd vocabulary, rows that are not whole tiles, a feature array
    that is not aligned to 16 bytes; what lies around the arrays is untouched and both alignments give the same bits."""
    print(f"outputs {name} {over}", flush=True)
    pair = Pair(name, **over)
    cfg, ctx = pair.cfg, pair.ctx
    ctx.prefill(make_prompt(cfg, n=40))
    tree = P.TreeArrays.from_lists([0, 5, 6, 7, 8], [-1, 0, 0, 1, 3])
    got = []
    for shift in (0, 1):
        lo = torch.full((2 * cfg.vocab + 5 * cfg.vocab,), -7.0, device="cuda")
        fe = torch.full((8 + 7 * cfg.d_model,), -7.0, device="cuda")
        lv, fv = lo[cfg.vocab:6 * cfg.vocab], fe[4 + shift:4 + shift + 5 * cfg.d_model]
        g = ctx.verify_tree(tree, logits_out=lv, feat_out=fv)[:5]
        torch.cuda.synchronize()
        assert (lo[:cfg.vocab] == -7).all() and (lo[6 * cfg.vocab:] == -7).all()
        assert (fe[:4 + shift] == -7).all() and (fe[4 + shift + 5 * cfg.d_model:] == -7).all()
        assert g.tolist() == lv.view(5, cfg.vocab).argmax(1).tolist()
        got.append((lv.clone(), fv.clone()))
        ctx.accept_and_commit()
        if shift == 0:                                     # the same state again
            ctx.reset()
            ctx.prefill(make_prompt(cfg, n=40))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    pair.close()


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("N,K", [(2944, 4096), (3072, 4096), (130, 24584)])
def test_many_rows_are_the_streaming_kernels_whatever_the_matrix_size(dtype, N, K):
    """More than 128 rows in a launch, matrices just below and at 24 MiB (how their weights are fetched changes there) and a thin
    one: a row's sums are those of a launch with fewer rows, bit for bit, and the float64 product's (float32 sums)."""
    print(f"many rows dtype={dtype} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + K)
    dt = torch.bfloat16 if dtype == 1 else torch.float16
    x = torch.empty(200, K, device="cuda").normal_(generator=g).to(dt)
    w = torch.empty(N, K, device="cuda").normal_(0.0, 0.02, generator=g).to(dt)
    y, _ = P.debug_gemm(dtype, x, w)
    for r0 in (0, 100):
        few, _ = P.debug_gemm(dtype, x[r0:r0 + 100].contiguous(), w)
        assert torch.equal(y[r0:r0 + 100], few)
    err = float((y.double() - x.double() @ w.double().T).abs().max())
    assert err < 2e-5 * np.sqrt(max(K, 256) / 256.0), err


@pytest.mark.parametrize("name", ["t_mid_bf16", "t_mid_f16"])
def test_keys_do_not_hang_on_how_many_rows_share_the_projection(name):
    """d_model 2048: up to 64 rows take the QKV kernel with the rotary embedding inside, more take the streaming kernel and its
    epilogue.  The first 30 tokens' keys and values of the first layer are the same bits either way (31 thousand keys a prompt: a
    rotation that one of them rounds once and the other twice, in fp16, shows in a few of them)."""
    pair = Pair(name, n_layers=1, d_model=2048, n_q_heads=8, n_kv_heads=8, head_dim=128, d_ffn=256, vocab=1000, n_specialists=1,
                positions_per_specialist=6)
    for seed in range(4):
        prompt = np.random.default_rng(seed).integers(0, pair.cfg.vocab, 90).astype(np.int32)
        got = []
        for n in (30, 60, 90):
            pair.ctx.reset()
            pair.ctx.prefill(prompt[:n])
            got.append(pair.ctx.debug_read_kv(-1, 0, 0, 30))
        for other in got[1:]:
            assert np.array_equal(got[0][0], other[0]) and np.array_equal(got[0][1], other[1]), seed
    pair.close()


# K splits of the QKV projection: one (512, 640 - a last chunk that is half padding), two (1024; 1192 - uneven, K ends inside a k-step),
# three (1536), four (2048; 1800); both head widths
@pytest.mark.parametrize("name,d_model,head_dim", [("t_mid_bf16", 512, 64), ("t_mid_f16", 640, 128), ("t_mid_bf16", 1024, 128),
                                                   ("t_mid_f16", 1192, 64), ("t_mid_bf16", 1536, 64), ("t_mid_f16", 2048, 64),
                                                   ("t_mid_bf16", 1800, 128)])
def test_projection_with_its_epilogue_inside_gives_the_streaming_kernels_bits(name, d_model, head_dim):
    """Keys and values of a prompt's first rows: up to 64 rows in a launch by the one-kernel form (row tiles of 16, 32 and 64 rows),
    120 rows by the streaming kernel and its epilogue; the same bits."""
    print(f"qkv {name} d_model={d_model} head_dim={head_dim}", flush=True)
    pair = Pair(name, n_layers=1, d_model=d_model, n_q_heads=4, n_kv_heads=2, head_dim=head_dim, d_ffn=256, vocab=300, n_specialists=1,
                positions_per_specialist=6)
    prompt = np.random.default_rng(d_model).integers(0, pair.cfg.vocab, 120).astype(np.int32)
    pair.ctx.prefill(prompt)
    want_k, want_v = pair.ctx.debug_read_kv(-1, 0, 0, 64)
    assert np.abs(want_k).max() > 0 and np.abs(want_v).max() > 0
    for n in (1, 15, 16, 17, 31, 32, 33, 47, 49, 63, 64):
        pair.ctx.reset()
        pair.ctx.prefill(prompt[:n])
        k, v = pair.ctx.debug_read_kv(-1, 0, 0, n)
        assert np.array_equal(k, want_k[:n]) and np.array_equal(v, want_v[:n]), n
    pair.close()


# equal numbers land in one block until its ids are gone; sharp distributions move every later target to a block that was not fetched ahead;
# the last two: one id holds nearly all the mass, and two blocks per share of the scan
@pytest.mark.parametrize("vocab,temperature,number", [(4100, 0.8, 0.5), (4100, 0.05, None), (70001, 0.1, 0.3), (128256, 0.02, None), (262401, 0.1, None)])
def test_draws_from_blocks_that_were_not_expected(vocab, temperature, number):
    """Children of the root against the float64 inverse CDF of what the earlier draws left (3e-5 of the interval, as above)."""
    print(f"draws from {vocab} ids at {temperature}", flush=True)
    pair = Pair("c0_tiny_f32", vocab=vocab, d_model=64, n_q_heads=1, n_kv_heads=1, d_ffn=64, n_layers=1, n_specialists=1,
                positions_per_specialist=1, depth=1, top_k=7, total_tokens=7)       # (every child is in the tree, in the order of the draws)
    cfg, ctx, k = pair.cfg, pair.ctx, pair.cfg.top_k
    ctx.prefill(make_prompt(cfg, n=12))
    ctx.set_sampling(temperature, np.zeros(cfg.depth + 1, np.float32))
    for seed in range(4):
        rng = np.random.default_rng(seed)
        UD = (rng.random((cfg.depth, k, k)) * 0.999).astype(np.float32)
        if number is not None:
            UD[:] = number
        ctx.set_draft_sampling(UD, (rng.random((cfg.depth + 1, k + 1)) * 0.999).astype(np.float32))
        d = ctx.draft_tree().as_dict()
        root = [i for i in range(1, d["n"]) if d["parent"][i] == 0]
        left = softmax_t(ctx.debug_draft_logits(0, 1)[0].cpu().numpy().astype(np.float64), temperature)
        for j, node in enumerate(root):
            c = d["token"][node]
            if left.sum() < 1e-6:                          # what is left is the rounding of a float32 sum
                break
            cdf = np.cumsum(left) / left.sum()
            lo, hi = (cdf[c - 1] if c else 0.0), cdf[c]
            assert lo - 3e-5 <= float(UD[0, 0, j]) < hi + 3e-5, (seed, j, c, lo, hi)
            left[c] = 0.0
        assert len(root) == k
    pair.close()


# 48 and 96 MiB of activation reads with one and two row tiles, the streaming kernel from 33 rows on; 320 column tiles on 256 CUs: always
@pytest.mark.parametrize("d_model,heads,rows", [(6144, (48, 8), (16, 17, 32, 33)), (2048, (48, 16), (1, 16, 33))])
def test_projections_at_the_line_between_the_two_kernels(d_model, heads, rows):
    """Keys and values of a prompt's first rows: the same bits on either side of where the one-kernel form stops."""
    print(f"qkv line d_model={d_model} heads={heads}", flush=True)
    pair = Pair("t_mid_bf16", n_layers=1, d_model=d_model, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=128, d_ffn=64, vocab=300,
                n_specialists=1, positions_per_specialist=6)
    prompt = np.random.default_rng(d_model).integers(0, pair.cfg.vocab, 120).astype(np.int32)
    pair.ctx.prefill(prompt)
    want_k, want_v = pair.ctx.debug_read_kv(-1, 0, 0, 64)
    assert np.abs(want_k).max() > 0 and np.abs(want_v).max() > 0
    for n in rows:
        pair.ctx.reset()
        pair.ctx.prefill(prompt[:n])
        k, v = pair.ctx.debug_read_kv(-1, 0, 0, n)
        assert np.array_equal(k, want_k[:n]) and np.array_equal(v, want_v[:n]), n
    pair.close()


@pytest.mark.parametrize("name,over", [
    ("t_mid_bf16", dict()),                                                                   # one K split of QKV
    ("t_mid_f16", dict()),                                                                    # K padded to whole chunks
    ("t_mid_bf16", dict(d_model=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, d_ffn=1000)),  # two splits, units that end inside a tile
    ("t_mid_f16", dict(d_model=1536, n_q_heads=12, n_kv_heads=4, d_ffn=1544)),                # three: the norm stays a kernel
    ("t_mid_bf16", dict(d_model=2048, n_q_heads=16, n_kv_heads=2, head_dim=128)),             # four, a wave each
    ("t_mid_f16", dict(d_model=4224, n_q_heads=4, n_kv_heads=1, d_ffn=4000)),                 # a second turn of the norm's groups, in gate/up alone (six)
])
def test_one_row_has_the_bits_of_a_tree_row(name, over):
    """A pass of one row forms its norms and merges its attention splits inside the products; a row of a wider tree (17 rows and more:
    neither) goes through kernels of their own.  Same logits and features, bit for bit, from one attention split to more than the
    merge inside takes; 2 and 16 rows (merge inside, norms not) as well."""
    over = dict(over, n_layers=2, vocab=1000, max_seq=4096, n_specialists=1)
    pair = Pair(name, **over)
    one_row_against_tree_rows(pair.cfg, pair.ctx, (20, 300, 600, 1300, 2500))
    pair.close()


# gemm_row_qkv_kernel<T, NP, NSL, NTW>: planes read at once, slots a wave forms, column tiles of a wave (2: four QKV splits, 1: fewer); its
# planes are the down projection's.  gemm_row_silu_kernel<T, NP, NSL>: its planes are the output projection's.
@pytest.mark.parametrize("name,over", [
    ("t_mid_f16", dict(d_model=2048, n_q_heads=16, n_kv_heads=2, head_dim=128, d_ffn=1024)),    # qkv <2, 4, 2> (2 planes), silu <4, 2> (4)
    ("t_mid_bf16", dict(d_ffn=4096)),                                                           # qkv <8, 4, 1> (8 planes), silu <2, 2> (1)
    ("t_mid_bf16", dict(d_model=4096, n_q_heads=32, n_kv_heads=8, head_dim=128, d_ffn=4096)),   # qkv <8, 4, 2>, silu <8, 2> (8 planes each): the 8B shape
    ("t_mid_f16", dict(d_model=5120, n_q_heads=40, n_kv_heads=40, head_dim=128, d_ffn=4096)),   # qkv <6, 5, 1> (6), silu <6, 3> (5): the 13B shape
    ("t_mid_bf16", dict(d_model=5120, n_q_heads=40, n_kv_heads=8, head_dim=128, d_ffn=4096)),   # qkv <6, 5, 2>, the same with grouped heads
    ("t_mid_f16", dict(d_model=5120, n_q_heads=40, n_kv_heads=40, head_dim=128, d_ffn=2048)),   # qkv <4, 5, 1> (4)
    ("t_mid_bf16", dict(d_model=4616, n_q_heads=40, n_kv_heads=8, head_dim=128, d_ffn=2048)),   # qkv <4, 5, 2>; a second turn of 130 groups, K padded
])
def test_one_row_at_every_number_of_planes_and_turns(name, over):
    """The same at plane counts, widths and QKV splits that lead to the other instantiations of the two kernels."""
    cfg = get_config(name, **dict(over, n_layers=2, vocab=1000, max_seq=2048, n_specialists=1))
    ctx = P.Poss(cfg, make_weights_on_device(cfg))
    one_row_against_tree_rows(cfg, ctx, (20, 1300))
    ctx.close()


def one_row_against_tree_rows(cfg, ctx, prompts):
    rs = np.random.RandomState(5)
    wide = [0] + [int(x) for x in rs.permutation(1000)[:16]]
    for n_prompt in prompts:
        prompt, got = rs.randint(0, 1000, n_prompt).astype(np.int32), []
        for rows in (17, 1, 2, 16):
            ctx.reset()
            ctx.prefill(prompt)
            logits, feats = torch.zeros(rows, 1000, device="cuda"), torch.zeros(rows, cfg.d_model, device="cuda")
            ctx.verify_tree(P.TreeArrays.from_lists(wide[:rows], [-1] + [0] * (rows - 1)), logits_out=logits, feat_out=feats)
            got.append((logits, feats))
        torch.cuda.synchronize()
        for logits, feats in got[1:]:
            n = logits.shape[0]
            assert torch.equal(logits, got[0][0][:n]) and torch.equal(feats, got[0][1][:n]), (n_prompt, n)
        assert torch.isfinite(got[0][0]).all()


@pytest.mark.parametrize("name,n_prompt", [("t_mid_bf16", 257), ("t_mid_f16", 257), ("t_mid_bf16", 1), ("t_mid_f16", 1)])
def test_prompt_whose_last_launch_is_one_row(name, n_prompt):
    """A streamed prompt's launches of 256 tokens can leave one row (a prompt of one token is one), whose norms are formed inside the products
    like a decoded row's.  Its keys and values in every layer are, bit for bit, those of a prompt of nine tokens more, where it shares a launch
    and the norms are kernels; its greedy token is the oracle's where two tolerances part the two best logits; the row behind it, which
    attends to it, has the oracle's logits and features (the storage type's tolerance)."""
    pair = Pair(name)
    ctx, o, layers = pair.ctx, pair.oracle(), range(pair.cfg.n_layers)
    longer = make_prompt(pair.cfg, n=n_prompt + 9)
    prompt = longer[:n_prompt]
    ctx.prefill(longer)
    shared = [ctx.debug_read_kv(-1, layer, 0, n_prompt) for layer in layers]
    ctx.reset()
    first = ctx.prefill(prompt)
    for layer, (k, v) in zip(layers, shared):
        alone_k, alone_v = ctx.debug_read_kv(-1, layer, 0, n_prompt)
        assert np.abs(k[-1]).max() > 0 and np.array_equal(alone_k, k) and np.array_equal(alone_v, v), layer
    assert o.prefill(prompt) == first or o.margins[-1] <= 2 * tol_for(pair.cfg)
    o.tokens[-1] = first
    logits, feats = torch.zeros(1, pair.cfg.vocab, device="cuda"), torch.zeros(1, pair.cfg.d_model, device="cuda")
    ctx.verify_tree(P.TreeArrays.from_lists([int(o.tokens[-1])], [-1]), logits_out=logits, feat_out=feats)
    _, want, want_f = o.verify_tree(Tree([int(o.tokens[-1])], [-1]))
    tol = tol_for(pair.cfg)
    assert np.abs(logits.cpu().numpy() - want).max() < tol
    assert np.abs(feats.cpu().numpy() - want_f).max() < tol * np.abs(want_f).max()
    pair.close()


@pytest.mark.parametrize("vocab,rows,shift", [(1000, 17, 0), (1001, 5, 0), (131, 40, 0), (1000, 9, 1), (8192, 1, 0)])
def test_logits_of_a_head_tile_in_the_callers_array(vocab, rows, shift):
    """Verified rows' logits leave the Head's tiles in pieces of four: vocabularies that are and are not multiples of 4 and end inside a
    tile, an array that is not aligned to 16 bytes.  The greedy choice is their argmax; nothing beyond the array's rows is written; the
    values are the oracle's within the storage type's tolerance."""
    pair = Pair("t_mid_bf16", vocab=vocab)
    ctx, o = pair.ctx, pair.oracle()
    prompt = make_prompt(pair.cfg, n=20)
    ctx.prefill(prompt)
    o.prefill(prompt)
    o.tokens[-1] = ctx.tokens()[-1]
    token, parent = [int(o.tokens[-1])] + list(range(1, rows)), [-1] + [0] * (rows - 1)
    buf = torch.full((rows * vocab + 8,), -7.0, device="cuda")
    logits = buf[shift:shift + rows * vocab].view(rows, vocab)
    g = ctx.verify_tree(P.TreeArrays.from_lists(token, parent), logits_out=logits)[:rows]
    assert g.tolist() == logits.argmax(1).tolist()
    assert (buf[:shift] == -7.0).all() and (buf[shift + rows * vocab:] == -7.0).all()
    _, want, _ = o.verify_tree(Tree(token, parent))
    assert np.abs(logits.cpu().numpy() - want).max() < tol_for(pair.cfg)
    pair.close()
