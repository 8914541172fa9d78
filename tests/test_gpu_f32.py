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
    from synth import make_prompt
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
