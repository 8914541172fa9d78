#!/usr/bin/env python3
"""Benchmark of the PosS draft-and-verify round on one MI355X.

A "step" is one round: poss_draft_tree -> poss_verify_tree -> poss_accept_and_commit through the
C ABI, on a synthetic random-init model of Llama-3-8B shape (3 specialists x 2 positions, tree
width 10, depth 6, 60 draft tokens, 512-token uniform-random prompt), everything resident in HBM.
Prints one JSON line.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "draft+verify round latency (ms), tokens/s and HBM GB/s, Llama-3-8B shape, bs=1"
HBM_PEAK_GBPS = 8000.0
# Table 1 of the paper, T=0, average over its six suites, drafter with 3 specialists x 2 positions
# (the paper's "PosS-2"; 13B: depth 7 in the paper, 6 here) and one specialist per position ("PosS-1")
PAPER_TAU = {"c1_llama3_8b_3x2": 4.55, "c2_llama3_8b_6x1": 4.54, "c3_llama2_13b_3x2": 5.36}
# HBM bytes per gemm_stream_kernel launch (average over the launches of a round) from rocprofv3 TCC
# counters, scaled by the reading of a plain 1 GiB copy (FETCH_SIZE x2.000, WRITE_SIZE x1.000);
# commands and raw sums: profiles/gemm_stream_kernel_c1_hbm_traffic.md.  The figures belong to one state of
# the sources that decide what the counted launches read and which launches there are - the products, the attention splits that
# some of them merge, the choice among them: they are quoted only while these still hash to the value recorded with them.
TRAFFIC_SOURCES = ("gemm.hip", "attn_merge.h", "attn_split.h", "attention.hip", "api.hip", "common.h", "device_utils.h")
MEASURED_TRAFFIC = {"c1_llama3_8b_3x2": dict(fetch_bytes=153.1e6, write_bytes=5.08e6,
                                             sources_sha256="92c2d862511fb1b8fa699347a4177b6b0865b79657bda854d8686993c5abf5ab")}


def traffic_source_hash(csrc=os.path.join(ROOT, "paper_2506_03566_amd", "csrc")):
    import hashlib
    h = hashlib.sha256()
    for name in TRAFFIC_SOURCES:
        with open(os.path.join(csrc, name), "rb") as f:
            h.update(name.encode() + b"\0" + hashlib.sha256(f.read()).digest())
    return h.hexdigest()


def measured_traffic(cfg_name):
    """(bytes per launch, None) if the recorded counters were taken on this build of the kernel, else (None, why)."""
    m = MEASURED_TRAFFIC.get(cfg_name)
    if not m:
        return None, "no counter run recorded for this workload"
    if m["sources_sha256"] != traffic_source_hash():
        return None, "counter run predates the current sources of the counted launches (recorded for %s...)" % m["sources_sha256"][:12]
    return m["fetch_bytes"] + m["write_bytes"], None


def round_bytes(cfg, t, a):
    """Algorithmic HBM bytes of one round: every weight of every GEMM once, plus the KV read."""
    es = 4 if cfg.dtype == 0 else 2
    d, qd, kd, F, V = cfg.d_model, cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim, cfg.d_ffn, cfg.vocab
    layer = (qd + 2 * kd) * d + d * qd + 2 * F * d + d * F + 2 * d
    head = V * d + d
    target = cfg.n_layers * layer + head
    draft = cfg.depth * (2 * d * d + d + layer + head)
    kv_target = cfg.n_layers * t * 2 * kd
    kv_draft = cfg.depth * t * 2 * kd
    return es * (target + draft + kv_target + kv_draft)


def cpu_baseline(cfg, n_layers_sample=16):
    """The CPU oracle timed on a bounded sample of the same round and scaled to a whole round:
    n_layers_sample of the target's layers and its Head over the tree rows at t = n_prompt, and one
    pass of every specialist with its Head over top_k rows."""
    import numpy as np
    from synth import make_weights
    from oracle.model import Weights, decoder_layer, head, specialist_pass
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] + [1])
    except Exception:
        cores = os.cpu_count() or 1
    act = None if cfg.dtype == 0 else cfg.dtype
    n_layers_sample = min(n_layers_sample, cfg.n_layers)
    names = ["layer%d." % l for l in range(n_layers_sample)] + ["lm_head", "final_norm", "embed"] + \
            ["spec%d." % s for s in range(cfg.n_specialists)]
    W = Weights(cfg, make_weights(cfg, names=names), cache=False)
    rng = np.random.default_rng(0)
    t, M, k = cfg.n_prompt, cfg.total_tokens + 1, cfg.top_k
    h = rng.normal(size=(M, cfg.d_model))
    kc = rng.normal(size=(t, cfg.n_kv_heads, cfg.head_dim))
    vc = rng.normal(size=(t, cfg.n_kv_heads, cfg.head_dim))
    allowed = np.ones((M, t + M), dtype=bool)
    allowed[:, t:] = np.tril(np.ones((M, M), dtype=bool))
    t0 = time.perf_counter()
    f = h
    for l in range(n_layers_sample):
        f, _, _ = decoder_layer(W, "layer%d." % l, cfg, f, np.arange(t, t + M), kc, vc, allowed, act)
    t_layers = time.perf_counter() - t0
    t0 = time.perf_counter()
    head(W, cfg, f, act)
    t_head_v = time.perf_counter() - t0
    n_seq = t + k
    toks = rng.integers(0, cfg.vocab, size=n_seq)
    feats = rng.normal(size=(n_seq, cfg.d_model))
    al = np.ones((k, n_seq), dtype=bool)
    t0 = time.perf_counter()
    for s in range(cfg.n_specialists):
        out = specialist_pass(W, cfg, s, toks, feats, np.arange(n_seq), al, list(range(t, n_seq)), act)
        head(W, cfg, out, act)
    t_spec = (time.perf_counter() - t0) / cfg.n_specialists
    round_s = cfg.n_layers * t_layers / n_layers_sample + t_head_v + cfg.depth * t_spec
    measured = t_layers + t_head_v + t_spec * cfg.n_specialists
    # the same oracle on ONE thread, on a smaller sample (one target layer, one specialist pass, both Heads)
    one = None
    try:
        from threadpoolctl import threadpool_limits
        with threadpool_limits(limits=1):
            t0 = time.perf_counter()
            f1, _, _ = decoder_layer(W, "layer0.", cfg, h, np.arange(t, t + M), kc, vc, allowed, act)
            t1_layer = time.perf_counter() - t0
            t0 = time.perf_counter()
            head(W, cfg, f1, act)
            t1_head_v = time.perf_counter() - t0
            t0 = time.perf_counter()
            out1 = specialist_pass(W, cfg, 0, toks, feats, np.arange(n_seq), al, list(range(t, n_seq)), act)
            head(W, cfg, out1, act)
            t1_spec = time.perf_counter() - t0
        r1 = cfg.n_layers * t1_layer + t1_head_v + cfg.depth * t1_spec
        one = dict(value=1.0 / r1, unit="tokens/s", cores=1, ms_per_round=r1 * 1e3,
                   sample="one target layer, the verification Head and one specialist pass + Head on one thread, "
                          "%.1f s measured, scaled to a round" % (t1_layer + t1_head_v + t1_spec))
    except Exception as exc:                              # threadpoolctl missing: the figure is left out, not guessed
        one = dict(error=str(exc))
    return dict(value=1.0 / round_s, unit="tokens/s", cores=int(cores), kind="oracle", one_thread=one,
                sample=("oracle timed on %d of %d target layers + Head over %d tree rows at t=%d, and one pass + "
                        "Head of each of the %d specialists over %d rows; scaled to a full round (%d layers, %d "
                        "draft passes) at 1 committed token per round; %.1f s measured, %.1f s per round extrapolated"
                        % (n_layers_sample, cfg.n_layers, M, t, cfg.n_specialists, k, cfg.n_layers, cfg.depth,
                           measured, round_s)),
                ms_per_round=round_s * 1e3)


def quick_measure(name, steps=10, warmup=3, vanilla_steps=10, batch=1):
    """Round latency, achieved fraction of the HBM peak and the plain-decoding step of another workload of
    the benchmark spec (same library, same timing rules as the headline: inputs resident, synchronised on both sides).
    batch > 1: that many sequences per round (other prompts of the same length), tokens/s over all of them; the
    bytes of the fraction are one round's weights, streamed once for all sequences."""
    import torch
    import paper_2506_03566_amd as P
    from synth import get_config, make_prompt
    from synth.gpu import make_weights_on_device
    cfg = get_config(name)
    weights = make_weights_on_device(cfg)
    ctx = P.Poss(cfg, weights, batch=batch)
    del weights
    torch.cuda.empty_cache()
    prompt = make_prompt(cfg)
    ctx.prefill(prompt)
    for b in range(1, batch):
        ctx.prefill(make_prompt(cfg.with_(prompt_seed=cfg.prompt_seed + 17 * b)), seq=b)

    def one_round():
        ctx.draft_tree(want_tree=False)
        ctx.verify_tree(None, want_argmax=False)
        return ctx.accept_and_commit()

    for _ in range(warmup):
        one_round()
    s0 = ctx.stats()
    t_begin = len(ctx.tokens()) - 1
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        one_round()
    torch.cuda.synchronize()
    ms_round = (time.perf_counter() - t0) * 1e3 / steps
    s1 = ctx.stats()
    committed = s1.committed_tokens - s0.committed_tokens
    t_mid = t_begin + committed // (2 * batch)
    bytes_round = round_bytes(cfg, t_mid, 1) + (batch - 1) * (round_bytes(cfg, t_mid, 1) - round_bytes(cfg, 0, 1))   # weights once, KV per sequence
    gbps = bytes_round / (ms_round * 1e-3) / 1e9
    out = dict(ms_per_round=round(ms_round, 4), hbm_frac=round(gbps / HBM_PEAK_GBPS, 4),
               draft_ms=round((s1.ms_draft - s0.ms_draft) / steps, 4), verify_ms=round((s1.ms_verify - s0.ms_verify) / steps, 4),
               tokens_per_s=round(committed / (ms_round * 1e-3 * steps), 2), steps=steps, n_prompt=cfg.n_prompt,
               depth=cfg.depth, total_tokens=cfg.total_tokens, dtype={0: "f32", 1: "bf16", 2: "f16"}[cfg.dtype])
    if batch > 1:
        out["batch"] = batch
    if vanilla_steps > 0 and batch == 1:
        ctx.reset()
        ctx.prefill(prompt)
        root = P.TreeArrays.from_lists([0], [-1])
        for _ in range(2):
            ctx.verify_tree(root, want_argmax=False)
            ctx.accept_and_commit()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(vanilla_steps):
            ctx.verify_tree(root, want_argmax=False)
            ctx.accept_and_commit()
        torch.cuda.synchronize()
        out["vanilla_ms"] = round((time.perf_counter() - t0) * 1e3 / vanilla_steps, 4)
    ctx.close()
    del ctx
    torch.cuda.empty_cache()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", default="c1_llama3_8b_3x2")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--gemm-wgs", type=int, default=0)
    ap.add_argument("--attn-split", type=int, default=0)
    ap.add_argument("--vanilla-steps", type=int, default=20,
                    help="tokens of plain autoregressive decoding (root-only rounds) timed after the main "
                         "measurement; 0 skips that leg")
    ap.add_argument("--depth", type=int, default=0, help="override the drafting depth L (sweeps)")
    ap.add_argument("--total-tokens", type=int, default=0, help="override the number of draft tokens N (sweeps)")
    ap.add_argument("--specialists", type=int, default=0, help="override the number of specialists S (sweeps)")
    ap.add_argument("--positions", type=int, default=0, help="override positions per specialist n (sweeps)")
    ap.add_argument("--batch", type=int, default=1,
                    help="sequences per round, up to 8 (the headline metric is quoted at 1); rows of the sequences share the weight "
                         "streams, 256 rows per launch (beyond that the passes run group by group)")
    ap.add_argument("--temperature", type=float, default=0.0,
                    help="> 0: verification draws the target's tokens at this temperature (sampler kernels "
                         "instead of argmax); the headline metric is quoted at 0")
    ap.add_argument("--drawn-children", action="store_true",
                    help="with --temperature: children drawn from the drafter's distribution and verified by the rejection "
                         "rule (poss_set_draft_sampling) instead of the deterministic tree")
    ap.add_argument("--no-other-configs", action="store_true",
                    help="skip the short measurements of the other workloads (6 specialists x 1, 13B fp16, 8192-token context) "
                         "that the default run appends as other_configs")
    ap.add_argument("--pmc-calibration", action="store_true",
                    help="also run a plain 1 GiB device copy, to scale rocprofv3 FETCH_SIZE / WRITE_SIZE readings")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (no sharding, no collectives); --gpus %d is not supported"
              % args.gpus, file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2506_03566_amd as P
    from synth import get_config, make_prompt
    from synth.gpu import make_weights_on_device

    over = {}
    if args.depth: over["depth"] = args.depth
    if args.total_tokens: over["total_tokens"] = args.total_tokens
    if args.specialists: over["n_specialists"] = args.specialists
    if args.positions: over["positions_per_specialist"] = args.positions
    cfg = get_config(args.config, **over)
    P.load_library()                                  # fail loudly if the HIP library is missing
    t0 = time.perf_counter()
    weights = make_weights_on_device(cfg)
    t_gen = time.perf_counter() - t0
    B = max(1, args.batch)
    ctx = P.Poss(cfg, weights, batch=B)
    del weights
    torch.cuda.empty_cache()
    if args.gemm_wgs or args.attn_split:
        ctx.set_tuning(args.gemm_wgs, args.attn_split)
    prompt = make_prompt(cfg)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ctx.prefill(prompt)
    torch.cuda.synchronize()
    t_prefill = time.perf_counter() - t0
    for b in range(1, B):                             # further sequences: other prompts of the same length
        ctx.prefill(make_prompt(cfg.with_(prompt_seed=cfg.prompt_seed + 17 * b)), seq=b)

    import numpy as np
    u_rng = np.random.default_rng(0)

    def one_round():
        if args.temperature > 0:
            ctx.set_sampling(args.temperature, u_rng.random(cfg.depth + 1).astype(np.float32))
            if args.drawn_children:
                ctx.set_draft_sampling(u_rng.random((cfg.depth, cfg.top_k, cfg.top_k)).astype(np.float32),
                                       u_rng.random((cfg.depth + 1, cfg.top_k + 1)).astype(np.float32))
        ctx.draft_tree(want_tree=False)
        ctx.verify_tree(None, want_argmax=False)
        return ctx.accept_and_commit()

    for _ in range(args.warmup):
        one_round()
    s0 = ctx.stats()
    base = (s0.rounds, s0.committed_tokens, s0.ms_draft, s0.ms_verify, s0.ms_commit)
    t_begin = len(ctx.tokens()) - 1
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        one_round()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    s1 = ctx.stats()
    rounds = (s1.rounds - base[0]) // B               # the statistics count one round per sequence and call
    committed = s1.committed_tokens - base[1]
    ms_round = wall * 1e3 / rounds
    t_mid = t_begin + committed // (2 * B)
    bytes_round = round_bytes(cfg, t_mid, 1) + (B - 1) * (round_bytes(cfg, t_mid, 1) - round_bytes(cfg, 0, 1))   # weights once, KV per sequence
    gbps = bytes_round / (ms_round * 1e-3) / 1e9

    # dominant kernel: the weight-streaming GEMM, timed per launch with HIP events on the library's stream
    ctx.profile_gemm(True)
    prof_rounds = min(3, args.steps)
    for _ in range(prof_rounds):
        one_round()
    launches, gemm_ms, gemm_bytes = ctx.gemm_profile()
    ctx.profile_gemm(False)
    achieved = gemm_bytes / (gemm_ms * 1e-3) / 1e9 if gemm_ms > 0 else 0.0
    roofline = dict(bound="hbm", kernel="gemm_stream_kernel", achieved=round(achieved, 1), peak=HBM_PEAK_GBPS,
                    unit="GB/s", frac=round(achieved / HBM_PEAK_GBPS, 4),
                    traffic=(measured_traffic(cfg.name)[0] if not over and B == 1 else None),
                    algorithmic_bytes_per_launch=round(gemm_bytes / max(launches, 1), 1),
                    launches_per_round=launches // max(prof_rounds, 1),
                    avg_launch_us=round(gemm_ms * 1e3 / max(launches, 1), 2),
                    weight_bytes_per_round=gemm_bytes / max(prof_rounds, 1))
    if roofline["traffic"] is None and not over and B == 1:
        roofline["traffic_note"] = measured_traffic(cfg.name)[1]

    out = dict(metric=METRIC, value=round(committed / wall, 2), unit="tokens/s", n_gpus=1, steps=rounds,
               warmup=args.warmup, ms_per_step=round(ms_round, 4), higher_is_better=True, scaling="weak",
               vs_baseline=None, dtype={0: "f32", 1: "bf16", 2: "f16"}[cfg.dtype], data="synthetic",
               config=dict(workload=cfg.name, target_layers=cfg.n_layers, d_model=cfg.d_model, vocab=cfg.vocab,
                           specialists=cfg.n_specialists, positions_per_specialist=cfg.positions_per_specialist,
                           top_k=cfg.top_k, depth=cfg.depth, total_tokens=cfg.total_tokens,
                           n_prompt=cfg.n_prompt, batch=B, t_at_timing=t_mid),
               round_latency_ms=round(ms_round, 4), hbm_gbps=round(gbps, 1), hbm_frac=round(gbps / HBM_PEAK_GBPS, 4),
               bytes_per_round=bytes_round, tau_gen=round(committed / (rounds * B), 3),
               phase_ms=dict(draft=round((s1.ms_draft - base[2]) / rounds, 4),
                             verify=round((s1.ms_verify - base[3]) / rounds, 4),
                             commit=round((s1.ms_commit - base[4]) / rounds, 4)),
               setup_s=dict(weights=round(t_gen, 1), prefill=round(t_prefill, 3)), roofline=roofline)
    # Plain autoregressive decoding of the same target through the same library: rounds whose tree is the
    # root alone (one target pass over one row, one committed token).  The denominator of the paper's
    # speed-up ratio (Table 2); measured, while the ratio at the paper's tau stays a projection.
    if args.vanilla_steps > 0:
        ctx.reset()
        if args.temperature > 0:
            ctx.set_draft_sampling(None)
            ctx.set_sampling(0.0)
        ctx.prefill(prompt)
        for b in range(1, B):
            ctx.prefill(make_prompt(cfg.with_(prompt_seed=cfg.prompt_seed + 17 * b)), seq=b)
        root = [P.TreeArrays.from_lists([0], [-1]) for _ in range(B)]     # one step = one token for every sequence
        for _ in range(3):
            ctx.verify_tree(root, want_argmax=False)
            ctx.accept_and_commit()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.vanilla_steps):
            ctx.verify_tree(root, want_argmax=False)
            ctx.accept_and_commit()
        torch.cuda.synchronize()
        ar_ms = (time.perf_counter() - t0) * 1e3 / args.vanilla_steps
        out["vanilla_ar"] = dict(ms_per_token=round(ar_ms, 4), tokens_per_s=round(B * 1e3 / ar_ms, 1),
                                 round_over_vanilla=round(ms_round / ar_ms, 3),
                                 break_even_tau=round(ms_round / ar_ms, 3),
                                 note="root-only rounds; speculative decoding is faster once tokens per round exceed "
                                      "round_over_vanilla")
    if over:
        out["config"]["overrides"] = over
    if args.temperature > 0:
        out["config"]["temperature"] = args.temperature
        out["config"]["drawn_children"] = bool(args.drawn_children)
    if cfg.name in PAPER_TAU and not over:
        # NOT a measurement: random-init drafters accept nothing (tau_gen = 1), so this only restates the
        # measured round latency at the acceptance length the paper reports for trained drafters.
        out["projection"] = dict(tokens_per_s_at_paper_tau=round(B * PAPER_TAU[cfg.name] / (ms_round * 1e-3), 1),
                                 paper_tau=PAPER_TAU[cfg.name],
                                 note="projection, not measured: paper's Table 1 tau (trained drafter, six suites, "
                                      "A100; bonus-token convention not stated) x this build's round latency")
    if "vanilla_ar" in out and "projection" in out:
        out["projection"]["speedup_vs_vanilla_at_paper_tau"] = round(
            PAPER_TAU[cfg.name] * out["vanilla_ar"]["ms_per_token"] / ms_round, 2)
    ctx.close()
    del ctx
    torch.cuda.empty_cache()
    # the other workloads of the benchmark spec, each measured briefly by the same rules (the headline fields above are C1's)
    if (not args.no_other_configs and args.config == "c1_llama3_8b_3x2" and not over and B == 1 and args.temperature == 0
            and not args.gemm_wgs and not args.attn_split):
        out["other_configs"] = {n: quick_measure(n) for n in ("c2_llama3_8b_6x1", "c3_llama2_13b_3x2", "c4_llama3_8b_long")}
        # four sequences per round at the headline shape: 4 x 61 rows verified in one weight stream
        out["other_configs"]["c1_llama3_8b_3x2_batch4"] = quick_measure("c1_llama3_8b_3x2", batch=4)
    if args.pmc_calibration:
        src = torch.zeros(1 << 28, dtype=torch.float32, device="cuda")       # 1 GiB read + 1 GiB written
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
