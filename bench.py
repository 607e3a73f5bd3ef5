#!/usr/bin/env python3
"""Benchmark of the QuickPrefill hot path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config NAME] [--no-cpu-baseline] [--grid] ...

One step = one pass of the whole path (group attention + scoring + top-k/compaction for every group of every layer)
over the named synthetic workload, through qp_prefill_video of the C ABI, inputs already resident in HBM. Without
--config the headline is the largest config, cfg5_7b_hour_stack (28 layers, every layer's inputs and pruned cache
resident), and all five configs are measured. Prints ONE JSON line on stdout, short enough to be kept whole by whatever
keeps the end of a program's output, with the headline and, per config, its time, rate and attention fraction
(`configs`); everything below goes to stderr before it, one line per section, "[bench] detail <section> <JSON>":
  value         video tokens prefilled per second per layer over the K timed steps
  roofline      the group-attention kernel (dominant): useful flops of a launch / its average duration (HIP events
                around every qp_group_attend launch of a serial replay of layer 0, on the stream the kernels run on)
                against the bf16 MFMA peak; whole_step_frac = all layers' attention flops / ms_per_step; traffic =
                HBM bytes per launch from the rocprofv3 counter summary under profiles/
  stages        per-stage times of the replay, the HBM-side figures of the score / top-k+compact kernels at their
                real per-group shapes and at a bandwidth-characterisation shape, the stages that consume the cache
  cpu_baseline  the fp64 oracle timed on the host on a bounded sample of the same workload (projected layer time)
  near_tie      kept sets of the GPU against the oracle's: identical / excused near-ties / mismatches
  configs       per config: ms per step, tokens/s/layer, attention fraction of peak, score and top-k GB/s, near-tie
                counts, final cache length, resident cache bytes, and the oracle's projected rate
  table2_grid   the points of the paper's Table 2 ablation grid as throughput on config 2's video
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0       # MI355X HBM3E
PEAK_EXP_PER_S = 256 * 4 * 4 * 2.4e9   # v_exp_f32: a wavefront instruction takes 16 cycles on a 16-lane SIMD

CAL_COPY_BYTES = 256 << 20


def attend_flops(w, c, n_g):
    """Useful flops of one group-attention launch: QK^T and PV over visible (row, key) pairs only."""
    return 4.0 * w.head_dim * w.n_q_heads * (n_g * c + n_g * (n_g + 1) / 2.0)


def score_bytes(w, rule, n_g):
    esz = 4 if w.dtype == "f32" else 2
    b = w.n_kv_heads * n_g * w.head_dim * esz + w.n_kv_heads * n_g * 4
    if rule.startswith("window"):
        b += w.n_window * w.n_q_heads * w.head_dim * esz
    return b


def topk_bytes(w, n_g, keep):
    esz = 4 if w.dtype == "f32" else 2
    return w.n_kv_heads * (n_g * 4 + keep * 4 + 2 * 2 * keep * w.head_dim * esz)


def characterise_hbm(torch, B, reps=6):
    """HBM-bound steps at a bandwidth-characterisation shape: the layers of the hour-long stack folded into
    the head axis (28 x 4 = 112 KV heads x 8192 tokens x 128, bf16), inputs rotated over three buffers
    (3 x 235 MB > the 256 MB Infinity Cache) so that the bytes come from HBM."""
    h, n_g, d, keep = 112, 8192, 128, 820
    layout = B.make_layout(h, h, d, "bf16")
    ks = [torch.randn(n_g, h, d, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    vs = [torch.randn(n_g, h, d, device="cuda", dtype=torch.bfloat16) for _ in range(3)]
    scores = torch.empty(h, n_g, dtype=torch.float32, device="cuda")
    cache = B.Cache(layout, keep)
    kept = torch.empty(h, keep, dtype=torch.int32, device="cuda")
    out = {}
    ev = lambda: torch.cuda.Event(enable_timing=True)
    # key-norm scores: read K once, write H*N_g floats
    for i in range(3):
        B.score_kv(layout, "key_norm_small", ks[i], None, None, scores)
    torch.cuda.synchronize()
    e0, e1 = ev(), ev()
    e0.record()
    for i in range(reps):
        B.score_kv(layout, "key_norm_small", ks[i % 3], None, None, scores)
    e1.record()
    torch.cuda.synchronize()
    t = e0.elapsed_time(e1) * 1e-3 / reps
    nbytes = h * n_g * d * 2 + h * n_g * 4
    out["score_norm"] = {"shape": f"{h} heads x {n_g} tokens x {d} bf16", "bytes": nbytes, "us": t * 1e6,
                         "GBps": nbytes / t / 1e9, "frac_of_hbm_peak": nbytes / t / 1e9 / PEAK_HBM_GBS}
    # top-k + compaction: read the scores, gather keep rows of K and V, write them + pos
    for i in range(3):
        cache.reset()
        B.topk_compact(layout, scores, ks[i], vs[i], keep, 0, cache, kept)
    torch.cuda.synchronize()
    e0, e1 = ev(), ev()
    e0.record()
    for i in range(reps):
        cache.reset()
        B.topk_compact(layout, scores, ks[i % 3], vs[i % 3], keep, 0, cache, kept)
    e1.record()
    torch.cuda.synchronize()
    t = e0.elapsed_time(e1) * 1e-3 / reps
    nbytes = h * (n_g * 4 + keep * 4 + 2 * 2 * keep * d * 2)
    out["topk_compact"] = {"shape": f"{h} heads x {n_g} tokens, keep {keep}", "bytes": nbytes, "us": t * 1e6,
                           "GBps": nbytes / t / 1e9, "frac_of_hbm_peak": nbytes / t / 1e9 / PEAK_HBM_GBS}
    # window-attention scores at the same folded shape: 7 query heads per KV head, 64 window rows; the two-pass
    # kernel does 2 x (2 H_q W N_g d) flops and reads K twice (the second time mostly from cache)
    r, win = 7, 64
    wl = B.make_layout(h * r, h, d, "bf16")
    qwin = torch.randn(win, h * r, d, device="cuda", dtype=torch.bfloat16) / d ** 0.5
    wws = B.make_workspace(wl, n_g, win)
    for i in range(3):
        B.score_kv(wl, "window_attn", ks[i], None, qwin, scores, wws)
    torch.cuda.synchronize()
    e0, e1 = ev(), ev()
    e0.record()
    for i in range(reps):
        B.score_kv(wl, "window_attn", ks[i % 3], None, qwin, scores, wws)
    e1.record()
    torch.cuda.synchronize()
    t = e0.elapsed_time(e1) * 1e-3 / reps
    # the softmax-free variant of that rule: one dot product per key, HBM-bound like the norms
    for i in range(3):
        B.score_kv(wl, "window_logit", ks[i], None, qwin, scores, wws)
    torch.cuda.synchronize()
    e0, e1 = ev(), ev()
    e0.record()
    for i in range(reps):
        B.score_kv(wl, "window_logit", ks[i % 3], None, qwin, scores, wws)
    e1.record()
    torch.cuda.synchronize()
    tl = e0.elapsed_time(e1) * 1e-3 / reps
    nbytes = h * n_g * d * 2 + h * n_g * 4 + win * h * r * d * 2
    out["score_window_logit"] = {"shape": f"{h} KV heads x {r} query heads x {win} window rows x {n_g} tokens",
                                 "bytes": nbytes, "us": tl * 1e6, "GBps": nbytes / tl / 1e9,
                                 "frac_of_hbm_peak": nbytes / tl / 1e9 / PEAK_HBM_GBS}
    flops = 2.0 * h * r * win * n_g * d          # the method's one-pass minimum; the kernels do two passes
    n_exp = 2.0 * h * r * win * n_g              # one exponential per (row, key) and pass
    out["score_window"] = {"shape": f"{h} KV heads x {r} query heads x {win} window rows x {n_g} tokens",
                           "flops_one_pass": flops, "us": t * 1e6, "one_pass_TFLOPs": flops / t / 1e12,
                           "frac_of_mfma_peak_one_pass": flops / t / 1e12 / PEAK_BF16_TFLOPS,
                           "bound": "alu (exp2 at a quarter of the vector rate: 256 CUs x 4 SIMDs x 4 lanes x 2.4 GHz)",
                           "exp_per_s": n_exp / t, "frac_of_exp_peak": n_exp / t / PEAK_EXP_PER_S, "bytes": nbytes,
                           "GBps": nbytes / t / 1e9, "frac_of_hbm_peak": nbytes / t / 1e9 / PEAK_HBM_GBS}
    return out


def characterise_after_prefill(torch, B, w, layout, cache, ws, reps=50):
    """The stages that consume the pruned cache (Sec. 2.1: text-token prefill, then decoding), through the same
    qp_group_attend: a chunk of W text tokens and a single token against the layer's final cache. Few rows
    against a long cache: HBM-bound on the cache's K and V. With scratch the cache is dealt to about one workgroup
    per CU (decode: the kernel whose wavefronts stream their own key blocks; text chunk: key split of the large
    kernel) and a second launch merges; without scratch a single workgroup per row block walks the whole cache."""
    out = {}
    d, esz = w.head_dim, 2
    cesz = cache.k.element_size()          # 1 for an 8-bit cache
    c = cache.len
    for name, n_g in (("decode_1_token", 1), ("text_prefill_%d_tokens" % max(w.n_window, 64), max(w.n_window, 64))):
        q = torch.randn(n_g, w.n_q_heads, d, device="cuda").to(torch.bfloat16) / d ** 0.5
        k = torch.randn(n_g, w.n_kv_heads, d, device="cuda").to(torch.bfloat16) / d ** 0.5
        v = torch.randn(n_g, w.n_kv_heads, d, device="cuda").to(torch.bfloat16)
        o = torch.empty_like(q)
        res = {}
        for label, scratch in (("us", ws), ("us_without_scratch", None)):
            for _ in range(3):
                B.group_attend(layout, q, k, v, cache, o, None, scratch)
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(reps):
                B.group_attend(layout, q, k, v, cache, o, None, scratch)
            e1.record()
            torch.cuda.synchronize()
            res[label] = e0.elapsed_time(e1) * 1e3 / reps
        nbytes = 2 * w.n_kv_heads * (c * cesz + n_g * esz) * d + 2 * n_g * w.n_q_heads * d * esz
        flops = 4.0 * d * w.n_q_heads * (n_g * c + n_g * (n_g + 1) / 2)
        t = res["us"] * 1e-6
        res.update({"cache_len": c, "bytes": nbytes, "GBps": nbytes / t / 1e9,
                    "frac_of_hbm_peak": nbytes / t / 1e9 / PEAK_HBM_GBS, "TFLOPs": flops / t / 1e12})
        out[name] = res
    out["note"] = "one layer's cache is a few tens of MB and stays in the 256 MB Infinity Cache between repeats"
    return out


def layer_dims_of(w):
    """The decoder-layer sizes that go with a config's head counts (None if there is no such model)."""
    from paper_2505_16175_amd.workload import LAYER_DIMS
    for dims in LAYER_DIMS.values():
        if (dims.n_q_heads, dims.n_kv_heads, dims.head_dim) == (w.n_q_heads, w.n_kv_heads, w.head_dim):
            return dims
    return None


def _time_us(torch, fn, reps):
    for _ in range(2):
        fn()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(reps):
        fn()
    e1.record()
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) * 1e3 / reps


def characterise_layer(torch, B, w, rule, cache_len, reps=10):
    """One group of the config through one decoder layer around the path (Sec. 3.2: a block's activations exist
    for one group at a time; Appendix D.1 prices them): RMSNorm, QKV projection + rotary embedding, the path
    (attention over a cache of cache_len entries per head, scoring, top-k, compaction), o_proj + residual,
    RMSNorm, fused gate/up + SwiGLU, down_proj + residual. Random-init weights of the model's shape."""
    from paper_2505_16175_amd import workload as W
    dims = layer_dims_of(w)
    if dims is None or w.dtype != "bf16":
        return None
    n_g, dm, dff, hq, hkv = w.group_tokens, dims.d_model, dims.d_ff, dims.n_q_heads, dims.n_kv_heads
    layout = B.make_layout(hq, hkv, 128, "bf16")
    shape = B.make_layer_shape(dm, dff, dims.rms_eps, dims.rope_theta, dims.mrope_section)
    wt = W.make_decoder_layer(dims, 0, device="cuda")
    weights = B.LayerWeights(**wt)
    x = W.make_hidden(w.group_frames, w.tokens_per_frame, dm, device="cuda")
    pos = W.video_positions(w.group_frames, w.tokens_per_frame, device="cuda", first_frame=w.n_frames // 2)
    windowed = rule.startswith("window")
    n_win = w.n_window if windowed else 0
    ws = B.make_layer_workspace(layout, shape, n_g, n_win)
    keep = B.keep_count(n_g, w.retention)
    cache = B.Cache(layout, cache_len + keep)
    cache.k.normal_()
    cache.v.normal_()
    q_win = None
    if windowed:
        q_win = torch.empty(n_win, hq, 128, dtype=torch.bfloat16, device="cuda")
        B.layer_window_queries(layout, shape, weights, W.make_hidden(1, n_win, dm, device="cuda", seed=77),
                               W.text_positions(n_win, w.n_frames, device="cuda"), q_win, ws)
    x_out = torch.empty_like(x)

    def whole():
        cache.c.len = cache_len
        B.layer_group(layout, shape, weights, x, pos, 0, 0, q_win, rule, keep, cache, x_out, None, ws)

    t_layer = _time_us(torch, whole, reps)
    # the parts, on buffers of their own
    h = torch.empty_like(x)
    cs = torch.empty(n_g, 64, 2, dtype=torch.float32, device="cuda")
    q = torch.empty(n_g, hq, 128, dtype=torch.bfloat16, device="cuda")
    k = torch.empty(n_g, hkv, 128, dtype=torch.bfloat16, device="cuda")
    v = torch.empty_like(k)
    attn = torch.empty_like(q)
    act = torch.empty(n_g, dff, dtype=torch.bfloat16, device="cuda")
    scores = torch.empty(hkv, n_g, dtype=torch.float32, device="cuda")
    B.rope_table(pos, 0, n_g, dims.rope_theta, dims.mrope_section, cs)
    B.rms_norm(x, wt["ln1_w"], h, dims.rms_eps)
    B.qkv_rope(layout, h, wt["w_qkv"], wt["b_qkv"], cs, q, k, v)
    pws = B.make_workspace(layout, n_g, n_win)

    def path_rest():
        cache.c.len = cache_len
        B.score_kv(layout, rule, k, v, q_win, scores, pws)
        B.topk_compact(layout, scores, k, v, keep, 0, cache, None, pws)

    def attend():
        cache.c.len = cache_len
        B.group_attend(layout, q, k, v, cache, attn, None, pws)

    parts = {
        "rms_norm": (lambda: B.rms_norm(x, wt["ln1_w"], h, dims.rms_eps), 0.0),
        "qkv_rope": (lambda: B.qkv_rope(layout, h, wt["w_qkv"], wt["b_qkv"], cs, q, k, v), 2.0 * n_g * dm * (hq + 2 * hkv) * 128),
        "group_attend": (attend, attend_flops(w, cache_len, n_g)),
        "score_topk_compact": (path_rest, 0.0),
        "o_proj_residual": (lambda: B.linear(attn.view(n_g, hq * 128), wt["w_o"], None, x, x_out), 2.0 * n_g * dm * hq * 128),
        "gate_up_swiglu": (lambda: B.swiglu_gate_up(h, wt["w_gate_up"], act), 2.0 * n_g * dm * 2 * dff),
        "down_residual": (lambda: B.linear(act, wt["w_down"], None, x, x_out), 2.0 * n_g * dm * dff),
    }
    out = {"shape": f"{n_g} tokens x d_model {dm}, d_ff {dff}, {hq}q/{hkv}kv heads, cache {cache_len} per head, rule {rule}",
           "layer_us": t_layer, "tokens_per_s": n_g / (t_layer * 1e-6), "parts": {}}
    proj_flops = proj_us = 0.0
    for name, (fn, flops) in parts.items():
        us = _time_us(torch, fn, reps)
        out["parts"][name] = {"us": us}
        if flops:
            out["parts"][name].update({"TFLOPs": flops / us / 1e6, "frac_of_mfma_peak": flops / us / 1e6 / PEAK_BF16_TFLOPS})
        if name in ("qkv_rope", "o_proj_residual", "gate_up_swiglu", "down_residual"):
            proj_flops += flops
            proj_us += us
    out["parts"]["rms_norm"]["us_both"] = 2 * out["parts"]["rms_norm"]["us"]
    out["projections"] = {"flops": proj_flops, "us": proj_us, "TFLOPs": proj_flops / proj_us / 1e6,
                          "frac_of_mfma_peak": proj_flops / proj_us / 1e6 / PEAK_BF16_TFLOPS}
    # the later stages of Sec. 2.1 through the same layer call: a text chunk and a single token against the cache
    # (nothing pruned); few tokens, so streaming the layer's weights once is the bound (HBM)
    weight_bytes = sum(t.numel() * t.element_size() for t in wt.values())
    out["after_prefill_through_layer"] = {}
    for label, n_t in (("decode_1_token", 1), (f"text_chunk_{max(w.n_window, 64)}_tokens", max(w.n_window, 64))):
        xt = W.make_hidden(1, n_t, dm, device="cuda", seed=31)
        pt = W.text_positions(n_t, w.n_frames, device="cuda")
        ot = torch.empty_like(xt)
        tcache = B.Cache(layout, cache_len + n_t)
        tcache.k.normal_()
        tcache.v.normal_()

        def small():
            tcache.c.len = cache_len
            B.layer_group(layout, shape, weights, xt, pt, 0, 0, None, "key_norm_small", n_t, tcache, ot, None, ws)

        us = _time_us(torch, small, 4 * reps)
        out["after_prefill_through_layer"][label] = {
            "us": us, "weight_bytes": weight_bytes, "weight_GBps": weight_bytes / us / 1e3,
            "frac_of_hbm_peak": weight_bytes / us / 1e3 / PEAK_HBM_GBS}
    # activation memory of the group against Appendix D.1's model (fp16/bf16 elements)
    act_bytes = B.layer_workspace_bytes(layout, shape, n_g, n_win) - B.workspace_bytes(layout, n_g, n_win)
    model_group = (3 * n_g * hq * 128 + hq * 1024 * 1024) * 2 + n_g * (2 * dm + 4 * dff) * 2
    model_video = (3 * w.n_tokens * hq * 128 + hq * 1024 * 1024) * 2 + w.n_tokens * (2 * dm + 4 * dff) * 2
    out["activation_bytes"] = {"workspace_of_one_group": act_bytes, "appendix_d1_model_one_group": model_group,
                               "appendix_d1_model_whole_video": model_video,
                               "note": "model: Q,K,V at the query head count + one 1024x1024 score block per head, and "
                                       "(2 d_model + 4 d_ff) per token for the MLP; the fused kernels keep one d_ff-wide "
                                       "tensor (gate, up and SiLU never reach memory) and K,V at the KV head count"}
    return out


def run_stack(torch, B, w, rule, n_layers, steps, warmup, feed_ms=None):
    """Group-major schedule of Sec. 3.2 through a stack of decoder layers: every group runs through all layers
    (layer l+1 consumes layer l's output) before the next group starts; each layer keeps its own pruned cache."""
    from paper_2505_16175_amd import workload as W
    dims = layer_dims_of(w)
    if dims is None or w.dtype != "bf16":
        print("bench.py --stack: the config has no decoder-layer shape", file=sys.stderr)
        sys.exit(2)
    dm, hq, hkv = dims.d_model, dims.n_q_heads, dims.n_kv_heads
    layout = B.make_layout(hq, hkv, 128, "bf16")
    shape = B.make_layer_shape(dm, dims.d_ff, dims.rms_eps, dims.rope_theta, dims.mrope_section)
    weights = [B.LayerWeights(**W.make_decoder_layer(dims, l, device="cuda")) for l in range(n_layers)]
    x = W.make_hidden(w.n_frames, w.tokens_per_frame, dm, device="cuda")
    pos = W.video_positions(w.n_frames, w.tokens_per_frame, device="cuda")
    windowed = rule.startswith("window")
    n_win = w.n_window if windowed else 0
    ws = B.make_layer_workspace(layout, shape, w.group_tokens, n_win)
    cap = B.cache_capacity(w.n_frames, w.tokens_per_frame, w.group_frames, w.retention)
    caches = [B.Cache(layout, cap) for _ in range(n_layers)]
    q_wins = [None] * n_layers
    if windowed:
        pw = W.text_positions(n_win, w.n_frames, device="cuda")
        for l in range(n_layers):
            q_wins[l] = torch.empty(n_win, hq, 128, dtype=torch.bfloat16, device="cuda")
            B.layer_window_queries(layout, shape, weights[l], W.make_hidden(1, n_win, dm, device="cuda", seed=900 + l),
                                   pw, q_wins[l], ws)
    bounds = B.group_bounds(w.n_frames, w.tokens_per_frame, w.group_frames)
    bufs = [torch.empty(w.group_tokens, dm, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    out = torch.empty_like(x)

    def step():
        for c in caches:
            c.reset()
        for base, n_g in bounds:
            cur = x[base:base + n_g]
            keep = B.keep_count(n_g, w.retention)
            for l in range(n_layers):
                nxt = out[base:base + n_g] if l == n_layers - 1 else bufs[l & 1][:n_g]
                B.layer_group(layout, shape, weights[l], cur, pos, base, base, q_wins[l], rule, keep, caches[l], nxt,
                              None, ws)
                cur = nxt

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step()
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    flops_proj = 2.0 * w.n_tokens * n_layers * (dm * (hq + 2 * hkv) * 128 + dm * hq * 128 + 3 * dm * dims.d_ff)
    fed = None
    if feed_ms is not None:
        # Sec. 3.3: the same stack fed group by group from host memory by a stand-in loader that delivers the first
        # group after feed_ms[0] ms and one more every feed_ms[1] ms; copies overlap the previous group's compute
        first_ms, group_ms = feed_ms
        x_host = x.cpu().pin_memory()
        sizes = [n * dm * 2 for _, n in bounds]
        land = [torch.empty(w.group_tokens, dm, dtype=torch.bfloat16, device="cuda") for _ in range(2)]

        def one_group(g, dev_ptr, nbytes):
            base, n_g = bounds[g]
            cur = (land[0] if dev_ptr == land[0].data_ptr() else land[1])[:n_g]
            keep = B.keep_count(n_g, w.retention)
            for l in range(n_layers):
                nxt = out[base:base + n_g] if l == n_layers - 1 else bufs[l & 1][:n_g]
                B.layer_group(layout, shape, weights[l], cur, pos, base, base, q_wins[l], rule, keep, caches[l], nxt,
                              None, ws)
                cur = nxt

        for c in caches:
            c.reset()
        torch.cuda.synchronize()
        feed = B.Feed(3, w.group_tokens * dm * 2)
        try:
            feed.stub_producer(x_host, sizes, int(first_ms * 1000), int(group_ms * 1000))
            stats = feed.consume(land[0], land[1], one_group)
            producer_ms = feed.stub_join()
        finally:
            feed.destroy()
        t_prefill = elapsed / steps * 1e3
        t_dec = first_ms + (len(bounds) - 1) * group_ms
        t_last = t_prefill / len(bounds)       # the last group is the longest (largest cache): a lower bound
        fed = {"loader": {"first_group_ms": first_ms, "per_group_ms": group_ms, "t_dec_ms": t_dec,
                          "producer_wall_ms": producer_ms},
               "t_prefill_ms": t_prefill, "t_total_ms": stats["total_ms"], "waited_for_loader_ms": stats["waited_ms"],
               "sequential_ms": t_dec + t_prefill,
               "overlap_equation_ms": max(t_dec + t_last, t_prefill + first_ms),
               "note": "overlap_equation_ms takes the average group time for t^g_prefill (the last group is slower); "
                       "delta covers that, one group's copy and the queue hand-offs"}
    # calibration copy for the HBM counters: a plain device-to-device copy of known size (outside all timing)
    cal_src = torch.empty(CAL_COPY_BYTES // 4, dtype=torch.float32, device="cuda").normal_()
    torch.empty_like(cal_src).copy_(cal_src)
    torch.cuda.synchronize()
    print(json.dumps({
        "metric": "video tokens prefilled/sec through the decoder stack (group-major; layer l+1 consumes layer l)",
        "value": w.n_tokens * steps / elapsed, "unit": "tokens/s", "n_gpus": 1, "steps": steps, "warmup": warmup,
        "ms_per_step": elapsed / steps * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": f"{w.name} as a stack: {n_layers} decoder layers (d_model {dm}, d_ff {dims.d_ff}, {hq}q/{hkv}kv "
                               f"heads), {w.n_frames} frames x {w.tokens_per_frame} tokens, group {w.group_frames} frames, "
                               f"retention {w.retention}, rule {rule}",
                   "n_tokens": w.n_tokens, "groups": len(bounds), "layers": n_layers,
                   "weight_bytes": n_layers * sum(t.numel() * 2 for t in weights[0].tensors.values()),
                   "resident_cache_bytes": sum(c.nbytes() for c in caches),
                   "group_workspace_bytes": ws.numel()},
        "projection_TFLOPs_over_whole_step": flops_proj * steps / elapsed / 1e12,
        **({"fed_from_host": fed} if fed is not None else {}),
    }))


def _blas_threads():
    try:
        from threadpoolctl import threadpool_info
        return int(max([p.get("num_threads", 1) for p in threadpool_info()] or [1]))
    except Exception:
        return int(os.cpu_count() or 1)


def _boundary_rows(n_g, n_rows, rng):
    """Group-token rows for the sampled oracle: first, last, both sides of tile boundaries, then random ones."""
    rows = {0, n_g - 1}
    for b in (32, 64, 128, 256, n_g // 2, n_g - 32):
        for r in (b - 1, b):
            if 0 <= r < n_g:
                rows.add(r)
    while len(rows) < min(n_g, n_rows):
        rows.add(int(rng.integers(0, n_g)))
    return sorted(rows)


def cpu_baseline(w, q, k, v, qw, rule, gpu_pos=None, rows_per_group=64, full_below=40000):
    """The oracle on the host, as it stands: every group scored and selected in full (scores need no attention), the
    attention of a sample of groups evaluated in full (short videos) or on sampled rows (first, last, tile-boundary
    and random rows of each sampled group), and the layer time projected from the measured (row, key) pairs per
    second. If gpu_pos (the GPU's cache positions of the same layer) is given, the kept sets are compared: per
    (group, head) identical, excused as a near-tie (every differing index has an oracle score within 1e-5 relative
    of the k-th), or a mismatch."""
    import numpy as np
    from oracle import qp_oracle as O
    from paper_2505_16175_amd.workload import to_f64
    cores = _blas_threads()
    k64, v64 = to_f64(k), to_f64(v)
    qw64 = None if qw is None else to_f64(qw)
    t0 = time.perf_counter()
    sel = O.select_all_groups(k64, v64, qw64, w.n_frames, w.tokens_per_frame, w.group_frames, w.retention, rule)
    t_sel = time.perf_counter() - t0
    bounds = [(b, n) for b, n, _, _ in sel]
    g = len(bounds)
    near = None
    if gpu_pos is not None:
        lo = identical = excused = mismatched = 0
        for base, n_g, idx, sc in sel:
            kk = idx.shape[1]
            got = gpu_pos[:, lo:lo + kk] - base
            lo += kk
            for h in range(idx.shape[0]):
                if np.array_equal(got[h], idx[h]):
                    identical += 1
                    continue
                diff = np.setxor1d(got[h], idx[h])
                s_k = np.sort(sc[h])[::-1][kk - 1]
                ok = diff.min() >= 0 and diff.max() < n_g and (np.abs(sc[h][diff] - s_k) < 1e-5 * abs(s_k)).all()
                excused += bool(ok)
                mismatched += not ok
        near = {"group_heads": g * k64.shape[1], "identical": identical, "near_tie_excused": excused,
                "mismatched": mismatched, "rule": "relative score gap < 1e-5 to the k-th oracle score"}
    # attention cost is linear in the group index; this sample's mean index equals the full run's
    sample = sorted({0, g - 1} | ({(g - 1) // 3, g - 1 - (g - 1) // 3} if g >= 4 else set())) if g > 1 else [0]
    rng = np.random.default_rng(7)
    full = w.n_tokens <= full_below
    t_att, pairs = 0.0, 0.0
    for gi in sample:
        base, n_g = bounds[gi]
        rows = None if full else _boundary_rows(n_g, rows_per_group, rng)
        ck, cv, _ = O.gather_cache(k64, v64, sel, gi)
        qg = to_f64(q[base:base + n_g])
        t0 = time.perf_counter()
        O.attend_group(qg, k64[base:base + n_g], v64[base:base + n_g], ck, cv, rows=rows)
        t_att += time.perf_counter() - t0
        c = ck.shape[1]
        pairs += (n_g * c + n_g * (n_g + 1) / 2.0) if rows is None else float(sum(c + r + 1 for r in rows))
    total_pairs, c = 0.0, 0
    for (base, n_g), (_, _, idx, _) in zip(bounds, sel):
        total_pairs += n_g * c + n_g * (n_g + 1) / 2.0
        c += idx.shape[1]
    projected = t_sel + t_att * total_pairs / pairs
    what = "attended in full" if full else f"attended on {rows_per_group} sampled rows each (first, last, tile-boundary, random)"
    out = {"value": w.n_tokens / projected, "unit": "tokens/s", "cores": cores, "kind": "oracle",
           "sample": f"fp64 numpy oracle, one layer: all {g} groups scored+selected ({t_sel:.2f} s), groups {sample} {what} "
                     f"({t_att:.2f} s); layer time projected by visible (row,key) pairs ({pairs:.3g} of {total_pairs:.3g})",
           "projected": True, "projected_layer_seconds": projected, "measured_seconds": t_sel + t_att}
    return out, near


def read_traffic_table():
    """HBM bytes per launch of the attention kernel per config, from the rocprofv3 counter summary kept under
    profiles/ (written by paper_2505_16175_amd/profile_summary.py from FETCH_SIZE / WRITE_SIZE runs of this file)."""
    path = os.path.join(ROOT, "profiles", "attend_hbm_traffic.txt")
    table = {}
    if os.path.exists(path):
        for line in open(path):
            parts = line.split("|")
            if len(parts) >= 2 and not line.startswith("#"):
                try:
                    table[parts[0].strip()] = float(parts[1])
                except ValueError:
                    pass
    return table


def measure_config(torch, B, w, rule, steps, warmup, n_layers, replay_steps, graph=False, traffic=None, cache_fmt=0):
    """Timed steps of the whole path on one config (every layer's inputs and pruned cache resident in HBM), then an
    instrumented serial replay of layer 0 with HIP events around every launch group. Returns (result, keep) where
    keep holds what the CPU-baseline leg needs (layer 0's inputs and cache positions)."""
    from paper_2505_16175_amd.workload import make_layer
    layers = [make_layer(w, layer=l, device="cuda") for l in range(n_layers)]
    q, k, v, qw = layers[0]
    layout = B.make_layout(w.n_q_heads, w.n_kv_heads, w.head_dim, w.dtype)
    cap = B.cache_capacity(w.n_frames, w.tokens_per_frame, w.group_frames, w.retention)
    caches = [B.Cache(layout, cap, fmt=cache_fmt) for _ in range(n_layers)]   # every layer's pruned cache stays resident
    cache = caches[0]
    ws = B.make_workspace(layout, min(w.group_tokens, w.n_tokens), w.n_window)
    out = torch.empty_like(q)                                  # the layer output is consumed and overwritten
    windowed = rule.startswith("window")
    qwin = qw if windowed else None

    def step():
        for (lq, lk, lv, lqw), c in zip(layers, caches):
            c.reset()
            B.prefill_video(layout, w.n_frames, w.tokens_per_frame, w.group_frames, w.retention, rule, lq, lk, lv,
                            lqw if windowed else None, c, out, ws)

    print(f"[bench] {w.name} ({rule}): {n_layers} layer(s) generated, warm-up", file=sys.stderr, flush=True)
    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    if graph:
        eager_step = step
        gobj = torch.cuda.CUDAGraph()
        with torch.cuda.graph(gobj):
            eager_step()
        step = gobj.replay
        step()
        torch.cuda.synchronize()
    marks = [torch.cuda.Event(enable_timing=True) for _ in range(steps + 1)]
    t0 = time.perf_counter()
    marks[0].record()
    for i in range(steps):
        step()
        marks[i + 1].record()     # on the caller's stream, which every step rejoins before it returns
        if n_layers > 1:          # long steps: say where the run is (the host runs at most a queue's depth ahead)
            print(f"[bench] {w.name}: step {i + 1}/{steps} enqueued, {time.perf_counter() - t0:.1f} s", file=sys.stderr,
                  flush=True)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    ms_per_step = elapsed / steps * 1e3
    per_step = sorted(marks[i].elapsed_time(marks[i + 1]) for i in range(steps))
    value = w.n_tokens * n_layers * steps / elapsed           # tokens per second per layer
    pos_layer0 = cache.pos[:, :cache.len].cpu().numpy()
    final_len = cache.len
    resident_cache_bytes = sum(c.nbytes() for c in caches)
    cache_bytes_per_layer = cache.nbytes()

    # ---- instrumented replay of layer 0, one launch group after the other on one stream: HIP events around each
    bounds = B.group_bounds(w.n_frames, w.tokens_per_frame, w.group_frames)
    score_bufs = {n: torch.empty(w.n_kv_heads, n, dtype=torch.float32, device="cuda") for _, n in set(bounds)}
    ev = []
    for _ in range(replay_steps):
        cache.reset()
        for base, n_g in bounds:
            sl = slice(base, base + n_g)
            e = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
            c_before = cache.len
            e[0].record()
            B.group_attend(layout, q[sl], k[sl], v[sl], cache, out[sl], None, ws)
            e[1].record()
            scores = score_bufs[n_g]
            B.score_kv(layout, rule, k[sl], v[sl], qwin, scores, ws)
            e[2].record()
            keep = B.keep_count(n_g, w.retention)
            B.topk_compact(layout, scores, k[sl], v[sl], keep, base, cache, None, ws)
            e[3].record()
            ev.append((e, c_before, n_g, keep))
    torch.cuda.synchronize()
    t_att = t_sc = t_tk = 0.0
    fl = sb = tb = 0.0
    for e, c_before, n_g, keep in ev:
        t_att += e[0].elapsed_time(e[1]) * 1e-3
        t_sc += e[1].elapsed_time(e[2]) * 1e-3
        t_tk += e[2].elapsed_time(e[3]) * 1e-3
        fl += attend_flops(w, c_before, n_g)
        sb += score_bytes(w, rule, n_g)
        tb += topk_bytes(w, n_g, keep)
    n_launch = len(ev)
    achieved = fl / t_att / 1e12
    flops_per_layer = fl / replay_steps
    whole_step = flops_per_layer * n_layers / (ms_per_step * 1e-3) / 1e12
    roofline = {"kernel": "attend_mfma_kernel (qp_group_attend)", "bound": "mfma", "achieved": achieved,
                "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s", "frac": achieved / PEAK_BF16_TFLOPS,
                "traffic": None if traffic is None else traffic.get(w.name),
                "traffic_source": "profiles/attend_hbm_traffic.txt (rocprofv3 FETCH_SIZE + WRITE_SIZE per launch, scaled "
                                  "by a plain copy; a snapshot taken with the committed kernels, not measured in this run)",
                "launches": n_launch, "avg_launch_us": t_att / n_launch * 1e6, "flops_per_launch_avg": fl / n_launch,
                "measured": f"HIP events around every qp_group_attend launch of a serial replay of layer 0 ({replay_steps} "
                            "step(s), one stream, after the timed steps); for groups of under two rounds of workgroups "
                            "the timed steps overlap consecutive groups' launches on two streams, so whole_step_frac "
                            "(all layers' attention flops / ms_per_step) can exceed frac",
                "whole_step_achieved": whole_step, "whole_step_frac": whole_step / PEAK_BF16_TFLOPS}
    if w.dtype == "f32":
        roofline.update({"kernel": "attend_scalar_kernel (qp_group_attend)", "bound": "alu", "peak": 157.3,
                         "frac": achieved / 157.3, "whole_step_frac": whole_step / 157.3})
    stages = {
        "attend_ms_per_step": t_att / replay_steps * 1e3 * n_layers,
        "score_ms_per_step": t_sc / replay_steps * 1e3 * n_layers,
        "topk_compact_ms_per_step": t_tk / replay_steps * 1e3 * n_layers,
        "score": {"bound": "mfma" if rule.startswith("window_attn") else "hbm", "avg_launch_us": t_sc / n_launch * 1e6,
                  "algorithmic_GBps": sb / t_sc / 1e9, "frac_of_hbm_peak": sb / t_sc / 1e9 / PEAK_HBM_GBS},
        "topk_compact": {"bound": "hbm", "avg_launch_us": t_tk / n_launch * 1e6,
                         "algorithmic_GBps": tb / t_tk / 1e9, "frac_of_hbm_peak": tb / t_tk / 1e9 / PEAK_HBM_GBS},
        "note": "serial replay of layer 0 scaled to the config's layers; score/top-k figures are at the real per-group "
                "shapes (a few MB per launch: latency-bound; the bandwidth figures are under hbm_characterisation)",
    }
    if rule.startswith("window_attn"):   # the method's one-pass minimum 2 H_q W N_g d; the kernels do two passes
        wf = sum(2.0 * w.n_q_heads * w.n_window * n_g * w.head_dim for _, _, n_g, _ in ev)
        stages["score"].update({"one_pass_TFLOPs": wf / t_sc / 1e12,
                                "frac_of_mfma_peak_one_pass": wf / t_sc / 1e12 / PEAK_BF16_TFLOPS})
    result = {
        "ms_per_step": ms_per_step, "ms_per_step_median": per_step[len(per_step) // 2], "ms_per_step_min": per_step[0],
        "value": value, "steps": steps, "warmup": warmup, "dtype": w.dtype,
        "config": {"workload": f"{w.name}: {w.n_q_heads}q/{w.n_kv_heads}kv heads x d{w.head_dim}, "
                               f"{w.n_frames} frames x {w.tokens_per_frame} tokens, group {w.group_frames} frames, "
                               f"retention {w.retention}, rule {rule}, window {w.n_window if windowed else 0}"
                               + (", pruned cache in 8-bit E4M3" if cache_fmt else ""),
                   "n_tokens": w.n_tokens, "groups": len(bounds), "layers": n_layers,
                   "final_cache_len_per_head": final_len, "cache_bytes_per_layer": cache_bytes_per_layer,
                   "resident_cache_bytes": resident_cache_bytes},
        "roofline": roofline, "stages": stages,
    }
    keep_for_cpu = dict(q=q, k=k, v=v, qw=qwin, pos=pos_layer0, layout=layout, cache=cache, ws=ws)
    return result, keep_for_cpu


TABLE2_GROUP_FRAMES = (4, 8, 16, 32, 64, 128)       # Table 2, "Varying Group Size" (rho 0.5)
TABLE2_RETENTION = (1.0, 0.1, 0.2, 0.4, 0.6, 0.8, 0.9)  # Table 2, "Varying Retention Ratio" (groups of 16 frames)


def table2_grid(torch, B, base_w, steps=10, warmup=2):
    """The points of the paper's Table 2 ablation (Key Norms (small); group size 4-128 frames at rho 0.5, rho
    0.1-1.0 at 16 frames) as throughput on config 2's synthetic video: what the grid costs, not what it scores
    (the accuracies need the benchmark datasets and trained weights)."""
    import dataclasses
    points = [(g, 0.5) for g in TABLE2_GROUP_FRAMES] + [(16, r) for r in TABLE2_RETENTION]
    out = []
    for gf, rho in points:
        w = dataclasses.replace(base_w, group_frames=gf, retention=rho)
        res, keep = measure_config(torch, B, w, "key_norm_small", steps, warmup, 1, 1)
        out.append({"group_frames": gf, "group_tokens": w.group_tokens, "retention": rho,
                    "ms_per_layer": res["ms_per_step"], "tokens_per_s_per_layer": res["value"],
                    "final_cache_len_per_head": res["config"]["final_cache_len_per_head"],
                    "attend_frac_of_mfma_peak": res["roofline"]["frac"],
                    "whole_step_frac_of_mfma_peak": res["roofline"]["whole_step_frac"]})
        del keep
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--config", default=None,
                    help="run this config only (default: the headline on cfg5_7b_hour_stack, the largest config, plus a "
                         "`configs` array with all five)")
    ap.add_argument("--rule", default=None)
    ap.add_argument("--layers", type=int, default=None,
                    help="layers of a stacked config to run per step (default: all of the config's; inputs and the "
                         "pruned cache of every layer stay resident in HBM)")
    ap.add_argument("--group-frames", type=int, default=None,
                    help="frames per group instead of the config's (the group-size axis of the paper's Table 2 grid)")
    ap.add_argument("--retention", type=float, default=None,
                    help="KV retention ratio rho instead of the config's (the other axis of that grid)")
    ap.add_argument("--grid", action="store_true",
                    help="run the points of the paper's Table 2 grid (group 4-128 frames at rho 0.5; rho 0.1-1.0 at 16 "
                         "frames; Key Norms (small)) on config 2's video and print them as one JSON line")
    ap.add_argument("--graph", action="store_true",
                    help="capture one step (every layer's qp_prefill_video, library streams included) into a HIP graph "
                         "and time its replays: removes the host's launch cost, which bounds configs of many small groups")
    ap.add_argument("--stack", type=int, default=None, metavar="LAYERS",
                    help="instead of the headline path, run the config's video through a stack of this many decoder "
                         "layers around the path (group-major, each layer feeding the next) and print that line")
    ap.add_argument("--feed", type=float, nargs=2, default=None, metavar=("FIRST_MS", "GROUP_MS"),
                    help="with --stack: also run the stack fed group by group from host memory by a stand-in loader "
                         "(first group after FIRST_MS, one more every GROUP_MS) and report the overlapped run time")
    ap.add_argument("--cache-format", choices=("same", "fp8_e4m3"), default="same",
                    help="element format of the pruned cache: the inputs' own (default) or 8-bit E4M3")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--headline-only", action="store_true",
                    help="skip the other configs, the characterisation stages and the grid (profiling runs)")
    ap.add_argument("--mfma-probe", action="store_true",
                    help="run the stand-alone matrix-pipe probe (bf16 MFMA rate with constant / random operands) and exit")
    args = ap.parse_args()
    if args.mfma_probe:
        import subprocess
        from paper_2505_16175_amd.build import PROBE_PATH
        sys.exit(subprocess.run([PROBE_PATH]).returncode)
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2505_16175_amd import binding as B
    from paper_2505_16175_amd.workload import CONFIG_ORDER, CONFIGS

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(2)
    torch.cuda.set_device(0)
    headline_name = args.config or "cfg5_7b_hour_stack"
    w = CONFIGS[headline_name]
    if args.group_frames is not None or args.retention is not None:
        import dataclasses
        w = dataclasses.replace(w, group_frames=args.group_frames or w.group_frames,
                                retention=args.retention or w.retention)
    rule = args.rule or w.rules[0]
    if args.stack is not None:
        run_stack(torch, B, w, rule, args.stack, min(args.steps, 3), min(args.warmup, 1), args.feed)
        return
    if args.grid:
        print(json.dumps({"metric": "video tokens prefilled/sec per layer over the Table 2 grid (Key Norms (small))",
                          "unit": "tokens/s", "n_gpus": 1, "data": "synthetic", "dtype": "bf16",
                          "config": {"workload": "cfg2_7b_32k video, group size and retention varied"},
                          "table2_grid": table2_grid(torch, B, CONFIGS["cfg2_7b_32k"])}))
        return
    traffic = read_traffic_table() if w == CONFIGS[headline_name] else None
    all_configs = args.config is None and not args.headline_only and args.group_frames is None and args.retention is None

    # the other configs first (small), so that the headline's 119 GB of inputs is not resident beside them
    configs = []
    if all_configs:
        for name in CONFIG_ORDER:
            if name == headline_name:
                configs.append(None)
                continue
            cw = CONFIGS[name]
            for crule in cw.rules:
                res, keep = measure_config(torch, B, cw, crule, 10, 2, cw.n_layers, 2, traffic=traffic)
                entry = _config_entry(name, crule, res)
                if not args.no_cpu_baseline:
                    entry["cpu_baseline"], entry["near_tie"] = cpu_baseline(cw, keep["q"], keep["k"], keep["v"], keep["qw"],
                                                                            crule, keep["pos"], rows_per_group=96)
                configs.append(entry)
                del keep
            torch.cuda.empty_cache()

    n_layers = args.layers or w.n_layers
    cache_fmt = B.QP_CACHE_FP8_E4M3 if args.cache_format == "fp8_e4m3" else B.QP_CACHE_SAME
    if cache_fmt:
        traffic, args.no_cpu_baseline = None, True     # the counter table and the oracle leg are for the default format
    res, keep = measure_config(torch, B, w, rule, args.steps, args.warmup, n_layers, 1 if n_layers > 1 else min(args.steps, 10),
                               graph=args.graph, traffic=traffic, cache_fmt=cache_fmt)
    result = {
        "metric": "video tokens prefilled/sec per layer (attend+score+prune)",
        "value": res["value"], "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": res["ms_per_step"], "ms_per_step_median": res["ms_per_step_median"],
        "ms_per_step_min": res["ms_per_step_min"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": w.dtype, "data": "synthetic", "launch": "hip_graph_replay" if args.graph else "eager",
        "config": res["config"], "roofline": res["roofline"], "stages": res["stages"],
    }
    if not args.no_cpu_baseline:
        print(f"[bench] {w.name}: timed steps done, oracle on the host", file=sys.stderr, flush=True)
        result["cpu_baseline"], near = cpu_baseline(w, keep["q"], keep["k"], keep["v"], keep["qw"], rule, keep["pos"],
                                                    rows_per_group=384)
        if near is not None:
            near["layers_checked"] = "layer 0 of %d (the GPU tests check every layer)" % n_layers
        result["near_tie"] = near
    if all_configs:
        head_entry = _config_entry(headline_name, rule, res)
        head_entry["cpu_baseline"] = result.get("cpu_baseline")
        head_entry["near_tie"] = result.get("near_tie")
        result["configs"] = [head_entry if c is None else c for c in configs]
    # calibration copy for the HBM counters: a plain device-to-device copy of known size (outside all timing)
    cal_src = torch.empty(CAL_COPY_BYTES // 4, dtype=torch.float32, device="cuda").normal_()
    cal_dst = torch.empty_like(cal_src)
    cal_dst.copy_(cal_src)
    torch.cuda.synchronize()
    del cal_src, cal_dst
    if not args.headline_only:
        print("[bench] characterisation stages", file=sys.stderr, flush=True)
        layout, cache, ws = keep["layout"], keep["cache"], keep["ws"]
        result["stages"]["hbm_characterisation"] = characterise_hbm(torch, B)
        if w.dtype == "bf16":
            result["stages"]["after_prefill"] = characterise_after_prefill(torch, B, w, layout, cache, ws)
            layer = characterise_layer(torch, B, w, rule, cache.len // 2)
            if layer is not None:
                result["stages"]["decoder_layer"] = layer
        if all_configs:
            del keep
            torch.cuda.empty_cache()
            result["table2_grid"] = table2_grid(torch, B, CONFIGS["cfg2_7b_32k"], steps=5, warmup=1)
            # the 8-bit cache variant on config 2: same path, kept rows stored in E4M3 and widened when read
            w2 = CONFIGS["cfg2_7b_32k"]
            r8, k8 = measure_config(torch, B, w2, w2.rules[0], 10, 2, 1, 2, cache_fmt=B.QP_CACHE_FP8_E4M3)
            result["stages"]["fp8_cache_variant"] = {
                "workload": r8["config"]["workload"], "ms_per_step": r8["ms_per_step"],
                "tokens_per_s_per_layer": r8["value"], "attend_frac_of_mfma_peak": r8["roofline"]["frac"],
                "resident_cache_bytes": r8["config"]["resident_cache_bytes"],
                "after_prefill": characterise_after_prefill(torch, B, w2, k8["layout"], k8["cache"], k8["ws"])}
    emit(result)


BRIEF = ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "ms_per_step_median", "ms_per_step_min",
         "higher_is_better", "scaling", "vs_baseline", "dtype", "data", "launch", "config")


def emit(result):
    """The full record to stderr, section by section, then the one line on stdout."""
    for section, value in result.items():
        if isinstance(value, list):
            for i, entry in enumerate(value):
                print(f"[bench] detail {section}[{i}] {json.dumps(entry)}", file=sys.stderr)
        elif isinstance(value, dict):
            print(f"[bench] detail {section} {json.dumps(value)}", file=sys.stderr)
    sys.stderr.flush()
    line = {key: result[key] for key in BRIEF}
    rf = result["roofline"]
    line["roofline"] = {key: rf.get(key) for key in ("bound", "achieved", "peak", "frac", "whole_step_frac", "avg_launch_us")}
    if result.get("near_tie"):
        line["near_tie"] = {key: v for key, v in result["near_tie"].items() if isinstance(v, int)}
    if result.get("cpu_baseline"):
        line["cpu_baseline"] = {key: v for key, v in result["cpu_baseline"].items() if key != "sample"}
    if "configs" in result:
        line["configs"] = [{"name": c["name"], "rule": c["rule"], "ms_per_step": c["ms_per_step"],
                            "tokens_per_s_per_layer": c["tokens_per_s_per_layer"], "attend_frac": c["attend"]["frac"]}
                           for c in result["configs"]]
    print(json.dumps(line))


def _config_entry(name, rule, res):
    """One line of the `configs` array: what the benchmark definition asks to be reported per config."""
    rf, st = res["roofline"], res["stages"]
    return {"name": name, "rule": rule, "workload": res["config"]["workload"], "layers": res["config"]["layers"],
            "ms_per_step": res["ms_per_step"], "tokens_per_s_per_layer": res["value"], "dtype": res["dtype"],
            "attend": {"bound": rf["bound"], "TFLOPs": rf["achieved"], "frac": rf["frac"],
                       "whole_step_frac": rf["whole_step_frac"], "avg_launch_us": rf["avg_launch_us"],
                       "traffic": rf["traffic"]},
            "score": st["score"], "topk_compact": st["topk_compact"],
            "final_cache_len_per_head": res["config"]["final_cache_len_per_head"],
            "resident_cache_bytes": res["config"]["resident_cache_bytes"]}


if __name__ == "__main__":
    main()
