"""Performance cases of the library: what its users have it do, through the public entry points of the binding.

Three kinds of calls, each over the range of sizes it meets:

  prefill  one layer of a video through `prefill_video`: all groups attended, scored, pruned and compacted
  layer    one group of tokens through a decoder layer with `layer_group`: a video group (pruned on the way), a text
           chunk or a single token (everything kept) over the cache the video left
  attend   `group_attend` alone for the stages after the video: a text chunk or a decoding step over the pruned cache,
           as an integration that brings its own projections calls it

`listed()` names the cases, `draw()` draws others from the same ranges. Inputs come from `workload.py`, the generators
that the tests and `bench.py` use; layer shapes are the ones of its configurations.
"""
import math

import torch

from paper_2505_16175_amd import binding as B
from paper_2505_16175_amd import workload as W

# head layouts of workload.py's configurations
LAYOUTS = {"tiny": (4, 2, 64, "f32"), "7b": (28, 4, 128, "bf16"), "72b": (64, 8, 128, "bf16")}
MAX_FLOPS = 1.75e14  # a drawn case costs no more than the hour-long layer


def _prefill(name, layout, frames, tokens, group, rho, rule, window=0, fp8=False, corr=0.9, sigma=0.5):
    return dict(name=name, kind="prefill", layout=layout, frames=frames, tokens_per_frame=tokens, group_frames=group,
                retention=rho, rule=rule, window=window, fp8_cache=fp8, corr=corr, key_sigma=sigma)


def _layer(name, layout, tokens, cache, rho, rule="key_norm_small", window=0):
    return dict(name=name, kind="layer", layout=layout, tokens=tokens, cache=cache, retention=rho, rule=rule, window=window)


def _attend(name, layout, tokens, cache, fp8=False):
    return dict(name=name, kind="attend", layout=layout, tokens=tokens, cache=cache, fp8_cache=fp8)


def listed():
    return [
        # the smallest video: eight tiny frames in f32, four groups; launches and waits are what it costs
        _prefill("tiny_f32", "tiny", 8, 16, 2, 0.5, "key_norm_small"),
        # four minutes at one frame a second through one layer, scored by the question's attention (config 2)
        _prefill("video_7b_32k", "7b", 256, 128, 16, 0.3, "window_attn", 64),
        # a short clip in odd sizes: frames of 11 x 11 tokens, small groups with a ragged last one, 8-bit cache
        _prefill("clip_7b_fp8", "7b", 99, 121, 4, 0.5, "value_norm", 0, True),
        # seventeen minutes of static scenes, the paper's default rule (config 3)
        _prefill("video_7b_128k", "7b", 1024, 128, 32, 0.2, "key_norm_small", 0, False, 0.95),
        # one layer of the large model over a 512-frame video (config 4)
        _prefill("video_72b_128k", "72b", 512, 256, 16, 0.25, "window_attn", 128, False, 0.9, 0.75),
        # one layer of the hour-long video (config 5): the largest
        _prefill("hour_7b", "7b", 3600, 128, 64, 0.1, "window_attn", 64),
        # a video group on its way through a whole decoder layer, in the middle of the video
        _layer("layer_video_7b", "7b", 2048, 4920, 0.3, "window_attn", 64),
        _layer("layer_video_72b", "72b", 4096, 16384, 0.25, "key_norm_small"),
        # the user's question after the video: a chunk of text through a layer over the hour-long cache
        _layer("layer_text_7b", "7b", 64, 46125, 1.0),
        # one token of the answer through a layer
        _layer("layer_decode_7b", "7b", 1, 46125, 1.0),
        # attention alone: a question of odd length over the four-minute cache, and an answer's token over an 8-bit one
        _attend("attend_text_7b", "7b", 77, 9840),
        _attend("attend_decode_72b", "72b", 1, 32768, True),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    while True:
        kind = rng.choice(("prefill", "prefill", "prefill", "layer", "layer", "layer", "attend"))
        big = rng.choice(("7b", "7b", "72b"))
        if kind == "prefill":
            rule = rng.choice(("key_norm_small", "value_norm", "window_attn", "window_attn"))
            window = _log_int(rng, 8, 128) if rule == "window_attn" else 0
            rho = round(rng.uniform(0.1, 0.9), 2)
            if rng.random() < 0.15:
                case = _prefill("", "tiny", rng.randint(4, 48), rng.randint(8, 32), rng.randint(1, 8), rho, rule, window)
            else:
                tokens = rng.choice((64, 81, 100, 121, 128, 128, 144, 169, 196, 256))
                group = _log_int(rng, 4, 64)
                case = _prefill("", big, _log_int(rng, 32, 3600), tokens, group, rho, rule, window, rng.random() < 0.25)
        elif kind == "layer":
            cache = _log_int(rng, 512, 60000)
            if rng.random() < 0.4:  # a video group
                rule = rng.choice(("key_norm_small", "value_norm", "window_attn"))
                case = _layer("", big, _log_int(rng, 512, 8192), min(cache, 32768), round(rng.uniform(0.1, 0.9), 2), rule,
                              _log_int(rng, 8, 128) if rule == "window_attn" else 0)
            else:  # text chunks down to single tokens
                case = _layer("", big, _log_int(rng, 1, 512), cache, 1.0)
        else:
            case = _attend("", big, _log_int(rng, 1, 256), _log_int(rng, 512, 120000), rng.random() < 0.35)
        del case["name"]
        if work(case)["flops"] <= MAX_FLOPS:
            return case


def _groups(case):
    """(tokens, kept) of every frame-aligned group: ceil(retention * tokens), as the entry points define it."""
    out = []
    for f in range(0, case["frames"], case["group_frames"]):
        n = min(case["group_frames"], case["frames"] - f) * case["tokens_per_frame"]
        out.append((n, max(1, min(n, math.ceil(case["retention"] * n - 1e-9)))))
    return out


def _keep(case):
    n = case["tokens"]
    return max(1, min(n, math.ceil(case["retention"] * n - 1e-9)))


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _filled_cache(layout, capacity, n, fp8, gen):
    """A cache as a video leaves it: n unit-scale keys and values per head, positions ascending with gaps."""
    cache = B.Cache(layout, capacity, fmt=B.QP_CACHE_FP8_E4M3 if fp8 else B.QP_CACHE_SAME)
    for t in (cache.k, cache.v):
        t[:, :n].copy_(torch.randn(layout.n_kv_heads, n, layout.head_dim, generator=gen, device="cuda").to(torch.bfloat16))
    cache.pos[:, :n] = torch.arange(0, 3 * n, 3, dtype=torch.int32, device="cuda")
    cache.c.len = n
    return cache


def prepare(case, seed):
    hq, hkv, d, dtype = LAYOUTS[case["layout"]]
    layout = B.make_layout(hq, hkv, d, dtype)
    if case["kind"] == "prefill":
        b = math.sqrt(1 - case["corr"] ** 2) if case["corr"] > 0.9 else 0.44
        w = W.Workload("case", dtype, hq, hkv, d, case["frames"], case["tokens_per_frame"], case["group_frames"],
                       case["retention"], (case["rule"],), case["window"], case["corr"], b, case["key_sigma"])
        q, k, v, qw = W.make_layer(w, 0, "cuda", seed=seed)
        capacity = B.cache_capacity(w.n_frames, w.tokens_per_frame, w.group_frames, w.retention)
        cache = B.Cache(layout, capacity, fmt=B.QP_CACHE_FP8_E4M3 if case["fp8_cache"] else B.QP_CACHE_SAME)
        ws = B.make_workspace(layout, min(w.group_tokens, w.n_tokens), w.n_window)
        return dict(case=case, layout=layout, q=q, k=k, v=v, qw=qw, cache=cache, out=torch.empty_like(q), ws=ws)
    gen = _gen(seed)
    n, c = case["tokens"], case["cache"]
    if case["kind"] == "layer":
        dims = W.LAYER_DIMS[case["layout"]]
        shape = B.make_layer_shape(dims.d_model, dims.d_ff, dims.rms_eps, dims.rope_theta, dims.mrope_section)
        weights = B.LayerWeights(**W.make_decoder_layer(dims, 0, "cuda", seed=seed))
        x = torch.randn(n, dims.d_model, generator=gen, device="cuda").to(torch.bfloat16)
        keep = _keep(case)
        if keep < n:
            frames = -(-n // 128)
            pos = W.video_positions(frames, 128, "cuda", 3 * c // 128)[:, :n].contiguous()
        else:
            pos = W.text_positions(n, 3 * c, "cuda")
        qw = None
        if case["window"]:
            qw = torch.randn(case["window"], hq, d, generator=gen, device="cuda").to(torch.bfloat16)
        cache = _filled_cache(layout, c + keep, c, False, gen)
        kept = torch.empty(hkv, keep, dtype=torch.int32, device="cuda")
        return dict(case=case, layout=layout, shape=shape, weights=weights, x=x, pos=pos, qw=qw, keep=keep, cache=cache,
                    kept=kept, out=torch.empty_like(x), ws=B.make_layer_workspace(layout, shape, n, case["window"]))
    q, k, v = (torch.randn(n, h, d, generator=gen, device="cuda").to(torch.bfloat16) for h in (hq, hkv, hkv))
    cache = _filled_cache(layout, c, c, case["fp8_cache"], gen)
    return dict(case=case, layout=layout, q=q, k=k, v=v, cache=cache, out=torch.empty_like(q),
                lse=torch.empty(hq, n, device="cuda"), ws=B.make_workspace(layout, n, 0))


def run(s):
    case, cache = s["case"], s["cache"]
    if case["kind"] == "prefill":
        cache.reset()
        B.prefill_video(s["layout"], case["frames"], case["tokens_per_frame"], case["group_frames"], case["retention"],
                        case["rule"], s["q"], s["k"], s["v"], s["qw"], cache, s["out"], s["ws"])
        return dict(out=s["out"], k=cache.k, v=cache.v, pos=cache.pos)
    if case["kind"] == "layer":
        cache.c.len = case["cache"]
        B.layer_group(s["layout"], s["shape"], s["weights"], s["x"], s["pos"], 0, 3 * case["cache"], s["qw"], case["rule"],
                      s["keep"], cache, s["out"], s["kept"], s["ws"])
        return dict(out=s["out"], k=cache.k, v=cache.v, pos=cache.pos, kept=s["kept"])
    B.group_attend(s["layout"], s["q"], s["k"], s["v"], cache, s["out"], s["lse"], s["ws"])
    return dict(out=s["out"], lse=s["lse"])


def work(case):
    """Bytes: every input read once, every output written once (a cache that the pass builds counts as an output only).
    Flops: the visible (row, key) pairs of the attention, the projections, one product per scored key."""
    hq, hkv, d, dtype = LAYOUTS[case["layout"]]
    e = 4 if dtype == "f32" else 2
    pair, kv_row = 4 * d * hq, 2 * hkv * d
    if case["kind"] == "prefill":
        ec = 1 if case["fp8_cache"] else e
        n = case["frames"] * case["tokens_per_frame"]
        c, flops = 0, 0
        for ng, keep in _groups(case):
            flops += pair * (ng * c + ng * (ng + 1) // 2)
            c += keep
        flops += n * d * 2 * (hq * case["window"] if case["window"] else hkv)
        return {"bytes": n * (2 * hq * d + kv_row) * e + case["window"] * hq * d * e + c * (kv_row * ec + 4 * hkv),
                "flops": flops}
    n, c = case["tokens"], case["cache"]
    pairs = n * c + n * (n + 1) // 2
    if case["kind"] == "attend":
        return {"bytes": (n * (2 * hq * d + kv_row)) * e + c * kv_row * (1 if case["fp8_cache"] else e) + 4 * hq * n,
                "flops": pair * pairs}
    dims, keep = W.LAYER_DIMS[case["layout"]], _keep(case)
    mats = dims.d_model * ((2 * hq + 2 * hkv) * d + 3 * dims.d_ff)
    score = 0 if keep == n else n * d * 2 * (hq * case["window"] if case["window"] else hkv)
    return {"bytes": 2 * (mats + 2 * n * dims.d_model + case["window"] * hq * d) + (c + keep) * kv_row * 2 + 8 * keep * hkv,
            "flops": 2 * n * mats + pair * pairs + score}


def tolerance(case):
    """About four times what was seen between the tiled and the scalar attention kernel, other tilings and splits of the
    projections, and double precision: bf16 rel 2.5e-3, max 2.5e-2 (the softmax numerators and the stored tensors are
    rounded to bf16); f32 rel 1e-7 on one group, more where a row meets many groups."""
    if LAYOUTS[case["layout"]][3] == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 1e-2, "max": 0.1}


# ---- the same results in 64 bits, from the definitions -------------------------------------------------------
MAX_EXACT_FLOPS = 4e13  # beyond this the 64-bit products take too long


def _attend64(q, k, v, ck, cv, out, lse=None):
    """Rows of a group over the kept entries and, causally, the group itself, head by head in blocks of rows."""
    n, hq, d = q.shape
    r, c = hq // k.shape[1], ck.shape[1]
    for h in range(hq):
        kk = torch.cat((ck[h // r].double(), k[:, h // r].double()))
        vv = torch.cat((cv[h // r].double(), v[:, h // r].double()))
        step = max(1, (1 << 27) // kk.shape[0])
        for t in range(0, n, step):
            e = min(n, t + step)
            s = (q[t:e, h].double() @ kk[:c + e].T) / math.sqrt(d)
            later = torch.arange(e, device=q.device)[None, :] > torch.arange(t, e, device=q.device)[:, None]
            s[:, c:].masked_fill_(later, -math.inf)
            if lse is not None:
                lse[h, t:e] = torch.logsumexp(s, -1)
            out[t:e, h] = torch.softmax(s, -1) @ vv[:c + e]


def _kept64(case, k, v, qw, keep):
    """Indices [h_kv][keep] that Eq. 2 keeps of a group, ascending."""
    if case["rule"] == "key_norm_small":
        s = -k.norm(dim=-1).T
    elif case["rule"] == "value_norm":
        s = v.norm(dim=-1).T
    else:
        w, hq, d = qw.shape
        hkv = k.shape[1]
        rows = qw.reshape(w, hkv, hq // hkv, d).permute(1, 0, 2, 3).reshape(hkv, -1, d)
        s = torch.softmax(torch.matmul(rows, k.permute(1, 2, 0).contiguous()) / math.sqrt(d), -1).sum(1)
    order = torch.sort(s, dim=-1, descending=True, stable=True).indices[:, :keep]
    return order.sort(-1).values


def _gather(x, idx):
    return torch.stack([x[idx[h], h] for h in range(idx.shape[0])])


def _cached64(t, fp8):
    """A kept row as the cache's format holds it (8-bit: nearest E4M3 value, saturating at 448)."""
    return t.clamp(-448, 448).float().to(torch.float8_e4m3fn).double() if fp8 else t


def _rms64(x, w, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * w.double()


def _rope64(x, pos, dims):
    """Rotary embedding with three position axes: halves of the head dimension pair up."""
    half = x.shape[-1] // 2
    axis = torch.tensor([0] * dims.mrope_section[0] + [1] * dims.mrope_section[1] + [2] * dims.mrope_section[2], device=x.device)
    freq = dims.rope_theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    ang = (pos.double()[axis].T * freq)[:, None, :]
    a, b = x[..., :half], x[..., half:]
    return torch.cat((a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()), -1)


def exact(case, seed):
    """What `run` returns, in 64 bits throughout. Where entries are pruned, the kept rows themselves are left out: at a
    near-tie more than one selection is right, and it shifts the rows behind it."""
    if work(case)["flops"] > MAX_EXACT_FLOPS:
        return None
    s = prepare(case, seed)
    hq, hkv, d, _ = LAYOUTS[case["layout"]]
    if case["kind"] == "prefill":
        q, k, v = s["q"], s["k"], s["v"]
        out = torch.empty(q.shape, dtype=torch.float64, device="cuda")
        ck = cv = torch.empty(hkv, 0, d, dtype=torch.float64, device="cuda")
        first = 0
        for n, keep in _groups(case):
            g = slice(first, first + n)
            _attend64(q[g], k[g], v[g], ck, cv, out[g])
            kg, vg = k[g].double(), v[g].double()
            idx = _kept64(case, kg, vg, s["qw"].double() if case["window"] else None, keep)
            ck = torch.cat((ck, _cached64(_gather(kg, idx), case["fp8_cache"])), 1)
            cv = torch.cat((cv, _cached64(_gather(vg, idx), case["fp8_cache"])), 1)
            first += n
        return dict(out=out, k=None, v=None, pos=None)
    cache, c, n = s["cache"], case["cache"], case["tokens"]
    ck, cv = cache.k[:, :c], cache.v[:, :c]
    if case["kind"] == "attend":
        out = torch.empty(s["q"].shape, dtype=torch.float64, device="cuda")
        lse = torch.empty(hq, n, dtype=torch.float64, device="cuda")
        _attend64(s["q"], s["k"], s["v"], ck, cv, out, lse)
        return dict(out=out, lse=lse)
    dims = W.LAYER_DIMS[case["layout"]]
    w, x = s["weights"].tensors, s["x"].double()
    qkv = (_rms64(x, w["ln1_w"], dims.rms_eps) @ w["w_qkv"].double().T + w["b_qkv"].double()).view(n, hq + 2 * hkv, d)
    q, k, v = _rope64(qkv[:, :hq], s["pos"], dims), _rope64(qkv[:, hq:hq + hkv], s["pos"], dims), qkv[:, hq + hkv:]
    att = torch.empty(n, hq, d, dtype=torch.float64, device="cuda")
    _attend64(q, k, v, ck, cv, att)
    x1 = x + att.view(n, hq * d) @ w["w_o"].double().T
    gate, up = (_rms64(x1, w["ln2_w"], dims.rms_eps) @ w["w_gate_up"].double().T).split(dims.d_ff, -1)
    out = x1 + (torch.nn.functional.silu(gate) * up) @ w["w_down"].double().T
    if s["keep"] < n:
        return dict(out=out, k=None, v=None, pos=None, kept=None)
    return dict(out=out, k=torch.cat((ck.double(), k.transpose(0, 1)), 1), v=torch.cat((cv.double(), v.transpose(0, 1)), 1),
                pos=None, kept=None)
