"""GPU parity of the 8-bit (E4M3) pruned-cache variant: what the compaction stores, what the attention reads, and the
whole path, against the fp64 oracle's cache_format="fp8_e4m3"."""
import numpy as np
import pytest
import torch

from helpers import assert_attn_close, compare_kept
from oracle import qp_oracle as O
from paper_2505_16175_amd import binding as B
from paper_2505_16175_amd import workload as W
from paper_2505_16175_amd.workload import CONFIGS, make_layer, scaled, to_f64

pytestmark = pytest.mark.gpu
DEV = "cuda"
FP8 = B.QP_CACHE_FP8_E4M3


def _decoded(t):
    """An E4M3 cache tensor as float64 (torch.float8_e4m3fn is the same format)."""
    return t.to(torch.float32).to(torch.float64).cpu().numpy()


@pytest.mark.parametrize("keep", [111, 300])
def test_compaction_stores_the_oracles_roundings(keep):
    """Kept rows enter the 8-bit cache rounded exactly as the oracle rounds them: ordinary activations, exact ties,
    values beyond the format's range (saturating), the subnormal range and zeros. keep = 300 keeps every token (the
    plain append)."""
    n_g, h_kv = 300, 3
    g = torch.Generator().manual_seed(5)
    k = torch.randn(n_g, h_kv, 128, generator=g) * 10.0 ** torch.randint(-4, 3, (n_g, h_kv, 1), generator=g).float()
    v = torch.randn(n_g, h_kv, 128, generator=g)
    special = torch.tensor([1.0625, 1.1875, 248.0, 448.0, 464.0, 1000.0, -7e4, 2.0 ** -9, 2.0 ** -10, 1.5 * 2.0 ** -9,
                            7.5 * 2.0 ** -9, 0.0, -0.0, 3.0e-5, -1.1, 0.00098])
    k[:, 0, :16] = special
    v[:, 1, 16:32] = -special
    k, v = k.to(torch.bfloat16), v.to(torch.bfloat16)
    s = torch.randn(h_kv, n_g, generator=g)
    layout = B.make_layout(h_kv, h_kv, 128, "bf16")
    cache = B.Cache(layout, keep + 7, fmt=FP8)
    assert cache.k.element_size() == 1
    cache.c.len = 7                                            # appended behind existing entries
    kept = torch.empty(h_kv, keep, dtype=torch.int32, device=DEV)
    B.topk_compact(layout, s.to(DEV), k.to(DEV), v.to(DEV), keep, 40, cache, kept)
    torch.cuda.synchronize()
    want = O.topk_select(s.double().numpy(), keep)
    np.testing.assert_array_equal(kept.cpu().numpy(), want)
    np.testing.assert_array_equal(cache.pos.cpu().numpy()[:, 7:7 + keep], 40 + want)
    k64, v64 = to_f64(k), to_f64(v)
    for h in range(h_kv):
        np.testing.assert_array_equal(_decoded(cache.k[h, 7:7 + keep]), O.fp8_e4m3_round(k64[want[h], h]))
        np.testing.assert_array_equal(_decoded(cache.v[h, 7:7 + keep]), O.fp8_e4m3_round(v64[want[h], h]))
    assert (cache.k[:, :7].view(torch.uint8) == 0).all()       # earlier entries untouched
    assert cache.nbytes() * 2 == 2 * h_kv * cache.len * 128 * 2  # half the bytes of a bf16 cache of the same length


@pytest.mark.parametrize("fmt", [B.QP_CACHE_SAME, FP8])
@pytest.mark.parametrize("n_g,h_q,h_kv,c", [(1, 64, 8, 32768), (4, 28, 4, 9840), (1, 28, 4, 700), (1, 6, 3, 50000), (77, 28, 4, 9840)])
def test_attend_writes_the_scratch_that_the_plan_reports(n_g, h_q, h_kv, c, fmt):
    """qp_attend_plan describes the launch over either cache format: the call writes every byte of scratch_bytes and none
    behind them, with scratch to spare and with exactly that much."""
    g = torch.Generator(device=DEV).manual_seed(c)
    bf = lambda *s: torch.randn(*s, generator=g, device=DEV).to(torch.bfloat16)
    q, k, v = bf(n_g, h_q, 128), bf(n_g, h_kv, 128), bf(n_g, h_kv, 128)
    layout = B.make_layout(h_q, h_kv, 128, "bf16")
    cache = B.Cache(layout, c, fmt=fmt)
    cache.k.copy_(bf(h_kv, c, 128))
    cache.v.copy_(bf(h_kv, c, 128))
    cache.c.len = c
    out = torch.empty_like(q)
    offered = 64 << 20
    scratch = B.attend_plan(layout, n_g, c, offered)["scratch_bytes"]
    assert 0 < scratch < offered
    for size in (offered, scratch):
        assert B.attend_plan(layout, n_g, c, size)["scratch_bytes"] == scratch
        seen = []
        for fill in (0x00, 0xff):                               # a byte that shows both fills was not written
            ws = torch.full((offered,), fill, dtype=torch.uint8, device=DEV)
            B.group_attend(layout, q, k, v, cache, out, None, ws[:size])
            torch.cuda.synchronize()
            seen.append(ws)
        untouched = (seen[0] == 0x00) & (seen[1] == 0xff)
        assert not untouched[:scratch].any() and untouched[scratch:].all()


@pytest.mark.parametrize("n_g,h_q,h_kv,c", [(300, 28, 4, 1000), (64, 28, 4, 5000), (1, 28, 4, 9840), (7, 8, 8, 77),
                                            (2048, 28, 4, 4920), (130, 64, 8, 0), (1, 64, 8, 40000), (4, 28, 4, 31),
                                            (3, 28, 4, 32), (1, 28, 4, 129), (2, 28, 4, 0), (4, 64, 8, 2051)])
def test_group_attend_reads_an_e4m3_cache(n_g, h_q, h_kv, c):
    """The attention over an 8-bit cache equals the oracle's attention over the cache's decoded values: large groups,
    key-split calls (text chunk), decode-shaped calls (a few rows per KV head: the small kernel widens the cache blocks
    itself; block counts below, at and above one block, ragged tails), an empty cache."""
    print(f"case n_g={n_g} h_q={h_q} h_kv={h_kv} c={c}", flush=True)
    g = torch.Generator().manual_seed(n_g * 7 + c)
    bf = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)
    q, k, v = bf(n_g, h_q, 128), bf(n_g, h_kv, 128), bf(n_g, h_kv, 128)
    layout = B.make_layout(h_q, h_kv, 128, "bf16")
    cache = B.Cache(layout, max(c, 1) + 3, fmt=FP8)
    ck = (torch.randn(h_kv, max(c, 1) + 3, 128, generator=g) * 2.0).to(torch.float8_e4m3fn)
    cv = (torch.randn(h_kv, max(c, 1) + 3, 128, generator=g) * 2.0).to(torch.float8_e4m3fn)
    cache.k.copy_(ck)
    cache.v.copy_(cv)
    cache.c.len = c
    ws = B.make_workspace(layout, max(n_g, 64), 0)
    out = torch.full((n_g, h_q, 128), float("nan"), dtype=torch.bfloat16, device=DEV)
    lse = torch.full((h_q, n_g), float("nan"), dtype=torch.float32, device=DEV)
    B.group_attend(layout, q.to(DEV), k.to(DEV), v.to(DEV), cache, out, lse, ws)
    torch.cuda.synchronize()
    want, want_lse = O.attend_group(to_f64(q), to_f64(k), to_f64(v), _decoded(ck)[:, :c], _decoded(cv)[:, :c],
                                    return_lse=True)
    assert_attn_close(to_f64(out), want, "bf16", f"fp8 cache n_g={n_g} c={c}")
    np.testing.assert_allclose(to_f64(lse), want_lse, atol=2e-3)


@pytest.mark.parametrize("rule", ["key_norm_small", "window_attn"])
def test_whole_path_with_an_e4m3_cache(rule):
    """qp_prefill_video with the 8-bit cache on a reduced config-2 shape: kept sets as the oracle's, the cache the
    oracle's rounded rows exactly, every output element against the oracle's run with cache_format="fp8_e4m3"."""
    w = scaled(CONFIGS["cfg2_7b_32k"], n_frames=14, tokens_per_frame=48, group_frames=4)    # ragged last group
    q, k, v, qw = make_layer(w, sharp=True)
    layout = B.make_layout(w.n_q_heads, w.n_kv_heads, w.head_dim, w.dtype)
    cap = B.cache_capacity(w.n_frames, w.tokens_per_frame, w.group_frames, w.retention)
    cache = B.Cache(layout, cap, fmt=FP8)
    ws = B.make_workspace(layout, w.group_tokens, w.n_window)
    out = torch.full_like(q, float("nan"), device=DEV)
    B.prefill_video(layout, w.n_frames, w.tokens_per_frame, w.group_frames, w.retention, rule, q.to(DEV), k.to(DEV),
                    v.to(DEV), qw.to(DEV) if rule.startswith("window") else None, cache, out, ws)
    torch.cuda.synchronize()
    q64, k64, v64, qw64 = to_f64(q), to_f64(k), to_f64(v), to_f64(qw)
    want, wck, wcv, wpos, sel = O.prefill_video(q64, k64, v64, qw64, w.n_frames, w.tokens_per_frame, w.group_frames,
                                                w.retention, rule, cache_format="fp8_e4m3")
    assert cache.len == wpos.shape[1]
    pos = cache.pos.cpu().numpy()[:, :cache.len]
    lo = near = 0
    sel_valid = []
    for base, n_g, idx, s in sel:
        kk = idx.shape[1]
        got = pos[:, lo:lo + kk] - base
        near += compare_kept(got, idx, s)
        sel_valid.append((base, n_g, got.astype(np.int64), s))
        lo += kk
    # the cache holds the rounded kept rows, bit for bit
    for h in range(w.n_kv_heads):
        np.testing.assert_array_equal(_decoded(cache.k[h, :cache.len]), O.fp8_e4m3_round(k64[pos[h], h]))
        np.testing.assert_array_equal(_decoded(cache.v[h, :cache.len]), O.fp8_e4m3_round(v64[pos[h], h]))
    if near:                                                   # the oracle attends over the validated choice
        want = np.zeros_like(q64)
        for gi, (base, n_g, _, _) in enumerate(sel_valid):
            gk, gv, _ = O.gather_cache(k64, v64, sel_valid, gi, cache_format="fp8_e4m3")
            sl = slice(base, base + n_g)
            want[sl] = O.attend_group(q64[sl], k64[sl], v64[sl], gk, gv)
    assert_attn_close(to_f64(out), want, "bf16", f"fp8 cache whole path {rule}")
    # and it differs from the bf16-cache run where the cache is visible (the rounding is really applied)
    full, *_ = O.prefill_video(q64, k64, v64, qw64, w.n_frames, w.tokens_per_frame, w.group_frames, w.retention, rule)
    assert np.abs(full[w.group_tokens:] - want[w.group_tokens:]).max() > 1e-3


def test_e4m3_cache_is_refused_where_no_kernel_reads_it():
    l32 = B.make_layout(4, 2, 128, "f32")
    with pytest.raises(B.QPError) as e:
        c = B.Cache(B.make_layout(4, 2, 128, "bf16"), 8, fmt=FP8)
        B.topk_compact(l32, torch.zeros(2, 16, device=DEV), torch.zeros(16, 2, 128, device=DEV),
                       torch.zeros(16, 2, 128, device=DEV), 4, 0, c, None)
    assert e.value.status == B.QP_ERR_UNSUPPORTED
    layout = B.make_layout(4, 2, 128, "bf16")
    cache = B.Cache(layout, 8, fmt=FP8)
    cache.c.len = 8
    q = torch.zeros(4, 4, 128, dtype=torch.bfloat16, device=DEV)
    kv = torch.zeros(4, 2, 128, dtype=torch.bfloat16, device=DEV)
    B.select_attend_kernel(B.QP_ATTEND_SCALAR)
    try:
        with pytest.raises(B.QPError) as e:
            B.group_attend(layout, q, kv, kv, cache, torch.empty_like(q))
        assert e.value.status == B.QP_ERR_UNSUPPORTED
    finally:
        B.select_attend_kernel(B.QP_ATTEND_AUTO)
    bad = B.Cache(layout, 8)
    bad.c.format = 9
    with pytest.raises(B.QPError) as e:
        B.group_attend(layout, q, kv, kv, bad, torch.empty_like(q))
    assert e.value.status == B.QP_ERR_INVALID_ARG


def test_refused_layer_call_leaves_cache_and_indices_alone():
    """An 8-bit cache that the pinned kernel does not read, every token kept: nothing behind the cache's length is written."""
    dims = W.LayerDims(256, 512, 8, 2)
    layout = B.make_layout(8, 2, 128, "bf16")
    shape = B.make_layer_shape(256, 512, dims.rms_eps, dims.rope_theta, dims.mrope_section)
    wt = {k_: v_.to(DEV) for k_, v_ in W.make_decoder_layer(dims, 0, seed=3).items()}
    cache = B.Cache(layout, 40, fmt=FP8)
    for t in (cache.k, cache.v):
        t.view(torch.uint8).fill_(0x2a)
    cache.c.len = 5
    for n_t in (1, 16):
        x = W.make_hidden(1, n_t, 256, seed=8).to(DEV)
        kept = torch.full((2, n_t), -3, dtype=torch.int32, device=DEV)
        B.select_attend_kernel(B.QP_ATTEND_SCALAR)
        try:
            with pytest.raises(B.QPError) as e:
                B.layer_group(layout, shape, B.LayerWeights(**wt), x, W.text_positions(n_t, 90).to(DEV), 0, 70, None,
                              "key_norm_small", n_t, cache, torch.empty_like(x), kept, B.make_layer_workspace(layout, shape, n_t, 0))
        finally:
            B.select_attend_kernel(B.QP_ATTEND_AUTO)
        torch.cuda.synchronize()
        assert e.value.status == B.QP_ERR_UNSUPPORTED and cache.len == 5
        assert (cache.k.view(torch.uint8) == 0x2a).all() and (cache.v.view(torch.uint8) == 0x2a).all()
        assert (cache.pos == -1).all() and (kept == -3).all()


@pytest.mark.parametrize("n_g,h_q,h_kv,c", [(1, 28, 4, 1), (4, 28, 4, 31), (2, 64, 8, 32), (1, 28, 4, 33), (3, 6, 3, 255), (4, 28, 4, 257),
                                            (1, 28, 4, 2015), (1, 28, 4, 2016), (1, 8, 8, 16384), (4, 28, 4, 32700)])
def test_decode_over_an_e4m3_cache_at_block_edges(n_g, h_q, h_kv, c):
    """Cache blocks stay bytes in LDS, two per wavefront under way, the group's own block beside them: caches that end in and
    at a block, chunks whose last block is the group's own, in the first wavefront and in later ones, and wavefronts of
    none, one, two and more blocks."""
    test_group_attend_reads_an_e4m3_cache(n_g, h_q, h_kv, c)
