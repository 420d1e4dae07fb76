"""GPU parity of verify_layer and lm_head_logits against the CPU checker."""
import numpy as np
import pytest
import torch

from oracle import verify_oracle as O
from paper_2505_10526_amd import synth, binding
from helpers import DEV, to_dev, i32, round_up, pad_rows, assert_close, max_rel_err, v_blocked_to_rows, k_cache_to_rows

pytestmark = pytest.mark.gpu

TOL_BF16 = 2e-2
TOL_F32 = 5e-5      # fp32 path; sums of up to 688 products, fp32 accumulation in a different order


def cfg_of(s):
    return binding.LayerConfig(s.hidden, s.n_q_heads, s.n_kv_heads, s.head_dim, s.mlp, s.act, s.qkv_bias,
                               s.norm_eps, s.rope_theta, window=s.window)


def run_layer(s, B, Q, kv_len, n_img, seed, kv_std=1.0, compress=True, w_std=0.02):
    w = synth.layer_weights(s, seed, std=w_std)
    kv = synth.kv_cache(s, B, Q, kv_len, n_img, seed, std=kv_std, hot_keys=1)
    x = synth.hidden_states(s, B, Q, seed)
    pos = synth.positions(kv.kv_len, kv.n_img, Q, compress_image=compress)
    y_ref, k_ref, v_ref = O.verify_layer(s, w, x, pos, kv.k, kv.v, kv.kv_len)
    lm = round_up(kv.l_max, 32)
    kd = binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), s.dtype))
    vd = binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), s.dtype))
    wd = binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in w.items()})
    xd = to_dev(x, s.dtype)
    binding.verify_layer(cfg_of(s), wd, xd, i32(pos), kd, vd, i32(kv.kv_len))
    torch.cuda.synchronize()
    tol = TOL_BF16 if s.dtype == "bf16" else TOL_F32
    assert_close(xd.float().cpu().numpy(), y_ref, tol, "layer output")
    kg = k_cache_to_rows(kd).float().cpu().numpy()
    vg = v_blocked_to_rows(vd).float().cpu().numpy()
    for b in range(B):
        L = int(kv.kv_len[b])
        assert_close(kg[b, :, L:L + Q], k_ref[b, :, L:L + Q], tol, "appended keys")
        assert_close(vg[b, :, L:L + Q], v_ref[b, :, L:L + Q], tol, "appended values")
        # the cached prefix is untouched
        assert np.array_equal(kg[b, :, :L], kv.k[b, :, :L])
        assert np.array_equal(vg[b, :, :L], kv.v[b, :, :L])
    return xd


def test_tiny_fp32_layer():
    """Config 1: hidden 256, 4/2 heads, d=64, SwiGLU 688, fp32, KV prefix 256 (64 image rows)."""
    run_layer(synth.TINY, 1, 6, [256], [64], seed=0, kv_std=0.02)
    run_layer(synth.TINY, 2, 6, [256, 100], [64, 30], seed=1, kv_std=1.0, w_std=0.05)


def test_tiny_bf16_layer():
    run_layer(synth.TINY_BF16, 1, 6, [256], [64], seed=2, w_std=0.05)
    run_layer(synth.TINY_BF16, 3, 4, [40, 0, 95], [8, 0, 64], seed=3, w_std=0.05)


def test_qwen7b_layer_b1():
    """Config 2: one Qwen2.5-VL-7B-shaped layer, B=1, gamma=5, KV 1024 (700 image rows)."""
    run_layer(synth.QWEN7B, 1, 6, [1024], [700], seed=4)


def test_qwen7b_layer_b8_ragged():
    """Config 3's layer shape: B=8 (M=48), ragged lengths.  Shorter caches than 1024-2048 keep the
    checker's run time in seconds; the full lengths are covered by the attention tests."""
    rng = np.random.default_rng(5)
    run_layer(synth.QWEN7B, 8, 6, rng.integers(100, 400, 8), rng.integers(20, 100, 8), seed=5)


def test_qwen7b_layer_b8_full_lengths():
    """Config 3's layer at its real sizes: B=8, gamma=5, per-sequence lengths U[1024, 2048] with 256-1024
    image rows -- the launch configuration bench.py times (same tile counts, K slabs and attention splits)."""
    rng = np.random.default_rng(0)
    run_layer(synth.QWEN7B, 8, 6, rng.integers(1024, 2049, 8), rng.integers(256, 1025, 8), seed=10)


def test_gemma12b_layer_b4_full_length():
    """Config 4 at its real sizes: B=4, KV length 4096 with 256 leading image rows."""
    run_layer(synth.GEMMA12B, 4, 6, [4096] * 4, [256] * 4, seed=11)


def test_qwen7b_layer_max_rows():
    """The largest row count the bf16 kernels take: B=8, gamma=7 -> M = 64 rows (four 16-row tiles),
    56 stacked query rows per KV head."""
    rng = np.random.default_rng(15)
    run_layer(synth.QWEN7B, 8, 8, rng.integers(40, 300, 8), rng.integers(8, 40, 8), seed=15)


def test_single_row_and_single_sequence():
    """Degenerate sizes: one query position (plain decoding), one sequence."""
    run_layer(synth.TINY_BF16, 1, 1, [33], [5], seed=16, w_std=0.05)
    run_layer(synth.TINY, 1, 1, [0], [0], seed=17, w_std=0.05)
    run_layer(synth.QWEN7B, 1, 1, [70], [20], seed=18)


def test_gemma12b_layer_b4():
    """Config 4's layer: hidden 3840, 16/8 heads, d=256, GeGLU 15360, no bias, B=4 (M=24)."""
    run_layer(synth.GEMMA12B, 4, 6, [300, 256, 50, 411], [256, 200, 10, 256], seed=6)


@pytest.mark.parametrize("shape,M", [(synth.TINY, 6), (synth.TINY_BF16, 6), (synth.TINY_BF16, 48)])
def test_lm_head_small(shape, M):
    lw = synth.lm_head_weights(shape, 7, std=0.05)
    x = synth.normal((M, shape.hidden), 1.0, 7, 60, dtype=shape.dtype)
    ref = O.lm_head_logits(x, lw["final_norm"], lw["w_lm"], shape.norm_eps)
    got = binding.lm_head_logits(to_dev(x, shape.dtype), to_dev(lw["final_norm"], shape.dtype),
                                 binding.weight_pack(to_dev(lw["w_lm"], shape.dtype)), shape.norm_eps)
    assert_close(got.cpu().numpy(), ref, TOL_BF16 if shape.dtype == "bf16" else TOL_F32, "logits")
    ref2 = O.lm_head_logits(x, None, lw["w_lm"], shape.norm_eps)
    got2 = binding.lm_head_logits(to_dev(x, shape.dtype), None, binding.weight_pack(to_dev(lw["w_lm"], shape.dtype)))
    assert_close(got2.cpu().numpy(), ref2, TOL_BF16 if shape.dtype == "bf16" else TOL_F32, "logits no norm")


@pytest.mark.parametrize("shape,M", [(synth.QWEN7B, 6), (synth.QWEN7B, 48), (synth.GEMMA12B, 24)])
def test_lm_head_full_vocab(shape, M):
    """lm_head at the real vocabulary (152064 / 262144 rows)."""
    lw = synth.lm_head_weights(shape, 8)
    x = synth.normal((M, shape.hidden), 1.0, 8, 60, dtype=shape.dtype)
    ref = O.lm_head_logits(x, lw["final_norm"], lw["w_lm"], shape.norm_eps)
    got = binding.lm_head_logits(to_dev(x, shape.dtype), to_dev(lw["final_norm"], shape.dtype),
                                 binding.weight_pack(to_dev(lw["w_lm"], shape.dtype)), shape.norm_eps)
    assert_close(got.cpu().numpy(), ref, TOL_BF16, "logits")


def run_stack(s, n_layers, B, Q, kv_len, n_img, seed, w_std=0.02):
    """n_layers layers through ONE massv_verify_layers call against the checker's layer-by-layer chain."""
    ws_h = [synth.layer_weights(s, seed, layer=l, std=w_std) for l in range(n_layers)]
    kvs = [synth.kv_cache(s, B, Q, kv_len, n_img, seed, layer=l, hot_keys=1) for l in range(n_layers)]
    x = synth.hidden_states(s, B, Q, seed)
    pos = synth.positions(kvs[0].kv_len, kvs[0].n_img, Q, compress_image=True)
    y_ref = x
    k_refs, v_refs = [], []
    for l in range(n_layers):
        y_ref, k_ref, v_ref = O.verify_layer(s, ws_h[l], y_ref, pos, kvs[l].k, kvs[l].v, kvs[l].kv_len)
        k_refs.append(k_ref); v_refs.append(v_ref)
    lm = round_up(kvs[0].l_max, 32)
    kds = [binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), s.dtype)) for kv in kvs]
    vds = [binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), s.dtype)) for kv in kvs]
    wds = [binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in w.items()}) for w in ws_h]
    stack = binding.LayerStack(wds, kds, vds)
    xd = to_dev(x, s.dtype)
    binding.verify_layers(cfg_of(s), stack, xd, i32(pos), i32(kvs[0].kv_len), lm)
    torch.cuda.synchronize()
    tol = TOL_BF16 if s.dtype == "bf16" else TOL_F32 * n_layers
    assert_close(xd.float().cpu().numpy(), y_ref, tol, "stack output")
    for l in range(n_layers):
        kg = k_cache_to_rows(kds[l]).float().cpu().numpy()
        vg = v_blocked_to_rows(vds[l]).float().cpu().numpy()
        for b in range(B):
            L = int(kvs[l].kv_len[b])
            assert_close(kg[b, :, L:L + Q], k_refs[l][b, :, L:L + Q], tol, f"layer {l} appended keys")
            assert_close(vg[b, :, L:L + Q], v_refs[l][b, :, L:L + Q], tol, f"layer {l} appended values")


def test_layer_stack_tiny():
    run_stack(synth.TINY, 3, 2, 6, [256, 100], [64, 30], seed=12, w_std=0.05)
    run_stack(synth.TINY_BF16, 3, 2, 6, [256, 100], [64, 30], seed=13, w_std=0.05)


def test_layer_stack_qwen7b_two_layers():
    """Two Qwen2.5-VL-7B-shaped layers, B=8 (M=48), in one call: the fused norm between layers."""
    rng = np.random.default_rng(14)
    run_stack(synth.QWEN7B, 2, 8, 6, rng.integers(100, 400, 8), rng.integers(20, 100, 8), seed=14)


CHAIN_LAYERS = 28


@pytest.fixture(scope="module")
def chain(request):
    """The headline workload at its real depth and sizes: 28 Qwen2.5-VL-7B-shaped layers, B=8, gamma=5 (M=48),
    per-sequence lengths U[1024, 2048] with 256-1024 image rows, every layer with its own weights and cache.
    Three runs against the checker's layer-by-layer chain:
      stepwise   layer l alone, fed the checker's output of layer l-1 (identical inputs on both sides);
      sequential the library's own output fed forward, one massv_verify_layer call per layer;
      one_call   the same through ONE massv_verify_layers call over all 28 layers.
    The host holds one layer's weights at a time (the next layer's are drawn while the checker works)."""
    from concurrent.futures import ThreadPoolExecutor
    capman = request.config.pluginmanager.getplugin("capturemanager")

    def say(msg):                                    # progress lines from the work itself: this runs for minutes
        with capman.global_and_fixture_disabled():
            print(msg, flush=True)

    s, N, B, Q, seed = synth.QWEN7B, CHAIN_LAYERS, 8, 6, 50
    rng = np.random.default_rng(0)
    kv_len, n_img = rng.integers(1024, 2049, B), rng.integers(256, 1025, B)
    x = synth.hidden_states(s, B, Q, seed)
    pos = synth.positions(kv_len, n_img, Q)
    lm = round_up(int(kv_len.max()) + Q, 32)
    pool = ThreadPoolExecutor(1)
    draw = lambda l: (synth.layer_weights(s, seed, layer=l, threads=6),
                      synth.kv_cache(s, B, Q, kv_len, n_img, seed, layer=l, hot_keys=1))
    nxt = pool.submit(draw, 0)
    wds, kds, vds = [], [], []
    y_ref, x_seq = x, to_dev(x, s.dtype)
    r = dict(stepwise=[], sequential=[], ref_max=[], layers=N)
    kvl_d, pos_d = i32(kv_len), i32(pos)
    for l in range(N):
        w, kv = nxt.result()
        if l + 1 < N:
            nxt = pool.submit(draw, l + 1)
        kds.append(binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), s.dtype)))
        vds.append(binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), s.dtype)))
        wds.append(binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in w.items()}))
        x_step = to_dev(y_ref, s.dtype)              # the checker's previous output: on the bf16 grid already
        y_ref, _, _ = O.verify_layer(s, w, y_ref, pos, kv.k, kv.v, kv.kv_len)
        del w, kv
        binding.verify_layer(cfg_of(s), wds[l], x_step, pos_d, kds[l], vds[l], kvl_d)
        binding.verify_layer(cfg_of(s), wds[l], x_seq, pos_d, kds[l], vds[l], kvl_d)     # rewrites the same cache rows
        torch.cuda.synchronize()
        for name, t in (("stepwise", x_step), ("sequential", x_seq)):
            got = t.float().cpu().numpy()
            assert np.all(np.isfinite(got)), f"layer {l} ({name}): non-finite output"
            r[name].append(max_rel_err(got, y_ref))
        r["ref_max"].append(float(np.max(np.abs(y_ref))))
        if l % 4 == 3:
            say(f"[chain] layer {l + 1}/{N}: stepwise {r['stepwise'][-1]:.2e}, sequential {r['sequential'][-1]:.2e}, "
                f"max |ref| {r['ref_max'][-1]:.1f}")
    pool.shutdown()
    stack = binding.LayerStack(wds, kds, vds)
    xd = to_dev(x, s.dtype)
    binding.verify_layers(cfg_of(s), stack, xd, pos_d, kvl_d, lm)      # rows kv_len .. kv_len+Q-1 are rewritten first
    torch.cuda.synchronize()
    r["one_call"] = max_rel_err(xd.float().cpu().numpy(), y_ref)
    say("[chain] stepwise error of each layer (max |err| / max |ref|): " + " ".join(f"{e:.2e}" for e in r["stepwise"]))
    say("[chain] sequential error after each layer: " + " ".join(f"{e:.2e}" for e in r["sequential"]))
    say("[chain] max |ref| after each layer: " + " ".join(f"{m:.1f}" for m in r["ref_max"]))
    say(f"[chain] one call over {N} layers: {r['one_call']:.3e}")
    return r


def test_every_layer_of_the_full_depth_stack_meets_the_bound(chain):
    """Each of the 28 layers, at the activation statistics of its own depth and with identical inputs on both
    sides, is within the bf16 bound."""
    assert max(chain["stepwise"]) <= TOL_BF16, chain["stepwise"]


def test_full_depth_chain_stays_consistent(chain):
    """Both sides feeding their own output forward: the library rounds the operands of every projection to bf16,
    the checker rounds only what the step stores, so the two drift apart with depth.  This is a guard against a
    defect that compounds (a wrong residual path, a stale workspace between layers), not the parity bound: the
    one call over all layers must agree with the layer-at-a-time run (same arithmetic, same inputs up to the fused
    norm between layers) and the drift must stay of the size that per-layer errors adding up explain."""
    seq, one = chain["sequential"][-1], chain["one_call"]
    assert abs(one - seq) <= 1e-2, (one, seq)
    budget = float(np.sum(np.array(chain["stepwise"]) * np.array(chain["ref_max"])) / chain["ref_max"][-1])
    assert one <= budget, (one, budget)


@pytest.mark.xfail(strict=False, reason="free-running 28-layer chain: bf16 operand rounding compounds with depth; "
                                        "the measured curve is reported, the bound is not raised")
def test_full_depth_chain_meets_the_single_layer_bound(chain):
    assert chain["one_call"] <= TOL_BF16, chain["one_call"]


def test_layer_repeatable_bits():
    s = synth.QWEN7B
    w = binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in synth.layer_weights(s, 9).items()})
    kv = synth.kv_cache(s, 2, 6, [64, 200], [10, 50], 9, junk_tail=False)
    pos = i32(synth.positions(kv.kv_len, kv.n_img, 6))
    outs = []
    for _ in range(2):
        lm = round_up(kv.l_max, 32)
        kd = binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), s.dtype))
        vd = binding.v_cache_pack(to_dev(np.nan_to_num(pad_rows(kv.v, lm)), s.dtype))
        x = to_dev(synth.hidden_states(s, 2, 6, 9), s.dtype)
        binding.verify_layer(cfg_of(s), w, x, pos, kd, vd, i32(kv.kv_len))
        outs.append((x.clone(), kd.clone(), vd.clone()))
    for a, b in zip(*outs):
        assert torch.equal(torch.nan_to_num(a.float()), torch.nan_to_num(b.float()))


@pytest.mark.parametrize("s", [synth.TINY, synth.TINY_BF16], ids=["f32", "bf16"])
def test_embed_tokens_gathers_rows(s):
    table = synth.embedding_table(s, 5)
    tokens = np.array([0, s.vocab - 1, 17, 17, -3, s.vocab, 1234], dtype=np.int32)
    ref = O.embed_tokens(table, tokens)
    got = binding.embed_tokens(to_dev(table, s.dtype), i32(tokens))
    assert np.array_equal(got.float().cpu().numpy(), ref)


# ---------------------------------------------------------------------------
# layer variants of the Gemma 3 targets: sliding window, query/key head norms, block-output norms
# ---------------------------------------------------------------------------
def test_gemma_style_tiny_layers():
    run_layer(synth.TINY_GEMMA, 2, 6, [256, 100], [64, 30], seed=31, w_std=0.05)
    run_layer(synth.TINY_GEMMA_BF16, 3, 4, [140, 0, 95], [8, 0, 64], seed=32, w_std=0.05)


def test_gemma12b_local_layer():
    """One Gemma3-12B-shaped sliding-window layer: d=256 heads with query/key norms, window 1024 over KV 4096,
    block-output norms, tanh-GELU MLP."""
    run_layer(synth.GEMMA12B_LOCAL, 4, 6, [4096, 3000, 1024, 500], [256, 256, 256, 100], seed=33)


def test_each_gemma_variant_alone():
    """Each optional step switched on by itself (a step wired to the wrong switch fails here)."""
    import dataclasses
    base = synth.TINY_BF16
    for kw in (dict(window=20), dict(qk_norm=True), dict(post_norms=True)):
        run_layer(dataclasses.replace(base, **kw), 2, 6, [100, 37], [30, 5], seed=34, w_std=0.05)


def test_layer_stack_interleaves_local_and_global_layers():
    """Four layers in one call, windows (24, 24, 0, 24) and rotary bases (1e4, 1e4, 1e6, 1e4) given per layer."""
    import dataclasses
    for base in (synth.TINY_GEMMA, synth.TINY_GEMMA_BF16):
        windows, thetas = [24, 24, 0, 24], [1e4, 1e4, 1e6, 1e4]
        shapes = [dataclasses.replace(base, window=w, rope_theta=t) for w, t in zip(windows, thetas)]
        B, Q, seed = 2, 6, 35
        ws_h = [synth.layer_weights(s, seed, layer=l, std=0.05) for l, s in enumerate(shapes)]
        kvs = [synth.kv_cache(base, B, Q, [200, 61], [64, 30], seed, layer=l, hot_keys=1) for l in range(4)]
        x = synth.hidden_states(base, B, Q, seed)
        pos = synth.positions(kvs[0].kv_len, kvs[0].n_img, Q, compress_image=True)
        y_ref = x
        for l in range(4):
            y_ref, _, _ = O.verify_layer(shapes[l], ws_h[l], y_ref, pos, kvs[l].k, kvs[l].v, kvs[l].kv_len)
        lm = round_up(kvs[0].l_max, 32)
        kds = [binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), base.dtype)) for kv in kvs]
        vds = [binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), base.dtype)) for kv in kvs]
        wds = [binding.pack_layer_weights({k: (None if v is None else to_dev(v, base.dtype)) for k, v in w.items()}) for w in ws_h]
        stack = binding.LayerStack(wds, kds, vds, windows=windows, rope_thetas=thetas)
        xd = to_dev(x, base.dtype)
        binding.verify_layers(cfg_of(base), stack, xd, i32(pos), i32(kvs[0].kv_len), lm)
        torch.cuda.synchronize()
        tol = TOL_BF16 if base.dtype == "bf16" else TOL_F32 * 4
        assert_close(xd.float().cpu().numpy(), y_ref, tol, "interleaved stack output")


# ---------------------------------------------------------------------------
# vocabulary projection fused with the temperature-0 accept rule (no logits written)
# ---------------------------------------------------------------------------
def greedy_case(s, B, gamma, seed, head_std=0.05, duplicate_rows=False):
    Q = gamma + 1
    head = synth.lm_head_weights(s, seed, std=head_std)
    if duplicate_rows:                                   # every logit appears twice: ties must go to the lower token id
        head["w_lm"][s.vocab // 2:] = head["w_lm"][: s.vocab // 2]
    x = synth.hidden_states(s, B, Q, seed)
    logits = O.lm_head_logits(x.reshape(B * Q, -1), head["final_norm"], head["w_lm"], s.norm_eps).reshape(B, Q, -1)
    # drafts: the checker's arg-max for a random-length prefix of every sequence, something else after it
    rng = np.random.default_rng(seed)
    drafts = np.argmax(logits[:, :gamma], axis=-1).astype(np.int32)
    for b in range(B):
        keep = int(rng.integers(0, gamma + 1))
        if keep < gamma:
            drafts[b, keep] = (drafts[b, keep] + 1 + int(rng.integers(0, s.vocab - 1))) % s.vocab
    xd = to_dev(x, s.dtype)
    norm, w = to_dev(head["final_norm"], s.dtype), binding.weight_pack(to_dev(head["w_lm"], s.dtype))
    return xd, norm, w, i32(drafts), logits, drafts


@pytest.mark.parametrize("s,B,gamma,dup", [(synth.TINY_BF16, 3, 5, False), (synth.TINY_BF16, 8, 5, True), (synth.TINY_BF16, 1, 0, False),
                                           (synth.TINY_BF16, 4, 15, False), (synth.QWEN7B, 8, 5, False), (synth.QWEN7B, 2, 3, True)],
                         ids=["tiny", "tiny-ties", "tiny-gamma0", "tiny-gamma15", "qwen7b", "qwen7b-ties"])
def test_lm_head_greedy_accept(s, B, gamma, dup):
    xd, norm, w, dtok, logits_ref, drafts = greedy_case(s, B, gamma, seed=41 + B + gamma, duplicate_rows=dup)
    n_f, out_f = binding.lm_head_greedy_accept(xd, norm, w, dtok if gamma else None, s.norm_eps)
    # the two separate calls on the same inputs: identical integers, ties included
    lg = binding.lm_head_logits(xd, norm, w, s.norm_eps).reshape(B, gamma + 1, -1)
    n_2, out_2 = binding.spec_accept(lg, None, dtok if gamma else None, None, 0.0)
    torch.cuda.synchronize()
    assert torch.equal(n_f, n_2) and torch.equal(out_f, out_2)
    if dup:
        assert int(out_f.max()) < s.vocab // 2
        return
    # the checker, wherever its arg-max is clear of the bf16 path's error
    top = np.sort(logits_ref, axis=-1)[..., -2:]
    clear = (top[..., 1] - top[..., 0]) > 5e-3 * np.max(np.abs(logits_ref))
    n_o, out_o, _ = O.spec_accept(logits_ref, None, drafts, None, 0.0)
    for b in range(B):
        if clear[b].all():
            assert int(n_f[b]) == n_o[b] and np.array_equal(out_f[b].cpu().numpy(), out_o[b])
    if gamma <= 5:
        assert clear.all(axis=1).sum() >= 1                 # the comparison with the checker is not vacuous
    if gamma >= 5 and B >= 3:
        assert len(set(n_o.tolist())) > 1


# ---------------------------------------------------------------------------
# vocabulary projection + accept rule in one call at T > 0 (row statistics formed in the projection's epilogue)
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("s,B,gamma,T,noise", [(synth.TINY_BF16, 3, 5, 1.0, 0.3), (synth.TINY_BF16, 1, 0, 0.7, 0.3),
                                               (synth.TINY_BF16, 4, 15, 1.0, 0.1), (synth.QWEN7B, 8, 5, 1.0, 0.5),
                                               (synth.QWEN7B, 8, 5, 0.7, 1.5), (synth.QWEN7B, 2, 3, 0.0, 1.0)],
                         ids=["tiny", "tiny-gamma0", "tiny-gamma15", "qwen7b", "qwen7b-T0.7", "qwen7b-T0"])
def test_lm_head_accept_one_call(s, B, gamma, T, noise):
    Q, seed = gamma + 1, 70 + B + gamma
    T = float(np.float32(T))
    head = synth.lm_head_weights(s, seed, std=0.05)
    xd = to_dev(synth.hidden_states(s, B, Q, seed), s.dtype)
    norm, w = to_dev(head["final_norm"], s.dtype), binding.weight_pack(to_dev(head["w_lm"], s.dtype))
    lg = binding.lm_head_logits(xd, norm, w, s.norm_eps)                   # the separate calls: logits first
    tl = lg.cpu().numpy().reshape(B, Q, -1)
    a = synth.accept_inputs(B, gamma, s.vocab, T, seed, noise_std=noise, target_logits=tl)   # drafts from the GPU's own logits
    dl = torch.from_numpy(a.draft_logits).cuda() if gamma else None
    dt = torch.from_numpy(a.draft_tokens).cuda() if gamma else None
    u = torch.from_numpy(a.uniforms).cuda()
    n_2, out_2 = binding.spec_accept(lg.view(B, Q, -1), dl if T > 0 else None, dt, u if T > 0 else None, T)
    n_f, out_f, lg_f = binding.lm_head_accept(xd, norm, w, dl, dt, u if T > 0 else None, T, s.norm_eps)
    torch.cuda.synchronize()
    if T > 0:
        assert torch.equal(lg_f, lg)                                        # the same projection arithmetic
    # the checker on the same fp32 logits
    n_o, out_o, margin = O.spec_accept(tl, a.draft_logits, a.draft_tokens, a.uniforms, T)
    clear = np.all(margin > 1e-5, axis=1)
    assert clear.sum() >= 0.5 * B, "pick another seed: too few decisions clear of rounding"
    for b in range(B):
        if clear[b]:
            for n_g, out_g in ((n_2, out_2), (n_f, out_f)):
                assert int(n_g[b]) == n_o[b] and np.array_equal(out_g[b].cpu().numpy(), out_o[b]), (b, out_g[b], out_o[b])
    if gamma >= 5 and T > 0:
        assert n_o.max() > 0                                                # drafts do get accepted in this case


# fp32 layers whose widths reach the corners of the f32 kernels: feature counts that no 16-byte load divides, head
# dimensions that leave threads over or take a workgroup whole, K of less than a load per lane and of more than four
# steps, rows that end inside a group of eight, a window that starts inside a block
F32_SHAPES = [(synth.LayerShape(90, 3, 1, 6, 35, 64, synth.ACT_SILU, True, dtype="f32"), 3, 3),
              (synth.LayerShape(132, 2, 2, 100, 1300, 64, synth.ACT_GELU_TANH, False, dtype="f32"), 1, 9),
              (synth.LayerShape(1284, 2, 1, 256, 68, 64, synth.ACT_SILU, True, dtype="f32", window=45), 2, 4),
              (synth.LayerShape(64, 4, 2, 32, 64, 64, synth.ACT_SILU, True, dtype="f32", window=7, post_norms=True), 5, 5)]


@pytest.mark.parametrize("s,B,Q", F32_SHAPES, ids=["odd", "d100", "d256_window", "post_norms"])
def test_fp32_layer_widths(s, B, Q):
    run_layer(s, B, Q, [(37 * b + 11) % 300 for b in range(B)], [3] * B, seed=40 + Q, w_std=0.05)


def test_fp32_layer_many_keys_and_unaligned_rows():
    """More keys than one tile of 256, and every operand one float off a multiple of 16 bytes (a slice of a larger
    buffer): the same bits."""
    s, B, Q, seed = synth.TINY, 2, 6, 45
    w = synth.layer_weights(s, seed, std=0.05)
    kv = synth.kv_cache(s, B, Q, [900, 513], [64, 30], seed, hot_keys=2)
    x, pos = synth.hidden_states(s, B, Q, seed), synth.positions(kv.kv_len, kv.n_img, Q)
    y_ref, _, _ = O.verify_layer(s, w, x, pos, kv.k, kv.v, kv.kv_len)
    lm = round_up(kv.l_max, 32)
    got = []
    for off in (0, 1):
        def put(a):
            t = to_dev(a, "f32")
            buf = torch.empty(t.numel() + 4, dtype=t.dtype, device=t.device)
            v = buf[off:off + t.numel()].view(t.shape)
            v.copy_(t)
            return v
        kd = put(pad_rows(kv.k, lm))
        vd = put(binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), "f32")).cpu().numpy())
        xd = put(x)
        binding.verify_layer(cfg_of(s), {k: (None if v is None else put(v)) for k, v in w.items()}, xd, i32(pos), kd, vd, i32(kv.kv_len))
        torch.cuda.synchronize()
        assert_close(xd.cpu().numpy(), y_ref, TOL_F32, f"offset {off}")
        got.append((xd, kd, vd))
    assert torch.equal(got[0][0], got[1][0])
    for a, b in zip(got[0][1:], got[1][1:]):                          # caches: bits, NaN in rows past the end
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("M,H,V", [(48, 512, 40960), (64, 160, 20512), (16, 64, 65600), (48, 512, 81328), (8, 96, 81328), (32, 64, 81328),
                                   (33, 544, 82000), (1, 32, 40976), (17, 96, 45072), (48, 96, 122240), (49, 32, 70000), (64, 32, 113888)])
def test_vocabulary_projection_in_shares(M, H, V):
    """Vocabularies that take a workgroup one (the first), two (the next five), three and up to seven shares (the last), most of
    unequal size, at every number of row tiles and of tile slots and down to hidden sizes that leave a wave without a
    single step (plain logits of few rows with empty slots go by a workgroup a share): logits against float64 (fp32 sums of H
    products), and the greedy rule's token, which carries its maximum across shares, against the arg-max of those logits."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M + V)
    x = torch.randn(M, H, generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn(V, H, generator=g, device="cuda").to(torch.bfloat16)
    wp = binding.weight_pack(w)
    got = binding.lm_head_logits(x, None, wp)
    tokens = binding.lm_head_greedy_accept(x.view(M, 1, H), None, wp, None)[1]
    ref = x.double() @ w.double().T
    torch.cuda.synchronize()
    assert_close(got.cpu().numpy(), ref.cpu().numpy(), 1e-5, "logits")
    assert torch.equal(tokens.view(-1).long(), got.argmax(-1))
    for T in (0.7, 1.0):
        u = torch.rand(M, 1, generator=g, device="cuda")
        _, drawn, logits = binding.lm_head_accept(x.view(M, 1, H), None, wp, None, None, u, T)
        apart = binding.spec_accept(got.view(M, 1, V), None, None, u, T)[1]
        torch.cuda.synchronize()
        assert torch.equal(logits, got)
        assert (drawn == apart).float().mean() >= 0.9              # a draw within rounding of a boundary may differ


def test_vocabulary_statistics_carried_across_shares_keep_small_terms():
    """The records (maximum, its column, sum of exp(x - maximum)) that the sampled projection leaves at the head of its
    workspace, behind the packed rows: one per workgroup, 256 where each works off several shares.  Four tokens in forty have
    logit 0, the others -17.25, so that a sum kept in fp32 takes on 4.0 and loses every small term after it (2.9e-7 of the
    total); the bound is the fp32 error of those terms, 2e-6 of that share."""
    H, V, T = 32, 152064, 1.0
    w = torch.zeros(V, H, device="cuda", dtype=torch.bfloat16)
    w[:, 0] = -17.25
    w[torch.arange(V, device="cuda") % 40 < 4, 0] = 0.0
    x = torch.zeros(1, 1, H, device="cuda", dtype=torch.bfloat16)
    x[..., 0] = 1.0
    ws = torch.full((binding.load().massv_lm_head_accept_workspace(1, 0, H, V, binding.BF16),), 255, dtype=torch.uint8, device="cuda")
    _, _, logits = binding.lm_head_accept(x, None, binding.weight_pack(w), None, None, torch.full((1, 1), 0.5, device="cuda"), T, ws=ws)
    torch.cuda.synchronize()
    head = 16 * H * 2
    rec = ws[head:head + 256 * 16].cpu().numpy().view(np.dtype([("m", "<f4"), ("arg", "<i4"), ("s", "<f8")]))
    assert np.all(rec["m"] == 0.0) and len(set(rec["arg"].tolist())) == 256
    n0 = sum(n % 40 < 4 for n in range(V))
    want = n0 + (V - n0) * np.exp(-17.25)
    assert abs(rec["s"].sum() / want - 1) <= 2e-6 * 2.9e-7 + 1e-12
    assert torch.equal(logits[0], w[:, 0].float())


@pytest.mark.parametrize("rising", [False, True], ids=["equal", "rising"])
@pytest.mark.parametrize("M", [5, 16, 17, 48, 64])
def test_vocabulary_maximum_that_never_and_always_moves(M, rising):
    """Statistics of rows whose logits are all equal (the first column holds the maximum from the start) and of rows that rise from each tile of 16
    columns to the next (every piece of every share brings a new maximum), at one to four row tiles and three shares a workgroup: the greedy
    token, and at T = 1 the same integers as from the logits themselves."""
    H, V = 64, 81328
    g = torch.Generator(device="cuda")
    g.manual_seed(M)
    x = torch.rand(M, H, generator=g, device="cuda").to(torch.bfloat16) + 0.25            # positive: a row's logits follow the weights
    w = torch.zeros(V, H, device="cuda")
    if rising:                # tile t = 72 c + f: c and f are exact in bf16, and 72 steps of the fine column are less than one of the coarse ones
        t = torch.arange(V, device="cuda") // 16
        w[:, 0], w[:, 1:] = (t % 72) / 512, (t // 72)[:, None] / 64
    else:
        w[:] = 1
    w = w.to(torch.bfloat16).contiguous()
    wp = binding.weight_pack(w)
    n, tok = binding.lm_head_greedy_accept(x.view(M, 1, H), None, wp, None)
    logits = binding.lm_head_logits(x, None, wp)
    assert torch.equal(tok.view(-1).long(), logits.argmax(-1)) and (rising or not tok.any())
    top = logits.view(M, V // 16, 16).amax(-1)
    assert (top[:, 1:] > top[:, :-1]).all() == rising
    u = torch.rand(M, 1, generator=g, device="cuda") * 0.999
    n1, t1, l1 = binding.lm_head_accept(x.view(M, 1, H), None, wp, None, None, u, 1.0)
    n2, t2 = binding.spec_accept(logits.view(M, 1, V), None, None, u, 1.0)
    assert torch.equal(l1.view(M, V), logits) and torch.equal(n1, n2) and torch.equal(t1, t2)


@pytest.mark.parametrize("M", [16, 17, 32, 33])
@pytest.mark.parametrize("V", [4096, 32000, 50000, 81328])
def test_logits_past_the_cache_and_through_it(M, V):
    """Two row tiles with one share a workgroup stay in L2 as plain logits and go past it beside the accept rule, and with more shares (or one row tile
    more) both go past it: the same bits, and against float64 within fp32 sums of H products (sqrt(H) roundings of 2^-24, four times)."""
    H = 256
    g = torch.Generator(device="cuda")
    g.manual_seed(M + V)
    x, w = (torch.randn(n, H, generator=g, device="cuda").to(torch.bfloat16) for n in (M, V))
    room = torch.full((M * V + 4096,), 7.0, device="cuda")
    wp = binding.weight_pack(w)
    logits = binding.lm_head_logits(x, None, wp, out=room[:M * V].view(M, V))
    assert (room[M * V:] == 7).all()
    ref = x.double() @ w.double().T
    assert (logits.double() - ref).abs().max() / ref.abs().max() <= 4 * H ** 0.5 * 2.0 ** -24
    assert torch.equal(binding.lm_head_accept(x.view(M, 1, H), None, wp, None, None, torch.full((M, 1), 0.5, device="cuda"), 1.0)[2].view(M, V), logits)


@pytest.mark.parametrize("H", [7, 64, 68, 252, 256, 260, 512, 700, 1028])
@pytest.mark.parametrize("M,V", [(1, 100), (2, 4097), (3, 33), (4, 5000), (5, 70), (8, 4096), (9, 4100), (17, 64)])
def test_fp32_logits_rows_and_widths(M, V, H):
    """1, 2, 4 or 8 rows a wave, single or 16-byte loads with one to four steps in flight, the norm in the product or ahead
    of it, against float64; the bound is the order of fp32 sums of H products (sqrt(H) roundings of 2^-24, four times)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(M * H + V)
    x, w = torch.randn(M, H, generator=g, device="cuda"), torch.randn(V, H, generator=g, device="cuda")
    gain = 1 + 0.1 * torch.randn(H, generator=g, device="cuda")
    for norm in (None, gain):
        got = binding.lm_head_logits(x, norm, w, 1e-6)
        y = x.double()
        if norm is not None:
            y = y / (y.square().mean(-1, keepdim=True) + 1e-6).sqrt() * norm.double()
        ref = y @ w.double().T
        err = (got.double() - ref).abs().max() / ref.abs().max()
        assert err <= 4 * H ** 0.5 * 2.0 ** -24, (norm is not None, err)


@pytest.mark.parametrize("s", [synth.TINY, synth.TINY_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("window", [0, 40])
def test_lengths_that_cannot_be_leave_the_caches_alone(s, window):
    """kv_len is read on the device; lengths at and past the end of the cache, up to the largest integer (where adding a
    row's number overflows), drop every new row: guard rows around the caches keep their bits.  Results are unspecified."""
    B, Q, l_max, dt = 4, 6, 64, (torch.float32 if s.dtype == "f32" else torch.bfloat16)
    kv_len = i32([64, 2 ** 31 - 1, 2 ** 31 - 3, 1 << 30])
    n = B * s.n_kv_heads * l_max * s.head_dim

    def guarded():
        buf = torch.randn(n + 2 * 65536, device="cuda").to(dt)
        return buf, buf[65536:65536 + n]
    (kb, k), (vb, v) = guarded(), guarded()
    k, v = k.view(B, s.n_kv_heads, l_max, s.head_dim), v.view(B, s.n_kv_heads, l_max // 32, s.head_dim, 32)
    before = kb.clone(), vb.clone()
    w = binding.pack_layer_weights({name: None if a is None else to_dev(a, s.dtype) for name, a in synth.layer_weights(s, 3, std=0.05).items()})
    pos = i32(np.arange(B * Q).reshape(B, Q))
    cfg = cfg_of(s)
    cfg.window = window
    binding.verify_layer(cfg, w, torch.randn(B, Q, s.hidden, device="cuda").to(dt), pos, k, v, kv_len)
    binding.verify_attention(torch.randn(B, Q, s.n_q_heads, s.head_dim, device="cuda").to(dt), k, v, kv_len, window=window)
    n_new = i32([Q] * B)
    qkv = torch.randn(B, Q, (s.n_q_heads + 2 * s.n_kv_heads) * s.head_dim, device="cuda").to(dt)
    q = binding.rope_append(qkv, pos, kv_len, n_new, k, v, s.n_q_heads, 1e6)
    o = binding.prefill_attention(torch.randn_like(q), k, v, kv_len, n_new, window=window)
    torch.cuda.synchronize()
    assert torch.equal(kb, before[0]) and torch.equal(vb, before[1])
    assert not q.any() and not o.any()


# ---------------------------------------------------------------------------
# projections that carry what follows them (whole K per workgroup): every kind, at the edges of its row range
# ---------------------------------------------------------------------------
WHOLE_SHAPES = {
    # q/k/v 256 -> 16 features x 256 workgroups at most; down has an odd number of 32-wide steps (352), O an even one
    "eight_pairs_odd_k": synth.LayerShape(128, 2, 1, 64, 352, 4096),
    # q/k/v 4608 features: 16 pairs a workgroup; gate / up 2 tiles a workgroup, one of them in some
    "sixteen_pairs": synth.LayerShape(96, 28, 4, 128, 2080, 4096, qkv_bias=False),
    # d = 256; hidden 2080: O and down by 16 features at any number of rows (260 workgroups of 8); gate / up 4 tiles
    "wide_rows": synth.LayerShape(2080, 2, 1, 256, 6176, 4096, synth.ACT_GELU_TANH, False),
}


@pytest.mark.parametrize("B,Q", [(1, 1), (8, 1), (9, 1), (4, 4), (17, 1), (8, 4), (11, 3), (8, 6), (7, 7)])
@pytest.mark.parametrize("name", WHOLE_SHAPES)
def test_projections_with_what_follows(name, B, Q):
    """Two layers in one call (rows * gains and their sums of squares handed from each projection to the next): 1, 8 | 9, 16 | 17,
    32 | 33, 48 | 49 rows."""
    # weights of unit gain: the bound is one layer's, and 0.05 at 2080 inputs (gain 2.3) amplifies the first layer's rounding
    # past it in the second (2.4e-2 at 32 rows, also without these kernels)
    s = WHOLE_SHAPES[name]
    rng = np.random.default_rng(B * 100 + Q)
    run_stack(s, 2, B, Q, rng.integers(1, 60, B), rng.integers(0, 2, B), seed=40 + B, w_std=min(0.05, s.hidden ** -0.5))


# every wave refills its slots: what the widths above, with a step or two a wave, do not reach
@pytest.mark.parametrize("s,layers,B,Q", [
    (synth.QWEN1P5B, 2, 8, 1),                                    # down: ten slots, 8 or 9 steps; gate / up 5 tiles, 6 steps
    (synth.QWEN1P5B, 2, 12, 1), (synth.QWEN1P5B, 2, 16, 1),       # O and down with eight slots, 3 and 17 or 18 steps
    (synth.GEMMA12B, 1, 1, 6),                                    # gate / up 8 tiles, 15 steps of four slots; 16 pairs, normalised as they are read
    (synth.LayerShape(2048, 4, 2, 64, 11008, 4096), 2, 8, 1),     # down: 10 or 11 steps of ten slots
    (synth.LayerShape(4096, 4, 2, 64, 10208, 4096), 2, 9, 1),     # gate / up 5, 6 and 7 tiles (4 to 6 in some workgroups), 16 steps
    (synth.LayerShape(4096, 4, 2, 64, 12256, 4096), 1, 2, 4),
    (synth.LayerShape(4096, 4, 2, 64, 14304, 4096), 1, 4, 4),
    (synth.LayerShape(4096, 8, 4, 64, 2080, 4096), 2, 8, 3),      # 8 pairs, two and three row tiles, 8 steps
    (synth.LayerShape(4096, 8, 4, 64, 2080, 4096), 2, 8, 6)], ids=lambda v: f"{v.hidden}x{v.mlp}" if isinstance(v, synth.LayerShape) else str(v))
def test_projections_with_what_follows_at_size(s, layers, B, Q):
    rng = np.random.default_rng(B * 10 + Q)
    run_stack(s, layers, B, Q, rng.integers(1, 60, B), rng.integers(0, 2, B), seed=70 + B, w_std=min(0.02, s.hidden ** -0.5))


LAYER_KINDS = {"plain": (), "head_norms": ("q_norm", "k_norm"), "query_norm": ("q_norm",), "attention_norm": ("post_attn_norm",),
               "mlp_norm": ("post_mlp_norm",)}


@pytest.mark.parametrize("second", LAYER_KINDS)
@pytest.mark.parametrize("first", LAYER_KINDS)
def test_rows_handed_between_layers_of_two_kinds(first, second):
    """Two layers in one call, each with its own selection of the optional norms: rows normalised by the kernel that closes a layer, or as
    row * gains with sums of squares, to a q/k/v projection that applies the scale or cannot (head norms), at one, two and three row tiles."""
    import dataclasses
    s = dataclasses.replace(synth.TINY_BF16, qk_norm=True, post_norms=True)
    norms = ("q_norm", "k_norm", "post_attn_norm", "post_mlp_norm")
    for B, Q in ((5, 1), (3, 4), (4, 6), (8, 5)):
        seed, ws_h = 80 + B, []
        for l, kind in enumerate((first, second)):
            w = synth.layer_weights(s, seed, layer=l, std=0.05)
            w.update({n: None for n in norms if n not in LAYER_KINDS[kind]})
            ws_h.append(w)
        kv_len = np.random.default_rng(seed).integers(1, 60, B)
        kvs = [synth.kv_cache(s, B, Q, kv_len, np.zeros(B, np.int32), seed, layer=l, hot_keys=1) for l in range(2)]
        x = synth.hidden_states(s, B, Q, seed)
        pos = synth.positions(kvs[0].kv_len, kvs[0].n_img, Q)
        y_ref, refs = x, []
        for w, kv in zip(ws_h, kvs):
            y_ref, k_ref, v_ref = O.verify_layer(s, w, y_ref, pos, kv.k, kv.v, kv.kv_len)
            refs.append((k_ref, v_ref))
        lm = round_up(kvs[0].l_max, 32)
        kds = [binding.k_cache_pack(to_dev(pad_rows(kv.k, lm), s.dtype)) for kv in kvs]
        vds = [binding.v_cache_pack(to_dev(pad_rows(kv.v, lm), s.dtype)) for kv in kvs]
        wds = [binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in w.items()}) for w in ws_h]
        xd = to_dev(x, s.dtype)
        binding.verify_layers(cfg_of(s), binding.LayerStack(wds, kds, vds), xd, i32(pos), i32(kvs[0].kv_len), lm)
        torch.cuda.synchronize()
        assert_close(xd.float().cpu().numpy(), y_ref, TOL_BF16, f"{B * Q} rows, output")
        for l in range(2):
            for got, ref, what in zip((k_cache_to_rows(kds[l]), v_blocked_to_rows(vds[l])), refs[l], ("keys", "values")):
                got = got.float().cpu().numpy()
                for b in range(B):
                    L = int(kv_len[b])
                    assert_close(got[b, :, L:L + Q], ref[b, :, L:L + Q], TOL_BF16, f"{B * Q} rows, layer {l}, appended {what}")


@pytest.mark.parametrize("name", WHOLE_SHAPES)
def test_norm_inside_the_query_projection(name):
    """Up to 16 rows the projection normalises its rows as it reads them, 17 rows have a launch for it: rows of very different size
    give the same bits in a batch and alone, and the same as rows of 2^k times the size (eps apart); the keys and values that a call of
    17 rows appends are the same but for rounding, and both are the checker's."""
    s = WHOLE_SHAPES[name]
    w_h = synth.layer_weights(s, 60, std=0.05)
    w = binding.pack_layer_weights({k: (None if v is None else to_dev(v, s.dtype)) for k, v in w_h.items()})
    cfg = cfg_of(s)
    cfg.norm_eps = 0.0
    n, lm = 16, 32
    x_h = synth.hidden_states(s, n + 1, 1, 61) * (2.0 ** (np.arange(n + 1, dtype=np.float32) - 8)).reshape(-1, 1, 1)
    pos_h = (3 + 7 * np.arange(n + 1)).reshape(-1, 1)
    x, pos, kv_len = to_dev(x_h, "bf16"), i32(pos_h), i32(np.zeros(n + 1))

    def keys(rows, scale=1.0):
        k = torch.zeros(rows.stop - rows.start, s.n_kv_heads, lm, s.head_dim, dtype=torch.bfloat16, device=DEV)
        v = torch.zeros(rows.stop - rows.start, s.n_kv_heads, lm // 32, s.head_dim, 32, dtype=torch.bfloat16, device=DEV)
        binding.verify_layer(cfg, w, (x[rows] * scale).contiguous(), pos[rows], k, v, kv_len[rows])
        return k, v

    whole = keys(slice(0, n))
    for rows in (slice(0, 1), slice(3, 12)):
        assert all(torch.equal(a[rows], b) for a, b in zip(whole, keys(rows)))
    assert all(torch.equal(a, b) for a, b in zip(whole, keys(slice(0, n), 16.0)))
    assert whole[0].abs().sum() > 0

    import dataclasses
    zeros = np.zeros((n + 1, s.n_kv_heads, lm, s.head_dim), np.float32)
    _, k_ref, v_ref = O.verify_layer(dataclasses.replace(s, norm_eps=0.0), w_h, x_h, pos_h, zeros, zeros, np.zeros(n + 1, np.int32))
    apart = keys(slice(0, n + 1))
    for got, ref in ((apart, slice(0, n + 1)), (whole, slice(0, n))):
        assert_close(k_cache_to_rows(got[0]).float().cpu().numpy()[:, :, 0], k_ref[ref, :, 0], TOL_BF16, "keys")
        assert_close(v_blocked_to_rows(got[1]).float().cpu().numpy()[:, :, 0], v_ref[ref, :, 0], TOL_BF16, "values")
    # each side rounds the operand of a sum over the inputs (relative 2^-9 at most, at random: 2^-9 / sqrt(3) of the sum's rms, sqrt(2) of that
    # between the two) and the result (2^-9 of it): five deviations of the first and two roundings stay under 1.2e-2 of the largest value
    for a, b in zip(whole, apart):
        assert_close(a.float().cpu().numpy(), b[:n].float().cpu().numpy(), 1.2e-2, "17 rows")


@pytest.mark.parametrize("mlp", [32, 2080, 4128, 6176, 8224, 10272, 12320, 16384, 16416])
def test_gated_projection_tiles(mlp):
    """1 to 8 tiles a workgroup of the gate / up projection, the last one missing in some workgroups, and one width past them."""
    run_layer(synth.LayerShape(64, 2, 1, 64, mlp, 4096), 3, 3, [40, 0, 7], [8, 0, 0], seed=50, w_std=0.05)
