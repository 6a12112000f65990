"""GPU parity: libpolystep (through its C ABI) against the CPU oracle, element by element, on
the same seeded inputs.  Bar: max |err| <= 2e-2 x RMS, applied by one rule to every case (final output
against the definition with bf16 contraction operands and, less the CPU-only gap, against the plain one;
every stage on its own per token row; see gpu_harness.py); integer results (slots written, untouched
cache) bit-exact."""
import numpy as np
import pytest
import torch

from paper_2507_17769_amd import binding as B
from paper_2507_17769_amd import workloads as W
from gpu_harness import TOL, Case, bits_to_dev, dev_to_bits, f32, rel_err
from oracle.bf16 import to_bits
from paper_2507_17769_amd.runner import Engine

pytestmark = pytest.mark.gpu


def _assert_errs(errs, tag=""):
    bad = {k: v for k, v in errs.items() if not v <= TOL}
    assert not bad, f"{tag} over tolerance: {bad} (all: {errs})"


def test_cfg0_tiny_mixed_batch_all_tensors():
    c = Case(W.config_batch(0, seed=0))
    errs = c.run()
    print("cfg0 errors", errs, "append mismatch frac", c.check_pool())
    _assert_errs(errs, "cfg0")
    assert c.stats.n_tokens == 68 and c.stats.total_kv == 128 + 17 + 64 + 100 + 128
    c.close()


@pytest.mark.parametrize("chunk,prefix,decodes", [
    (1, 0, []), (1, 1, [1]), (3, 15, [2, 16]), (15, 0, [17]), (16, 16, [31, 32, 33]), (17, 100, [1, 1, 1]),
    (33, 1, [64]), (100, 37, [5, 250]), (0, 0, [1]), (0, 0, [1, 2, 3, 15, 16, 17, 18, 255, 256, 257]),
    (130, 0, []), (257, 300, [300]),
    (70, 5, [3, 9]), (88, 0, [1, 2, 3, 4, 5, 6]),     # 72 and 94 tokens: five and six row tiles in the weight-streaming GEMM
    (112, 9, []), (120, 0, [3] * 8), (140, 1, [2, 2, 2, 2]), (150, 0, [7] * 10), (151, 0, [7] * 10),   # 112, 128, 144, 160 | 161 tokens: seven to ten row tiles | tiled again
    (64, 0, []), (65, 0, []), (90, 2, [4] * 6), (91, 2, [4] * 6),   # 64 | 65 and 96 | 97 tokens: a full fourth row tile | the first of a fifth, the last batch of the streaming GEMM | the first of the tiled one
])
def test_ragged_shapes_tiny_model(chunk, prefix, decodes):
    b = W.custom_batch("tiny", 11, chunk, prefix, decodes, name="ragged")
    c = Case(b)
    errs = c.run()
    _assert_errs(errs, f"chunk={chunk} prefix={prefix} decodes={decodes}")
    c.check_pool()
    c.close()


def test_long_contexts_tiny_model():
    """KV spans of thousands of pages: many 64-page blocks per work item, one sequence cut over hundreds of
    workers (merge groups with far more than eight partials), rotary positions up to 1e5."""
    b = W.custom_batch("tiny", 31, 40, 70000, [100001, 65537, 1025], name="long")
    c = Case(b)
    errs = c.run()
    print("long-context errors", errs, flush=True)
    _assert_errs(errs, "long contexts")
    c.check_pool()
    c.close()


def test_many_short_decodes_tiny_model():
    """700 one-token requests with 1..50 cached tokens: more sequences than attention workers would each get a
    page pair of, every work item a whole sequence, and a token count that is no multiple of any tile."""
    kv = 1 + (np.arange(700) * 37) % 50
    b = W.custom_batch("tiny", 41, 0, 0, kv, name="many")
    c = Case(b)
    errs = c.run()
    print("many-decodes errors", {k: round(v, 5) for k, v in errs.items()}, flush=True)
    _assert_errs(errs, "many short decodes")
    c.check_pool()
    c.close()


def test_unit_scale_branches():
    # weights of std 1/sqrt(hidden) make the attention and FFN branches as large as the residual
    # stream, so an error in the O or down projection cannot hide behind it in `out`
    b = W.custom_batch("tiny", 21, 48, 80, [1, 30, 200, 700], name="unit")
    c = Case(b, weight_std=1.0 / 16.0)
    errs = c.run()
    print("unit-scale errors", errs)
    _assert_errs(errs, "unit scale")
    c.close()


@pytest.mark.parametrize("n_q,n_kv,d", [(4, 4, 64), (8, 4, 128), (8, 2, 64), (8, 1, 128), (16, 1, 64), (16, 1, 128)])
def test_gqa_group_sizes_and_head_dims(n_q, n_kv, d):
    model = dict(hidden=256, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=320, rope_base=10000.0, n_layers=1)
    W.MODELS["_t"] = model
    try:
        b = W.custom_batch("_t", 5, 21, 40, [1, 17, 90], name="gqa")
        c = Case(b)
        errs = c.run()
        _assert_errs(errs, f"nq={n_q} nkv={n_kv} d={d}")
        c.check_pool()
        c.close()
    finally:
        del W.MODELS["_t"]


def test_split_plans_agree_and_runs_are_deterministic():
    b = W.custom_batch("tiny", 3, 40, 200, [1, 33, 500, 1000], name="splits")
    outs = []
    for split, teams in ((0, 0), (1, 0), (3, 0), (16, 0), (100, 0), (5000, 0), (0, 1), (0, 3), (0, 400)):
        c = Case(b, options={"attn_workers": split, "attn_teams": teams})
        errs = c.run()
        b_run = c.batch      # the case's own copy of the batch (page ids shifted past the guard page)
        _assert_errs(errs, f"split={split} teams={teams}")
        first = c.out_bits.copy()
        # same plan twice: bitwise identical
        x_dev = bits_to_dev(c.x_bits, c.eng.device)
        again, _ = c.eng.step(b_run.seqs, x_dev)
        c.eng.ctx.sync()
        assert np.array_equal(dev_to_bits(again), first)
        outs.append(c.out32.copy())
        c.close()
    for o in outs[1:]:
        assert rel_err(o, outs[0]) <= TOL


@pytest.mark.parametrize("chunk,prefix,decodes", [(512, 2048, [1024] * 128), (0, 0, [700] * 64), (2048, 0, []), (48, 0, [200] * 64), (200, 8192, [1000])])
def test_a_context_without_a_device_plans_what_the_device_launches(chunk, prefix, decodes):
    m = W.MODELS["8b"]
    b = W.custom_batch("8b", 17, chunk, prefix, decodes, name="plan")
    desc = (m["hidden"], m["n_q"], m["n_kv"], m["head_dim"], m["ffn"], 1, 16384)
    dev, host = B.Context(*desc), B.Context(*desc, host_only=True)
    assert np.array_equal(dev.plan_attention(b.seqs), host.plan_attention(b.seqs))
    dev.destroy()
    host.destroy()


@pytest.mark.parametrize("d", [64, 128])
def test_team_softmax_weights_at_large_scores(d):
    """Scores of some 5e5 in units of the exponent, where one rounding of the reference maximum is 3 % of a weight, that grow by
    less than one from one pair of pages to the next.  The reference a pair's weights are taken against and the rescaling of what
    came before must round alike.  Scores are exact: every query is 1024 and 1 in the two slowest dimensions (which a base of 1e30
    does not rotate), the keys of pair p are 4096 and 2p there and zero elsewhere, the values of pair p are one in dimension p.
    Left to differ by are the weights' bf16 rounding, 2^-8 of each and of their sum, and the output's: 2.5 x 2^-8."""
    model = dict(hidden=256, n_q=4, n_kv=1, head_dim=d, ffn=320, rope_base=1e30, n_layers=1)
    n_new, pairs = 48, 16
    W.MODELS["_s"] = model
    try:
        b = W.custom_batch("_s", 1, n_new, 32 * pairs, [], name="scores")
        w = W.layer_weights(model, 1)
    finally:
        del W.MODELS["_s"]
    bits = lambda a: to_bits(np.asarray(a, dtype=np.float32))
    qkv = np.zeros((256, 6, d), dtype=np.float32)
    qkv[0, :4, d // 2 - 1], qkv[0, :4, d // 2 - 2] = 1024.0, 1.0
    w["w_qkv"] = bits(qkv.reshape(256, 6 * d))
    k, v = (np.zeros((32 * pairs, 1, d), dtype=np.float32) for _ in range(2))
    pair = np.arange(32 * pairs) // 32
    k[:, 0, d // 2 - 1], k[:, 0, d // 2 - 2] = 4096.0, 2.0 * pair
    v[np.arange(32 * pairs), 0, pair] = 1.0
    eng = Engine(model, b.n_pool_pages, 1, 1, max_position=32 * pairs + 64)
    eng.ctx.set_option("attn_workers", 1)      # one team goes through all pairs
    eng.load_layer(0, w)
    eng.write_kv(0, b.seqs[0].pages, 0, bits(k), bits(v))
    taps = eng.alloc_taps(n_new)
    eng.ctx.set_taps(0, q=taps["q"].data_ptr(), attn=taps["attn"].data_ptr())
    eng.step(b.seqs, bits_to_dev(bits(np.ones((n_new, 256))), eng.device))
    eng.ctx.sync()
    q, got = f32(dev_to_bits(taps["q"])), f32(dev_to_bits(taps["attn"])).astype(np.float64).reshape(n_new, 4, d)
    eng.close()
    assert (q[:, :, d // 2 - 1] == 1024).all() and (q[:, :, d // 2 - 2] == 1).all()
    score = 2.0 * np.arange(pairs) / np.sqrt(d)
    want = np.exp(score - score.max())
    want /= want.sum()
    rel = np.abs(got[:, :, :pairs] / want - 1.0).max()
    assert rel <= 2.5 * 2.0 ** -8, rel
    assert not got[:, :, pairs:].any()


def test_chunked_prefill_on_gpu_matches_one_shot_and_oracle():
    # Sec. 2.4 / 4.7: any chunking of a prompt must give the same cache and outputs
    L = 150
    base = W.custom_batch("tiny", 9, L, 0, [], name="oneshot")
    one = Case(base)
    errs = one.run()
    pages = one.batch.seqs[0].pages      # as the case holds them (shifted past the guard page)
    _assert_errs(errs, "one-shot")
    x_bits = one.x_bits
    ref = f32(one.out_bits)
    hb = 2.0 ** -8        # the hand-driven chunks below produce bf16 output: allow its storage rounding
    for chunks in ([1, 149], [64, 64, 22], [17, 1, 100, 32]):
        c = Case(base)                       # same pages, weights; we drive the chunks by hand
        outs, done = [], 0
        for n in chunks:
            seqs = [(7, n, done + n, pages)]
            x_dev = bits_to_dev(x_bits[done:done + n], c.eng.device)
            o, _ = c.eng.step(seqs, x_dev)
            c.eng.ctx.sync()
            outs.append(f32(dev_to_bits(o)))
            done += n
        got = np.concatenate(outs)
        w64 = one.want.astype(np.float64)
        rms = np.sqrt(np.mean(w64 * w64))
        assert np.all(np.abs(got - w64) <= TOL * rms + hb * np.abs(w64))
        assert np.all(np.abs(got - ref) <= TOL * rms + 2 * hb * np.abs(ref))
        k1, v1 = one.eng.read_kv(0, pages, 0, L)
        k2, v2 = c.eng.read_kv(0, pages, 0, L)
        # both caches hold bf16 roundings of fp32 sums of the same products (the normalised input does not depend on
        # the chunking): one rounding flip plus twice the rounding-error bound of such a sum
        for a_, b_, bound in zip((k1, v1), (k2, v2), one.kv_sum_bounds()):
            fa, fb = f32(a_).astype(np.float64), f32(b_).astype(np.float64)
            assert np.all(np.abs(fa - fb) <= 2.0 ** -7 * np.abs(fa) + 2 * bound)
        c.close()
    one.close()


def test_decode_with_kv_len_one_returns_v():
    b = W.custom_batch("tiny", 2, 0, 0, [1, 1, 1], name="kv1")
    c = Case(b)
    b = c.batch
    T = 3
    taps = c.eng.alloc_taps(T)
    c.eng.ctx.set_taps(0, **{k: t.data_ptr() for k, t in taps.items()})
    x_dev = bits_to_dev(c.x_bits, c.eng.device)
    c.eng.step(b.seqs, x_dev)
    c.eng.ctx.sync()
    attn = dev_to_bits(taps["attn"]).reshape(T, 4, 64)
    for i, s in enumerate(b.seqs):
        k, v = c.eng.read_kv(0, s.pages, 0, 1)
        for h in range(4):
            assert np.array_equal(attn[i, h], v[0, h // 2])          # softmax of one logit is exactly 1
    c.close()


def test_three_layer_stack_with_two_kv_slots():
    b = W.custom_batch("tiny", 4, 20, 30, [1, 40], name="stack")
    c = Case(b, n_layers=3, n_kv_layers=3)
    errs = c.run(tap_layer=2)
    _assert_errs(errs, "stack")
    c.check_pool()
    c.close()


def test_kv_write_read_roundtrip_is_exact():
    b = W.custom_batch("tiny", 6, 0, 0, [77], name="rt")
    c = Case(b)
    b = c.batch
    rng = np.random.default_rng(0)
    k = rng.integers(0, 0x7F80, size=(50, 2, 64)).astype(np.uint16)
    v = rng.integers(0, 0x7F80, size=(50, 2, 64)).astype(np.uint16)
    pages = b.seqs[0].pages
    # the whole span first, then positions 13..62 over it: neither start nor end falls on a group of four positions,
    # and what the partial groups leave alone must still be there
    k_all = rng.integers(0, 0x7F80, size=(77, 2, 64)).astype(np.uint16)
    v_all = rng.integers(0, 0x7F80, size=(77, 2, 64)).astype(np.uint16)
    c.eng.write_kv(0, pages, 0, k_all, v_all)
    c.eng.write_kv(0, pages, 13, k, v)
    k2, v2 = c.eng.read_kv(0, pages, 13, 50)
    assert np.array_equal(k, k2) and np.array_equal(v, v2)
    k_all[13:63], v_all[13:63] = k, v
    k3, v3 = c.eng.read_kv(0, pages, 0, 77)
    assert np.array_equal(k_all, k3) and np.array_equal(v_all, v3)
    for p0, n in ((1, 1), (2, 3), (3, 6), (15, 2), (60, 17)):
        k4, v4 = c.eng.read_kv(0, pages, p0, n)
        assert np.array_equal(k_all[p0:p0 + n], k4) and np.array_equal(v_all[p0:p0 + n], v4), (p0, n)
    with pytest.raises(B.PolystepError) as e:
        c.eng.read_kv(0, pages, 70, 20)
    assert e.value.status == B.PS_ERANGE
    c.close()


@pytest.mark.parametrize("pos0,n", [(0, 4096), (0, 4097), (13, 4083), (13, 4084), (4095, 2), (5, 8400)])
def test_kv_copies_of_more_pages_than_one_launch_takes(pos0, n):
    # a launch takes the ids of 256 pages; spans that end with them, one position later, and that need three launches
    c = Case(W.custom_batch("tiny", 7, 0, 0, [8416], name="long copy"))
    rng = np.random.default_rng(n)
    k_all, v_all = (rng.integers(0, 0x7F80, size=(8416, 2, 64)).astype(np.uint16) for _ in range(2))
    pages = c.batch.seqs[0].pages
    for at in range(0, 8416, 526):   # small spans, a single launch each
        c.eng.write_kv(0, pages, at, k_all[at:at + 526], v_all[at:at + 526])
    k, v = c.eng.read_kv(0, pages, pos0, n)
    assert np.array_equal(k, k_all[pos0:pos0 + n]) and np.array_equal(v, v_all[pos0:pos0 + n])
    k_new, v_new = (rng.integers(0, 0x7F80, size=(n, 2, 64)).astype(np.uint16) for _ in range(2))
    c.eng.write_kv(0, pages, pos0, k_new, v_new)
    k_all[pos0:pos0 + n], v_all[pos0:pos0 + n] = k_new, v_new
    for at in range(0, 8416, 526):
        k, v = c.eng.read_kv(0, pages, at, 526)
        assert np.array_equal(k, k_all[at:at + 526]) and np.array_equal(v, v_all[at:at + 526]), at
    c.close()


def test_state_errors_and_empty_step():
    m = W.MODELS["tiny"]
    ctx = B.Context(m["hidden"], m["n_q"], m["n_kv"], m["head_dim"], m["ffn"], 1, 256, 1e-5, 1e4)
    x = torch.zeros((4, 256), dtype=torch.int16, device="cuda")
    with pytest.raises(B.PolystepError) as e:
        ctx.step([(1, 1, 1, [0])], x.data_ptr(), x.data_ptr())
    assert e.value.status == B.PS_ESTATE and "pool" in str(e.value)
    ctx.kv_alloc(4, 1, 0)
    with pytest.raises(B.PolystepError) as e:
        ctx.step([(1, 1, 1, [0])], x.data_ptr(), x.data_ptr())
    assert e.value.status == B.PS_ESTATE and "weights" in str(e.value)
    w = W.layer_weights("tiny", 0)
    dev = {k: bits_to_dev(v, "cuda") for k, v in w.items()}
    ctx.init_layer(0, **{k: t.data_ptr() for k, t in dev.items()})
    st = ctx.step([], 0, 0, want_stats=True)
    assert st.n_tokens == 0
    with pytest.raises(B.PolystepError) as e:          # invalid batch: nothing launched, pool untouched
        ctx.step([(1, 1, 1, [9])], x.data_ptr(), x.data_ptr())
    assert e.value.status == B.PS_ERANGE
    ctx.step([(1, 1, 1, [0])], x.data_ptr(), x.data_ptr())
    ctx.sync()
    ctx.destroy()


def test_profile_grid_small():
    from paper_2507_17769_amd.runner import Engine
    eng = Engine("tiny", 400, max_position=1024)
    eng.load_layer(0, W.layer_weights("tiny", 0))
    x = torch.zeros((80, 256), dtype=torch.int16, device="cuda")
    y = torch.zeros_like(x)
    cells = [(0, 0, [0, 0], np.zeros((2, 0))), (64, 4, [64, 10], [[17, 64, 100, 128], [1, 2, 3, 400]]), (0, 16, [0], [list(range(100, 116))])]
    out = eng.ctx.profile_grid(cells, x.data_ptr(), y.data_ptr(), warmup=1, iters=3)
    assert out[0].n_tokens == 0 and out[1].n_tokens == 68 and out[2].n_tokens == 16
    assert out[1].median_ms > 0 and out[1].total_kv in (128 + 309, 74 + 406)
    assert abs(sum(out[2].stage_ms) - out[2].median_ms) < 5 * out[2].median_ms
    assert eng.ctx.kv_free_pages() == 400
    eng.close()


def test_teacher_forced_layer_inside_an_aliased_stack():
    # 4 layers on 2 KV slots (layers 0,2 share slot 0; 1,3 share slot 1).  The whole stack is checked
    # against the oracle (which models the same aliasing), then layer 2 on its own: the x_in tap, that
    # layer's weights and its slot's cached prefix go to the oracle, the result must match the x_out tap.
    from oracle import run as orun
    b = W.custom_batch("tiny", 8, 24, 40, [1, 33, 70], name="alias")
    c = Case(b, n_layers=4, n_kv_layers=2)
    errs = c.run(tap_layer=3)
    _assert_errs(errs, "aliased stack")
    b = c.batch
    eng, T, H = c.eng, b.n_tokens, 256
    xin = torch.zeros((T, H), dtype=torch.float32, device=eng.device)
    xout = torch.zeros((T, H), dtype=torch.float32, device=eng.device)
    eng.ctx.set_taps(2, x_in=xin.data_ptr(), x_out=xout.data_ptr())
    x_dev = bits_to_dev(c.x_bits, eng.device)
    eng.step(b.seqs, x_dev)
    eng.ctx.sync()
    eng.ctx.set_taps(0)
    pool = orun.make_pool(c.model, b.n_pool_pages, 1)
    for i, s in enumerate(b.seqs):
        k, v = b.prefix_kv(i, 0)                      # slot 0 = layer 2's slot
        pool.write_bits(0, [int(p) for p in s.pages], 0, k, v)
    want = orun.run_layer_from(c.model, c.layers[2], b.seqs, xin.cpu().numpy(), pool, 0)
    assert rel_err(xout.cpu().numpy(), want) <= TOL
    c.close()


def test_wide_hidden_70b_like_shape_small_ffn():
    # hidden 8192 with 64 query / 8 KV heads (group size 8) as in the 70B-shaped layer, small FFN and batch.
    # With N(0, 0.02) weights at this width the attention logits have twice the spread of the 8B-shaped
    # layer, the softmax turns peaky, and rounding the contraction operands to bf16 moves the definition
    # itself by more than the bar (printed: the CPU-only gap).  Two weight scales, N(0, 0.02) and
    # 1.28/sqrt(hidden), which keeps the logits' spread of the 8B shape; the same rule for both.
    model = dict(hidden=8192, n_q=64, n_kv=8, head_dim=128, ffn=1024, rope_base=500000.0, n_layers=1)
    W.MODELS["_w"] = model
    try:
        for spec in ((70, 30, [1, 40, 300]), (0, 0, [5, 17, 64, 100] * 4)):
            b = W.custom_batch("_w", 13, *spec, name="wide")
            for std in (1.28 / 8192 ** 0.5, W.WEIGHT_STD):
                c = Case(b, weight_std=std)
                errs = c.run()
                print(f"wide spec={spec} std={std:.4f}: {c.report}", flush=True)
                _assert_errs(errs, f"wide spec={spec} std={std}")
                c.check_pool()
                c.close()
    finally:
        del W.MODELS["_w"]


def test_every_stage_on_its_own_tiny_and_mixed():
    # the same stage-by-stage check on the tiny model: prefill chunk with ragged tiles + decodes
    for spec in ((100, 37, [5, 250]), (257, 300, [300, 1, 17])):
        c = Case(W.custom_batch("tiny", 19, *spec, name="stages"))
        errs = c.run()
        assert sum(k.startswith("stage ") for k in errs) == 8, errs      # seven stages and the appended cache entries
        _assert_errs(errs, f"stages spec={spec}")
        c.close()


@pytest.mark.parametrize("tile,split,tails", [(128, 0, 0), (128, 1, 0), (128, 3, 0), (256, 0, 0), (256, 1, 0), (256, 2, 0), (256, 8, 0),
                                              (128, 1, 2), (256, 1, 2), (0, 0, 2), (128, 1, 1)])
def test_tiled_gemm_tile_sizes_and_k_splits(tile, split, tails):
    # more than 64 tokens take the tiled GEMM: both block tiles, automatic and forced K splits, on token
    # counts that leave ragged row tiles (65: one row past a 64-row wavefront tile; 300: 256 + 44;
    # 530: two full 256-row tiles + 18) and on widths that leave ragged column tiles (704-wide FFN:
    # 1408 = 5.5 x 256 gate/up columns; 256-wide hidden = one column tile); tails: 2 = every last, partial wave of tiles has
    # its K loops cut over all blocks (parked pieces, arrival counters, the last block adds them up), 1 = none has
    for chunk, decodes in ((65, []), (280, [7] * 20), (500, [40] * 30)):
        b = W.custom_batch("tiny", 17, chunk, 32, decodes, name="tiles")
        c = Case(b, options={"gemm_tile": tile, "gemm_split_k": split, "gemm_whole_tiles": tails})
        errs = c.run()
        _assert_errs(errs, f"tile={tile} split={split} tails={tails} T={b.n_tokens}")
        c.check_pool()
        c.close()


@pytest.mark.parametrize("tokens", [65, 97, 113, 129, 161, 209, 257, 289, 321])
def test_weights_in_registers_gemm_row_blocks(tokens):
    # a shape whose gate/up, QKV or down projection reaches the weights-in-registers GEMM by the automatic choice; the token counts
    # leave one row in the last 16-row tile.  test_host_gemm_plan.py asserts that the kernel is chosen; every block shape is
    # tested below
    W.MODELS["_r"] = dict(hidden=2048, n_q=16, n_kv=8, head_dim=128, ffn=12288, rope_base=500000.0, n_layers=1)
    try:
        c = Case(W.custom_batch("_r", 29, tokens - 5, 40, [1, 16, 17, 90, 200], name="row blocks"))
        errs = c.run()
        _assert_errs(errs, f"row blocks T={tokens}")
        c.check_pool()
        c.close()
    finally:
        del W.MODELS["_r"]


def _wreg_case(model, tokens, options):
    W.MODELS["_b"] = model
    try:
        c = Case(W.custom_batch("_b", 31, tokens - 4, 24, [1, 16, 17, 90], name="block"), options=dict(options, poison_workspaces=1))
        errs = c.run()
        _assert_errs(errs, f"T={tokens} {options}")
        c.check_pool()
        c.close()
    finally:
        del W.MODELS["_b"]


@pytest.mark.parametrize("nc", [2, 4])
@pytest.mark.parametrize("tm", [5, 6, 7, 8, 9, 10])
def test_weights_in_registers_gemm_every_block(tm, nc):
    # every block shape for all four projections: one row block (weights streamed past the caches), whose last tile has one
    # row, and three row blocks that share the weights, with one and two K splits.  QKV's 18 column groups leave two of a
    # block's four without work.  The small shape adds a last block with one group of two or four (three groups of QKV) and
    # two of four (42 of gate/up); its O and down projections are not divisible and stay with the other kernels.
    model = dict(hidden=1024, n_q=16, n_kv=1, head_dim=64, ffn=2048, rope_base=10000.0, n_layers=1)
    _wreg_case(model, 16 * tm - 15, {"gemm_wreg": 10 * tm + nc})
    for split in (1, 2):
        _wreg_case(model, 32 * tm + 1, {"gemm_wreg": 10 * tm + nc, "gemm_split_k": split})
    small = dict(hidden=1024, n_q=1, n_kv=1, head_dim=64, ffn=1344, rope_base=10000.0, n_layers=1)
    _wreg_case(small, 16 * tm + 1, {"gemm_wreg": 10 * tm + nc})


@pytest.mark.parametrize("tokens", [5, 16, 17, 48, 49, 64, 65, 97, 160])
def test_streaming_gemm_two_k_shares(tokens):
    # O (and QKV from 33 to 64 tokens) on weight streaming with two K shares in a block: one row tile, which one share keeps, to ten;
    # K of 36 blocks, cut into three splits of 12, and of 32 in four of 8, and one split alone
    _wreg_case(dict(hidden=1152, n_q=18, n_kv=9, head_dim=64, ffn=1344, rope_base=10000.0, n_layers=1), tokens, {})
    for split in (0, 1):
        _wreg_case(dict(hidden=1024, n_q=16, n_kv=1, head_dim=64, ffn=1024, rope_base=10000.0, n_layers=1), tokens, {"gemm_split_k": split})


@pytest.mark.parametrize("tokens", [5, 16, 17, 33, 64, 65, 97, 160])
def test_streaming_gemm_rotates_and_appends(tokens):
    # QKV of head dim 64 in one split, which the GEMM itself rotates and appends: one K share (34 k-blocks; with 15 heads the last
    # block of two column groups has one) and two (32), pairs of query, key and value heads in one block; by default where the
    # shape gives one split (shallow, 192 heads).  Head dim 128 in one split, and what other kernels serve, rotate separately
    for hidden, n_q, n_kv in ((1088, 8, 2), (1088, 5, 5), (1024, 14, 7), (1024, 1, 1)):
        _wreg_case(dict(hidden=hidden, n_q=n_q, n_kv=n_kv, head_dim=64, ffn=320, rope_base=10000.0, n_layers=1), tokens, {"gemm_split_k": 1})
    _wreg_case(dict(hidden=256, n_q=64, n_kv=64, head_dim=64, ffn=320, rope_base=10000.0, n_layers=1), tokens, {})
    _wreg_case(dict(hidden=256, n_q=4, n_kv=1, head_dim=128, ffn=320, rope_base=10000.0, n_layers=1), tokens, {"gemm_split_k": 1})


@pytest.mark.parametrize("chunk,splits", [(0, [1, 2, 8]), (0, [9, 16, 17]), (40, [2, 64, 65]), (40, [128, 129, 257])])
def test_merge_groups_with_different_numbers_of_splits(chunk, splits):
    # decodes of 128 tokens per split (workers take at least four pairs of pages each) next to each other and to a chunk in few
    # splits: a wavefront's batch of eight full and one over, one wavefront per pass to all sixteen, and more than their batches hold
    b = W.custom_batch("tiny", 37, chunk, 300 if chunk else 0, [128 * n for n in splits], name="merge")
    c = Case(b, options={"attn_workers": 100000})
    errs = c.run()
    _assert_errs(errs, f"chunk={chunk} splits={splits}")
    c.check_pool()
    c.close()


@pytest.mark.parametrize("tokens", [63, 64, 65, 127, 128, 129, 200])
def test_row_kernels_visit_every_row(tokens):
    # from 64 rows on a block's row is a permutation of its index over whole rounds of 64; the buffers start as NaN, so a row
    # that no block takes shows in the output
    c = Case(W.custom_batch("tiny", 43, tokens - 3, 21, [1, 16, 50], name="rows"), options={"poison_workspaces": 1})
    errs = c.run()
    _assert_errs(errs, f"rows T={tokens}")
    c.check_pool()
    c.close()


def test_only_layer_runs_that_layer_as_the_whole_model():
    # a 3-layer context restricted to layer 1 gives bit for bit what a 1-layer context with layer 1's weights gives
    b = W.custom_batch("tiny", 23, 40, 20, [3, 60, 129], name="only")
    ws = [W.layer_weights(W.MODELS["tiny"], 5, l) for l in range(3)]
    x = bits_to_dev(b.activations(), "cuda:0")
    outs = []
    for layers, only in (([ws[0], ws[1], ws[2]], 1), ([ws[1]], -1)):
        eng = Engine(W.MODELS["tiny"], b.n_pool_pages, len(layers), 1, max_position=256)
        for l, w in enumerate(layers):
            eng.load_layer(l, w)
        eng.load_prefixes(b)
        eng.ctx.set_option("only_layer", only)
        out, _ = eng.step(b.seqs, x)
        eng.ctx.sync()
        outs.append(dev_to_bits(out))
        with pytest.raises(B.PolystepError):
            eng.ctx.set_option("only_layer", len(layers))
        eng.close()
    assert np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("chunks,decodes", [
    ([(1023, 0), (1, 2049)], [5, 300]),                 # a budget already filled with 1023 tokens takes one token of the next request
    ([(17, 3), (64, 100), (5, 0), (130, 31)], [1, 16, 17]),   # four prefill requests of ragged sizes and offsets
    ([(512, 0)] * 4, []),                               # prefill-only step of 2048 tokens from four fresh requests
    ([(2048, 0)], []),                                  # one 2048-token prompt in one step
])
def test_steps_with_several_prefill_requests(chunks, decodes):
    b = W.multi_batch("tiny", 41, chunks, decodes)
    c = Case(b)
    errs = c.run()
    _assert_errs(errs, f"chunks={chunks} decodes={decodes}")
    c.check_pool()
    c.close()


def test_prefill_decode_handoff_through_kv_read_and_write():
    # Prefill on one context, decode on another: the keys and values of the prompt are the hand-off payload
    # (ps_kv_read on the prefill side, ps_kv_write into freshly reserved pages on the decode side).  The decode
    # step there gives bit for bit what the same step gives on the context that ran the prefill.
    m = W.MODELS["tiny"]
    w = W.layer_weights(m, 9, 0)
    prompt = 100
    pre = W.multi_batch("tiny", 43, [(prompt, 0)], [])
    x_pre = bits_to_dev(pre.activations(), "cuda:0")
    a = Engine(m, 64, max_position=256)
    a.load_layer(0, w)
    a.step(pre.seqs, x_pre)
    a.ctx.sync()
    pages_a = pre.seqs[0].pages
    k, v = a.read_kv(0, pages_a, 0, prompt)
    # decode side: its own pool and allocator
    bctx = Engine(m, 40, max_position=256, perm_seed=77)
    bctx.load_layer(0, w)
    pages_b = bctx.ctx.kv_reserve(req_id=5, kv_len=prompt + 1)
    bctx.write_kv(0, pages_b, 0, k, v)
    x_dec = bits_to_dev(W.normal_bf16(np.random.default_rng(1), (1, m["hidden"])), "cuda:0")
    seq_b = [W.SeqSpec(req_id=5, n_new=1, kv_len=prompt + 1, pages=pages_b)]
    out_b, _ = bctx.step(seq_b, x_dec)
    bctx.ctx.sync()
    # the same decode step where the prefill ran (one more page may be needed for position `prompt`)
    need = (prompt + 1 + 15) // 16
    pages_a2 = np.concatenate([pages_a, np.setdiff1d(np.arange(64, dtype=np.int32), pages_a)[:need - len(pages_a)]]).astype(np.int32)
    seq_a = [W.SeqSpec(req_id=pre.seqs[0].req_id, n_new=1, kv_len=prompt + 1, pages=pages_a2)]
    out_a, _ = a.step(seq_a, x_dec)
    a.ctx.sync()
    assert np.array_equal(dev_to_bits(out_a), dev_to_bits(out_b))
    ka, va = a.read_kv(0, pages_a2, 0, prompt + 1)
    kb, vb = bctx.read_kv(0, pages_b, 0, prompt + 1)
    assert np.array_equal(ka, kb) and np.array_equal(va, vb)
    a.close(); bctx.close()


@pytest.mark.gpu
def test_clock_under_load_reading_is_consistent():
    """The diagnostic's three figures must agree with each other: the matrix rate is the shader clock times the
    flop per tick that back-to-back MFMAs give, and neither exceeds the device's nominal figures."""
    b = W.custom_batch("tiny", 0, 0, 0, [16])
    c = Case(b)
    try:
        with pytest.raises(RuntimeError):
            c.eng.ctx.clock_under_load(100, 2)
        with pytest.raises(RuntimeError):
            c.eng.ctx.clock_under_load(100000, 3)
        for wps in (1, 2):
            r = c.eng.ctx.clock_under_load(100000, wps)
            assert r["compute_units"] == 256 and r["wavefronts_per_simd"] == wps
            assert 500.0 < r["shader_mhz"] <= 2400.0 * 1.02
            assert r["ticks_per_mfma"] >= 32.0 * 0.99                # a 32x32x16 bf16 MFMA occupies its SIMD for 32 ticks
            if wps == 1:
                assert r["ticks_per_mfma"] <= 32.0 * 1.5             # (nearly) alone on its SIMD a wavefront issues them back to back
            assert 0.0 < r["mfma_tflops"] <= 2500.0 * 1.02
            # 4 SIMDs x 256 CUs, one MFMA (32768 flop) per 32 ticks each
            from_clock = r["shader_mhz"] * 1e6 * 1024 * 32768 / 32 / 1e12
            assert r["mfma_tflops"] <= from_clock * 1.05
    finally:
        c.close()


@pytest.mark.gpu
def test_hbm_read_rate_reading_is_plausible():
    b = W.custom_batch("tiny", 0, 0, 0, [16])
    c = Case(b)
    try:
        for bad in ((1 << 29, 2), ((1 << 30) + 4096, 2), (1 << 30, 0), (1 << 30, 17)):
            with pytest.raises(B.PolystepError):
                c.eng.ctx.hbm_read_rate(*bad)
        r = c.eng.ctx.hbm_read_rate(1 << 30, 2)
        assert 1000.0 < r <= 8000.0 * 1.02      # between a fraction of and the nominal HBM rate, GB/s
    finally:
        c.close()


def _random_shape(rng):
    kind = int(rng.integers(0, 4))
    if kind == 0:    # decode-only, up to 100 tokens: every row-tile count of the streaming GEMM and the first tiled sizes
        return 0, 0, [int(x) for x in rng.integers(1, 400, size=rng.integers(1, 101))]
    if kind == 1:    # mixed
        return int(rng.integers(1, 150)), int(rng.integers(0, 300)), [int(x) for x in rng.integers(1, 600, size=rng.integers(0, 30))]
    if kind == 2:    # prefill only
        return int(rng.integers(1, 300)), int(rng.integers(0, 500)), []
    return int(rng.integers(1, 20)), int(rng.integers(0, 2000)), [int(x) for x in rng.integers(500, 3000, size=rng.integers(1, 4))]


@pytest.mark.gpu
@pytest.mark.parametrize("seed,random_heads", [(7, False), (8, True)])
def test_random_batches_tiny_models(seed, random_heads):
    """Seeded random batch shapes (and, in the second run, head layouts and FFN widths): all tensors of the step and the
    cache against the oracle, as in the ragged cases above."""
    rng = np.random.default_rng(seed)
    layouts = [(4, 4, 64), (8, 4, 128), (8, 2, 64), (8, 1, 128), (16, 1, 64), (16, 1, 128), (4, 2, 128), (2, 2, 64)]
    try:
        for it in range(30):
            chunk, prefix, decodes = _random_shape(rng)
            name = "tiny"
            if random_heads:
                n_q, n_kv, d = layouts[int(rng.integers(0, len(layouts)))]
                W.MODELS["_r"] = dict(hidden=256, n_q=n_q, n_kv=n_kv, head_dim=d, ffn=int(rng.choice([192, 320, 448])),
                                      rope_base=10000.0, n_layers=1)
                name = "_r"
            b = W.custom_batch(name, int(rng.integers(0, 1000)), chunk, prefix, decodes, name="random")
            c = Case(b)
            try:
                _assert_errs(c.run(), f"seed={seed} case={it} chunk={chunk} prefix={prefix} decodes={decodes} model={W.MODELS[name]}")
                c.check_pool()
            finally:
                c.close()
    finally:
        W.MODELS.pop("_r", None)
