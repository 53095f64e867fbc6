"""End-to-end parity of the HIP path with the CPU oracle (through the C ABI)."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import RTOL, assert_hit_paths_compared, plant_both_forms, compare_step, make_oracle, tails_of, teacher_forced
from oracle import spd_oracle as O

pytestmark = pytest.mark.gpu


def P():
    import paper_2405_18400_amd as pkg
    return pkg


def session(shape, weights, max_ctx=64, k_max=8, kv_dtype="fp32"):
    return P().Session(shape, weights, max_ctx=max_ctx, k_max=k_max, kv_dtype=kv_dtype)


def planted_tables(shape, weights, base, prefix, k, n_tokens, seed=0, tau=1.0):
    """Insert n-grams along the paths an alpha = 0 oracle run visits, so lookups hit."""
    lm = make_oracle(shape, weights)
    _, recs = O.generate(lm, None, prefix, O.DecodeCfg(k, 0.0, tau), n_tokens)
    visits = []
    for rec in recs[1:]:
        for i in range(k):
            for tok in rec.top_ids:
                visits.append((tuple(rec.state_in.history(i)), int(tok)))
    return synth.plant_ngrams(base, visits, shape.vocab, seed=seed, frac=0.5)


@pytest.fixture(scope="module")
def tiny():
    shape = synth.TINY
    w = synth.make_weights(shape, seed=0)
    tabs = synth.make_ngram_tables_uniform(shape.vocab, {2: 50_000, 3: 50_000}, seed=0)
    prefix = synth.make_prefix_uniform(shape.vocab, 16, seed=0)
    return shape, w, tabs, prefix


@pytest.fixture(params=["fused", "per_operator"])
def forward_path(request):
    """Both ways the library can run the transformer forward: one persistent kernel, or one
    kernel per matrix-vector product."""
    return request.param


def select_path(sess, path):
    if path == "fused":
        assert sess.spd_get_fused(), "no fused forward kernel was selected for this shape"
    else:
        sess.spd_set_fused(False)
        assert not sess.spd_get_fused()


def run_teacher_forced(shape, w, tabs, lambdas, prefix, k, alpha, n_tokens, tau=1.0, delta=0.1, max_ctx=64,
                       path="fused", kv_dtype="fp32", dense=None):
    pkg = P()
    sess = session(shape, w, max_ctx=max_ctx, kv_dtype=kv_dtype)
    try:
        select_path(sess, path)
        if dense is not None:
            sess.spd_set_dense_prefill(dense)
        if tabs is not None:
            sess.spd_load_ngrams(tabs, lambdas)
        dc = pkg.SpdDecodeCfg(k, alpha, tau, delta)
        cfg = O.DecodeCfg(k, alpha, tau, delta, tuple(lambdas))
        lm = make_oracle(shape, w)
        state, recs, stats = teacher_forced(sess, lm, tabs, lambdas, prefix, cfg, n_tokens, RTOL[shape.dtype], dc)
        assert sess.spd_position() == len(prefix) + n_tokens - 1
        return state, recs, stats
    finally:
        sess.close()


@pytest.mark.parametrize("dense", [True, False])
def test_tiny_config_as_specified(tiny, forward_path, dense):
    """2-layer fp32 model of the smallest workload, bigram+trigram tables, k = 3, 10 tokens, alpha 0.5; its prefix as a chunk and token by
    token through the forward."""
    shape, w, tabs, prefix = tiny
    lam = (0.01, 0.04, 0.0, 0.0, 0.0)
    _, recs, stats = run_teacher_forced(shape, w, tabs, lam, prefix, 3, 0.5, 10, path=forward_path, dense=dense)
    assert sum(s.get("vocab_decisive", False) for s in stats) >= 8


def test_tiny_config_with_planted_hits(tiny, forward_path):
    shape, w, tabs, prefix = tiny
    lam = (0.01, 0.04, 0.0, 0.0, 0.0)
    planted = planted_tables(shape, w, tabs, prefix, 3, 10)
    _, recs, stats = run_teacher_forced(shape, w, planted, lam, prefix, 3, 0.5, 10, path=forward_path)
    assert any(c.overlap for r in recs[1:] for c in r.candidates), "planting produced no n-gram hit"
    assert any(not c.overlap for r in recs[1:] for c in r.candidates)


@pytest.mark.parametrize("k", [1, 2, 5, 8])
@pytest.mark.parametrize("alpha", [0.0, 0.54])
@pytest.mark.parametrize("tau", [0.7, 0.06])
def test_tiny_k_sweep_all_orders(tiny, k, alpha, tau):
    """k from 1 to 8, with and without the n-gram stage, at a mild temperature and at the one the
    paper tuned for its generation experiments (Appendix B, "Hyperparameter Choices": 0.06)."""
    shape, w, _, prefix = tiny
    base = synth.make_ngram_tables_zipf(shape.vocab, 40_000, seed=3)
    planted = planted_tables(shape, w, base, prefix, k, 6, seed=k, tau=tau)
    _, _, stats = run_teacher_forced(shape, w, planted, synth.PAPER_LAMBDAS, prefix, k, alpha, 6, tau=tau)
    if alpha > 0 and k > 1:
        assert_hit_paths_compared(stats)


def test_bf16_small_model_gqa(forward_path):
    shape = synth.ModelShape("small-bf16", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=5)
    prefix = synth.make_prefix_zipf(shape.vocab, 37, seed=5)
    base = synth.make_ngram_tables_zipf(shape.vocab, 30_000, seed=5)
    planted = planted_tables(shape, w, base, prefix, 3, 8)
    _, _, stats = run_teacher_forced(shape, w, planted, synth.PAPER_LAMBDAS, prefix, 3, 0.54, 8, path=forward_path)
    assert sum(bool(s.get("fully_compared")) for s in stats) == 8
    assert_hit_paths_compared(stats, need_penalty=False)   # vocabulary of 2048: every draft finds some overlap


@pytest.mark.parametrize("dense", [True, False])
def test_long_prefix_crosses_attention_chunks(forward_path, dense):
    shape = synth.ModelShape("small-fp32", 2, 256, 4, 2, 512, 1024, "fp32")
    w = synth.make_weights(shape, seed=6)
    prefix = synth.make_prefix_uniform(shape.vocab, 300, seed=6)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 3, 0.0, 4, max_ctx=600, path=forward_path, dense=dense)


def test_many_attention_items(forward_path):
    """More (query head, chunk) items than a quarter of the fused kernel's blocks: the blocks
    that hold an item also take rows of the O projection and ask for them behind the item's
    own loads; the last chunk is ragged, so some waves of a block have no position in it."""
    shape = synth.ModelShape("heads32-fp32", 2, 512, 32, 8, 512, 1024, "fp32")
    w = synth.make_weights(shape, seed=9)
    prefix = synth.make_prefix_uniform(shape.vocab, 261, seed=9)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 3, 0.0, 4, max_ctx=400, path=forward_path)


def test_vocabulary_of_140k_tokens(forward_path):
    """A vocabulary larger than 128 slices of 1024 entries: more than four entries per thread of a slice, and the slices in a launch of
    their own; k = 5 of 140000."""
    shape = synth.ModelShape("vocab140k-fp32", 1, 128, 2, 2, 256, 140000, "fp32")
    w = synth.make_weights(shape, seed=14)
    prefix = synth.make_prefix_uniform(shape.vocab, 7, seed=14)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 5, 0.0, 4, path=forward_path)


def test_many_small_kv_heads(forward_path):
    """128 key/value heads of d_head 16: four lanes per cached position, and more heads than a
    wave has lanes."""
    shape = synth.ModelShape("heads128-fp32", 2, 2048, 128, 128, 1024, 1024, "fp32")
    w = synth.make_weights(shape, seed=12)
    prefix = synth.make_prefix_uniform(shape.vocab, 19, seed=12)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 3, 0.0, 4, path=forward_path)


def test_wide_ffn_three_pass_rows(forward_path):
    """d_ffn wider than one block pass (bf16: 4096 columns), ragged against the pass width,
    like the 7B shape's 11008: exercises the multi-pass rows of the fused kernel."""
    shape = synth.ModelShape("wide-ffn-bf16", 2, 512, 4, 4, 4096 * 2 + 1416, 1024, "bf16")
    w = synth.make_weights(shape, seed=7)
    prefix = synth.make_prefix_uniform(shape.vocab, 21, seed=7)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 2, 0.0, 5, path=forward_path)


def test_two_pass_ffn_rows(forward_path):
    """d_ffn between one and two block passes."""
    shape = synth.ModelShape("ffn2-bf16", 2, 512, 4, 4, 4096 + 2056, 1024, "bf16")
    w = synth.make_weights(shape, seed=8)
    prefix = synth.make_prefix_uniform(shape.vocab, 9, seed=8)
    run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 2, 0.0, 4, path=forward_path)


def _layer_truncated(shape, n_layers, prefix_len, k, n_tokens, seed, forward_path, alpha=0.54, kv_dtype="fp32"):
    """A published shape with its real widths and head layout but few layers (the oracle runs on
    the host): weights drawn on the GPU, n-gram tables planted along the oracle's path."""
    pkg = P()
    shape = shape.truncated(n_layers)
    wdev = synth.make_weights_device(shape, seed=seed)
    host = {k_: synth.host_view(v) for k_, v in wdev.items() if not k_.endswith("wqkv")}
    prefix = synth.make_prefix_zipf(shape.vocab, prefix_len, seed=seed)
    base = synth.make_ngram_tables_zipf(shape.vocab, 100_000, seed=seed)
    lm = make_oracle(shape, host)
    _, recs0 = O.generate(lm, None, prefix, O.DecodeCfg(k, 0.0), n_tokens)
    tabs = plant_both_forms(base, recs0, k, shape.vocab, seed + 1)
    sess = pkg.Session(shape, wdev, max_ctx=prefix_len + n_tokens + 8, k_max=8, kv_dtype=kv_dtype)
    try:
        select_path(sess, forward_path)
        sess.spd_load_ngrams(tabs, synth.PAPER_LAMBDAS)
        dc = pkg.SpdDecodeCfg(k, alpha, 1.0, 0.1)
        cfg = O.DecodeCfg(k, alpha, 1.0, 0.1, synth.PAPER_LAMBDAS)
        _, recs, stats = teacher_forced(sess, lm, tabs, synth.PAPER_LAMBDAS, prefix, cfg, n_tokens, RTOL["bf16"], dc)
        print(shape.name, "scaled logit errors:", [f"{s['logit_err']:.2e}" for s in stats if "logit_err" in s])
        name = shape.name + (" (fp16 cache)" if kv_dtype == "fp16" else "")
        report_decisions(name, stats, n_tokens)
        return stats
    finally:
        sess.close()


REPORT = []   # one line per large-shape test, printed once past pytest's capture when the module ends


@pytest.fixture(scope="module", autouse=True)
def _print_report(request):
    yield
    if REPORT:
        capman = request.config.pluginmanager.getplugin("capturemanager")
        with capman.global_and_fixture_disabled():
            print()
            for line in REPORT:
                print("  " + line)


def report_decisions(name, stats, n_steps):
    """Every step's decision stage was compared exactly (on the GPU's own logits), and with the
    planted tables both the interpolated and the penalty form of an option occurred."""
    full = sum(bool(s.get("fully_compared")) for s in stats)
    line = (f"{name}: {full}/{n_steps} steps compared exactly on the GPU's own logits; options in both distributions: "
            f"{sum(s.get('own_overlap', 0) for s in stats)}, penalty form: {sum(s.get('own_penalty', 0) for s in stats)}, "
            f"dropped: {sum(s.get('own_dropped', 0) for s in stats)}; steps decisive against the oracle's logits: "
            f"{sum(bool(s.get('vocab_decisive')) for s in stats)}; worst scaled logit error "
            f"{max(s['logit_err'] for s in stats):.1e}")
    print(line)
    REPORT.append(line)
    assert full == n_steps
    assert_hit_paths_compared(stats)


@pytest.mark.timeout(600)
def test_7b_shape_two_layers_context_of_two_load_batches(forward_path):
    """Llama-2-7B widths (32 heads of 128), two layers, 200 cached positions: past the 160 rows
    a block's lanes hold per batch of loads, so the fused kernel's single attention item per
    head walks two batches (the per-operator path cuts the context into two chunks instead)."""
    _layer_truncated(synth.LLAMA7B, 2, 200, 3, 3, 8, forward_path)


@pytest.mark.timeout(600)
def test_7b_shape_two_layers_config3_context(forward_path):
    """The benchmark's longest context and largest k at the 7B widths, two layers: a 1030-token
    prefix (dense prefix pass over a chunk boundary of its token arena), attention cut into
    chunks that are merged across blocks, k = 8."""
    _layer_truncated(synth.LLAMA7B, 2, 1030, 8, 3, 7, forward_path)


@pytest.mark.timeout(600)
def test_13b_shape_two_layers(forward_path):
    """The 13B widths (d_model 5120, 40 heads, FFN 13824: rows of 1.25 and 3.375
    block passes), k = 5, two of its 40 layers."""
    _layer_truncated(synth.LLAMA13B, 2, 140, 5, 4, 13, forward_path)


@pytest.mark.timeout(600)
def test_70b_shape_one_layer(forward_path):
    """The 70B widths (d_model 8192, 64 query heads on 8 key/value heads, FFN
    28672), k = 3, one of its 80 layers; the prefix crosses an attention chunk."""
    _layer_truncated(synth.LLAMA70B, 1, 131, 3, 3, 70, forward_path)


@pytest.mark.parametrize("m", [8, 31, 33, 64, 96, 160, 257, 300, 531, 1043])
def test_dense_prefix_pass_matches_the_oracle_and_the_token_by_token_pass(m):
    """The prefix pass on the matrix cores (1024 tokens per weight pass) against the oracle's
    full-sequence forward and against the token-by-token pass: logits after the prefix, and
    three timesteps on top of the cache it filled.  Sizes straddle the products' tiles of 32, 64
    and 128 tokens and the 1024-token chunk (1043 = one full chunk + a short one at a non-zero
    position); grouped key/value heads."""
    pkg = P()
    shape = synth.ModelShape("small-bf16-dense", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=21)
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    lm = make_oracle(shape, w)
    cfg = O.DecodeCfg(3, 0.0)
    dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
    logits = {}
    for dense in (True, False):
        sess = session(shape, w, max_ctx=m + 16)
        try:
            assert sess.spd_get_dense_prefill()
            sess.spd_set_dense_prefill(dense)
            state, recs, stats = teacher_forced(sess, lm, None, synth.PAPER_LAMBDAS, prefix, cfg, 4, RTOL["bf16"], dc)
            assert max(s["logit_err"] for s in stats if "logit_err" in s) < 1e-4      # far inside the bf16 tolerance
            sess.spd_prefill(prefix)
            logits[dense] = sess.spd_read_logits()
        finally:
            sess.close()
    assert np.max(np.abs(logits[True] - logits[False])) <= 1e-4 * np.max(np.abs(logits[False]))


@pytest.mark.parametrize("layers,heads,kv_heads", [(1, 4, 1), (2, 16, 1), (1, 6, 6), (2, 64, 4)])
@pytest.mark.parametrize("m", [8, 65, 1024, 1025, 1029, 1040])
@pytest.mark.parametrize("kv_dtype,bound", [("fp32", 1e-4), ("fp16", 1e-3)])
def test_last_layer_of_the_prefix_pass_runs_for_the_last_token(layers, heads, kv_heads, m, kv_dtype, bound):
    """Key and value rows of the last layer for every token, with the query rows or without them (then 64 .. 768 rows: less than a tile,
    ragged), the rest of it for the prefix's last token, in a chunk's last row, alone or among a few in a chunk of its own (from 1025): the
    logits are those of the token-by-token pass (bounds as above: 16-bit activations, an fp16 cache's roundings), and so are a
    timestep's on top of the cache and those behind a committed draft of ten tokens, a chunk at a position that is no multiple of anything."""
    shape = synth.ModelShape("tail-bf16", layers, 384 if heads == 6 else 512, heads, kv_heads, 640, 512, "bf16")
    w = synth.make_weights(shape, seed=m)
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    sess = session(shape, w, max_ctx=m + 24, kv_dtype=kv_dtype)
    dc, got = P().SpdDecodeCfg(2, 0.0, 1.0, 0.1), {}
    try:
        for mode in (2, 1, None):
            sess.spd_set_dense_prefill(mode is not None)
            if mode is not None:
                assert all(sess.spd_test_force_last_query(mode, T) == (mode == 2) for T in (1, 8, 1024))
            sess.spd_prefill(prefix)
            got[mode] = [sess.spd_read_logits()]
            sess.spd_step(dc)
            sess.spd_set_state(np.tile(prefix[:5], (2, 1)).astype(np.int32), np.array([-1.0, -2.0], np.float32))
            sess.spd_step(dc)
            got[mode].append(sess.spd_read_logits())
        # a draft committed behind the prefix: its tokens are passed again from position m on; the whole text, one by one
        for mode in (2, 1):
            sess.spd_set_dense_prefill(True)
            sess.spd_test_force_last_query(mode, 10)
            sess.spd_prefill(prefix)
            for _ in range(10):
                sess.spd_step(dc)
            _, toks = sess.spd_commit(0.0)
            assert len(toks) == 10
            got[mode].append(sess.spd_read_logits())
            sess.spd_set_dense_prefill(False)
            sess.spd_prefill(np.concatenate([prefix, toks]))
            got[mode, "text"] = sess.spd_read_logits()
    finally:
        sess.close()
    for mode in (1, 2):
        for x, y in zip(got[mode], [*got[None], got[mode, "text"]], strict=True):
            assert np.max(np.abs(x - y)) <= bound * np.max(np.abs(y))


def test_last_query_goes_with_the_others_up_to_a_size():
    """The rule itself, on both sides of its line: 178 and 179 tokens of 4096 x 4096."""
    shape = synth.ModelShape("wide-query-bf16", 1, 4096, 32, 1, 128, 512, "bf16")
    w = synth.make_weights(shape, seed=6)
    sess = session(shape, w, max_ctx=1216, kv_dtype="fp16")
    try:
        assert [sess.spd_test_force_last_query(0, T) for T in (178, 179, 1024)] == [False, True, True]
        logits = []
        for dense in (True, False):
            sess.spd_set_dense_prefill(dense)
            for m in (178, 179, 1024 + 180):
                sess.spd_prefill(synth.make_prefix_zipf(shape.vocab, m, seed=m))
                logits.append(sess.spd_read_logits())
    finally:
        sess.close()
    for x, y in zip(logits[:3], logits[3:], strict=True):
        assert np.max(np.abs(x - y)) <= 1e-3 * np.max(np.abs(y))


FP32_CHUNKS = [synth.ModelShape("fp32-256", 2, 256, 4, 4, 1024, 512, "fp32"), synth.ModelShape("fp32-gqa", 3, 512, 8, 2, 1008, 512, "fp32"),
               synth.ModelShape("fp32-128", 1, 384, 3, 1, 464, 512, "fp32"), synth.ModelShape("fp32-one-head-64", 2, 64, 1, 1, 208, 512, "fp32"),
               synth.ModelShape("fp32-one-head-128", 2, 128, 1, 1, 464, 512, "fp32")]


@pytest.mark.parametrize("shape", FP32_CHUNKS, ids=lambda s: s.name)
@pytest.mark.parametrize("m", [2, 3, 5, 9, 15, 16, 17, 32, 33, 64, 100, 1025])
def test_fp32_prefix_pass_matches_the_token_by_token_pass(shape, m):
    """An fp32 model's prefix as chunks (one and two pieces of 16 tokens, ragged; 1025: a token in a chunk of its own; gate and up ragged
    against a batch of pieces; one head: its rotary table is the larger part of what the pass sets up): logits as token by token, and those
    of a timestep on top of the cache.  Either pass is 2 .. 7e-7 from 64 bits, which the oracle's sums are for up to 33 tokens here: 2e-6
    of the largest logit leaves room for one, 5e-6 for both."""
    w = synth.make_weights(shape, seed=m)
    prefix = synth.make_prefix_uniform(shape.vocab, m, seed=m)
    sess = session(shape, w, max_ctx=m + 4)
    got = []
    try:
        for chunks in (True, False):
            sess.spd_set_dense_prefill(chunks)
            sess.spd_set_kernel_timing(True)
            sess.spd_prefill(prefix)
            assert sess.spd_get_dense_prefill() == chunks and sess.spd_get_kernel_timing()["fused_forward"][1] == (0 if chunks else m)
            sess.spd_set_kernel_timing(False)
            got.append([sess.spd_read_logits()])
            sess.spd_step(P().SpdDecodeCfg(2, 0.0, 1.0, 0.1))
            sess.spd_set_state(np.resize(prefix, (2, 5)).astype(np.int32), np.array([-1.0, -2.0], np.float32))
            sess.spd_step(P().SpdDecodeCfg(2, 0.0, 1.0, 0.1))
            got[-1].append(sess.spd_read_logits())
    finally:
        sess.close()
    for x, y in zip(*got):
        assert np.max(np.abs(x - y)) <= 5e-6 * np.max(np.abs(y))
    if m <= 33:
        lm = make_oracle(shape, w, np.float64)
        want = lm.forward(lm.embedding_rows(prefix))
        for x, _ in got:
            assert np.max(np.abs(x - want)) <= 2e-6 * np.max(np.abs(want))


@pytest.mark.parametrize("layers,d,heads,ffn,fused,chunk", [
    (4, 1152, 9, 4112, True, False), (3, 1152, 9, 4112, True, True), (4, 1024, 8, 4112, True, True), (4, 1152, 9, 4096, True, True), (4, 1152, 9, 4112, False, True),
    (4, 128, 2, 6160, False, False), (3, 128, 2, 6160, False, True), (4, 256, 4, 2048, False, True),
    (8, 640, 10, 3072, True, False), (7, 640, 10, 3072, True, True), (8, 640, 10, 3088, True, True), (8, 576, 9, 3072, True, True), (8, 1024, 8, 256, True, False),
    (8, 1152, 9, 2048, True, False), (7, 1152, 9, 2048, True, True), (8, 1152, 9, 2064, True, True), (8, 640, 10, 1024, False, True)])
def test_fp32_prefix_of_two_tokens_goes_the_faster_way(layers, d, heads, ffn, fused, chunk):
    """Either side of every line of the rule, with the persistent forward and with a kernel per product (feed-forwards past 6144 have no
    other): two tokens are one chunk, which makes no launch of the forward, or two forwards; three are always a chunk."""
    shape = synth.ModelShape("two", layers, d, heads, heads, ffn, 512, "fp32")
    sess = session(shape, synth.make_weights(shape, seed=2))
    try:
        if not fused:
            sess.spd_set_fused(False)
        for m, forwards in ((2, 0 if chunk else 2), (3, 0)):
            sess.spd_set_kernel_timing(True)
            sess.spd_prefill(np.arange(m, dtype=np.int32))
            t = sess.spd_get_kernel_timing()
            assert t["fused_forward"][1] == (forwards if fused else 0) and t["gemv_qkv"][1] == (0 if fused else forwards * layers)
            assert np.isfinite(sess.spd_read_logits()).all()
    finally:
        sess.close()


PREFIX_TILES = [(32, 256), (64, 256), (64, 384), (128, 256), (128, 384), (64, 128), (32, 128)]
QKV, ATTN_OUT, GATE_UP, DOWN = range(4)


@pytest.mark.parametrize("kv_dtype,bound", [("fp32", 1e-4), ("fp16", 1e-3)])
@pytest.mark.parametrize("m", [70, 230])
def test_prefix_products_of_every_tile_shape(m, kv_dtype, bound):
    """Every tile shape of the prefix products, with its epilogue in the product and as partial sums of one to five blocks per k
    range, asked for one product at a time whatever the estimate would choose: the logits are those of the token-by-token
    pass (whose activations are not cut to 16 bits; with an fp16 cache some entries go to the other neighbour).
    m: token tiles of 32, 64 and 128 that end ragged, one to eight of them; columns: QKV 896, gate and up 1408 each, ragged in
    tiles of 256 and 384; five query heads share a cached one."""
    shape = synth.ModelShape("ragged-bf16", 3, 640, 10, 2, 1408, 1024, "bf16")
    w = synth.make_weights(shape, seed=17)
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    sess = session(shape, w, max_ctx=m + 8, kv_dtype=kv_dtype)
    seen = set()
    try:
        sess.spd_set_dense_prefill(False)
        sess.spd_prefill(prefix)
        want = sess.spd_read_logits()
        sess.spd_set_dense_prefill(True)
        for product in (QKV, ATTN_OUT, GATE_UP, DOWN):
            for tile, size in enumerate(PREFIX_TILES):
                for splits in (1, 2, 3, 4, 5):
                    cut = sess.spd_test_force_prefill_cut(product, tile, splits, m)
                    if cut[:3] != (*size, splits):      # too few steps for that many blocks (or, gate and up, no room for the sums)
                        assert splits > (5 if product == DOWN else 2 if product == GATE_UP and m == 230 else 3), cut
                        continue
                    sess.spd_prefill(prefix)
                    err = np.max(np.abs(sess.spd_read_logits() - want)) / np.max(np.abs(want))
                    assert err <= bound, f"product {product}, tile {size}, {splits} blocks per k range: {err:.2e}"
                    seen.add((product, size, cut[3]))
            sess.spd_test_force_prefill_cut(product, -1, 0, m)
    finally:
        sess.close()
    fused = {(QKV, t, True) for t in PREFIX_TILES} | {(GATE_UP, t, True) for t in PREFIX_TILES if t not in [(32, 256), (64, 384), (128, 384)]}
    assert seen == fused | {(p, t, False) for p in (QKV, ATTN_OUT, GATE_UP, DOWN) for t in PREFIX_TILES}


GATE_UP_TILES = [(64, 96), (64, 192), (128, 192), (128, 320), (128, 384), (192, 192), (192, 256)]


@pytest.mark.parametrize("m", [30, 70, 193, 230, 385])
def test_gate_and_up_of_every_tile_shape(m):
    """The shapes only gate and up has, asked for one after the other, as one block per k range with its epilogue and as partial sums: token tiles
    of 64, 128 and 192 that end ragged; 1408 units in halves of 48 .. 192, ragged in most.  Bound as above.  For other products they do not exist."""
    shape = synth.ModelShape("ragged-bf16", 3, 640, 10, 2, 1408, 1024, "bf16")
    w = synth.make_weights(shape, seed=19)
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    sess = session(shape, w, max_ctx=m + 8)
    seen = set()
    try:
        sess.spd_set_dense_prefill(False)
        sess.spd_prefill(prefix)
        want = sess.spd_read_logits()
        sess.spd_set_dense_prefill(True)
        for tile, size in enumerate(GATE_UP_TILES, len(PREFIX_TILES)):
            for splits in (1, 2, 3):
                cut = sess.spd_test_force_prefill_cut(GATE_UP, tile, splits, m)
                if cut[:3] != (*size, splits):
                    continue
                assert cut[3] == (splits == 1)
                sess.spd_prefill(prefix)
                err = np.max(np.abs(sess.spd_read_logits() - want)) / np.max(np.abs(want))
                assert err <= 1e-4, f"tile {size}, {splits} blocks per k range: {err:.2e}"
                seen.add((size, cut[3]))
            sess.spd_test_force_prefill_cut(GATE_UP, -1, 0, m)
            for product in (QKV, ATTN_OUT, DOWN):
                assert sess.spd_test_force_prefill_cut(product, tile, 1, m)[:2] in PREFIX_TILES
                sess.spd_test_force_prefill_cut(product, -1, 0, m)
    finally:
        sess.close()
    assert {s for s, fused in seen if fused} == set(GATE_UP_TILES) and (m > 230 or {s for s, fused in seen if not fused} == set(GATE_UP_TILES))


@pytest.mark.parametrize("m", [9, 32, 61])
def test_prefix_products_that_start_inside_their_k_range(m):
    """Rows of 8 KB and one token tile: blocks start an eighth of their k range apart and wrap round, with 4 to 64 steps per
    block (less than an eighth's worth, ragged eighths, a last split shorter than the others); bound as above."""
    shape = synth.ModelShape("rotated-bf16", 2, 4096, 32, 4, 4096, 512, "bf16")
    w = synth.make_weights(shape, seed=3)
    sess, seen = session(shape, w, max_ctx=m + 8), set()
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    try:
        sess.spd_set_dense_prefill(False)
        sess.spd_prefill(prefix)
        want = sess.spd_read_logits()
        sess.spd_set_dense_prefill(True)
        for product in (QKV, ATTN_OUT, GATE_UP, DOWN):
            for tile, size in enumerate(PREFIX_TILES):
                for splits in (1, 3, 6, 7, 11, 16):
                    if size[0] > 64 or size[0] < m or sess.spd_test_force_prefill_cut(product, tile, splits, m)[:3] != (*size, splits):
                        continue
                    seen.add((product, size, splits))
                    sess.spd_prefill(prefix)
                    err = np.max(np.abs(sess.spd_read_logits() - want)) / np.max(np.abs(want))
                    assert err <= 1e-4, f"product {product}, tile {size}, {splits} blocks per k range: {err:.2e}"
            sess.spd_test_force_prefill_cut(product, -1, 0, m)
    finally:
        sess.close()
    # (61 tokens' partial sums of QKV in 16 splits have no room)
    assert seen == {(p, t, n) for p in (QKV, ATTN_OUT, GATE_UP, DOWN) for t in PREFIX_TILES for n in (1, 3, 6, 7, 11, 16)
                    if m <= t[0] <= 64 and not (m == 61 and p == QKV and n == 16)}


@pytest.mark.timeout(600)
@pytest.mark.parametrize("m", [66, 531])
def test_prefix_products_at_7b_widths(m):
    """As the estimate cuts them: 66 tokens (split k ranges throughout) and 531 (QKV, gate and up without)."""
    _layer_truncated(synth.LLAMA7B, 1, m, 2, 2, 31, "fused")


# ---- the fp16 key/value cache a bf16 model may ask for (spd_model_cfg.kv_dtype): every kernel that
# writes or reads the cache, against the same oracle (which keeps its keys and values unrounded), to
# the bf16 tolerance; the rounding of the cache is the only difference to the fp32-cache cases above,
# whose tighter bounds pin the logic.
FP16_CACHE_LOGIT_ERR = 8e-3   # of the largest |logit|: 11 significant bits in every cached key and value


def test_fp16_cache_small_model_gqa(forward_path):
    shape = synth.ModelShape("small-bf16", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=5)
    prefix = synth.make_prefix_zipf(shape.vocab, 37, seed=5)
    base = synth.make_ngram_tables_zipf(shape.vocab, 30_000, seed=5)
    planted = planted_tables(shape, w, base, prefix, 3, 8)
    _, _, stats = run_teacher_forced(shape, w, planted, synth.PAPER_LAMBDAS, prefix, 3, 0.54, 8, path=forward_path, kv_dtype="fp16")
    assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR


@pytest.mark.timeout(600)
@pytest.mark.parametrize("prefix_len,k", [(40, 3), (200, 3), (300, 5), (1030, 8)])
def test_fp16_cache_7b_shape_two_layers(forward_path, prefix_len, k):
    """Llama-2-7B widths, two layers, fp16 cache: a short context, one attention item per head in
    two batches of loads (200), chunks merged across blocks (300, and the benchmark's 1030
    with k = 8, whose prefix also crosses a chunk of the dense prefix pass)."""
    stats = _layer_truncated(synth.LLAMA7B, 2, prefix_len, k, 3, 8, forward_path, kv_dtype="fp16")
    assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR


@pytest.mark.timeout(600)
def test_fp16_cache_13b_shape_two_layers():
    stats = _layer_truncated(synth.LLAMA13B, 2, 140, 5, 4, 13, "fused", kv_dtype="fp16")
    assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR


@pytest.mark.timeout(600)
def test_fp16_cache_70b_shape_one_layer():
    """Grouped key/value heads (8 query heads per cached head) over an attention chunk boundary."""
    stats = _layer_truncated(synth.LLAMA70B, 1, 131, 3, 3, 70, "fused", kv_dtype="fp16")
    assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR


@pytest.mark.parametrize("m", [8, 33, 96, 300, 1043])
def test_fp16_cache_dense_prefix_pass(m):
    """The prefix pass on the matrix cores and the token-by-token pass fill the fp16 cache with the
    same roundings of (nearly) the same values: their logits agree far more closely than either
    agrees with the oracle."""
    shape = synth.ModelShape("small-bf16-dense", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=21)
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    lm = make_oracle(shape, w)
    cfg = O.DecodeCfg(3, 0.0)
    dc = P().SpdDecodeCfg(3, 0.0, 1.0, 0.1)
    logits = {}
    for dense in (True, False):
        sess = session(shape, w, max_ctx=m + 16, kv_dtype="fp16")
        try:
            sess.spd_set_dense_prefill(dense)
            state, recs, stats = teacher_forced(sess, lm, None, synth.PAPER_LAMBDAS, prefix, cfg, 4, RTOL["bf16"], dc)
            assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR
            sess.spd_prefill(prefix)
            logits[dense] = sess.spd_read_logits()
        finally:
            sess.close()
    assert np.max(np.abs(logits[True] - logits[False])) <= 1e-3 * np.max(np.abs(logits[False]))


@pytest.mark.parametrize("heads,m", [(4, 65), (8, 131)])
def test_fp16_cache_prefix_attention_does_not_depend_on_the_scale_of_queries(heads, m):
    """The prefix pass's attention over the fp16 cache splits a query's row into two fp16 numbers after scaling it by
    a power of two.  Queries 2^-8 and 2^4 times as large against keys scaled the other way leave the scores as they are,
    up to the fp16 rounding of keys that become subnormal (6e-8 in a few of them)."""
    pkg = P()
    shape = synth.ModelShape("small-bf16-dense", 2, 512, heads, heads, 1408, 1024, "bf16")
    prefix = synth.make_prefix_zipf(shape.vocab, m, seed=m)
    logits = []
    for q_scale, k_scale in ((0, 0), (-8, 8), (4, -4)):
        w = synth.make_weights(shape, seed=3)
        for l in range(shape.n_layers):
            for name, scale in (("wq", q_scale), ("wk", k_scale)):
                key = f"layers.{l}.{name}"
                w[key] = synth.bf16_bits(synth.bf16_widen(w[key]) * np.float32(2.0 ** scale)).reshape(w[key].shape)
        sess = session(shape, w, max_ctx=m + 4, kv_dtype="fp16")
        try:
            sess.spd_prefill(prefix)
            logits.append(sess.spd_read_logits())
        finally:
            sess.close()
    for z in logits[1:]:
        assert np.max(np.abs(z - logits[0])) <= 1e-5 * np.max(np.abs(logits[0]))


def test_fp16_cache_head_width_32_plain_prefix_attention():
    """d_head 32: the prefix pass uses its plain (not matrix-core) attention kernel."""
    shape = synth.ModelShape("small-bf16-dh32", 2, 256, 8, 4, 512, 1024, "bf16")
    w = synth.make_weights(shape, seed=23)
    prefix = synth.make_prefix_zipf(shape.vocab, 150, seed=23)
    _, _, stats = run_teacher_forced(shape, w, None, synth.PAPER_LAMBDAS, prefix, 3, 0.0, 4, max_ctx=200, kv_dtype="fp16")
    assert max(s["logit_err"] for s in stats if "logit_err" in s) < FP16_CACHE_LOGIT_ERR


def test_fp16_cache_generation_repeats_its_bits_across_the_switch_of_reading_widths():
    """A free-running generation of the persistent forward whose context passes 160 positions (where it goes from 8-byte to
    16-byte pieces of the fp16 cache) gives the same bits each time, whatever the graph switch says; the per-operator
    forward agrees to rounding."""
    pkg = P()
    shape = synth.ModelShape("small-bf16", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=5)
    prefix = synth.make_prefix_zipf(shape.vocab, 150, seed=9)
    dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
    sess = session(shape, w, max_ctx=200, kv_dtype="fp16")
    try:
        select_path(sess, "fused")
        drafts, scores = sess.spd_generate(prefix, dc, 24)
        logits = sess.spd_read_logits()
        for graph in (False, True):
            sess.spd_set_graph(graph)
            drafts2, scores2 = sess.spd_generate(prefix, dc, 24)
            assert np.array_equal(drafts, drafts2) and np.array_equal(scores, scores2)
            assert np.array_equal(logits, sess.spd_read_logits())
        # the same prefix and the same first timesteps through one kernel per operator
        sess.spd_prefill(prefix)
        sess.spd_step(dc)
        sess.spd_step(dc)
        fused = sess.spd_read_logits()
        sess.spd_set_fused(False)
        sess.spd_prefill(prefix)
        sess.spd_step(dc)
        sess.spd_step(dc)
        per_op = sess.spd_read_logits()
        np.testing.assert_allclose(fused, per_op, rtol=0, atol=2e-5 * np.abs(per_op).max())
    finally:
        sess.close()


@pytest.mark.parametrize("n_prefix", [150, 500])
def test_fp16_cache_graph_replay_of_the_per_operator_forward(n_prefix):
    """bf16 weights, an fp16 cache, four query heads per cached head of 64: one captured timestep is replayed while the context grows, from
    500 tokens on past the 512 positions that are one attention chunk.  Each generation has the bits of plain launches."""
    pkg = P()
    shape = synth.ModelShape("small-bf16", 3, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=5)
    prefix = synth.make_prefix_zipf(shape.vocab, n_prefix, seed=9)
    dc, sc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1), pkg.SpdSampleCfg(0.9, 1.0)
    sess = session(shape, w, max_ctx=n_prefix + 30, kv_dtype="fp16")
    try:
        select_path(sess, "per_operator")
        runs = []
        for graph in (False, True, True, False, True):
            sess.spd_set_graph(graph)
            drafts, scores = sess.spd_generate(prefix, dc, 24)
            logits = sess.spd_read_logits()
            sess.spd_prefill(prefix)
            sampled = [sess.spd_nucleus_step(sc, float(u)) for u in np.linspace(0.05, 0.95, 20)]
            runs.append((drafts.tolist(), scores.tolist(), logits.tolist(), sampled, sess.spd_read_logits().tolist()))
        assert all(r == runs[0] for r in runs)
    finally:
        sess.close()


@pytest.mark.parametrize("shape", [synth.ModelShape("fp32-heads-of-16", 2, 336, 21, 7, 1008, 512, "fp32"), synth.ModelShape("bf16-320", 1, 320, 5, 5, 640, 512, "bf16")], ids=lambda s: s.name)
def test_dense_prefix_pass_is_refused_where_it_does_not_exist(shape):
    sess = session(shape, synth.make_weights(shape, seed=1))
    try:
        assert not sess.spd_get_dense_prefill()
        with pytest.raises(P().SpdError):
            sess.spd_set_dense_prefill(True)
        sess.spd_set_dense_prefill(False)
        assert not sess.spd_get_dense_prefill()
    finally:
        sess.close()


@pytest.mark.parametrize("max_ctx", [40, 1500])
def test_fp32_workspace_without_the_chunk_pass(max_ctx, monkeypatch):
    """A workspace that has no room for the chunk's rows (all but its last byte, none) makes a context without that pass, with the logits of
    the token-by-token one; a byte less than the rest is refused."""
    from paper_2405_18400_amd import binding
    shape = synth.ModelShape("small-workspace", 2, 256, 4, 2, 512, 512, "fp32")
    w, prefix = synth.make_weights(shape, seed=4), synth.make_prefix_uniform(shape.vocab, 30, seed=4)
    whole, rows = binding.spd_workspace_bytes(binding.model_cfg(shape, max_ctx, 8)), min(max_ctx, 1024)
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    chunk = 3 * up(rows * 256 * 4) + up(rows * 512 * 4) + up(rows * 32 * 8)
    logits = []
    for size in (whole, whole - 1, whole - chunk):
        monkeypatch.setattr(binding, "spd_workspace_bytes", lambda cfg: size)
        sess = session(shape, w, max_ctx=max_ctx)
        try:
            assert sess.spd_get_dense_prefill() == (size == whole)
            if size == whole:
                sess.spd_set_dense_prefill(False)
            else:
                with pytest.raises(P().SpdError):
                    sess.spd_set_dense_prefill(True)
            sess.spd_prefill(prefix)
            logits.append(sess.spd_read_logits())
        finally:
            sess.close()
    assert all(np.array_equal(z, logits[0]) for z in logits)
    monkeypatch.setattr(binding, "spd_workspace_bytes", lambda cfg: whole - chunk - 1)
    with pytest.raises(P().SpdError):
        session(shape, w, max_ctx=max_ctx)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
def test_dense_prefix_pass_is_switched_off_and_on_again(dtype):
    """What the getter says is what runs (a token-by-token pass of m tokens is m launches of the forward, the dense one none), and setting
    what it said restores it: the logits are those of the pass before, bit for bit."""
    shape = synth.ModelShape("switch", 2, 256, 4, 4, 512, 512, dtype)
    prefix = synth.make_prefix_uniform(shape.vocab, 20, seed=3)
    sess = session(shape, synth.make_weights(shape, seed=3))
    try:
        seen = []
        for _ in range(2):
            was = sess.spd_get_dense_prefill()
            for on in (was, False, was):
                sess.spd_set_dense_prefill(on)
                assert sess.spd_get_dense_prefill() == on
                sess.spd_set_kernel_timing(True)
                sess.spd_prefill(prefix)
                launches = sess.spd_get_kernel_timing()["fused_forward"][1]
                sess.spd_set_kernel_timing(False)
                assert launches == (0 if on else len(prefix))
                seen.append((on, sess.spd_read_logits()))
        for on, z in seen:
            assert np.array_equal(z, next(y for o, y in seen if o == on))
        assert {on for on, _ in seen} == {True, False}
    finally:
        sess.close()


def test_fused_and_per_operator_forward_agree(tiny):
    """Same inputs through both forward paths, from the prefix on: logits agree to fp32 rounding."""
    shape, w, tabs, prefix = tiny
    pkg = P()
    out = {}
    for path in ("fused", "per_operator"):
        sess = session(shape, w)
        try:
            select_path(sess, path)
            sess.spd_set_dense_prefill(False)
            sess.spd_prefill(prefix)
            logits = sess.spd_read_logits()
            drafts, scores = sess.spd_generate(prefix, pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1), 6)
            out[path] = (logits, drafts, scores)
        finally:
            sess.close()
    np.testing.assert_allclose(out["fused"][0], out["per_operator"][0], rtol=0, atol=2e-5 * np.abs(out["fused"][0]).max())


@pytest.mark.parametrize("dtype,d,heads,kv_heads,ffn", [
    ("fp32", 32, 2, 1, 40), ("fp32", 256, 4, 2, 1024), ("fp32", 256, 4, 4, 1028), ("fp32", 272, 17, 17, 1024), ("fp32", 1024, 8, 8, 3072), ("fp32", 1024, 8, 2, 3076),
    ("fp32", 1040, 65, 13, 3072), ("bf16", 512, 8, 8, 2048), ("bf16", 512, 8, 2, 2056), ("bf16", 528, 33, 33, 2048), ("bf16", 2048, 16, 4, 6144),
    ("bf16", 2048, 16, 16, 6152), ("bf16", 2064, 129, 129, 6144)])
def test_persistent_forward_of_one_four_and_eight_waves_to_a_row(dtype, d, heads, kv_heads, ffn):
    """Either side of every line between one, four and eight waves to a row (the last widths that one and four waves hold, and the first
    that they do not), rows far narrower than one wave, a vocabulary that leaves the last tiles ragged: prefix token by token, then
    timesteps, against the forward of one kernel per product.  Both are fp32 sums of the same products in another order."""
    pkg = P()
    shape = synth.ModelShape("waves", 2, d, heads, kv_heads, ffn, 518, dtype)
    w = synth.make_weights(shape, seed=d)
    prefix = synth.make_prefix_uniform(shape.vocab, 5, seed=ffn)
    dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
    for kv_dtype in ("fp32", "fp16")[:1 if dtype == "fp32" else 2]:
        sess = session(shape, w, max_ctx=12, kv_dtype=kv_dtype)
        try:
            sess.spd_set_dense_prefill(False)
            logits = []
            for path in ("fused", "per_operator"):
                select_path(sess, path)
                sess.spd_prefill(prefix)
                got = [sess.spd_read_logits()]
                sess.spd_step(dc)
                for t in range(3):
                    sess.spd_set_state(np.resize(prefix + t, (3, 5)).astype(np.int32) % shape.vocab, np.array([-1.0, -2.0, -2.5], np.float32))
                    sess.spd_step(dc)
                    got.append(sess.spd_read_logits())
                logits.append(got)
            for x, y in zip(*logits):
                np.testing.assert_allclose(x, y, rtol=0, atol=(2e-5 if kv_dtype == "fp32" else 1e-3) * np.abs(y).max())   # (1e-3: keys and values that round to the other fp16 neighbour)
        finally:
            sess.close()


@pytest.mark.parametrize("max_ctx", [512, 513])
def test_per_operator_attention_where_the_merge_begins(max_ctx):
    """Four query heads per cached head of 64 in fp16: up to 512 positions the longest context is one chunk and attention one
    launch, one position more and a merge follows it.  Up to the last position, against the persistent kernel."""
    pkg = P()
    shape = synth.ModelShape("small-bf16", 2, 512, 8, 2, 1408, 2048, "bf16")
    w = synth.make_weights(shape, seed=5)
    prefix = synth.make_prefix_zipf(shape.vocab, max_ctx - 2, seed=9)
    dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
    sess = session(shape, w, max_ctx=max_ctx, kv_dtype="fp16")
    try:
        logits = []
        for path in ("fused", "per_operator"):
            select_path(sess, path)
            sess.spd_prefill(prefix)
            for _ in range(3):
                sess.spd_step(dc)
            logits.append(sess.spd_read_logits())
        np.testing.assert_allclose(logits[0], logits[1], rtol=0, atol=2e-5 * np.abs(logits[1]).max())
    finally:
        sess.close()


@pytest.mark.parametrize("dense", [True, False])
def test_generate_free_running_matches_until_first_undecided_step(tiny, dense):
    shape, w, tabs, prefix = tiny
    pkg = P()
    lam = (0.01, 0.04, 0.0, 0.0, 0.0)
    planted = planted_tables(shape, w, tabs, prefix, 3, 10)
    sess = session(shape, w)
    try:
        sess.spd_set_dense_prefill(dense)
        sess.spd_load_ngrams(planted, lam)
        dc = pkg.SpdDecodeCfg(3, 0.5, 1.0, 0.1)
        drafts, scores = sess.spd_generate(prefix, dc, 10)
        lm = make_oracle(shape, w)
        state, recs = O.generate(lm, O.NgramTables(planted), prefix, O.DecodeCfg(3, 0.5, 1.0, 0.1, lam), 10)
        tol = RTOL["fp32"] * max(float(np.max(np.abs(r.logits))) for r in recs)
        decided = 0
        for r in recs:
            if r.gap_vocab <= 4 * tol or r.gap_prune <= 4 * tol:
                break
            decided += 1
        assert decided >= 5, "synthetic case too close to ties to say anything"
        if decided == len(recs):
            assert drafts.tolist() == state.drafts
            np.testing.assert_allclose(scores, state.logscores, atol=1e-3)
        else:
            # up to the first undecided step both sides hold the same set of drafts; whatever the
            # GPU kept later descends from that set
            upto = {tuple(d) for d in recs[decided].state_in.drafts}
            assert {tuple(d[:decided]) for d in drafts.tolist()} <= upto
        # and so does a second generation (determinism, counters reset, state reset), plainly launched and, with one kernel
        # per product, replayed from a graph
        for fused in (True, False):
            sess.spd_set_fused(fused)
            runs = [(drafts.tolist(), scores.tolist())] if fused else []
            for graph in (False, True, True):
                sess.spd_set_graph(graph)
                again, scores2 = sess.spd_generate(prefix, dc, 10)
                runs.append((again.tolist(), scores2.tolist()))
            assert all(r == runs[0] for r in runs)
    finally:
        sess.close()


def test_graph_replay_of_the_per_operator_forward_equals_plain_launches(tiny):
    """The graphs (timestep, nucleus timestep, prefix token) are the per-operator forward's: replayed several times, with a new prefix and
    the program's own calls between, and each time the bits of plain launches; with the persistent forward the switch changes nothing."""
    shape, w, tabs, prefix = tiny
    pkg = P()
    dc, sc = pkg.SpdDecodeCfg(3, 0.5, 1.0, 0.1), pkg.SpdSampleCfg(0.9, 1.0)
    sess = session(shape, w)
    try:
        sess.spd_load_ngrams(tabs, (0.01, 0.04, 0.0, 0.0, 0.0))
        sess.spd_set_dense_prefill(False)
        for fused in (False, True):
            sess.spd_set_fused(fused)
            runs = []
            for graph in (False, True, True, False, True):
                sess.spd_set_graph(graph)
                drafts, scores = sess.spd_generate(prefix, dc, 7)
                logits = sess.spd_read_logits()
                sess.spd_prefill(prefix[:9])
                sampled = [sess.spd_nucleus_step(sc, u) for u in (0.2, 0.9, 0.4, 0.6)]
                runs.append((drafts.tolist(), scores.tolist(), logits.tolist(), sampled))
            assert all(r == runs[0] for r in runs)
    finally:
        sess.close()


@pytest.mark.parametrize("fused", [True, False])
def test_logits_that_are_no_numbers_give_tokens_that_exist(tiny, fused):
    """Fewer numbers among the logits than drafts are kept: the numbers first, in their order, and for the rest ids of the vocabulary
    (they were 2^31 - 1, which the next forward looked up in the embeddings); scores are NaN, and stay so through the timesteps."""
    shape, w, _, prefix = tiny
    pkg = P()
    dc = pkg.SpdDecodeCfg(4, 0.0, 1.0, 0.1)
    sess = session(shape, w)
    try:
        sess.spd_set_fused(fused)
        for numbers in ([], [5], [9, 3, shape.vocab - 1]):
            z = torch.full((shape.vocab,), float("nan"))
            z[numbers] = torch.arange(len(numbers), 0, -1, dtype=torch.float32)
            z = z.cuda()
            sess.spd_prefill(prefix)
            for t in range(2):
                sess.spd_expand_prune(dc, z, t == 0)
                ids = sess.spd_get_step_info(4)[0]
                tails, scores, _ = sess.spd_get_state()
                assert ids[:len(numbers)].tolist() == numbers and np.all((ids >= 0) & (ids < shape.vocab))
                assert np.all((tails[:, -1] >= 0) & (tails[:, -1] < shape.vocab)) and np.isnan(scores).all()
            for _ in range(2):
                tok, _, sc = sess.spd_step(dc)
                assert np.all((tok >= 0) & (tok < shape.vocab)) and np.isnan(sc).all()
            sess.spd_prefill(prefix)
            sess.spd_nucleus_sample(pkg.SpdSampleCfg(0.9, 1.0), 0.5, z, True)
            assert 0 <= sess.spd_get_state()[0][0, -1] < shape.vocab
        sess.spd_prefill(prefix)                   # and a prefix pass starts from numbers again
        assert np.isfinite(sess.spd_step(dc)[2]).all()
    finally:
        sess.close()


def test_k1_is_greedy_on_the_gpu(tiny):
    shape, w, _, prefix = tiny
    pkg = P()
    sess = session(shape, w)
    try:
        drafts, _ = sess.spd_generate(prefix, pkg.SpdDecodeCfg(1, 0.0, 1.0, 0.1), 8)
        lm = make_oracle(shape, w)
        logits = lm.forward(lm.embedding_rows(prefix))
        for t in range(8):
            srt = np.sort(logits)[::-1]
            if srt[0] - srt[1] < 1e-3:
                break
            assert drafts[0, t] == int(np.argmax(logits))
            logits = lm.forward(lm.embedding_rows([int(np.argmax(logits))]))
    finally:
        sess.close()


@pytest.mark.parametrize("vocab,k", [(64, 16), (1026, 16), (4098, 7), (32000, 1), (32000, 16), (140000, 16)])
def test_kept_tokens_and_log_softmax_of_masked_logits(vocab, k):
    """KeepTopK and the log-softmax from given logits: whole slices masked with -inf, whole slices equal, +0 and -0
    tied, more candidates than one pass of the merge takes (k = 16 of 32000 and more), slices of more than 1024."""
    pkg = P()
    shape = synth.ModelShape("select", 1, 128, 2, 2, 256, vocab, "fp32")
    rng = np.random.default_rng(vocab + k)
    z = np.round(rng.standard_normal(vocab) * 2, 2).astype(np.float32)      # many exact ties
    if vocab > 2048:
        z[1000:2100] = -np.inf
        z[2100:3300] = 1.25
    z[:40] = np.where(np.arange(40) % 2, np.float32(-0.0), np.float32(0.0))
    cases = [z, np.where(np.arange(vocab) % 40 == 3, z, -np.inf).astype(np.float32) if vocab >= 40 * k else z,
             np.where(np.abs(z) > 0, -1.0, z).astype(np.float32)]           # only the zeros stand out
    sess = pkg.Session(shape, synth.make_weights(shape, seed=1), max_ctx=16, k_max=16)
    try:
        sess.spd_prefill(np.zeros(2, np.int32))
        for x in cases:
            sess.spd_expand_prune(pkg.SpdDecodeCfg(k, 0.0, 1.0, 0.1), torch.from_numpy(x).cuda(), True)
            ids, logp, _, _, _ = sess.spd_get_step_info(k)
            want = np.lexsort((np.arange(vocab), -x.astype(np.float64)))[:k]
            assert ids.tolist() == want.tolist()
            x64 = x.astype(np.float64)
            lse = x64.max() + np.log(np.exp(x64 - x64.max()).sum())
            np.testing.assert_allclose(logp, x64[want] - lse, atol=4e-6)   # a few fp32 roundings of numbers below 16
    finally:
        sess.close()


def test_expand_prune_on_scripted_logits_with_ties(tiny):
    """Decision logic alone: crafted logits (exact ties included) fed straight to the
    post-forward kernels; everything here is integer- or fp32-exact, so results are compared
    without a gap allowance."""
    shape, w, tabs, prefix = tiny
    pkg = P()
    lam = synth.PAPER_LAMBDAS
    rng = np.random.default_rng(0)
    sess = session(shape, w)
    try:
        k = 4
        corpus = rng.integers(0, 12, size=600)
        from collections import Counter
        ctabs = {}
        for n in range(2, 7):
            c = Counter(tuple(corpus[i:i + n]) for i in range(len(corpus) - n + 1))
            ctabs[n] = (np.array(list(c.keys()), np.int32).reshape(-1, n), np.array(list(c.values()), np.uint32))
        sess.spd_load_ngrams(ctabs, lam)
        otabs = O.NgramTables(ctabs)
        pre = corpus[:7].astype(np.int32)
        sess.spd_prefill(pre)
        for alpha in (0.54, 0.0):
            dc = pkg.SpdDecodeCfg(k, alpha, 1.0, 0.1)
            cfg = O.DecodeCfg(k, alpha, 1.0, 0.1, lam)
            state = None
            for step in range(6):
                z = np.full(shape.vocab, -8.0, np.float32)
                z[:14] = rng.integers(0, 4, size=14).astype(np.float32)      # many exact ties among 14 tokens
                if state is None:
                    state, rec = O.first_step(z, pre, cfg)
                else:
                    state, rec = O.expand_and_prune(state, z, otabs, cfg)
                sess.spd_expand_prune(dc, torch.from_numpy(z).cuda(), first=(step == 0))
                tails, sc, gamma = sess.spd_get_state()
                ids, lp, cs, cv, cp = sess.spd_get_step_info(k)
                assert list(ids) == list(rec.top_ids)
                np.testing.assert_allclose(lp, rec.top_logp, rtol=2e-6)
                assert np.array_equal(tails, tails_of(state))
                np.testing.assert_allclose(sc, state.logscores, rtol=1e-5, atol=1e-5)
                np.testing.assert_allclose(gamma, O.superposition_weights(state.logscores), rtol=1e-5)
                assert abs(float(gamma.sum()) - 1.0) < 1e-6
                if step > 0 and alpha > 0:
                    np.testing.assert_allclose(cp, rec.pngram, rtol=1e-6)
                    assert rec.pngram.max() > 0
                # keep both sides on identical scores so ties stay ties
                sess.spd_set_state(tails_of(state), state.logscores)
    finally:
        sess.close()


def test_many_small_hash_tables_against_the_oracle(tiny):
    """The n-gram probabilities of the k x k options on 150 different tiny tables (about a
    hundred keys in about two hundred slots each): clusters of displaced keys occur all over
    such a table, at its end too, where the probe sequence wraps round to slot 0; the oracle
    looks the same n-grams up in plain dictionaries.  Exact comparison (counts are integers,
    the mixture of Eq. 3 is a handful of fp32 operations in a fixed order)."""
    shape, w, _, _ = tiny
    pkg = P()
    lam = synth.PAPER_LAMBDAS
    from collections import Counter
    sess = session(shape, w)
    try:
        k = 3
        dc = pkg.SpdDecodeCfg(k, 0.54, 1.0, 0.1)
        cfg = O.DecodeCfg(k, 0.54, 1.0, 0.1, lam)
        hits = 0
        for seed in range(150):
            rng = np.random.default_rng(1000 + seed)
            corpus = rng.integers(0, 6, size=16)
            ctabs = {}
            for n in range(2, 7):
                c = Counter(tuple(corpus[i:i + n]) for i in range(len(corpus) - n + 1))
                ctabs[n] = (np.array(list(c.keys()), np.int32).reshape(-1, n), np.array(list(c.values()), np.uint32))
            sess.spd_load_ngrams(ctabs, lam)
            otabs = O.NgramTables(ctabs)
            pre = corpus[:6].astype(np.int32)
            sess.spd_prefill(pre)
            state = None
            for step in range(3):
                z = np.full(shape.vocab, -8.0, np.float32)
                z[:6] = rng.permutation(6).astype(np.float32)   # distinct: no ties, top-k inside the corpus alphabet
                if state is None:
                    state, rec = O.first_step(z, pre, cfg)
                else:
                    state, rec = O.expand_and_prune(state, z, otabs, cfg)
                sess.spd_expand_prune(dc, torch.from_numpy(z).cuda(), first=(step == 0))
                ids, lp, cs, cv, cp = sess.spd_get_step_info(k)
                assert list(ids) == list(rec.top_ids), f"table {seed} step {step}"
                if step > 0:
                    np.testing.assert_allclose(cp, rec.pngram, rtol=1e-6, err_msg=f"table {seed} step {step}")
                    hits += int(np.count_nonzero(rec.pngram))
                sess.spd_set_state(tails_of(state), state.logscores)
        assert hits > 300   # the tables were hit, not merely missed consistently
    finally:
        sess.close()


def test_error_paths(tiny):
    shape, w, tabs, prefix = tiny
    pkg = P()
    sess = session(shape, w, max_ctx=20, k_max=4)
    try:
        dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_step(dc)
        assert e.value.code == -2
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_prefill(np.arange(20))
        assert e.value.code == -3
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_prefill([0, shape.vocab])
        assert e.value.code == -1
        sess.spd_prefill(prefix)                      # 16 positions of 20
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_step(pkg.SpdDecodeCfg(5, 0.0, 1.0, 0.1))      # k > k_max
        assert e.value.code == -1
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_step(pkg.SpdDecodeCfg(3, 0.5, 1.0, 0.1))      # alpha > 0 without tables
        assert e.value.code == -1
        for _ in range(5):                            # first step + 4 forwards fill the cache
            sess.spd_step(dc)
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_step(dc)
        assert e.value.code == -3
        bad = {2: (np.array([[1, 2], [1, 2]], np.int32), np.array([1, 1], np.uint32))}
        with pytest.raises(pkg.SpdError) as e:
            sess.spd_load_ngrams(bad, synth.PAPER_LAMBDAS)
        assert e.value.code == -5 and "duplicate" in str(e.value)
        for keys, counts in (([[1, shape.vocab]], [1]), ([[1, 2]], [0])):
            with pytest.raises(pkg.SpdError) as e:
                sess.spd_load_ngrams({2: (np.array(keys, np.int32), np.array(counts, np.uint32))}, synth.PAPER_LAMBDAS)
            assert e.value.code == -5
    finally:
        sess.close()


@pytest.mark.timeout(900)
@pytest.mark.parametrize("kv_dtype", ["fp16", "fp32"])
def test_full_size_7b_shape_teacher_forced(kv_dtype):
    """The headline workload at its real size and in the launch configuration the benchmark times
    (persistent forward, fp16 cache; and with the fp32 cache): Llama-2-7B shape, bf16,
    64-token Zipf prefix, k = 3, alpha = 0.54, synthetic n = 2..6 tables.  The oracle runs the
    full model on the host (a few seconds per step), so three timesteps are compared,
    teacher-forced."""
    pkg = P()
    shape = synth.LLAMA7B
    wdev = synth.make_weights_device(shape, seed=0)
    host = {k: synth.host_view(v) for k, v in wdev.items() if not k.endswith("wqkv")}
    prefix = synth.make_prefix_zipf(shape.vocab, 64, seed=0)
    base = synth.make_ngram_tables_zipf(shape.vocab, 200_000, seed=0)
    lm = make_oracle(shape, host)
    _, recs0 = O.generate(lm, None, prefix, O.DecodeCfg(3, 0.0), 3)
    tabs = plant_both_forms(base, recs0, 3, shape.vocab, 1)
    sess = pkg.Session(shape, wdev, max_ctx=128, k_max=8, kv_dtype=kv_dtype)
    try:
        assert sess.spd_get_fused()
        sess.spd_load_ngrams(tabs, synth.PAPER_LAMBDAS)
        dc = pkg.SpdDecodeCfg(3, 0.54, 1.0, 0.1)
        cfg = O.DecodeCfg(3, 0.54, 1.0, 0.1, synth.PAPER_LAMBDAS)
        _, recs, stats = teacher_forced(sess, lm, tabs, synth.PAPER_LAMBDAS, prefix, cfg, 3, RTOL["bf16"], dc)
        assert all("logit_err" in s for s in stats)
        print("7B scaled logit errors:", [f"{s['logit_err']:.2e}" for s in stats])
        report_decisions(f"7B full size ({kv_dtype} cache)", stats, 3)
    finally:
        sess.close()


def test_device_error_word_reaches_the_caller(tiny):
    """The getters (and every call that fetches results) report SPD_EHIP once the device-side
    error word is set; here it is written by a fill kernel after the work has finished -- no
    wait fails, no kernel runs while it is set -- and the next prefix pass clears it."""
    shape, w, _, prefix = tiny
    pkg = P()
    sess = session(shape, w)
    try:
        dc = pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1)
        sess.spd_prefill(prefix)
        sess.spd_step(dc)
        sess.spd_step(dc)
        sess.spd_get_state()
        sess.spd_test_poke_err(1)
        for call in (sess.spd_get_state, lambda: sess.spd_get_step_info(3)):
            with pytest.raises(pkg.SpdError) as e:
                call()
            assert e.value.code == -6 and "barrier" in str(e.value)
        sess.spd_prefill(prefix)
        tok, par, sc = sess.spd_step(dc)
        assert len(tok) == 3
        sess.spd_get_state()
    finally:
        sess.close()
