"""Nucleus (top-p) sampling pass on the GPU against the oracle, through the C ABI."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import RTOL, assert_close_scaled, make_oracle
from oracle import spd_oracle as O

pytestmark = pytest.mark.gpu


def P():
    import paper_2405_18400_amd as pkg
    return pkg


def acceptable(logits, top_p, tau, u, token, tol):
    """Is `token` what nucleus sampling returns for SOME cumulative probabilities within `tol`
    of the exact ones?  (Both sides sum probabilities in floating point; a draw that lands
    within rounding of a boundary may legitimately select either neighbour.)"""
    lp = O.log_softmax_tau(np.asarray(logits, np.float64), tau, np.float64)
    p = np.exp(lp)
    order = np.lexsort((np.arange(p.size), -p))
    cs = np.cumsum(p[order])
    n = int(min(np.searchsorted(cs, top_p, side="left"), p.size - 1))
    masses = {float(cs[n])}
    if n > 0 and cs[n - 1] >= top_p - tol: masses.add(float(cs[n - 1]))
    if n + 1 < p.size and cs[n] < top_p + tol: masses.add(float(cs[n + 1]))
    j = int(np.nonzero(order == token)[0][0])
    lo = cs[j - 1] if j > 0 else 0.0
    return any(lo - tol <= u * m <= cs[j] + tol for m in masses)


def check_draw(sess, rec, top_p, tau, u, got_token, got_logp, tol):
    decisive = rec.margin_sample > tol + (u * rec.p_edge if rec.margin_nucleus <= tol else 0.0)
    if decisive:
        assert got_token == rec.token, (got_token, rec.token, rec.margin_sample)
        assert abs(got_logp - rec.logp) <= tol * max(1.0, abs(rec.logp)) + 1e-4
    else:
        assert acceptable(rec.logits, top_p, tau, u, got_token, tol)
    return decisive


# Cumulative probabilities are fp32 sums of up to a few thousand terms on the GPU and fp64 sums
# in the oracle, from logits that agree to about 1e-6 of their scale: a draw closer than this
# to a boundary is not held to the oracle's choice, only to a valid one.
TOL = 1e-5


@pytest.fixture(scope="module")
def tiny():
    shape = synth.TINY
    return shape, synth.make_weights(shape, seed=0), synth.make_prefix_uniform(shape.vocab, 16, seed=0)


@pytest.mark.parametrize("top_p,tau", [(0.9, 1.0), (0.5, 0.7), (1.0, 1.3)])
def test_pass_teacher_forced(tiny, top_p, tau):
    """The benchmark's comparison decoder on the tiny model: 12 tokens, seeded draws; after
    every token the oracle's token is written back so each step is compared on its own."""
    shape, w, prefix = tiny
    pkg = P()
    us = np.random.default_rng(11).random(12).astype(np.float32)
    lm = make_oracle(shape, w)
    toks, total, recs = O.nucleus_generate(lm, prefix, top_p, tau, [float(u) for u in us], keep_logits=True)
    sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
    try:
        sc = pkg.SpdSampleCfg(top_p, tau)
        sess.spd_prefill(prefix)
        n_decisive, run_total, tail = 0, 0.0, [-1] * 5
        tail = ([-1] * 5 + list(prefix))[-5:]
        for t, rec in enumerate(recs):
            tok, lp = sess.spd_nucleus_step(sc, float(us[t]))
            assert_close_scaled(sess.spd_read_logits(), rec.logits, RTOL[shape.dtype], "logits")
            n_decisive += check_draw(sess, rec, top_p, tau, float(us[t]), tok, lp, TOL)
            size, mass, _ = sess.spd_get_nucleus_info()
            assert abs(mass - rec.nucleus_mass) < 1e-4
            if rec.margin_nucleus > 1e-4:
                assert size == rec.nucleus_size
            run_total += rec.logp
            tail = tail[1:] + [rec.token]
            sess.spd_set_state(np.array([tail], np.int32), np.array([run_total], np.float32))   # teacher forcing
        assert n_decisive >= len(recs) - 4
        assert sess.spd_position() == len(prefix) + len(recs) - 1
    finally:
        sess.close()


def test_free_running_pass_and_graph_replay_agree(tiny):
    """Replayed from a graph (the forward of one kernel per product; the persistent one is launched plainly whatever the switch says) and
    plainly launched: the same tokens and log-probabilities."""
    shape, w, prefix = tiny
    pkg = P()
    us = np.random.default_rng(12).random(10).astype(np.float32)
    for fused in (False, True):
        out = []
        for graph in (True, False, True):
            sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
            try:
                sess.spd_set_fused(fused)
                sess.spd_set_graph(graph)
                sc = pkg.SpdSampleCfg(0.9, 1.0)
                sess.spd_prefill(prefix)
                out.append([sess.spd_nucleus_step(sc, float(u)) for u in us])
                assert abs(sess.spd_get_nucleus_info()[2] - sum(lp for _, lp in out[-1])) < 1e-3
            finally:
                sess.close()
        assert out[0] == out[1] == out[2]


def _sample_only(sess, sc, logits, u, first=True):
    sess.spd_nucleus_sample(sc, u, torch.tensor(logits, dtype=torch.float32, device="cuda"), first)
    tails, _, _ = sess.spd_get_state()
    return int(tails[0, -1])


def test_sampler_on_scripted_logits_ties_and_limits(tiny):
    shape, w, prefix = tiny
    pkg = P()
    sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
    try:
        sess.spd_prefill(prefix)
        V = shape.vocab
        base = np.full(V, -30.0, np.float32)
        # four tokens carry all the mass: ids 7 and 900 tie at 0.3, id 3 has 0.2, id 2000 has 0.2
        lg = base.copy()
        lg[[7, 900, 3, 2000]] = np.log([0.3, 0.3, 0.2, 0.2]).astype(np.float32)
        sc = pkg.SpdSampleCfg(1.0, 1.0)
        want = lambda u, p=1.0: O.nucleus_sample(lg, p, 1.0, u).token
        for u in (0.0, 0.1, 0.29, 0.31, 0.59, 0.61, 0.79, 0.81, 0.99):
            assert _sample_only(sess, sc, lg, u) == want(u), u
        assert _sample_only(sess, sc, lg, 0.0) == 7 and _sample_only(sess, sc, lg, 0.45) == 900    # lower id first
        assert _sample_only(sess, sc, lg, 0.7) == 3 and _sample_only(sess, sc, lg, 0.9) == 2000
        # nucleus that ends inside the tie: p = 0.25 keeps only id 7; p = 0.55 keeps 7 and 900
        assert all(_sample_only(sess, pkg.SpdSampleCfg(0.25, 1.0), lg, u) == 7 for u in (0.0, 0.5, 0.99))
        got = {_sample_only(sess, pkg.SpdSampleCfg(0.55, 1.0), lg, u) for u in np.linspace(0, 0.99, 23)}
        assert got == {7, 900}
        assert sess.spd_get_nucleus_info()[0] == 2
        # tiny top_p: greedy whatever the draw
        rng = np.random.default_rng(5)
        rl = (rng.normal(size=V) * 3).astype(np.float32)
        for p in (1e-6, 2.0 ** -40, 1e-13, 1e-30):      # (down to masses below the sampler's unit, 2^-40)
            assert all(_sample_only(sess, pkg.SpdSampleCfg(p, 1.0), rl, u) == int(np.argmax(rl)) for u in (0.0, 0.5, 0.999))
            assert sess.spd_get_nucleus_info()[0] == 1
        # random logits, many draws, both temperatures: equal to the oracle wherever it is decisive
        for tau in (1.0, 0.4):
            n_dec = 0
            for u in rng.random(60):
                rec = O.nucleus_sample(rl, 0.9, tau, float(np.float32(u)), keep_logits=True)
                tok = _sample_only(sess, pkg.SpdSampleCfg(0.9, tau), rl, float(np.float32(u)))
                n_dec += check_draw(sess, rec, 0.9, tau, float(np.float32(u)), tok, rec.logp, 1e-5)
            assert n_dec >= 45
    finally:
        sess.close()


def test_draws_on_a_grid_follow_the_renormalised_distribution(tiny):
    shape, w, prefix = tiny
    pkg = P()
    sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
    try:
        sess.spd_prefill(prefix)
        rng = np.random.default_rng(6)
        lg = (rng.normal(size=shape.vocab) * 3).astype(np.float32)
        p = np.exp(lg.astype(np.float64) - lg.max()); p /= p.sum()
        order = np.argsort(-p, kind="stable")
        n = int(np.searchsorted(np.cumsum(p[order]), 0.8))
        keep = order[: n + 1]
        N = 400
        counts = np.zeros(shape.vocab)
        sc = pkg.SpdSampleCfg(0.8, 1.0)
        for i in range(N):
            counts[_sample_only(sess, sc, lg, (i + 0.5) / N)] += 1
        want = np.zeros(shape.vocab); want[keep] = p[keep] / p[keep].sum()
        assert counts[np.setdiff1d(np.arange(shape.vocab), keep)].sum() == 0
        assert np.max(np.abs(counts / N - want)) <= 1.5 / N
    finally:
        sess.close()


@pytest.mark.parametrize("vocab", [40000, 70000])
def test_draws_from_large_vocabularies(vocab):
    """More than 32768 entries: eight pieces of bucket numbers per thread, and beyond 65536 all of them read again for each question."""
    pkg = P()
    shape = synth.ModelShape("bigvocab", 1, 64, 2, 2, 128, vocab, "fp32")
    w = synth.make_weights(shape, seed=2)
    sess = pkg.Session(shape, w, max_ctx=32, k_max=8)
    try:
        sess.spd_prefill([1, 2, 3])
        rng = np.random.default_rng(7)
        lg = (rng.normal(size=shape.vocab) * 4).astype(np.float32)
        n_dec = 0
        for u in rng.random(20):
            rec = O.nucleus_sample(lg, 0.9, 1.0, float(np.float32(u)), keep_logits=True)
            tok = _sample_only(sess, pkg.SpdSampleCfg(0.9, 1.0), lg, float(np.float32(u)))
            n_dec += check_draw(sess, rec, 0.9, 1.0, float(np.float32(u)), tok, rec.logp, 1e-5)
        assert n_dec >= 12
    finally:
        sess.close()


@pytest.mark.parametrize("vocab", [66, 1024, 1026, 4098, 32768, 32770])
def test_neighbouring_entries_in_one_bucket_and_the_next(vocab):
    """The entries of a bucket are found two bucket numbers at a time: ids side by side that share a bucket, that lie in buckets whose numbers
    differ in the last bit alone, and at random; slices of one to 32 blocks, ragged ones, the last vocabulary of four
    pieces of bucket numbers per thread and the first beyond."""
    pkg = P()
    shape = synth.ModelShape("buckets", 1, 64, 2, 2, 128, vocab, "fp32")
    sess = pkg.Session(shape, synth.make_weights(shape, seed=2), max_ctx=32, k_max=8)
    try:
        sess.spd_prefill([1, 2, 3])
        rng = np.random.default_rng(vocab)
        i = np.arange(vocab)
        width = 8.0 / 2048                                                          # of a bucket, the logits spanning 8
        for lg in (rng.normal(size=vocab) * 2, np.repeat(rng.random(vocab // 2 + 1), 2)[:vocab] * 8, ((i * 7919) % 2048 // 2 * 2 + i % 2) * width, 8.0 - (i % 2048) * width):
            lg = lg.astype(np.float32)
            n_dec = 0
            for u in (0.03, 0.31, 0.62, 0.97):
                rec = O.nucleus_sample(lg, 0.7, 1.0, float(np.float32(u)), keep_logits=True)
                tok = _sample_only(sess, pkg.SpdSampleCfg(0.7, 1.0), lg, float(np.float32(u)))
                n_dec += check_draw(sess, rec, 0.7, 1.0, float(np.float32(u)), tok, rec.logp, 1e-5)
            assert n_dec >= 1 or vocab > 4098
    finally:
        sess.close()


@pytest.mark.parametrize("vocab", [32766, 32770, 65534, 65536, 65538, 131072, 140002])
def test_vocabularies_around_the_bucket_numbers_a_thread_holds(vocab):
    """Four pieces of eight bucket numbers per thread, eight, or all read again per walk; a last piece that the vocabulary ends in; slices of
    1024 entries and longer ones; buckets that fit the list, and ties by the thousand that do not (cut again by key)."""
    pkg = P()
    shape = synth.ModelShape("pieces", 1, 64, 2, 2, 128, vocab, "fp32")
    sess = pkg.Session(shape, synth.make_weights(shape, seed=2), max_ctx=32, k_max=8)
    try:
        sess.spd_prefill([1, 2, 3])
        rng = np.random.default_rng(vocab)
        ends = np.full(vocab, -12.0)
        ends[[0, 7, 8, vocab // 2, vocab - 2, vocab - 1]] = [0.5, 1.0, 0.2, 0.7, 0.9, 1.1]      # the mass at the array's ends
        for lg in (rng.normal(size=vocab) * 3, rng.integers(0, 6, vocab) * 1.5, ends, np.zeros(vocab)):
            lg = lg.astype(np.float32)
            for u in (0.0, 0.35, 0.8, 0.995):
                u = float(np.float32(u))
                rec = O.nucleus_sample(lg, 0.93, 1.0, u, keep_logits=True)
                tok = _sample_only(sess, pkg.SpdSampleCfg(0.93, 1.0), lg, u)
                check_draw(sess, rec, 0.93, 1.0, u, tok, rec.logp, 1e-5)
                if rec.margin_nucleus > 1e-5:
                    assert sess.spd_get_nucleus_info()[0] == rec.nucleus_size
    finally:
        sess.close()


@pytest.mark.parametrize("vocab", [2050, 32000, 40000, 65538])
def test_masked_logits(vocab):
    """Tokens excluded with -inf, the type's lowest value or a large negative one, next to live entries from the likeliest down to
    probabilities of 1e-9: many more entries between two keys than are ranked pairwise, keys up to the last one that a
    64-bit word holds (a range of keys that ends there used to come out empty, its answer an entry that nothing had written)."""
    pkg = P()
    shape = synth.ModelShape("masked", 1, 64, 2, 2, 128, vocab, "fp32")
    sess = pkg.Session(shape, synth.make_weights(shape, seed=2), max_ctx=32, k_max=8)
    try:
        sess.spd_prefill([1, 2, 3])
        rng = np.random.default_rng(vocab)
        few = 1200.0 / vocab
        for mask in (-np.inf, float(np.finfo(np.float32).min), -1e9):
            tail = np.full(vocab, mask)
            tail[rng.permutation(vocab)[:1000]] = -9.0 - rng.random(1000)      # one likely entry, the rest of the mass spread thin
            tail[vocab // 3] = 0.0
            vectors = [tail, np.full(vocab, mask)]
            vectors[1][vocab - 1] = 1.0                                        # a single live entry
            for live in (0.5, few):
                lg = rng.normal(size=vocab) * 3
                lg[rng.random(vocab) >= live] = mask
                vectors.append(lg)
            lg = np.full(vocab, mask)
            lg[:700] = rng.normal(size=700) * 3                               # whole slices without an entry
            vectors.append(lg)
            vectors.append(rng.normal(size=vocab) * 30)                        # no mask, most probabilities zero in 40 bits all the same
            for lg in vectors:
                lg, n_dec = lg.astype(np.float32), 0
                for top_p, u in ((0.5, 0.3), (0.9, 0.05), (0.9, 0.97), (0.98, 0.6), (0.9999, 0.93), (1.0, 0.02), (1.0, 0.875), (1.0, 0.99)):
                    u = float(np.float32(u))
                    rec = O.nucleus_sample(lg, top_p, 1.0, u, keep_logits=True)
                    tok = _sample_only(sess, pkg.SpdSampleCfg(top_p, 1.0), lg, u)
                    assert lg[tok] > -1e8
                    n_dec += check_draw(sess, rec, top_p, 1.0, u, tok, rec.logp, 1e-5)
                    size, mass, _ = sess.spd_get_nucleus_info()
                    assert abs(mass - rec.nucleus_mass) <= 1e-5 + rec.p_edge * (rec.margin_nucleus <= 1e-5) and size <= vocab
                    if rec.margin_nucleus > 1e-5:
                        assert size == rec.nucleus_size
                assert n_dec >= 4
    finally:
        sess.close()


def test_error_paths(tiny):
    shape, w, prefix = tiny
    pkg = P()
    sess = pkg.Session(shape, w, max_ctx=64, k_max=8)
    try:
        sc = pkg.SpdSampleCfg(0.9, 1.0)
        with pytest.raises(pkg.SpdError): sess.spd_nucleus_step(sc, 0.5)              # before prefill
        sess.spd_prefill(prefix)
        for bad in (pkg.SpdSampleCfg(0.0, 1.0), pkg.SpdSampleCfg(1.5, 1.0), pkg.SpdSampleCfg(0.9, 0.0)):
            with pytest.raises(pkg.SpdError): sess.spd_nucleus_step(bad, 0.5)
        for u in (-0.1, 1.0):
            with pytest.raises(pkg.SpdError): sess.spd_nucleus_step(sc, u)
        sess.spd_step(pkg.SpdDecodeCfg(3, 0.0, 1.0, 0.1))
        with pytest.raises(pkg.SpdError): sess.spd_nucleus_step(sc, 0.5)              # SPD generation in progress
        sess.spd_prefill(prefix)
        assert sess.spd_nucleus_step(sc, 0.5)[0] >= 0
    finally:
        sess.close()
