"""Per-kernel parity: each HIP operator against the oracle's matching sub-function."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import (PREFIX_ATTENTION_BOUND, PREFIX_ATTENTION_CASES, RTOL, assert_close_scaled, prefix_attention64, prefix_attention_inputs,
                        relative_error)
from oracle import spd_oracle as O

pytestmark = pytest.mark.gpu


def P():
    import paper_2405_18400_amd as pkg
    return pkg


def mat(rows, cols, dtype, seed, std=0.02):
    rng = np.random.default_rng(seed)
    w = (rng.standard_normal((rows, cols), dtype=np.float32) * std).astype(np.float32)
    if dtype == "bf16":
        bits = synth.bf16_bits(w).reshape(rows, cols)
        return bits, synth.bf16_widen(bits)
    if dtype == "fp16":      # key/value cache only: numpy's own binary16 rounding (to nearest even)
        h = w.astype(np.float16)
        return h, h.astype(np.float32)
    return w, w


def dev(a, dtype):
    if dtype == "fp16":
        return torch.from_numpy(a).cuda()
    return P().binding.to_device(a, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,cols", [(4096, 4096), (4096, 11008), (6, 40), (258, 520), (2, 2048 + 8), (1024, 256)])
@pytest.mark.parametrize("norm,resid", [(False, False), (True, False), (False, True)])
def test_gemv(dtype, rows, cols, norm, resid):
    Wst, W = mat(rows, cols, dtype, 1)
    gst, g = mat(1, cols, dtype, 2, std=1.0)
    rng = np.random.default_rng(3)
    x = rng.standard_normal(cols, dtype=np.float32)
    r = rng.standard_normal(rows, dtype=np.float32)
    xin = O.rmsnorm(x, g[0], 1e-5).astype(np.float32) if norm else x
    want = W.astype(np.float64) @ xin.astype(np.float64) + (r if resid else 0)
    y = torch.from_numpy(r.copy()).cuda() if resid else torch.zeros(rows, device="cuda")
    P().spd_op_gemv(dtype, dev(Wst, dtype), torch.from_numpy(x).cuda(), y,
                    gain=dev(gst.reshape(-1), dtype) if norm else None, eps=1e-5, residual=y if resid else None)
    torch.cuda.synchronize()
    assert_close_scaled(y.cpu().numpy(), want, 2e-5, "gemv")   # fp32 accumulation of exact products


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,cols,shift", [(2, 8, 0), (130, 512, 0), (4098, 520, 0), (8192, 4096, 0), (66, 4104, 0), (4100, 8200, 0),
                                             (40, 16384, 0), (38, 16392, 0), (20, 32768, 0), (6, 32776, 0), (34, 520, 1), (34, 4096, 1)])
def test_gemv_pieces_and_waves_per_row(dtype, rows, cols, shift):
    """Rows that end at, before and past a whole number of 1 KB pieces, one to eight waves per row, more rows
    than one round takes; rows too wide for registers and operands off the 16-byte grid (`shift` floats)."""
    rng = np.random.default_rng(rows + cols)
    Wst, W = mat(rows, cols, dtype, 31)
    gst, g = mat(1, cols, dtype, 32, std=1.0)
    x, r = rng.standard_normal(cols, dtype=np.float32), rng.standard_normal(rows, dtype=np.float32)
    xin = O.rmsnorm(x, g[0], 1e-5).astype(np.float64)
    xd = torch.zeros(cols + 8, device="cuda")[shift:shift + cols]
    xd.copy_(torch.from_numpy(x))
    Wd, gd, y, u = dev(Wst, dtype), dev(gst.reshape(-1), dtype), torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    P().spd_op_gemv(dtype, Wd, xd, y, gain=gd, eps=1e-5, residual=torch.from_numpy(r).cuda())
    P().spd_op_swiglu(dtype, Wd, Wd, xd, u, eps=1e-5)
    torch.cuda.synchronize()
    W64 = W.astype(np.float64)
    assert_close_scaled(y.cpu().numpy(), W64 @ xin + r, 2e-5, "gemv")      # fp32 accumulation of exact products
    z = W64 @ x.astype(np.float64)
    assert_close_scaled(u.cpu().numpy(), z / (1 + np.exp(-z)) * z, 2e-5, "swiglu")


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("rows,cols", [(11008, 4096), (7, 24), (1025, 264)])
def test_swiglu(dtype, rows, cols):
    Gst, G = mat(rows, cols, dtype, 4, std=0.05)
    Ust, U = mat(rows, cols, dtype, 5, std=0.05)
    gst, g = mat(1, cols, dtype, 6, std=1.0)
    x = np.random.default_rng(7).standard_normal(cols, dtype=np.float32)
    xn = O.rmsnorm(x.astype(np.float64), g[0].astype(np.float64), 1e-5)
    want = O.silu(G.astype(np.float64) @ xn) * (U.astype(np.float64) @ xn)
    u = torch.zeros(rows, device="cuda")
    P().spd_op_swiglu(dtype, dev(Gst, dtype), dev(Ust, dtype), torch.from_numpy(x).cuda(), u, gain=dev(gst.reshape(-1), dtype), eps=1e-5)
    torch.cuda.synchronize()
    assert_close_scaled(u.cpu().numpy(), want, 2e-5, "swiglu")


@pytest.mark.parametrize("dtype,dh", [("bf16", 128), ("fp32", 64), ("bf16", 64), ("fp32", 128), ("fp16", 128), ("fp16", 64), ("fp16", 32)])
@pytest.mark.parametrize("heads,kv", [(4, 4), (8, 1), (8, 2)])
@pytest.mark.parametrize("n_ctx,cap", [(1, 8), (7, 300), (128, 128), (129, 300), (256, 256), (257, 600), (1044, 1100)])
def test_attention(dtype, dh, heads, kv, n_ctx, cap):
    rng = np.random.default_rng(n_ctx + heads)
    Kst, K = mat(kv * cap, dh, dtype, 11, std=1.0)
    Vst, V = mat(kv * cap, dh, dtype, 12, std=1.0)
    q = rng.standard_normal((heads, dh), dtype=np.float32)
    Kt = torch.from_numpy(K.reshape(kv, cap, dh)[:, :n_ctx].astype(np.float64)).repeat_interleave(heads // kv, 0)
    Vt = torch.from_numpy(V.reshape(kv, cap, dh)[:, :n_ctx].astype(np.float64)).repeat_interleave(heads // kv, 0)
    want = torch.nn.functional.scaled_dot_product_attention(
        torch.from_numpy(q.astype(np.float64))[:, None, :], Kt, Vt)[:, 0, :].numpy()
    out = torch.zeros(heads, dh, device="cuda")
    P().spd_op_attention(dtype, torch.from_numpy(q).cuda(), dev(Kst, dtype).view(kv, cap, dh), dev(Vst, dtype).view(kv, cap, dh), out, n_ctx)
    torch.cuda.synchronize()
    assert_close_scaled(out.cpu().numpy(), want, 1e-5, "attention")
    # a second call reuses zeroed counters and gives the same bits
    out2 = torch.zeros(heads, dh, device="cuda")
    P().spd_op_attention(dtype, torch.from_numpy(q).cuda(), dev(Kst, dtype).view(kv, cap, dh), dev(Vst, dtype).view(kv, cap, dh), out2, n_ctx)
    assert torch.equal(out, out2)


# Where the kernels change hands: the vector path (up to two query heads per key/value head, or a
# head size the matrix-core path has no tile for) and the matrix-core path (tiles of 16 query heads,
# turns of 128 positions), one chunk (128 KB of keys per head, 64 KB for larger groups) or several.
# The rows behind the context hold NaN: nothing may read them into a result.
@pytest.mark.parametrize("dtype,dh,heads,kv,n_ctx,cap", [
    ("fp32", 128, 8, 8, 256, 260), ("fp32", 128, 8, 8, 257, 700), ("fp16", 128, 4, 4, 512, 520), ("fp16", 128, 4, 4, 513, 520),
    ("bf16", 8, 6, 3, 77, 90), ("bf16", 256, 4, 2, 300, 400), ("fp32", 256, 3, 3, 1500, 1500), ("fp16", 64, 300, 300, 2100, 2100),
    ("fp32", 128, 6, 2, 127, 130), ("fp32", 128, 6, 2, 128, 130), ("fp32", 128, 6, 2, 129, 400), ("fp16", 64, 34, 2, 16, 20),
    ("fp16", 64, 34, 2, 1025, 1030), ("bf16", 256, 16, 4, 1, 3), ("bf16", 256, 16, 4, 2049, 2049), ("fp16", 128, 16, 1, 5000, 5000)])
def test_attention_where_its_kernels_change_hands(dtype, dh, heads, kv, n_ctx, cap):
    g = torch.Generator(device="cuda").manual_seed(n_ctx + heads)
    tdt = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}[dtype]
    K, V = (torch.randn(kv, cap, dh, generator=g, device="cuda").to(tdt) for _ in range(2))
    K[:, n_ctx:], V[:, n_ctx:] = float("nan"), float("nan")
    q = torch.randn(heads, dh, generator=g, device="cuda")
    out = torch.full((heads, dh), float("nan"), device="cuda")
    print(f"attention {dtype} d_head={dh} heads={heads}/{kv} n_ctx={n_ctx} cap={cap}", flush=True)
    P().spd_op_attention(dtype, q, K, V, out, n_ctx)
    Kd, Vd = K[:, :n_ctx].double(), V[:, :n_ctx].double()
    want = torch.stack([((Kd[h * kv // heads] @ q[h].double()) / dh ** 0.5).softmax(-1) @ Vd[h * kv // heads] for h in range(heads)])
    # fp32 sums of at most 5000 terms: about sqrt(5000) 2^-24 = 4e-6 of the scale
    assert_close_scaled(out.cpu().numpy(), want.cpu().numpy(), 1e-5, "attention")


@pytest.mark.parametrize("vocab", [131072, 131074, 262144, 262146, 524290])
def test_top_k_where_the_entries_per_thread_change(vocab):
    """A slice's entries per thread: 4, 8, 16 and 32, the last and the first vocabulary of each; ties and the two ends included."""
    pkg = P()
    shape = synth.ModelShape("one-head", 1, 64, 1, 1, 128, vocab, "fp32")
    k = 16
    sess = pkg.Session(shape, synth.make_weights(shape, seed=1), max_ctx=32, k_max=k)
    try:
        sess.spd_prefill(np.arange(4))
        z = np.random.default_rng(vocab).standard_normal(vocab).astype(np.float32)
        z[[0, vocab - 1, 12345, 12346, vocab // 2]] = 9.0
        sess.spd_expand_prune(pkg.SpdDecodeCfg(k, 0.0, 1.0, 0.1), torch.from_numpy(z).cuda(), True)
        ids, logp, _, _, _ = sess.spd_get_step_info(k)
        want = np.argsort(-z, kind="stable")[:k]
        z64 = z.astype(np.float64)
        lse = 9.0 + np.log(np.exp(z64 - 9.0).sum())
        assert list(ids) == list(want)
        np.testing.assert_allclose(logp, z64[want] - lse, atol=2e-5, rtol=0)   # fp32 sums of 131072 .. 524290 terms
    finally:
        sess.close()


@pytest.mark.parametrize("kv_dtype", ["fp16", "fp32"])
@pytest.mark.parametrize("case", PREFIX_ATTENTION_CASES + [(6, 3, 32, 70, 20, 1.0)])
def test_prefix_attention_against_64_bits(case, kv_dtype):
    """Both halves of queries and probabilities arrive (fp16 cache), the fp32 products keep theirs (fp32 cache); 32: the plain
    kernel.  The bound, and that it notices a lost half: test_bound_on_the_prefix_attention_notices_a_lost_half."""
    q, K, V = prefix_attention_inputs(case)
    cache = torch.float16 if kv_dtype == "fp16" else torch.float32
    hi, lo = P().spd_test_prefill_attention(kv_dtype, torch.from_numpy(q).cuda(), torch.from_numpy(K).cuda().to(cache), torch.from_numpy(V).cuda().to(cache),
                                            case[4])
    err = relative_error(hi.double().cpu().numpy() + lo.double().cpu().numpy(), prefix_attention64(q, K, V, case[4]))
    assert err < PREFIX_ATTENTION_BOUND, err


@pytest.mark.parametrize("kv_dtype", ["fp16", "fp32"])
@pytest.mark.parametrize("case", [(18, 6, 64, 97, 0, 1.0), (12, 3, 128, 161, 250, 2.0), (1, 1, 128, 64, 0, 1.0)])
def test_prefix_attention_where_heads_and_tiles_share_an_xcd(case, kv_dtype):
    """Query tiles are placed longest first over all heads of an XCD, whose last round of heads is ragged here; up to four tiles
    of keys per wave.  Every (query, head) is written: the bound is that of the test above."""
    q, K, V = prefix_attention_inputs(case)
    cache = torch.float16 if kv_dtype == "fp16" else torch.float32
    hi, lo = P().spd_test_prefill_attention(kv_dtype, torch.from_numpy(q).cuda(), torch.from_numpy(K).cuda().to(cache), torch.from_numpy(V).cuda().to(cache),
                                            case[4])
    got, want = hi.double().cpu().numpy() + lo.double().cpu().numpy(), prefix_attention64(q, K, V, case[4])
    for h in range(case[0]):
        assert relative_error(got[:, h], want[:, h]) < PREFIX_ATTENTION_BOUND, h


def test_operators_run_on_the_callers_current_stream():
    """The handle the operators launch on is torch's current stream, inside and outside a stream context and per thread."""
    import threading
    from paper_2405_18400_amd import binding
    same = lambda: binding._stream_ptr() == torch.cuda.current_stream().cuda_stream  # noqa: E731
    side, seen = torch.cuda.Stream(), []
    with torch.cuda.stream(side):
        seen += [same(), binding._stream_ptr() == side.cuda_stream]
        other = threading.Thread(target=lambda: seen.extend([same(), binding._stream_ptr() != side.cuda_stream]))
        other.start()
        other.join()
    seen += [same(), binding._stream_ptr() != side.cuda_stream]
    assert all(seen) and len(seen) == 6
