"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same
seeded inputs, at sizes the oracle finishes in seconds.  Codes, blob bytes, routing and
permutation are compared bit for bit; outputs within the floating-point bar."""
import numpy as np
import pytest
import torch

import oracle as O
from helpers import (MAX_ABS_TOL, assert_output_close, check_bucket, compare_routing, dev, dev_bf16)
from workloads import CONFIGS, f32_to_bf16_bits, make_case, make_weight

pytestmark = pytest.mark.gpu


def tokens(T, K, seed, scale_channels=True):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((T, K)).astype(np.float32)
    if scale_channels and K >= 256:
        x[:, rng.choice(K, size=max(1, K // 100), replace=False)] *= 20.0
    return f32_to_bf16_bits(x)


# ----------------------------------------------------------------------------- encode
@pytest.mark.parametrize("N,K", [(16, 256), (3, 128), (40, 384), (130, 1280), (2048, 2048)])
def test_encode_blob_is_bit_exact(mbq, N, K):
    print(f"[case] encode N={N} K={K}", flush=True)
    W = make_weight(N, K, [7, N, K], 4.0)
    if N >= 40:
        W[1, :128] = 0.0                # an all-zero group
        W[2, 128:256] = 0.3125          # a constant group
    codes, s0, z0 = O.encode(W)
    blob = mbq.mbq_encode(dev(W))
    torch.cuda.synchronize()
    got = blob.cpu().numpy()
    want = O.pack_blob(codes, s0, z0)
    assert got.size == want.size
    assert np.array_equal(got, want)
    c, s, z = mbq.mbq_unpack(blob, N, K)
    assert np.array_equal(c.cpu().numpy(), codes)
    assert np.array_equal(s.cpu().numpy(), s0) and np.array_equal(z.cpu().numpy(), z0)
    for p in range(4):
        What = mbq.mbq_dequant(blob, N, K, p).cpu().numpy().astype(np.float64)
        ref = O.dequant(codes, s0, z0, p)
        np.testing.assert_allclose(What, ref, rtol=2e-7, atol=1e-12)


@pytest.mark.parametrize("offset", [0.0, -128.0, 1000.0, -3.0])
@pytest.mark.parametrize("ulps", [0, 1, -1])
def test_encode_weights_on_code_boundaries(mbq, offset, ulps):
    """Weights on the boundaries between two codes of some slice (every multiple of 1/64 of the first step), or one
    float next to them, with small and large zero points: the blob is the recursion's, bit for bit."""
    N, K = 18, 384
    rng = np.random.default_rng([N, K, 5])
    m = rng.integers(0, 257, size=(N, K // 128, 128))
    m[..., 3], m[..., 77] = 0, 256  # both ends of the range in every group
    step = np.exp2(rng.integers(-9, -5, size=(N, K // 128, 1)))
    W = (offset + m / 64.0 * step).astype(np.float32)
    if ulps:
        moved = np.nextafter(W, np.float32(np.inf if ulps > 0 else -np.inf), dtype=np.float32)
        W = np.where(rng.random(W.shape) < 0.5, moved, W)
    W = W.reshape(N, K)
    codes, s0, z0 = O.encode(W)
    blob = mbq.mbq_encode(dev(W))
    torch.cuda.synchronize()
    assert np.array_equal(blob.cpu().numpy(), O.pack_blob(codes, s0, z0))
    Wg = W.reshape(N, K // 128, 128)
    s0 = ((Wg.max(axis=2) - Wg.min(axis=2)) / np.float32(8.0)).astype(np.float32)  # half the weights saturate
    z0 = (-Wg.min(axis=2) / s0 - np.float32(1.0)).astype(np.float32)
    codes, _, _ = O.encode(W, s0, z0)
    blob = mbq.mbq_encode_with_params(dev(W), dev(s0), dev(z0))
    assert np.array_equal(blob.cpu().numpy(), O.pack_blob(codes, s0, z0))


@pytest.mark.parametrize("N,K,keep", [(3, 128, 0.7), (130, 1280, 0.6), (272, 4096, 0.9)])
def test_encode_with_external_parameters(mbq, N, K, keep):
    """Calibrated (clipped) base-slice parameters handed in: blob bit-exact with the oracle's, weights outside the range
    saturated, and the routed linear over such a blob within tolerance of the oracle's."""
    print(f"[case] encode with params N={N} K={K} keep={keep}", flush=True)
    W = make_weight(N, K, [53, N, K], 4.0)
    Wg = W.reshape(N, K // 128, 128)
    lo = (Wg.min(axis=2) * np.float32(keep)).astype(np.float32)
    hi = (Wg.max(axis=2) * np.float32(keep)).astype(np.float32)
    s0 = ((hi - lo) / np.float32(4.0)).astype(np.float32)
    z0 = ((-lo) / s0).astype(np.float32)
    codes, _, _ = O.encode(W, s0, z0)
    blob = mbq.mbq_encode_with_params(dev(W), dev(s0), dev(z0))
    torch.cuda.synchronize()
    assert np.array_equal(blob.cpu().numpy(), O.pack_blob(codes, s0, z0))
    c, s, z = mbq.mbq_unpack(blob, N, K)
    assert np.array_equal(c.cpu().numpy(), codes)
    assert np.array_equal(s.cpu().numpy(), s0) and np.array_equal(z.cpu().numpy(), z0)
    T = 16
    xb = tokens(T, K, [N, K, 59])
    prec = np.random.default_rng([N, K]).integers(0, 4, size=T).astype(np.int32)
    perm, offsets = O.bucket(prec)
    Y = mbq.mbq_linear(dev_bf16(xb).reshape(T, K), blob, N, K, dev(prec), dev(perm), dev(offsets))
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"linear over clipped blob N={N} K={K}")


@pytest.mark.parametrize("meta", ["float16", "bfloat16"])
def test_sixteen_bit_parameter_values_through_external_parameters(mbq, meta):
    """App. C.1's pipeline may keep the per-group scale and zero point in 16 bits.  The blob stores fp32 pairs, but the
    NUMBERS of such a setting pass through unchanged: parameters rounded to fp16 / bf16 before they are handed in give
    the oracle's codes for exactly those parameters, and every stored value is a 16-bit number."""
    N, K, T = 70, 1024, 16
    print(f"[case] encode with {meta} parameter values N={N} K={K}", flush=True)
    W = make_weight(N, K, [57, N, K], 4.0)
    _, s_fit, z_fit = O.encode(W)
    if meta == "float16":
        s0, z0 = s_fit.astype(np.float16).astype(np.float32), z_fit.astype(np.float16).astype(np.float32)
    else:
        def to_bf16(a):
            u = a.view(np.uint32).astype(np.uint64)
            u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
            return u.astype(np.uint32).view(np.float32)
        s0, z0 = to_bf16(s_fit), to_bf16(z_fit)
    codes, _, _ = O.encode(W, s0, z0)
    blob = mbq.mbq_encode_with_params(dev(W), dev(s0), dev(z0))
    torch.cuda.synchronize()
    assert np.array_equal(blob.cpu().numpy(), O.pack_blob(codes, s0, z0))
    c, s, z = mbq.mbq_unpack(blob, N, K)
    assert np.array_equal(s.cpu().numpy(), s0) and np.array_equal(z.cpu().numpy(), z0)
    xb = tokens(T, K, [N, K, 61])
    prec = np.random.default_rng([N, K, 3]).integers(0, 4, size=T).astype(np.int32)
    perm, offsets = O.bucket(prec)
    Y = mbq.mbq_linear(dev_bf16(xb).reshape(T, K), blob, N, K, dev(prec), dev(perm), dev(offsets))
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"linear, {meta} parameter values")


# ------------------------------------------------------------------------------ route
@pytest.mark.parametrize("T,K", [(0, 256), (1, 128), (5, 384), (16, 4096), (16, 11008), (28, 8192), (29, 8320),
                                 (32, 2048), (64, 4096), (65, 1024), (100, 2304), (128, 4096), (129, 512), (1023, 256), (1024, 256), (1025, 256),
                                 (4100, 512)])
def test_route_and_bucket_are_bit_exact(mbq, T, K):
    print(f"[case] route T={T} K={K}", flush=True)
    rng = np.random.default_rng([T, K])
    xb = tokens(T, K, [T, K, 1])
    Wr = (rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32)
    br = np.array([0.3, 0.1, -0.1, -0.4], dtype=np.float32)
    S, prec_ref, gap = O.route(xb, Wr, br)
    prec, perm, offsets, logits = mbq.mbq_route(dev_bf16(xb).reshape(T, K), dev(Wr), dev(br), want_logits=True)
    torch.cuda.synchronize()
    prec, perm, offsets = prec.cpu().numpy(), perm.cpu().numpy(), offsets.cpu().numpy()
    if T:
        np.testing.assert_allclose(logits.cpu().numpy(), S, rtol=0, atol=1e-10)
    compare_routing(prec, prec_ref, gap, f"route T={T} K={K}")
    check_bucket(prec, perm, offsets)          # permutation of the GPU's own choices: unique answer
    assert offsets[4] == T


# ------------------------------------------------------------- the paper's router (2-layer MLP + threshold)
@pytest.mark.parametrize("T,K,H", [(0, 256, 8), (1, 128, 1), (16, 4096, 64), (37, 384, 13), (513, 512, 32),
                                   (2048, 1024, 64), (300, 256, 512), (290, 384, 21)])
def test_route_mlp_matches_oracle(mbq, T, K, H):
    """Scores to fp64 rounding, precisions bit-exact away from the threshold, permutation exact; a sweep of the
    threshold over one set of parameters switches precisions without touching anything else."""
    from workloads import make_mlp_router
    print(f"[case] route_mlp T={T} K={K} H={H}", flush=True)
    xb = tokens(T, K, [T, K, H])
    W1, b1, W2, b2 = make_mlp_router(K, H, [T, K, H])
    X = dev_bf16(xb).reshape(T, K)
    d = [dev(a) for a in (W1, b1, W2, b2)]
    avgs = []
    for delta in (-1e3, -0.75, 0.0, 0.4, 1e3):
        S, prec_ref, margin = O.route_mlp(xb, W1, b1, W2, b2, delta)
        prec, perm, offsets, scores = mbq.mbq_route_mlp(X, *d, delta, want_scores=True)
        torch.cuda.synchronize()
        prec, perm, offsets = prec.cpu().numpy(), perm.cpu().numpy(), offsets.cpu().numpy()
        if T:
            np.testing.assert_allclose(scores.cpu().numpy(), S, rtol=0, atol=1e-10)
        compare_routing(prec, prec_ref, margin, f"route_mlp T={T} K={K} H={H} delta={delta}")
        check_bucket(prec, perm, offsets)
        assert offsets[4] == T
        avgs.append(O.avg_bits(prec))
    if T:
        assert avgs[0] == 8.0 and avgs[-1] == 2.0 and all(a >= b for a, b in zip(avgs, avgs[1:]))


def test_threshold_quantile_is_exact(mbq):
    """The calibration quantile is an order statistic: fed the oracle's scores it must return the same double."""
    rng = np.random.default_rng(23)
    S = rng.standard_normal((1000, 4)) * 3.0
    S[5, 1] = S[9, 2]                      # a tie among the residual scores
    Sd = dev(S)
    for rho in (0.0, 1.0 / 6.0, 1.0 / 3.0, 0.5, 0.77, 1.0):
        want = O.threshold_quantile(S, rho)
        got = float(mbq.mbq_threshold_quantile(Sd, rho).cpu().numpy()[0])
        assert got == want, (rho, got, want)
    with pytest.raises(mbq.MbqError):
        mbq.mbq_threshold_quantile(Sd, 1.5)


def test_route_mlp_target_bits_and_linear(mbq):
    """Layer-wise calibration end to end (App. C.2): scores of a calibration batch -> threshold for a target of
    4 average bits -> routing of a fresh batch -> routed linear against the oracle with the same routing."""
    from workloads import make_mlp_router
    N, K, H, T = 272, 512, 16, 200
    W = make_weight(N, K, [29], 4.0)
    W1, b1, W2, b2 = make_mlp_router(K, H, [29])
    d = [dev(a) for a in (W1, b1, W2, b2)]
    cal = tokens(4096, K, [29, 1])
    *_, cal_scores = mbq.mbq_route_mlp(dev_bf16(cal).reshape(-1, K), *d, 0.0, want_scores=True)
    rho = (4.0 - 2.0) / 6.0
    delta = float(mbq.mbq_threshold_quantile(cal_scores, rho).cpu().numpy()[0])
    S_cal, _, _ = O.route_mlp(cal, W1, b1, W2, b2, 0.0)
    active = float(np.mean(S_cal[:, 1:] - delta > 0))
    assert abs(active - rho) < 2e-3                       # the requested fraction of residual slices is active
    xb = tokens(T, K, [29, 2])
    X = dev_bf16(xb).reshape(T, K)
    prec, perm, offsets = mbq.mbq_route_mlp(X, *d, delta)
    S, prec_ref, margin = O.route_mlp(xb, W1, b1, W2, b2, delta)
    compare_routing(prec.cpu().numpy(), prec_ref, margin, "route_mlp calibrated")
    blob = mbq.mbq_encode(dev(W))
    codes, s0, z0 = O.encode(W)
    for algo in (1, 3):
        Y = mbq.mbq_linear(X, blob, N, K, prec, perm, offsets, algo=algo)
        assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec.cpu().numpy()), f"mlp-routed linear algo={algo}")


@pytest.mark.parametrize("T,K,n", [(1, 4096, 3), (16, 4096, 3), (28, 1280, 4), (16, 11008, 1), (40, 512, 2), (97, 4096, 2), (128, 1024, 3), (130, 512, 2),
                                   (0, 256, 2)])
def test_route_group_equals_separate_calls(mbq, T, K, n):
    """Several routers over one X: against the oracle, and bit for bit against mbq_route; called
    twice on one workspace that starts out full of ones (the call clears its counters itself)."""
    print(f"[case] route group T={T} K={K} n={n}", flush=True)
    rng = np.random.default_rng([T, K, n])
    xb = tokens(T, K, [T, K, 2])
    X = dev_bf16(xb).reshape(T, K)
    Wrs = [(rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32) for _ in range(n)]
    brs = [rng.normal(0, 0.2, size=4).astype(np.float32) for _ in range(n)]
    ws = mbq.route_workspace(T, K, "cuda").fill_(0xFF)
    for _ in range(2):
        outs = mbq.mbq_route_group(X, [dev(w) for w in Wrs], [dev(b) for b in brs], ws=ws)
        torch.cuda.synchronize()
        for i in range(n):
            S, prec_ref, gap = O.route(xb, Wrs[i], brs[i])
            prec, perm, offsets = (t.cpu().numpy() for t in outs[i])
            compare_routing(prec, prec_ref, gap, f"group router {i}")
            check_bucket(prec, perm, offsets)
            single = mbq.mbq_route(X, dev(Wrs[i]), dev(brs[i]))
            for a, b in zip(single, outs[i]):
                assert torch.equal(a, b)


@pytest.mark.parametrize("T", [1, 16, 28, 29, 128, 129, 700])
def test_route_workspace_contents_do_not_matter(mbq, T):
    """A workspace left in any state (say by a call that was cut short) gives the same routing as a clean one,
    for the linear router, the 2-layer router and the routed stage."""
    from workloads import make_mlp_router
    K, H, N = 512, 16, 64
    print(f"[case] dirty route workspace T={T}", flush=True)
    rng = np.random.default_rng([T, 91])
    xb = tokens(T, K, [T, 91])
    X = dev_bf16(xb).reshape(T, K)
    Wr = dev((rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32))
    br = dev(rng.normal(0, 0.2, size=4).astype(np.float32))
    clean = mbq.mbq_route(X, Wr, br, ws=mbq.route_workspace(T, K, "cuda").zero_())
    for fill in (0xFF, 0x01, 0x80):
        dirty = mbq.mbq_route(X, Wr, br, ws=mbq.route_workspace(T, K, "cuda").fill_(fill))
        torch.cuda.synchronize()
        for a, b in zip(clean, dirty):
            assert torch.equal(a, b), (T, fill)
    m = [dev(a) for a in make_mlp_router(K, H, [T, 92])]
    clean = mbq.mbq_route_mlp(X, *m, 0.1, ws=mbq.route_mlp_workspace(T, K, H, "cuda").zero_())
    dirty = mbq.mbq_route_mlp(X, *m, 0.1, ws=mbq.route_mlp_workspace(T, K, H, "cuda").fill_(0xFF))
    torch.cuda.synchronize()
    for a, b in zip(clean, dirty):
        assert torch.equal(a, b), T
    blob = mbq.mbq_encode(dev(make_weight(N, K, [T, 93])))
    outs = []
    for fill in (0x00, 0xFF):
        ws = mbq.route_workspace(T, K, "cuda").fill_(fill)
        outs.append(mbq.mbq_routed_linear_group(X, [Wr], [br], [blob], [N], ws_route=ws))
        torch.cuda.synchronize()
    for a, b in zip(outs[0][0][0] + (outs[0][1][0],), outs[1][0][0] + (outs[1][1][0],)):
        assert torch.equal(a, b), T


def test_route_small_and_general_kernels_agree(mbq):
    T, K = 16, 4096
    xb = tokens(T, K, 77)
    rng = np.random.default_rng(77)
    Wr = (rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32)
    br = np.zeros(4, dtype=np.float32)
    a = mbq.mbq_route(dev_bf16(xb), dev(Wr), dev(br), want_logits=True)
    mbq.set_knob(4, 1)
    try:
        b = mbq.mbq_route(dev_bf16(xb), dev(Wr), dev(br), want_logits=True)
    finally:
        mbq.set_knob(4, 0)
    for u, v in zip(a[:3], b[:3]):
        assert torch.equal(u, v)
    np.testing.assert_allclose(a[3].cpu().numpy(), b[3].cpu().numpy(), rtol=0, atol=1e-10)


def test_route_ties_and_single_bucket(mbq):
    T, K = 70, 256
    xb = tokens(T, K, 3)
    Wr = np.zeros((4, K), dtype=np.float32)
    br = np.zeros(4, dtype=np.float32)            # every logit ties: first index wins
    prec, perm, offsets = mbq.mbq_route(dev_bf16(xb), dev(Wr), dev(br))
    assert prec.cpu().numpy().tolist() == [0] * T
    assert offsets.cpu().numpy().tolist() == [0, T, T, T, T]
    assert perm.cpu().numpy().tolist() == list(range(T))
    br[2] = 1.0
    prec, perm, offsets = mbq.mbq_route(dev_bf16(xb), dev(Wr), dev(br))
    assert prec.cpu().numpy().tolist() == [2] * T
    assert offsets.cpu().numpy().tolist() == [0, 0, 0, T, T]


# ----------------------------------------------------------------------------- linear
def run_linear(mbq, W, xb, prec, algo):
    N, K = W.shape
    T = xb.shape[0]
    blob = mbq.mbq_encode(dev(W))
    perm, offsets = O.bucket(prec)
    Y = mbq.mbq_linear(dev_bf16(xb).reshape(T, K), blob, N, K, dev(prec.astype(np.int32)), dev(perm),
                       dev(offsets), algo=algo)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


ALGOS = {"simple": 1, "decode": 2, "prefill": 3}


@pytest.mark.parametrize("algo", ["simple", "decode", "prefill"])
@pytest.mark.parametrize("N,K,T", [(16, 256, 1), (40, 384, 5), (130, 1280, 16), (272, 512, 33), (64, 2048, 64)])
def test_linear_small_shapes(mbq, algo, N, K, T):
    print(f"[case] linear {algo} N={N} K={K} T={T}", flush=True)
    W = make_weight(N, K, [11, N, K], 4.0)
    xb = tokens(T, K, [N, K, T])
    prec = np.random.default_rng([N, T]).integers(0, 4, size=T).astype(np.int32)
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, ALGOS[algo])
    assert_output_close(Y, Yref, f"{algo} N={N} K={K} T={T}")


@pytest.mark.parametrize("algo", ["decode", "prefill"])
@pytest.mark.parametrize("p", [0, 1, 2, 3])
def test_linear_single_precision_is_a_dense_gemm(mbq, algo, p):
    """All tokens at one precision: three empty buckets; equals X What^T (dense library matmul)."""
    N, K, T = 96, 768, 16 if algo == "decode" else 150
    print(f"[case] linear {algo} uniform p={p}", flush=True)
    W = make_weight(N, K, [13, p], 4.0)
    xb = tokens(T, K, [p, 5])
    prec = np.full(T, p, dtype=np.int32)
    codes, s0, z0 = O.encode(W)
    dense = torch.from_numpy(O.bf16_bits_to_f64(xb)) @ torch.from_numpy(O.dequant_merged(codes, s0, z0, p)).T
    Y = run_linear(mbq, W, xb, prec, ALGOS[algo])
    assert_output_close(Y, dense.numpy(), f"{algo} uniform p={p}")


@pytest.mark.parametrize("N,K,T,mix", [
    (300, 128, 70, None),            # one group (no rescale), N not a multiple of 16 or 256, one ragged tile per bucket
    (520, 1152, 513, None),          # odd group count (tail pairs end on a single group), three column tiles
    (272, 512, 300, (0.9, 0.1, 0.0, 0.0)),   # full 128-row tiles plus a ragged rest in bucket 0, an empty bucket
    (256, 768, 600, (0.0, 0.0, 0.5, 0.5)),   # full tiles at precisions 2 and 3 (8-bit operand path)
])
def test_prefill_tile_shapes(mbq, N, K, T, mix):
    """Full and ragged tiles, group-boundary rescale, the fp32 zero-point tail, column padding."""
    print(f"[case] prefill tiles N={N} K={K} T={T} mix={mix}", flush=True)
    W = make_weight(N, K, [17, N, K], 4.0)
    xb = tokens(T, K, [N, K, T, 1])
    rng = np.random.default_rng([N, T, 3])
    prec = (rng.integers(0, 4, size=T) if mix is None else rng.choice(4, size=T, p=mix)).astype(np.int32)
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, ALGOS["prefill"])
    assert_output_close(Y, Yref, f"prefill N={N} K={K} T={T}")


@pytest.mark.parametrize("counts", [(1, 16, 17, 32), (33, 64, 65, 96), (97, 128, 129, 1), (0, 0, 200, 257), (127, 0, 191, 63)])
@pytest.mark.parametrize("Ns,K", [((257,), 128), ((16, 300), 2048), ((1, 255, 64), 4352)])
@pytest.mark.parametrize("parts", [0, 1, 2])
def test_prefill_remainders_and_groups(mbq, counts, Ns, K, parts):
    """Buckets that end at the edges of the 16-, 32-, 64-, 96- and 128-row tiles, several matrices with orders of their own
    in one launch.  In one part: K of one group, of exactly one pass of the zero-point update and of two passes and a
    rest; in two: passes half way through 8 groups and behind 16 with one group left; cut as the library chooses (0)."""
    T = sum(counts)
    xb = tokens(T, K, [T, K, 71])
    X = dev_bf16(xb).reshape(T, K)
    blobs, routing, refs = [], [], []
    for i, N in enumerate(Ns):
        W = make_weight(N, K, [71, N, K, i], 4.0)
        codes, s0, z0 = O.encode(W)
        prec = np.repeat(np.arange(4), np.roll(counts, i)).astype(np.int32)
        np.random.default_rng([71, T, i]).shuffle(prec)
        perm, offsets = O.bucket(prec)
        blobs.append(mbq.mbq_encode(dev(W)))
        routing.append((dev(prec), dev(perm), dev(offsets)))
        refs.append(O.linear(xb, codes, s0, z0, prec))
    mbq.set_knob(5, parts)
    try:
        Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, algo=ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    torch.cuda.synchronize()
    for i in range(len(Ns)):
        assert_output_close(Ys[i].cpu().numpy(), refs[i], f"prefill group matrix {i}, {parts} parts")


def test_prefill_above_four_gibibytes_of_activations(mbq):
    """Row offsets of the tile kernel are 32-bit; from 4 GiB of activations on it reads a sorted copy instead."""
    T, K, N = 131200, 16384, 40
    assert T * K * 2 > 2 ** 32
    W = make_weight(N, K, [73, N], 4.0)
    blob = mbq.mbq_encode(dev(W))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(73)
    X = torch.empty((T, K), dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 8200):
        X[t:t + 8200] = torch.randn((8200, K), generator=gen, device="cuda").to(torch.bfloat16)
    prec = torch.randint(0, 4, (T,), generator=gen, device="cuda", dtype=torch.int32)
    perm = torch.sort(prec.long(), stable=True)[1].int()
    offsets = torch.stack([(prec < q).sum() for q in range(5)]).int()
    Y = mbq.mbq_linear(X, blob, N, K, prec, perm, offsets, algo=ALGOS["prefill"])
    pick = torch.cat([torch.arange(0, 40), torch.arange(60000, 60040), torch.arange(T - 40, T)]).cuda()
    for p in range(4):
        rows = pick[prec[pick] == p]
        ref = X[rows].double() @ mbq.mbq_dequant(blob, N, K, p).double().T
        assert_output_close(Y[rows].cpu().numpy(), ref.cpu().numpy(), f"precision {p}")


@pytest.mark.parametrize("T,K,N,parts", [(131200, 16384, 40, 2), (16384, 131072, 256, 0)])
def test_prefill_sorted_copy_in_two_parts(mbq, T, K, N, parts):
    """From 4 GiB of activations on, two parts of K add into outputs that the launch ahead clears: forced, and a shape that takes
    two by itself.  Whatever the outputs held before, and again on the outputs of the call before."""
    assert T * K * 2 > 2 ** 32 - 1
    gen = torch.Generator(device="cuda")
    gen.manual_seed(157)
    blob = mbq.mbq_encode(0.02 * torch.randn((N, K), generator=gen, device="cuda"))
    X = torch.empty((T, K), dtype=torch.bfloat16, device="cuda")
    for t in range(0, T, 2050):
        X[t:t + 2050] = torch.randn((min(2050, T - t), K), generator=gen, device="cuda").to(torch.bfloat16)
    prec = torch.randint(0, 4, (T,), generator=gen, device="cuda", dtype=torch.int32)
    r = (prec, torch.sort(prec.long(), stable=True)[1].int(), torch.stack([(prec < q).sum() for q in range(5)]).int())
    Y = torch.full((T, N), float("nan"), device="cuda")
    mbq.set_knob(5, parts)
    try:
        mbq.mbq_linear(X, blob, N, K, *r, Y=Y, algo=ALGOS["prefill"])
        first = Y.clone()
        mbq.mbq_linear(X, blob, N, K, *r, Y=Y, algo=ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    assert torch.equal(first, Y)
    pick = torch.cat([torch.arange(0, 40), torch.arange(T // 2, T // 2 + 40), torch.arange(T - 40, T)]).cuda()
    for p in range(4):
        rows = pick[prec[pick] == p]
        ref = X[rows].double() @ mbq.mbq_dequant(blob, N, K, p).double().T
        assert_output_close(Y[rows].cpu().numpy(), ref.cpu().numpy(), f"precision {p}")


@pytest.mark.parametrize("T,K,n", [(129, 128, 1), (257, 640, 3), (1024, 384, 2), (1025, 128, 4), (1041, 4224, 1), (2064, 640, 3)])
def test_route_group_above_128_tokens(mbq, T, K, n):
    """The general routers on both sides of their token limits, odd token counts, one 128-column block (most wavefronts
    of a tile without work) and odd numbers of blocks: precisions, order and offsets of every router of the call."""
    xb = tokens(T, K, [T, K, 79])
    rng = np.random.default_rng([T, K, 79])
    Wr = [(rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32) for _ in range(n)]
    br = [rng.standard_normal(4).astype(np.float32) * 0.3 for _ in range(n)]
    got = mbq.mbq_route_group(dev_bf16(xb).reshape(T, K), [dev(w) for w in Wr], [dev(b) for b in br])
    torch.cuda.synchronize()
    for i in range(n):
        _, prec_ref, gap = O.route(xb, Wr[i], br[i])
        prec = got[i][0].cpu().numpy()
        compare_routing(prec, prec_ref, gap, f"router {i}")
        check_bucket(prec, got[i][1].cpu().numpy(), got[i][2].cpu().numpy())


@pytest.mark.parametrize("splits", [2, 3, 4, 7])
def test_prefill_k_split(mbq, splits):
    """The K range of a tile cut into workgroups: two that add into a cleared Y, more with arrays of their own."""
    N, K, T = 272, 2304, 300     # 18 groups: uneven ranges, at least four groups each (seven parts become four)
    print(f"[case] prefill K split {splits}", flush=True)
    W = make_weight(N, K, [19, splits], 4.0)
    xb = tokens(T, K, [N, K, T, 2])
    prec = np.random.default_rng([splits, 5]).integers(0, 4, size=T).astype(np.int32)
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    mbq.set_knob(5, splits)
    try:
        Y = run_linear(mbq, W, xb, prec, ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    assert_output_close(Y, Yref, f"prefill K split {splits}")


@pytest.mark.parametrize("parts", [3, 4, 5, 6, 8])
@pytest.mark.parametrize("T,Ns", [(301, (999,)), (301, (1999,)), (70, (272, 17)), (130, (5, 1001, 300))])
def test_prefill_parts_in_arrays_of_their_own(mbq, parts, T, Ns):
    """More than two parts along K go to arrays of the workspace and are added in order: one or two parts an array, as
    many arrays as there is room for (301 tokens: 5 and 3 of them, Y included, T N not a multiple of four), several
    matrices in one launch, an output that allows 16-byte accesses and one that does not; the same bits on every call."""
    K = 4608  # 36 groups: eight parts of four or five
    xb = tokens(T, K, [T, K, 101])
    X = dev_bf16(xb).reshape(T, K)
    blobs, routing, refs = [], [], []
    for i, N in enumerate(Ns):
        W = make_weight(N, K, [101, N, i], 4.0)
        codes, s0, z0 = O.encode(W)
        prec = np.random.default_rng([101, T, i]).integers(0, 4, size=T).astype(np.int32)
        perm, offsets = O.bucket(prec)
        blobs.append(mbq.mbq_encode(dev(W)))
        routing.append((dev(prec), dev(perm), dev(offsets)))
        refs.append(O.linear(xb, codes, s0, z0, prec))
    mbq.set_knob(5, parts)
    try:
        Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, algo=ALGOS["prefill"])
        shifted = [torch.full((T * N + 1,), float("nan"), device="cuda")[1:].view(T, N) for N in Ns]
        again = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, Y=shifted, algo=ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    torch.cuda.synchronize()
    for i in range(len(Ns)):
        assert_output_close(Ys[i].cpu().numpy(), refs[i], f"{parts} parts, matrix {i}")
        assert torch.equal(Ys[i], again[i]), i


@pytest.mark.parametrize("groups", [1, 2, 8, 9, 15, 16, 17, 32, 33])
@pytest.mark.parametrize("parts", [1, 2])
def test_prefill_windows_of_row_sums(mbq, groups, parts):
    """The rows' sums come in windows of 16 groups: lengths around one and two windows, parts that begin inside a window,
    every row-tile count, outputs that allow 16-byte stores and the same numbers where they do not.  (The zero-point term
    of parts of at most 8 groups comes in fp32, of longer ones in bf16 pieces.)"""
    K, N, T = 128 * groups, 276, 1 + 40 + 70 + 128
    xb = tokens(T, K, [T, K, 131])
    W = make_weight(N, K, [131, K], 4.0)
    codes, s0, z0 = O.encode(W)
    prec = np.random.default_rng([131]).permutation(np.repeat(np.arange(4), (1, 40, 70, 128))).astype(np.int32)
    perm, offsets = O.bucket(prec)
    X, blob, r = dev_bf16(xb).reshape(T, K), mbq.mbq_encode(dev(W)), (dev(prec), dev(perm), dev(offsets))
    shifted = torch.full((T * N + 1,), float("nan"), device="cuda")[1:].view(T, N)
    mbq.set_knob(5, parts)
    try:
        Y = mbq.mbq_linear(X, blob, N, K, *r, algo=ALGOS["prefill"])
        mbq.mbq_linear(X, blob, N, K, *r, Y=shifted, algo=ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    torch.cuda.synchronize()
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"{groups} groups, {parts} parts")
    assert torch.equal(Y, shifted)


@pytest.mark.parametrize("p", [0, 1, 2, 3])
def test_prefill_many_windows_of_row_sums(mbq, p):
    """Each window's sums take the place of those before: many windows, tiles with every number of row tiles, the zero-point
    term in either form; three calls give the same bits, and those are the oracle's within the bar."""
    K, N = 128 * 90, 272
    counts = np.roll((128, 70, 33, 20), p)
    T = int(counts.sum())
    xb = tokens(T, K, [T, K, 151])
    W = make_weight(N, K, [151, N], 4.0)
    codes, s0, z0 = O.encode(W)
    prec = np.random.default_rng([151, p]).permutation(np.repeat(np.arange(4), counts)).astype(np.int32)
    perm, offsets = O.bucket(prec)
    X, blob, r = dev_bf16(xb).reshape(T, K), mbq.mbq_encode(dev(W)), (dev(prec), dev(perm), dev(offsets))
    mbq.set_knob(5, 1)
    try:
        Y, *again = [mbq.mbq_linear(X, blob, N, K, *r, algo=ALGOS["prefill"]) for _ in range(3)]
    finally:
        mbq.set_knob(5, 0)
    torch.cuda.synchronize()
    assert all(torch.equal(Y, y) for y in again)
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"rows {counts}")


@pytest.mark.parametrize("N", [16, 48, 272, 300])
@pytest.mark.parametrize("turn", [0, 1, 2, 3])
def test_prefill_pairs_of_code_tiles(mbq, N, turn):
    """The tile kernel takes columns in pairs of code tiles and rows by 32: odd numbers of code tiles (the last pair's second
    tile is past the matrix), every number of row tiles at every precision, first and last rows of a row tile."""
    K, sizes = 384, np.roll((1, 33, 96, 97), turn)
    T = int(sizes.sum())
    xb = tokens(T, K, [T, N, 137])
    W = make_weight(N, K, [137, N], 4.0)
    codes, s0, z0 = O.encode(W)
    prec = np.random.default_rng([137, turn]).permutation(np.repeat(np.arange(4), sizes)).astype(np.int32)
    perm, offsets = O.bucket(prec)
    X, blob = dev_bf16(xb).reshape(T, K), mbq.mbq_encode(dev(W))
    Y = mbq.mbq_linear(X, blob, N, K, dev(prec), dev(perm), dev(offsets), algo=ALGOS["prefill"])
    torch.cuda.synchronize()
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"N={N}, rows {sizes}")


@pytest.mark.parametrize("parts", [0, 2, 6])
@pytest.mark.parametrize("T,K,Ns", [(129, 2304, (300, 530)), (256, 384, (272,)), (257, 4608, (999, 64, 130)),
                                    (1024, 640, (260, 36)), (1025, 1152, (530,)), (1041, 4608, (72, 300, 130, 16))])
def test_stage_call_whose_router_launch_prepares_the_prefill(mbq, T, K, Ns, parts):
    """Above 128 tokens the stage's router launch also forms the row sums and clears the arrays that parts add into: the same
    bits as the two calls, whatever outputs and workspace held before, at the token counts where the router changes."""
    xb = tokens(T, K, [T, K, 139])
    X = dev_bf16(xb).reshape(T, K)
    rng = np.random.default_rng([T, K, 139])
    Wr = [dev((rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32)) for _ in Ns]
    br = [dev(rng.normal(0, 0.3, size=4).astype(np.float32)) for _ in Ns]
    Ws = [make_weight(N, K, [139, N, i], 4.0) for i, N in enumerate(Ns)]
    blobs = [mbq.mbq_encode(dev(W)) for W in Ws]
    ws_linear = mbq.linear_workspace(T, max(Ns), K, "cuda")
    ws_linear.fill_(255)  # floats of NaN
    Y = [torch.full((T, N), float("nan"), device="cuda") for N in Ns]
    mbq.set_knob(5, parts)
    try:
        routing, Ys = mbq.mbq_routed_linear_group(X, Wr, br, blobs, list(Ns), Y=Y, ws_linear=ws_linear, algo=ALGOS["prefill"])
        again = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, algo=ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    torch.cuda.synchronize()
    routing2 = mbq.mbq_route_group(X, Wr, br)
    for i, N in enumerate(Ns):
        for a, b in zip(routing[i], routing2[i]):
            assert torch.equal(a, b), i
        assert torch.equal(Ys[i], again[i]), i
    codes, s0, z0 = O.encode(Ws[0])
    want = O.linear(xb, codes, s0, z0, routing[0][0].cpu().numpy())
    assert_output_close(Ys[0].cpu().numpy(), want, f"T={T}, {parts} parts")


@pytest.mark.parametrize("parts", [2, 6])
def test_prefill_parts_replay_from_a_hip_graph(mbq, parts):
    """A captured call that clears arrays, adds into them and adds them up, replayed with eager work of the same kind in
    its workspace and outputs between the replays: the eager call's bits every time."""
    N, K, T = 999, 4608, 301
    xb = tokens(T, K, [T, K, 107])
    X = dev_bf16(xb).reshape(T, K)
    blob = mbq.mbq_encode(dev(make_weight(N, K, [107], 4.0)))
    prec = np.random.default_rng([107]).integers(0, 4, size=T).astype(np.int32)
    perm, offsets = O.bucket(prec)
    r = (dev(prec), dev(perm), dev(offsets))
    X2, r2 = X.flip(0).contiguous(), tuple(dev(v) for v in (prec[::-1].copy(), *O.bucket(prec[::-1])))
    Y, ws = torch.empty((T, N), dtype=torch.float32, device="cuda"), mbq.linear_workspace(T, N, K, "cuda")
    mbq.set_knob(5, parts)
    try:
        want = mbq.mbq_linear(X, blob, N, K, *r, algo=ALGOS["prefill"])
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side):
            mbq.mbq_linear(X, blob, N, K, *r, Y=Y, ws=ws, algo=ALGOS["prefill"])
        torch.cuda.current_stream().wait_stream(side)
        with torch.cuda.graph(g):
            mbq.mbq_linear(X, blob, N, K, *r, Y=Y, ws=ws, algo=ALGOS["prefill"])
        for _ in range(4):
            mbq.mbq_linear(X2, blob, N, K, *r2, Y=Y, ws=ws, algo=ALGOS["prefill"])
            torch.cuda.synchronize()
            assert not torch.equal(Y, want)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(Y, want)
    finally:
        mbq.set_knob(5, 0)


@pytest.mark.parametrize("Ns,K,T", [
    ((14336, 14336), 4096, 96), ((14336, 14336), 4096, 256), ((11008, 11008), 4096, 384), ((11008, 11008), 4096, 777),
    ((13824, 13824), 5120, 256), ((4096, 4096), 4096, 512), ((11008,), 4096, 96), ((11008,), 4096, 256),
    ((4096,), 11008, 96), ((4096,), 14336, 128), ((4096,), 11008, 777), ((8192,), 28672, 256)])
def test_prefill_bits_do_not_depend_on_the_call(mbq, Ns, K, T):
    """The automatic cut along K: three equal calls give the same bits, and a call for several matrices those of separate
    calls (each of these takes one or two parts alone).  Nothing but the bits is compared."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(103 + T)
    X = torch.randn((T, K), generator=gen, device="cuda").to(torch.bfloat16)
    blobs, routing = [], []
    for N in Ns:
        blobs.append(mbq.mbq_encode(0.02 * torch.randn((N, K), generator=gen, device="cuda")))
        prec = torch.randint(0, 4, (T,), generator=gen, device="cuda", dtype=torch.int32)
        perm = torch.sort(prec.long(), stable=True)[1].int()
        routing.append((prec, perm, torch.stack([(prec < q).sum() for q in range(5)]).int()))
    first = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, algo=ALGOS["prefill"])
    for _ in range(2):
        for a, b in zip(first, mbq.mbq_linear_group(X, blobs, list(Ns), K, routing, algo=ALGOS["prefill"])):
            assert torch.equal(a, b)
    for i, N in enumerate(Ns):
        assert torch.equal(first[i], mbq.mbq_linear(X, blobs[i], N, K, *routing[i], algo=ALGOS["prefill"])), i


@pytest.mark.parametrize("K", [768, 2048, 4096, 5120, 11008])
@pytest.mark.parametrize("pmax", [0, 1, 2, 3])
@pytest.mark.parametrize("T", [7, 16, 40])
def test_decode_every_highest_precision(mbq, K, pmax, T):
    """The decode kernels are specialised on the highest precision present and on the number of
    column blocks (4, 8 or 16 wavefronts, one or several K chunks): cover every combination."""
    N = 80
    print(f"[case] decode pmax={pmax} K={K} T={T}", flush=True)
    W = make_weight(N, K, [19, K], 4.0)
    xb = tokens(T, K, [K, pmax, T])
    prec = np.random.default_rng([K, pmax, T]).integers(0, pmax + 1, size=T).astype(np.int32)
    prec[T // 2] = pmax
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, ALGOS["decode"])
    assert_output_close(Y, Yref, f"decode pmax={pmax} K={K} T={T}")


@pytest.mark.parametrize("K,N,T,pmax", [(8448, 80, 16, 3), (11008, 272, 16, 3), (11008, 4096, 13, 2), (14336, 130, 1, 3),
                                        (16384, 64, 16, 1), (9216, 2064, 7, 3), (12288, 16, 16, 0), (16384, 16500, 5, 3)])
def test_decode_one_token_tile_long_rows(mbq, K, N, T, pmax):
    """8192 < K <= 16384 at up to 16 tokens: the loader kernel works through each of its two parts in two chunks and
    keeps the tiles' sums of the first chunk in LDS (few enough tiles per workgroup), else the kernel that streams the
    activations with the weights takes over (the last case: 1032 row tiles); outputs also identical from call to call."""
    print(f"[case] decode long rows K={K} N={N} T={T} pmax={pmax}", flush=True)
    W = make_weight(N, K, [53, N, K], 4.0)
    xb = tokens(T, K, [K, N, T])
    prec = np.random.default_rng([K, N, T]).integers(0, pmax + 1, size=T).astype(np.int32)
    prec[T // 2] = pmax
    blob = mbq.mbq_encode(dev(W))
    perm, offsets = O.bucket(prec)
    X = dev_bf16(xb).reshape(T, K)
    args = (X, blob, N, K, dev(prec), dev(perm), dev(offsets))
    Y = mbq.mbq_linear(*args, algo=ALGOS["decode"])
    Y2 = mbq.mbq_linear(*args, algo=ALGOS["decode"])
    torch.cuda.synchronize()
    assert torch.equal(Y, Y2)
    rows = np.arange(N) if N <= 4096 else np.random.default_rng(3).choice(N, 2048, replace=False)
    codes, s0, z0 = O.encode(W[rows])
    assert_output_close(Y.cpu().numpy()[:, rows], O.linear(xb, codes, s0, z0, prec), f"long rows K={K} N={N} T={T}")


@pytest.mark.parametrize("T,K,N", [(17, 4096, 130), (31, 2304, 48), (32, 4096, 64), (33, 1024, 272), (48, 4096, 40),
                                   (49, 2048, 130), (64, 4096, 2064), (64, 256, 16)])
def test_decode_several_token_tiles(mbq, T, K, N):
    """17..64 tokens: one pass over the weights per 16 precision-sorted tokens, each reading the slices of
    ITS highest precision; mixes chosen so that the passes differ."""
    print(f"[case] decode token tiles T={T} K={K} N={N}", flush=True)
    W = make_weight(N, K, [37, N, K], 4.0)
    xb = tokens(T, K, [T, K, 41])
    rng = np.random.default_rng([T, K, N])
    prec = rng.integers(0, 4, size=T).astype(np.int32)
    prec[:32] = np.minimum(prec[:32], 2)      # first window: at most 6 bits
    prec[5] = 2
    if T > 40:
        prec[40] = 3
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, ALGOS["decode"])
    assert_output_close(Y, Yref, f"decode token tiles T={T} K={K} N={N}")


def reference64(X, blob, N, K, prec):
    """The routed output in 64 bits from the weights that mbq_dequant gives (itself pinned against the oracle)."""
    import paper_2602_20191_amd as pkg

    Y = torch.zeros((X.shape[0], N), dtype=torch.float64, device="cuda")
    for p in range(4):
        rows = torch.nonzero(prec == p).flatten()
        if len(rows):
            Y[rows] = X[rows].double() @ pkg.mbq_dequant(blob, N, K, p).double().T
    return Y


@pytest.mark.parametrize("T,mix", [(33, (0, 1, 2, 3)), (48, (16, 16, 16, 0)), (49, (0, 0, 49, 0)), (63, (5, 30, 1, 27)), (64, (16, 16, 16, 16)),
                                   (64, (0, 0, 0, 64)), (40, (40, 0, 0, 0)), (64, (31, 0, 32, 1))])
@pytest.mark.parametrize("Ns,K", [((10240,), 128), ((10243, 10300), 640), ((10240, 10240), 4096), ((3072,), 8448), ((3075, 3072), 8320)])
def test_decode_wide_matrices_and_long_rows(mbq, T, mix, Ns, K):
    """33 to 64 tokens on the shapes of the kernel that unpacks once for all tokens: precisions that begin on a row tile
    and inside one, absent ones, a last block of one group, parts along K, columns past the matrix.  Against 64 bits (32-bit
    sums: 4e-5), a group against single calls and a stage against its two calls bit for bit, an output that is not 16-byte
    aligned against one that is."""
    counts = mix if sum(mix) == T else (T - sum(mix[1:]), *mix[1:])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(149 + T + K)
    X = torch.randn((T, K), generator=gen, device="cuda")
    X[:, torch.randperm(K, generator=gen, device="cuda")[: K // 100]] *= 20.0
    X = X.to(torch.bfloat16)
    blobs, routing = [], []
    for i, N in enumerate(Ns):
        blobs.append(mbq.mbq_encode(0.02 * torch.randn((N, K), generator=gen, device="cuda")))
        prec = np.random.default_rng([149, T, i]).permutation(np.repeat(np.arange(4), counts)).astype(np.int32)
        routing.append((dev(prec), *[dev(v) for v in O.bucket(prec)]))
    Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing)
    for i, N in enumerate(Ns):
        ref = reference64(X, blobs[i], N, K, routing[i][0])
        assert float((Ys[i].double() - ref).norm() / ref.norm()) < 4e-5, i
        assert torch.equal(Ys[i], mbq.mbq_linear(X, blobs[i], N, K, *routing[i])), i
        shifted = torch.full((T * N + 1,), float("nan"), device="cuda")[1:].view(T, N)
        assert torch.equal(Ys[i], mbq.mbq_linear(X, blobs[i], N, K, *routing[i], Y=shifted)), i
    Wr = [torch.randn((4, K), generator=gen, device="cuda") / K ** 0.5 for _ in Ns]
    br = [torch.zeros(4, device="cuda") for _ in Ns]
    stage_routing, stage_Y = mbq.mbq_routed_linear_group(X, Wr, br, blobs, list(Ns))
    separate = mbq.mbq_route_group(X, Wr, br)
    for a, b in zip(stage_routing, separate):
        assert all(torch.equal(x, y) for x, y in zip(a, b))
    for a, b in zip(stage_Y, mbq.mbq_linear_group(X, blobs, list(Ns), K, separate)):
        assert torch.equal(a, b)


@pytest.mark.parametrize("T,mix", [(33, (8, 9, 8, 8)), (48, (0, 17, 31, 0)), (49, (48, 0, 0, 1)), (64, (16, 15, 17, 16))])
@pytest.mark.parametrize("Ns,K", [((10740,), 128), ((10752, 10740), 384), ((10750, 13312), 896), ((11250,), 1408), ((11264, 11267), 1536),
                                  ((16384,), 1664), ((11300,), 2432), ((12800, 13000), 3328), ((12800,), 3456), ((13001,), 3968),
                                  ((16300, 12790), 4096), ((24570,), 1536), ((24580,), 3840)])
def test_decode_wide_matrices_in_halves(mbq, T, mix, Ns, K):
    """Wide matrices are the sum of two halves of K, formed at a time by one workgroup where the matrix is alone and in turn
    in a group or where it has more columns: the same bits.  Halves of the same and of different lengths, a last block of one
    group, both sides of the range's bounds in rows and columns."""
    test_decode_wide_matrices_and_long_rows(mbq, T, mix, Ns, K)


@pytest.mark.parametrize("T,mix", [(33, (8, 9, 8, 8)), (64, (16, 15, 17, 16))])
@pytest.mark.parametrize("Ns,K", [((1040, 3072), 8448), ((3072, 600, 3080, 513), 8320), ((3072, 80, 1040), 8448), ((12800, 272), 1536),
                                  ((33, 11270), 2048)])
def test_decode_groups_of_two_kernels(mbq, T, mix, Ns, K):
    """Groups of which only some matrices take the kernel of wide matrices and long rows: a launch for those of each kernel, one
    by one where a third is needed; outputs of the others that are added into (K = 8448) and that are not."""
    test_decode_wide_matrices_and_long_rows(mbq, T, mix, Ns, K)


@pytest.mark.parametrize("K,T,Ns", [(4096, 16, (96, 32, 130)), (4096, 1, (64, 64)), (2048, 7, (80, 48, 16, 33)),
                                    (768, 16, (40,)), (3072, 5, (48, 96)), (5120, 16, (48, 32)), (1024, 40, (48, 32)),
                                    (4096, 64, (1040, 130, 256)), (2304, 33, (272, 48, 16, 640)), (4352, 48, (2064, 16))])
def test_linear_group_equals_separate_calls(mbq, K, T, Ns):
    """Several matrices over one X, each with its own routing: against the oracle and bit for bit
    against mbq_linear (17..64 tokens: one launch of the register-stationary kernel for all matrices when
    each would take it, else per-matrix kernels inside the group call - the last shape)."""
    print(f"[case] linear group K={K} T={T} Ns={Ns}", flush=True)
    xb = tokens(T, K, [K, T, 9])
    X = dev_bf16(xb).reshape(T, K)
    blobs, routing, refs = [], [], []
    for i, N in enumerate(Ns):
        W = make_weight(N, K, [23, N, K, i], 4.0)
        codes, s0, z0 = O.encode(W)
        rng = np.random.default_rng([K, T, i])
        prec = rng.integers(0, (i % 4) + 1 if i else 4, size=T).astype(np.int32)   # different highest precisions
        perm, offsets = O.bucket(prec)
        blobs.append(mbq.mbq_encode(dev(W)))
        routing.append((dev(prec), dev(perm), dev(offsets)))
        refs.append(O.linear(xb, codes, s0, z0, prec))
    Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing)
    torch.cuda.synchronize()
    for i, N in enumerate(Ns):
        assert_output_close(Ys[i].cpu().numpy(), refs[i], f"group matrix {i}")
        single = mbq.mbq_linear(X, blobs[i], N, K, *routing[i])
        assert torch.equal(single, Ys[i])


@pytest.mark.parametrize("K,T,Ns", [(4096, 16, (96, 32, 130)), (2048, 1, (64, 48)), (1280, 9, (40,)), (5120, 16, (48, 32)),
                                    (1024, 40, (48, 32)),
                                    # 29..64 tokens: the linear launch sorts the tokens; last shape: one matrix takes
                                    # another kernel, so the stage falls back to the two calls
                                    (4096, 64, (1040, 130)), (2304, 33, (272, 48, 16)), (512, 17, (40,)), (4352, 48, (2064, 16)),
                                    # 65..128 tokens under the automatic choice: the same path, two tokens per sorting lane
                                    (4096, 65, (272, 130)), (2304, 128, (1040, 48, 16)), (1024, 100, (40, 300)),
                                    # many row tiles: the whole chip takes part, K in one part, two parts and streamed
                                    (1024, 5, (1024, 528)), (4096, 16, (1040, 512, 512)), (9216, 3, (1600,)), (2304, 16, (640, 130))])
def test_routed_linear_stage_equals_route_then_linear(mbq, K, T, Ns):
    """One block stage in one call: same routing and the same outputs, bit for bit, as mbq_route_group
    followed by mbq_linear_group, and within tolerance of the oracle; run twice on the same workspaces,
    which the calls must leave zeroed."""
    print(f"[case] stage K={K} T={T} Ns={Ns}", flush=True)
    rng = np.random.default_rng([K, T, len(Ns)])
    xb = tokens(T, K, [K, T, 31])
    X = dev_bf16(xb).reshape(T, K)
    Wrs = [(rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32) for _ in Ns]
    brs = [rng.normal(0, 0.3, size=4).astype(np.float32) for _ in Ns]
    Ws = [make_weight(N, K, [29, N, K, i], 4.0) for i, N in enumerate(Ns)]
    blobs = [mbq.mbq_encode(dev(W)) for W in Ws]
    ws_r = mbq.route_workspace(T, K, "cuda").fill_(0xA5)
    ws_l = mbq.linear_workspace(T, max(Ns), K, "cuda")
    dWr, dbr = [dev(w) for w in Wrs], [dev(b) for b in brs]
    for _ in range(2):
        routing, Ys = mbq.mbq_routed_linear_group(X, dWr, dbr, blobs, list(Ns), ws_route=ws_r, ws_linear=ws_l)
        torch.cuda.synchronize()
        routing2 = mbq.mbq_route_group(X, dWr, dbr)
        Ys2 = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing2)
        for i, N in enumerate(Ns):
            for a, b in zip(routing[i], routing2[i]):
                assert torch.equal(a, b)
            assert torch.equal(Ys[i], Ys2[i])
            S, prec_ref, gap = O.route(xb, Wrs[i], brs[i])
            prec = routing[i][0].cpu().numpy()
            compare_routing(prec, prec_ref, gap, f"stage router {i}")
            check_bucket(prec, routing[i][1].cpu().numpy(), routing[i][2].cpu().numpy())
            codes, s0, z0 = O.encode(Ws[i])
            assert_output_close(Ys[i].cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"stage matrix {i}")


@pytest.mark.parametrize("algo,T", [("decode", 12), ("decode", 40), ("prefill", 300)])
def test_linear_special_activation_rows(mbq, algo, T):
    """Rows that stress the activation handling: all zeros, all tiny (1e-30), one element 2^20 times the rest of
    its block, negative zeros, a constant row, an outlier in another 256-column block than the small values, bf16
    subnormals (alone in their block and next to normal values); every row is held to the bar on its own as well."""
    N, K = 130, 1280
    print(f"[case] special rows {algo} T={T}", flush=True)
    W = make_weight(N, K, [43, T], 4.0)
    rng = np.random.default_rng([43, T])
    x = rng.standard_normal((T, K)).astype(np.float32)
    x[0] = 0.0
    x[1] *= 1e-30
    x[2] *= 1e-3
    x[2, 300] = 1e3
    x[3, ::2] = -0.0
    x[4] = 0.75
    x[5] *= 1e-4
    x[5, 256:512] *= 1e8                      # block 1 of the row is 10^8 times its other blocks
    x[6] *= 1e-3
    x[6, :256] = rng.standard_normal(256) * 2.0 ** -130      # a block of subnormals only (bf16 keeps 2^-133)
    x[6, 600:640] = rng.standard_normal(40) * 2.0 ** -128    # subnormals among normal values
    x[7] = rng.standard_normal(K) * 2.0 ** -131               # a whole row of subnormals
    xb = f32_to_bf16_bits(x)
    assert (xb[7] & 0x7F80).max() == 0 and (xb[7] & 0x7F).max() > 0   # really subnormal, and not all zero
    prec = rng.integers(0, 4, size=T).astype(np.int32)
    prec[:8] = [3, 2, 3, 1, 0, 3, 3, 2]
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, ALGOS[algo])
    assert np.all(np.isfinite(Y))
    assert_output_close(Y, Yref, f"special rows {algo} T={T}")
    assert not Y[0].any(), "an all-zero token must give an all-zero output row"
    for i in range(1, 7):
        assert_output_close(Y[i:i + 1], Yref[i:i + 1], f"special row {i}")
    if algo == "decode" and T <= 16:
        # The two-FP8-piece split cannot scale a block below 2^-122 (the block scale is an 8-bit exponent and the
        # second piece sits 4 binades lower): elements of a block whose largest is under 2^-115 are rounded to
        # multiples of 2^-135, an eighth of bf16's subnormal spacing.  Row 7 is held to that bound element by
        # element: |dY[n]| <= 2^-136 sum_k |W^(p)[n, k]|, plus the ordinary bar for the fp32 accumulation.
        What = O.dequant(codes, s0, z0, int(prec[7]))
        bound = 2.0 ** -136 * np.abs(What).sum(axis=1) + MAX_ABS_TOL * np.sqrt(np.mean(Yref[7] ** 2))
        err = np.abs(Y[7].astype(np.float64) - Yref[7])
        print(f"[parity] special row 7 (subnormals): max err/bound {float((err / bound).max()):.3f}", flush=True)
        assert np.all(err <= bound)
    else:
        assert_output_close(Y[7:8], Yref[7:8], "special row 7")


@pytest.mark.parametrize("T", [16, 64])
def test_stage_call_replays_from_a_hip_graph(mbq, T):
    """The stage call captured once and replayed with new activations in the same buffers (eager work and
    synchronisation between the replays): every replay equals the eager call bit for bit.  K = 4096 takes the
    two-part kernels at both token counts, whose outputs the router launch zeroes with a kernel (not a memset
    node); at 64 tokens the linear launch also sorts the tokens."""
    K, Ns = 4096, (272, 130)
    print(f"[case] stage call under graph replay T={T}", flush=True)
    rng = np.random.default_rng(47)
    Wrs = [dev((rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32)) for _ in Ns]
    brs = [dev(rng.normal(0, 0.3, size=4).astype(np.float32)) for _ in Ns]
    blobs = [mbq.mbq_encode(dev(make_weight(N, K, [47, N], 4.0))) for N in Ns]
    X = dev_bf16(tokens(T, K, [47, 0])).reshape(T, K)
    ws_r = mbq.route_workspace(T, K, "cuda")
    ws_l = mbq.linear_workspace(T, max(Ns), K, "cuda")
    routing = [(torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty(T, dtype=torch.int32, device="cuda"),
                torch.empty(5, dtype=torch.int32, device="cuda")) for _ in Ns]
    Ys = [torch.empty((T, N), dtype=torch.float32, device="cuda") for N in Ns]

    def call():
        mbq.mbq_routed_linear_group(X, Wrs, brs, blobs, list(Ns), routing=routing, Y=Ys, ws_route=ws_r, ws_linear=ws_l)

    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for rep in range(4):
        X.copy_(dev_bf16(tokens(T, K, [47, rep + 1])).reshape(T, K))
        call()
        torch.cuda.synchronize()
        want = [[t.clone() for t in r] for r in routing], [y.clone() for y in Ys]
        for y in Ys:
            y.fill_(float("nan"))
        for r in routing:
            for t in r:
                t.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        for i in range(len(Ns)):
            for a, b in zip(want[0][i], routing[i]):
                assert torch.equal(a, b), (rep, i)
            assert torch.equal(want[1][i], Ys[i]), (rep, i)


def test_stage_calls_on_drawn_shapes(mbq):
    """Stage calls on seeded random shapes (1..4 matrices, 1..64 tokens, K up to 6144, ragged N): routing,
    permutation and outputs against the oracle.  Covers the launch arithmetic of the grouped kernels (shares of
    workgroups per matrix, K parts, token passes) beyond the hand-picked shapes above."""
    rng = np.random.default_rng(2027)
    for case in range(14):
        n = int(rng.integers(1, 5))
        T = int(rng.choice([1, 7, 16, 17, 29, 33, 48, 63, 64]))
        K = 128 * int(rng.integers(1, 49))
        Ns = [int(rng.integers(1, 700)) for _ in range(n)]
        print(f"[case] drawn stage {case}: T={T} K={K} Ns={Ns}", flush=True)
        xb = tokens(T, K, [2027, case])
        X = dev_bf16(xb).reshape(T, K)
        Wrs = [(rng.standard_normal((4, K)) / np.sqrt(K)).astype(np.float32) for _ in Ns]
        brs = [rng.normal(0, 0.3, size=4).astype(np.float32) for _ in Ns]
        Ws = [make_weight(N, K, [53, case, i], 4.0) for i, N in enumerate(Ns)]
        blobs = [mbq.mbq_encode(dev(W)) for W in Ws]
        routing, Ys = mbq.mbq_routed_linear_group(X, [dev(w) for w in Wrs], [dev(b) for b in brs], blobs, Ns)
        torch.cuda.synchronize()
        for i, N in enumerate(Ns):
            S, prec_ref, gap = O.route(xb, Wrs[i], brs[i])
            prec = routing[i][0].cpu().numpy()
            compare_routing(prec, prec_ref, gap, f"drawn stage {case} router {i}")
            check_bucket(prec, routing[i][1].cpu().numpy(), routing[i][2].cpu().numpy())
            codes, s0, z0 = O.encode(Ws[i])
            assert_output_close(Ys[i].cpu().numpy(), O.linear(xb, codes, s0, z0, prec), f"drawn stage {case} matrix {i}")


def test_prefill_on_drawn_shapes(mbq):
    """mbq_linear above 64 tokens on seeded random shapes, automatic launch choice (including the K split that
    launches with few tiles take): outputs against the oracle."""
    rng = np.random.default_rng(2029)
    shapes = [(int(rng.integers(65, 700)), int(rng.integers(1, 600)), 128 * int(rng.integers(1, 40))) for _ in range(6)]
    shapes += [(130, 272, 8192), (600, 520, 9216), (257, 40, 12288)]
    for case, (T, N, K) in enumerate(shapes):
        print(f"[case] drawn prefill {case}: T={T} N={N} K={K}", flush=True)
        W = make_weight(N, K, [59, case], 4.0)
        xb = tokens(T, K, [2029, case])
        prec = rng.choice(4, size=T, p=[0.4, 0.3, 0.2, 0.1]).astype(np.int32)
        codes, s0, z0 = O.encode(W)
        Yref = O.linear(xb, codes, s0, z0, prec)
        Y = run_linear(mbq, W, xb, prec, 0)
        assert_output_close(Y, Yref, f"drawn prefill {case}")


@pytest.mark.parametrize("T,K,Ns", [(65, 4096, (130,)), (96, 2304, (48,)), (128, 4096, (272,)), (100, 1024, (40,)),
                                    (128, 4352, (2064,)), (96, 4096, (272, 130, 16)), (127, 512, (48, 300)),
                                    (80, 4352, (2064, 16)), (192, 4096, (130, 272)), (161, 2304, (48,)), (500, 1024, (300,)),
                                    (129, 4352, (2064, 16, 2080)), (150, 2048, (4112, 40)), (300, 4352, (40, 2064, 300)),
                                    (200, 4352, (2064, 16))])
def test_automatic_choice_above_64_tokens(mbq, T, K, Ns):
    """Above 64 tokens the automatic choice still takes the register-stationary kernel (one pass per 32 sorted
    tokens, the tokens dealt evenly to the passes) up to 128 tokens, 512 for small matrices, 161..256 for matrices with
    more columns than rows, alone or as one launch for a group.  A matrix of more than 2048 code blocks (2064 x 4352 has
    2193, 4112 x 2048 has 2056) takes the prefill kernel at 129..160 and above 256 tokens: those groups mix the two, the
    prefill matrices in one launch ahead of the others.  Group and single calls against the oracle and each other."""
    print(f"[case] automatic choice T={T} K={K} Ns={Ns}", flush=True)
    xb = tokens(T, K, [T, K, 61])
    X = dev_bf16(xb).reshape(T, K)
    blobs, routing, refs = [], [], []
    for i, N in enumerate(Ns):
        W = make_weight(N, K, [61, N, K, i], 4.0)
        codes, s0, z0 = O.encode(W)
        prec = np.random.default_rng([T, K, i]).integers(0, 4, size=T).astype(np.int32)
        perm, offsets = O.bucket(prec)
        blobs.append(mbq.mbq_encode(dev(W)))
        routing.append((dev(prec), dev(perm), dev(offsets)))
        refs.append(O.linear(xb, codes, s0, z0, prec))
    Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing)
    torch.cuda.synchronize()
    for i, N in enumerate(Ns):
        assert_output_close(Ys[i].cpu().numpy(), refs[i], f"automatic choice matrix {i}")
        single = mbq.mbq_linear(X, blobs[i], N, K, *routing[i])
        # (no bit-for-bit claim here: a matrix that goes to the prefill kernel may be cut into fewer parts along K in
        # company than alone, where it takes more than two)
        assert_output_close(single.cpu().numpy(), refs[i], f"automatic choice matrix {i}, single call")


@pytest.mark.parametrize("T", [129, 160, 161, 200, 256])
@pytest.mark.parametrize("mix", [(0.8, 0.15, 0.05, 0.0), (0.25, 0.25, 0.25, 0.25), (0.0, 0.0, 0.1, 0.9)])
def test_automatic_choice_from_129_to_256_tokens_on_every_mix(mbq, T, mix):
    """129..256 tokens on a matrix that is not small and has more columns than rows: the prefill kernel up to 160 tokens,
    the stationary kernel from there, whatever the mix (few slices, all of them, an empty bucket)."""
    N, K = 2064, 4352
    print(f"[case] automatic choice T={T} mix={mix}", flush=True)
    W = make_weight(N, K, [67, T], 4.0)
    xb = tokens(T, K, [67, T, 1])
    prec = np.random.default_rng([67, T]).choice(4, size=T, p=mix).astype(np.int32)
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    Y = run_linear(mbq, W, xb, prec, 0)
    assert_output_close(Y, Yref, f"automatic choice T={T} mix={mix}")


def test_linear_zero_tokens_and_bad_arguments(mbq):
    N, K = 32, 256
    W = make_weight(N, K, [17], 4.0)
    blob = mbq.mbq_encode(dev(W))
    empty = torch.empty((0, K), dtype=torch.bfloat16, device="cuda")
    z32 = torch.zeros(0, dtype=torch.int32, device="cuda")
    off = torch.zeros(5, dtype=torch.int32, device="cuda")
    Y = mbq.mbq_linear(empty, blob, N, K, z32, z32, off)
    assert Y.shape == (0, N)
    xb = tokens(70, K, 1)
    prec = np.zeros(70, dtype=np.int32)
    perm, offsets = O.bucket(prec)
    with pytest.raises(mbq.MbqError):       # the decode kernel refuses more than 64 tokens
        mbq.mbq_linear(dev_bf16(xb), blob, N, K, dev(prec), dev(perm), dev(offsets), algo=2)
    with pytest.raises(mbq.MbqError):       # workspace too small
        mbq.mbq_linear(dev_bf16(xb), blob, N, K, dev(prec), dev(perm), dev(offsets),
                       ws=torch.empty(16, dtype=torch.uint8, device="cuda"))


def test_config0_end_to_end(mbq):
    """BASELINE config 0: 2048 x 2048, 32 tokens, {40,30,20,10}% mix; full comparison, every kernel."""
    cfg = CONFIGS[0]
    case = make_case(cfg, 0, 32)
    W, xb, Wr, br = case["W"], case["X"], case["Wr"], case["br"]
    N, K = W.shape
    codes, s0, z0 = O.encode(W)
    S, prec_ref, gap = O.route(xb, Wr, br)
    X = dev_bf16(xb)
    blob = mbq.mbq_encode(dev(W))
    assert np.array_equal(blob.cpu().numpy(), O.pack_blob(codes, s0, z0))
    prec, perm, offsets = mbq.mbq_route(X, dev(Wr), dev(br))
    compare_routing(prec.cpu().numpy(), prec_ref, gap, "config 0")
    check_bucket(prec.cpu().numpy(), perm.cpu().numpy(), offsets.cpu().numpy())
    Yref = O.linear(xb, codes, s0, z0, prec.cpu().numpy())
    for name, algo in ALGOS.items():
        Y = mbq.mbq_linear(X, blob, N, K, prec, perm, offsets, algo=algo)
        assert_output_close(Y.cpu().numpy(), Yref, f"config 0 {name}")
    # the layer fed with the oracle's routing as well
    perm_ref, off_ref = O.bucket(prec_ref)
    Y = mbq.mbq_linear(X, blob, N, K, dev(prec_ref), dev(perm_ref), dev(off_ref))
    assert_output_close(Y.cpu().numpy(), O.linear(xb, codes, s0, z0, prec_ref), "config 0 oracle routing")


@pytest.mark.parametrize("rows_of", ["one", "every"])
@pytest.mark.parametrize("parts", [1, 2])
def test_prefill_rows_of_small_numbers(mbq, rows_of, parts):
    """Rows of tiny, subnormal and large activations in tiles whose zero-point term is formed in bf16 pieces (parts of more
    than eight groups; three of the four precisions): each row is held to the bar on its own."""
    N, K, T = 130, 128 * 34, 48
    rng = np.random.default_rng([173, parts])
    W = make_weight(N, K, [173, parts], 4.0)
    x = rng.standard_normal((T, K)).astype(np.float32)
    scales = [1.0, 2.0 ** -100, 2.0 ** -110, 2.0 ** -118, 2.0 ** -122, 2.0 ** -126, 2.0 ** -129, 2.0 ** -131, 2.0 ** 90, 2.0 ** 110]
    for t in range(T):
        if rows_of == "every" or t % 4 == 0:
            x[t] *= np.float32(scales[t % 12 if t % 12 < len(scales) else 0])
    x[47, :2048] *= np.float32(2.0 ** -126)   # groups of small numbers beside ordinary ones
    xb = f32_to_bf16_bits(x)
    prec = (np.arange(T) % 3).astype(np.int32) if rows_of == "one" else np.repeat(np.arange(4), 12).astype(np.int32)
    codes, s0, z0 = O.encode(W)
    Yref = O.linear(xb, codes, s0, z0, prec)
    mbq.set_knob(5, parts)
    try:
        Y = run_linear(mbq, W, xb, prec, ALGOS["prefill"])
    finally:
        mbq.set_knob(5, 0)
    bad = []
    for t in range(T):
        err = np.abs(Y[t].astype(np.float64) - Yref[t])
        rms = np.sqrt(np.mean(Yref[t] ** 2))
        print(f"[parity] row {t}: precision {prec[t]}, largest activation 2^{np.log2(np.abs(x[t]).max()):.0f}, "
              f"rel {np.linalg.norm(err) / np.linalg.norm(Yref[t]):.1e}, max {err.max() / rms:.1e}", flush=True)
        if not (np.linalg.norm(err) <= 1e-3 * np.linalg.norm(Yref[t]) and err.max() <= MAX_ABS_TOL * rms):
            bad.append(t)
    assert not bad, bad


ROW_KERNELS = [((11270,), 1536, 48), ((12800, 12810), 3328, 33), ((3072,), 8448, 64), ((3072, 600), 8320, 40), ((300,), 4352, 300)]


@pytest.mark.parametrize("Ns,K,T", ROW_KERNELS)
def test_rows_do_not_meet(mbq, Ns, K, T):
    """Rows of NaN, of an infinity, of the largest numbers and of zeros: every other row has the bits that it has beside
    ordinary ones, zeros give zeros, and tiny and subnormal rows are held to the bar on their own.  Row 0 is among the former:
    kernels read it in the place of rows past the last."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(179 + T + K)
    X = torch.randn((T, K), generator=gen, device="cuda")
    small = {3: 2.0 ** -110, 7: 2.0 ** -126, 12: 2.0 ** -131, 20: 2.0 ** 90}
    for t, scale in small.items():
        X[t] *= scale
    X[9] = 0.0
    X = X.to(torch.bfloat16)
    blobs = [mbq.mbq_encode(0.02 * torch.randn((N, K), generator=gen, device="cuda")) for N in Ns]
    routing = []
    for i in range(len(Ns)):
        prec = np.random.default_rng([179, T, i]).integers(0, 4, size=T).astype(np.int32)
        routing.append((dev(prec), *[dev(v) for v in O.bucket(prec)]))
    Ys = mbq.mbq_linear_group(X, blobs, list(Ns), K, routing)
    odd = X.clone()
    odd[0] = float("nan")
    odd[5, K // 2] = float("inf")
    odd[11] = 3.3e38
    odd[T - 1] = -float("inf")
    others = torch.tensor([t for t in range(T) if t not in (0, 5, 11, T - 1)], device="cuda")
    for i, (a, b) in enumerate(zip(Ys, mbq.mbq_linear_group(odd, blobs, list(Ns), K, routing))):
        assert torch.equal(a[others], b[others]), i
        assert bool(a.isfinite().all()) and not bool(a[9].any()) and bool(b[0].isnan().all()), i
        ref = reference64(X, blobs[i], Ns[i], K, routing[i][0])
        for t in (0, *small):
            err = (a[t].double() - ref[t]).norm() / ref[t].norm()
            assert float(err) < 4e-5, (i, t, float(err))


@pytest.mark.parametrize("Ns,K,T", ROW_KERNELS)
def test_stages_of_these_kernels_replay_from_a_hip_graph(mbq, Ns, K, T):
    """A captured stage, replayed with new activations and eager work in between, gives the eager call's bits every time."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(181 + T + K)
    Wr = [torch.randn((4, K), generator=gen, device="cuda") / K ** 0.5 for _ in Ns]
    br = [torch.zeros(4, device="cuda") for _ in Ns]
    blobs = [mbq.mbq_encode(0.02 * torch.randn((N, K), generator=gen, device="cuda")) for N in Ns]
    X = torch.randn((T, K), generator=gen, device="cuda").to(torch.bfloat16)
    kept = dict(routing=[(torch.empty(T, dtype=torch.int32, device="cuda"), torch.empty(T, dtype=torch.int32, device="cuda"),
                          torch.empty(5, dtype=torch.int32, device="cuda")) for _ in Ns],
                Y=[torch.empty((T, N), device="cuda") for N in Ns],
                ws_route=mbq.route_workspace(T, K, "cuda"), ws_linear=mbq.linear_workspace(T, max(Ns), K, "cuda"))

    def call():
        mbq.mbq_routed_linear_group(X, Wr, br, blobs, list(Ns), **kept)

    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for rep in range(4):
        X.copy_(torch.randn((T, K), generator=gen, device="cuda").to(torch.bfloat16))
        call()
        want = [[t.clone() for t in r] for r in kept["routing"]], [y.clone() for y in kept["Y"]]
        torch.cuda.synchronize()
        kept["ws_linear"].fill_(255)
        for y in kept["Y"]:
            y.fill_(float("nan"))
        for r in kept["routing"]:
            for t in r:
                t.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        for i in range(len(Ns)):
            assert all(torch.equal(a, b) for a, b in zip(want[0][i], kept["routing"][i])), (rep, i)
            assert torch.equal(want[1][i], kept["Y"][i]), (rep, i)
