"""GPU parity of the weight-only setting (W4A16, the paper's appendix on weight-only
quantization): sq_rotate_fp16 and sq_w4a16_gemm through the C ABI against the CPU oracle.

Bars.  Rotated rows: the fp32 result is within 1e-5 of the row maximum (the bar of the W4A4 path)
and is then rounded once to fp16, so |gpu - oracle| <= 1e-5 max_k|row| + one fp16 spacing at the
oracle's value.  GEMM: products of fp16 values and codes are exact, the sums run in fp32 in the
matrix cores' own order, the step and the final rounding follow, so the value the library rounds
is within slack = (K + 2) 2^-24 sw sum_k|x q| of the exact one.  The oracle's Y is that exact
value rounded to fp16, the library's is the perturbed value rounded to fp16: two roundings of two
reals that far apart land on the same fp16 number, or -- when the exact value lies within slack
of a rounding boundary -- on neighbours.  Hence |gpu - oracle| <= one fp16 spacing at the
oracle's value + slack, and, since a flip needs the exact value within slack of a boundary, the
number of entries that differ at all is bounded by the sum of 2 slack / spacing (a kernel that
truncated, or rounded twice, would differ on half of them).  Whole layer: per token row
||dY|| / ||Y|| <= 1e-2."""
import numpy as np
import pytest

from paper_2511_22316_amd import synth
from parity_util import Y_ROW_TOL, dev, host

pytestmark = pytest.mark.gpu


def run_rotate_fp16(L, X=None, ldo=None):
    import torch
    import paper_2511_22316_amd as sq
    X = L.X if X is None else X
    T, K = X.shape
    out = torch.full((T, ldo or K), 7.0, dtype=torch.float16, device="cuda")
    sq.sq_rotate_fp16(dev(X), L.giv_i, L.giv_j, L.giv_theta, dev(L.R1), dev(L.R2), out[:, :K])
    torch.cuda.synchronize()
    return host(out)


def check_rotated_f16(got, want, xr):
    """got, want fp16 [T, K]; xr the oracle's fp64 rotated rows."""
    g, o = got.astype(np.float64), want.astype(np.float64)
    assert np.all(np.isfinite(g) == np.isfinite(o))
    fin = np.isfinite(o)
    spacing = np.maximum(np.abs(np.nextafter(want, np.float16(np.inf)).astype(np.float64) - o),
                         np.abs(o - np.nextafter(want, np.float16(-np.inf)).astype(np.float64)))
    bound = 1e-5 * np.max(np.abs(xr), axis=1, keepdims=True) + np.where(fin, spacing, 0.0)
    excess = np.where(fin, np.abs(g - o) - bound, 0.0)
    assert excess.max() <= 0, f"rotated fp16 rows: worst excess {excess.max():.3e}"
    return float(np.mean(got == want))


@pytest.mark.parametrize("name,T", [("tiny", 16), ("attn_proj", 70), ("mlp_down", 37), ("decode", 8),
                                    ("large_prefill", 33)])
def test_rotate_fp16_matches_oracle(oracle, name, T):
    print(f"case rotate_fp16 {name} T={T}", flush=True)
    L = synth.layer(synth.CONFIGS[name], T)
    got = run_rotate_fp16(L)
    xr = oracle.rotate(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    want = oracle.rotate_f16(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    same = check_rotated_f16(got, want, xr)
    print(f"  {same:.4f} of the entries are the oracle's fp16 value exactly", flush=True)
    assert same > 0.8


def test_rotate_fp16_other_shapes_and_edges(oracle):
    print("case rotate_fp16 plain-kernel shape, strided output, no tokens", flush=True)
    import torch
    import paper_2511_22316_amd as sq
    # a shape only the plain-FMA kernel takes
    cfg = synth.LayerConfig("w16_12x8", 9, 12, 8, 16, 3, "normal", 1, 50.0, 0.02, 20.0, 0.02, 77)
    L = synth.layer(cfg)
    xr = oracle.rotate(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    check_rotated_f16(run_rotate_fp16(L), oracle.rotate_f16(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2), xr)
    # strided output: the padding is not written
    L = synth.layer(synth.CONFIGS["tiny"])
    out = run_rotate_fp16(L, ldo=L.X.shape[1] + 40)
    assert np.all(out[:, L.X.shape[1]:] == 7.0)
    xr = oracle.rotate(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    check_rotated_f16(out[:, : L.X.shape[1]], oracle.rotate_f16(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2), xr)
    # identity rotation, no list: the input comes back bit for bit
    n1, n2 = 16, 32
    Li = synth.Layer(L.cfg, L.X, L.giv_i[:0], L.giv_j[:0], L.giv_theta[:0], np.eye(n1, dtype=np.float16),
                     np.eye(n2, dtype=np.float16), None, None)
    assert np.array_equal(run_rotate_fp16(Li), L.X)
    # no tokens
    e = torch.empty((0, 512), dtype=torch.float16, device="cuda")
    sq.sq_rotate_fp16(e, L.giv_i, L.giv_j, L.giv_theta, dev(L.R1), dev(L.R2), torch.empty_like(e))


def run_w4a16(X, Qw, sw, ldy=None):
    import torch
    import paper_2511_22316_amd as sq
    T, N = X.shape[0], Qw.shape[0]
    Y = torch.full((T, ldy or N), -9.0, dtype=torch.float16, device="cuda")
    sq.sq_w4a16_gemm(dev(X), dev(Qw), dev(sw), Y[:, :N])
    torch.cuda.synchronize()
    return host(Y)


def check_w4a16(Yg, Yo, m, K):
    g, o = Yg.astype(np.float64), Yo.astype(np.float64)
    assert np.all(np.isfinite(g))
    spacing = np.maximum(np.abs(np.nextafter(Yo, np.float16(np.inf)).astype(np.float64) - o),
                         np.abs(o - np.nextafter(Yo, np.float16(-np.inf)).astype(np.float64)))
    slack = (K + 2) * 2.0 ** -24 * m
    excess = np.abs(g - o) - (spacing + slack)
    assert excess.max() <= 0, f"w4a16 Y: worst excess {excess.max():.3e}"
    flips, expected = int(np.count_nonzero(g != o)), float(np.sum(2.0 * slack / spacing))
    assert flips <= expected + 3, f"w4a16 Y: {flips} entries differ from the oracle's, at most {expected:.1f} expected"


@pytest.mark.parametrize("T,K,N", [(1, 64, 1), (16, 512, 512), (77, 128, 300), (130, 320, 257), (300, 2048, 130),
                                   (256, 4096, 384), (129, 64, 129),
                                   # at most 32 tokens and K % 256 == 0: the decode-shaped kernel, both launch
                                   # shapes, one and two token blocks, ragged channel tails, one slice only;
                                   # K % 256 != 0: the tile kernel on few tokens
                                   (8, 1024, 24700), (32, 768, 10300), (20, 256, 50), (16, 8192, 300), (17, 2048, 33),
                                   (1, 4096, 4096), (16, 320, 100),
                                   # just past the decode-shaped kernel's 32 tokens; fewer channels than a fragment
                                   (33, 64, 5), (33, 256, 31)])
def test_w4a16_gemm_random_operands(oracle, T, K, N):
    print(f"case w4a16 gemm random T={T} K={K} N={N}", flush=True)
    g = np.random.default_rng(T + 3 * K + 5 * N)
    X = (g.standard_normal((T, K)) * g.choice([0.1, 1.0, 30.0], size=(T, 1))).astype(np.float16)
    Qw = synth.random_codes(N, K, 300 + N)           # all 16 codes, -8 included
    sw = g.uniform(1e-4, 5e-3, N).astype(np.float32)
    Yo, m = oracle.gemm_w4a16(X, Qw, sw, want_abs_sum=True)
    Yg = run_w4a16(X, Qw, sw)
    check_w4a16(Yg, Yo, m, K)
    # exactly representable case: small integers, step 1/4 -> no rounding anywhere, equal bits
    Xi = g.integers(-3, 4, size=(T, K)).astype(np.float16)
    s4 = np.full(N, 0.25, np.float32)
    Yi = oracle.gemm_w4a16(Xi, Qw, s4)
    if np.max(np.abs(Yi.astype(np.float64))) < 2048:
        assert np.array_equal(run_w4a16(Xi, Qw, s4), Yi)


@pytest.mark.parametrize("T,K,N", [(3, 1024, 16400), (16, 2048, 16384), (2, 3072, 16390), (9, 4096, 20000), (8, 8192, 16400),
                                   (1, 6144, 33000), (4, 16384, 16390), (2, 24576, 16400)])
def test_w4a16_gemm_walks_that_begin_anywhere(oracle, T, K, N):
    """Few tokens and many channels, rounds of four or eight slices (one round, several, several blocks of channels a wave):
    where K is a multiple of 8192 neighbouring workgroups begin their walk over K in different ones.  One-hot rows in every round and small integers: sums
    without rounding, equal bits."""
    print(f"case w4a16 gemm turned walks T={T} K={K} N={N}", flush=True)
    g = np.random.default_rng(T + K + N)
    Qw, s4 = synth.random_codes(N, K, 71), np.full(N, 0.25, np.float32)
    X = np.zeros((T, K), np.float16)
    X[np.arange(T), g.permutation(K)[:T]] = 1.0
    X[0] = g.integers(-3, 4, K)
    Y = oracle.gemm_w4a16(X, Qw, s4)
    assert np.max(np.abs(Y.astype(np.float64))) < 2048
    assert np.array_equal(run_w4a16(X, Qw, s4), Y)


@pytest.mark.parametrize("shape", [1, 2])
@pytest.mark.parametrize("T,K,N", [(16, 512, 512), (130, 320, 257), (300, 2048, 130), (257, 128, 520), (1, 64, 1)])
def test_w4a16_gemm_every_tile_kernel(oracle, shape, T, K, N):
    """The kernel for many tokens with 128 x 256 and with 256 x 256 tiles, each forced onto shapes
    with few tokens, ragged token and channel tails, strided output."""
    print(f"case w4a16 gemm launch shape {shape} T={T} K={K} N={N}", flush=True)
    import paper_2511_22316_amd as sq
    g = np.random.default_rng(shape + T + 3 * K + 5 * N)
    X = (g.standard_normal((T, K)) * g.choice([0.1, 1.0, 30.0], size=(T, 1))).astype(np.float16)
    Qw = synth.random_codes(N, K, 400 + N)
    sw = g.uniform(1e-4, 5e-3, N).astype(np.float32)
    Yo, m = oracle.gemm_w4a16(X, Qw, sw, want_abs_sum=True)
    Xi = g.integers(-3, 4, size=(T, K)).astype(np.float16)
    s4 = np.full(N, 0.25, np.float32)
    Yi = oracle.gemm_w4a16(Xi, Qw, s4)
    sq.sq_debug_set_option(sq.binding.SQ_DEBUG_W4A16_LAUNCH_SHAPE, shape)
    try:
        got = run_w4a16(X, Qw, sw, ldy=N + 3)          # odd leading dimension: no 16-byte stores
        got8 = run_w4a16(X, Qw, sw, ldy=N + 8 - N % 8 if N % 8 else N)
        goti = run_w4a16(Xi, Qw, s4)
    finally:
        sq.sq_debug_set_option(sq.binding.SQ_DEBUG_W4A16_LAUNCH_SHAPE, 0)
    check_w4a16(got[:, :N], Yo, m, K)
    assert np.all(got[:, N:] == -9.0)
    check_w4a16(got8[:, :N], Yo, m, K)
    assert np.all(got8[:, N:] == -9.0)
    if np.max(np.abs(Yi.astype(np.float64))) < 2048:
        assert np.array_equal(goti, Yi)


# one K tile per group, an odd number, more than the ring holds; ragged tails of both small tiles
@pytest.mark.parametrize("T,K,N", [(1, 128, 1), (33, 384, 130), (65, 256, 129), (129, 640, 257), (200, 1152, 1000)])
@pytest.mark.parametrize("shape", [3, 4])
def test_w4a16_gemm_two_k_groups(oracle, shape, T, K, N):
    test_w4a16_gemm_every_tile_kernel(oracle, shape, T, K, N)


def test_w4a16_gemm_seeded_random_shapes(oracle):
    """Twenty shapes drawn from a seed (T up to 400, K a multiple of 64 up to 1536, N up to 1500,
    a third of them with at most 32 tokens), whatever kernel the dispatcher picks."""
    g = np.random.default_rng(1122)
    for case in range(20):
        T = int(g.integers(1, 33)) if case % 3 == 0 else int(g.integers(33, 400))
        K = 64 * int(g.integers(1, 25))
        N = int(g.integers(1, 1500))
        print(f"case w4a16 seeded shape {case}: T={T} K={K} N={N}", flush=True)
        X = (g.standard_normal((T, K)) * g.choice([0.1, 1.0, 30.0], size=(T, 1))).astype(np.float16)
        Qw = synth.random_codes(N, K, 900 + case)
        sw = g.uniform(1e-4, 5e-3, N).astype(np.float32)
        Yo, m = oracle.gemm_w4a16(X, Qw, sw, want_abs_sum=True)
        check_w4a16(run_w4a16(X, Qw, sw), Yo, m, K)


def test_w4a16_gemm_strided_and_empty(oracle):
    print("case w4a16 gemm strided output / input, empty", flush=True)
    import torch
    import paper_2511_22316_amd as sq
    g = np.random.default_rng(4)
    T, K, N = 40, 192, 72
    X = g.standard_normal((T, K)).astype(np.float16)
    Qw, sw = synth.random_codes(N, K, 2), np.full(N, 0.01, np.float32)
    Yo, m = oracle.gemm_w4a16(X, Qw, sw, want_abs_sum=True)
    got = run_w4a16(X, Qw, sw, ldy=N + 10)
    check_w4a16(got[:, :N], Yo, m, K)
    assert np.all(got[:, N:] == -9.0)
    wide = torch.zeros((T, K + 64), dtype=torch.float16, device="cuda")
    wide[:, :K] = dev(X)
    Y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    sq.sq_w4a16_gemm(wide[:, :K], dev(Qw), dev(sw), Y)
    torch.cuda.synchronize()
    check_w4a16(host(Y), Yo, m, K)
    sq.sq_w4a16_gemm(wide[:0, :K], dev(Qw), dev(sw), Y[:0])
    # the decode-shaped kernel on a strided input and output
    T, K, N = 9, 512, 40
    X = g.standard_normal((T, K)).astype(np.float16)
    Qw, sw = synth.random_codes(N, K, 3), np.full(N, 0.01, np.float32)
    Yo, m = oracle.gemm_w4a16(X, Qw, sw, want_abs_sum=True)
    wide = torch.full((T, K + 24), 1000.0, dtype=torch.float16, device="cuda")
    wide[:, :K] = dev(X)
    Y = torch.full((T, N + 5), -9.0, dtype=torch.float16, device="cuda")
    sq.sq_w4a16_gemm(wide[:, :K], dev(Qw), dev(sw), Y[:, :N])
    torch.cuda.synchronize()
    check_w4a16(host(Y)[:, :N], Yo, m, K)
    assert np.all(host(Y)[:, N:] == -9.0)


@pytest.mark.parametrize("name,T,N", [("tiny", 16, 512), ("attn_proj", 96, 300), ("mlp_down", 40, 130)])
def test_weight_only_layer_end_to_end(oracle, name, T, N):
    """GPU pipeline (rotation to fp16, offline weight path, W4A16 GEMM: its own values on both
    operands) against the oracle pipeline."""
    print(f"case weight-only layer {name} T={T} N={N}", flush=True)
    import torch
    import paper_2511_22316_amd as sq
    cfg = synth.CONFIGS[name]
    L = synth.layer(cfg, T)
    Wt = synth.weights_t(cfg, N)
    xo = oracle.rotate_f16(L.X, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    Qwo, swo = oracle.prepare_weights(Wt, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    Yo = oracle.gemm_w4a16(xo, Qwo, swo).astype(np.float64)
    dR1, dR2 = dev(L.R1), dev(L.R2)
    Qw = torch.empty((N, cfg.K // 2), dtype=torch.uint8, device="cuda")
    sw = torch.empty((N,), dtype=torch.float32, device="cuda")
    sq.sq_rotate_quantize(dev(Wt), L.giv_i, L.giv_j, L.giv_theta, dR1, dR2, Qw, sw)
    Xr = torch.empty((T, cfg.K), dtype=torch.float16, device="cuda")
    sq.sq_rotate_fp16(dev(L.X), L.giv_i, L.giv_j, L.giv_theta, dR1, dR2, Xr)
    Y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    sq.sq_w4a16_gemm(Xr, Qw, sw, Y)
    torch.cuda.synchronize()
    d = host(Y).astype(np.float64) - Yo
    rel = np.linalg.norm(d, axis=1) / np.linalg.norm(Yo, axis=1)
    print(f"  worst row error {rel.max():.3e}", flush=True)
    assert rel.max() <= Y_ROW_TOL
    # and the point of the variant: with 16-bit activations the layer is closer to X W than W4A4
    ref = L.X.astype(np.float64) @ Wt.astype(np.float64).T
    e16 = np.linalg.norm(host(Y).astype(np.float64) - ref) / np.linalg.norm(ref)
    Qx = torch.empty((T, cfg.K // 2), dtype=torch.uint8, device="cuda")
    sx = torch.empty((T,), dtype=torch.float32, device="cuda")
    sq.sq_rotate_quantize(dev(L.X), L.giv_i, L.giv_j, L.giv_theta, dR1, dR2, Qx, sx)
    Y4 = torch.empty((T, N), dtype=torch.float16, device="cuda")
    sq.sq_w4a4_gemm(Qx, sx, Qw, sw, Y4)
    torch.cuda.synchronize()
    e4 = np.linalg.norm(host(Y4).astype(np.float64) - ref) / np.linalg.norm(ref)
    print(f"  error against X W: W4A16 {e16:.3f}, W4A4 {e4:.3f}", flush=True)
    assert e16 < e4


def test_weight_only_full_size_attn_proj_sampled_rows(oracle):
    """Full attn_proj layer in the configuration the benchmark times; sampled token rows x all N
    against the oracle pipeline."""
    print("case weight-only attn_proj full size", flush=True)
    import torch
    import paper_2511_22316_amd as sq
    cfg = synth.CONFIGS["attn_proj"]
    L = synth.layer(cfg)
    T, K, N = cfg.T, cfg.K, cfg.N
    Wt = synth.weights_t(cfg)
    dR1, dR2 = dev(L.R1), dev(L.R2)
    Qw = torch.empty((N, K // 2), dtype=torch.uint8, device="cuda")
    sw = torch.empty((N,), dtype=torch.float32, device="cuda")
    sq.sq_rotate_quantize(dev(Wt), L.giv_i, L.giv_j, L.giv_theta, dR1, dR2, Qw, sw)
    Xr = torch.empty((T, K), dtype=torch.float16, device="cuda")
    sq.sq_rotate_fp16(dev(L.X), L.giv_i, L.giv_j, L.giv_theta, dR1, dR2, Xr)
    Y = torch.empty((T, N), dtype=torch.float16, device="cuda")
    sq.sq_w4a16_gemm(Xr, Qw, sw, Y)
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([[0, T - 1], np.random.default_rng(23).integers(0, T, 48)]))
    xr = oracle.rotate(L.X[rows], L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    xo = oracle.rotate_f16(L.X[rows], L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    check_rotated_f16(host(Xr)[rows], xo, xr)
    Qwo, swo = oracle.prepare_weights(Wt, L.giv_i, L.giv_j, L.giv_theta, L.R1, L.R2)
    Yo = oracle.gemm_w4a16(xo, Qwo, swo).astype(np.float64)
    d = host(Y)[rows].astype(np.float64) - Yo
    rel = np.linalg.norm(d, axis=1) / np.linalg.norm(Yo, axis=1)
    print(f"  worst row error {rel.max():.3e} over {len(rows)} rows", flush=True)
    assert rel.max() <= Y_ROW_TOL
    # the GEMM alone on the GPU's own operands: element-wise bound
    Yo2, m = oracle.gemm_w4a16(host(Xr)[rows], host(Qw), host(sw), want_abs_sum=True)
    check_w4a16(host(Y)[rows], Yo2, m, K)
