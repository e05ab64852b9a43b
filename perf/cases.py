"""The measured cases of this library: the work that a program which serves or prepares SingleQuant
layers has it do, through the public entry points of ``paper_2511_22316_amd``.

A case is one pass through one linear layer's path, named by ``path``:

  w4a4        rotation + quantizer, then the W4A4 GEMM on the canonical weight codes (prefill)
  w4a4_decode the same for at most 32 tokens, weights kept in the decode layout
  single      both steps in one launch (``sq_decode_layer``)
  w4a16       weight-only setting: rotation to fp16, then the W4A16 GEMM
  w3a16       the same on three-bit weight storage
  weights     offline: rotation and quantization of a weight matrix
  rotation    offline: the closed-form rotation from calibration activations

T tokens (calibration rows for ``rotation``), K = n1 * n2 channels, N output channels, P Givens
pairs.  Activations follow the benchmark's recipe: a Gaussian or Student-t body, a few channels of
massive outliers on every token, a share of moderate outliers.  Weight codes are what
round-to-nearest makes of Gaussian weights (a rotated Gaussian matrix is Gaussian again).
"""
import math

import numpy as np
import torch

import paper_2511_22316_amd as sq
from paper_2511_22316_amd import synth


def _case(name, path, T, n1, n2, N, P, body="normal", massive=4, scale=1000.0, frac=0.01, bits=4, clip=1.0):
    return {"name": name, "path": path, "T": T, "n1": n1, "n2": n2, "N": N, "P": P, "body": body, "massive": massive,
            "scale": scale, "frac": frac, "bits": bits, "clip": clip}


def listed():
    return [
        # the smallest layer of the benchmark: launches and the host path are all there is
        _case("tiny_layer", "w4a4_decode", 16, 16, 32, 512, 8, massive=2, scale=500.0),
        # one token through an attention projection with one call per layer, the way a loop bound by its host does it
        _case("one_token_single_launch", "single", 1, 64, 64, 4096, 32),
        # decoding a small batch through an up projection: one pass over the weights
        _case("decode", "w4a4_decode", 8, 64, 128, 28672, 32, frac=0.0),
        # a short prompt of odd length, a 5120-wide layer
        _case("short_prompt", "w4a4", 333, 80, 64, 13824, 24),
        # a 3072-wide layer, factors from sq_kron_factor, a batch of odd length
        _case("narrow_batch", "w4a4", 1001, 48, 64, 9216, 16),
        # prefill of an attention projection, the benchmark's headline layer
        _case("attn_proj", "w4a4", 2048, 64, 64, 4096, 32),
        # prefill of a down projection, heavy-tailed activations
        _case("mlp_down", "w4a4", 2048, 86, 128, 4096, 16, body="student_t3", massive=2, scale=2000.0, frac=0.0),
        # a large prefill batch through an up projection: the largest case
        _case("large_prefill", "w4a4", 8192, 64, 128, 28672, 64, massive=8, frac=0.005),
        # weight-only setting, prefill and decode
        _case("weight_only_prefill", "w4a16", 2048, 64, 64, 4096, 32),
        _case("weight_only_decode", "w4a16", 8, 64, 128, 28672, 32, frac=0.0),
        # offline: the weights of a down projection, and the rotation of an attention projection
        _case("offline_weights", "weights", 0, 86, 128, 4096, 16),
        _case("offline_rotation", "rotation", 2048, 64, 64, 0, 32),
    ]


# the factor pairs of the benchmark's layers and of the other layer widths that the tests cover
_PAIRS = [(16, 32), (32, 32), (32, 64), (64, 64), (80, 64), (64, 128), (86, 128), (128, 64), (108, 128), (112, 128)]
_SINGLE = [(16, 32), (32, 32), (32, 64), (64, 64), (64, 128)]      # what sq_decode_layer covers
_LARGEST = 8192 * 8192 * 28672


def _log_int(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    path = rng.choice(["w4a4", "w4a4", "w4a4", "w4a4_decode", "w4a4_decode", "single", "w4a16", "w4a16", "w3a16",
                       "weights", "rotation"])
    # half of the layer widths from the list, half any multiple of 128 (256 where the path asks for it),
    # split by the paper's Alg. 1
    small = 256 if path in ("w4a4_decode", "w3a16") else 128
    if path == "single":
        n1, n2 = rng.choice(_SINGLE)
    elif path == "rotation" or rng.random() < 0.5:
        n1, n2 = rng.choice(_PAIRS)
        while (n1 * n2) % small:
            n1, n2 = rng.choice(_PAIRS)
    else:
        n1, n2 = sq.sq_kron_factor(small * _log_int(rng, 512 // small, 14336 // small))
        while n1 > 128:
            n1, n2 = sq.sq_kron_factor(small * _log_int(rng, 512 // small, 14336 // small))
    K = n1 * n2
    N = _log_int(rng, 256, 28672)
    if rng.random() < 0.75:
        N = (N + 63) // 64 * 64
    most = {"w4a4": 8192, "w4a4_decode": 32, "single": 32, "w4a16": 2048, "w3a16": 32, "weights": 1, "rotation": 8192}
    T = _log_int(rng, {"w4a4": 33, "rotation": 64}.get(path, 1), most[path])
    if path in ("w4a4", "w4a16"):        # no more than half of the largest listed case's products
        T = max(1, min(T, _LARGEST // 2 // (K * N)))
    P = rng.choice([0, 8, 16, 24, 32, 48, 64])
    case = _case("", path, T, n1, n2, N, P, body=rng.choice(["normal", "student_t3"]), massive=rng.randint(1, 8),
                 scale=rng.choice([500.0, 1000.0, 2000.0]), frac=rng.choice([0.0, 0.005, 0.01]))
    if path in ("w4a4", "weights") and rng.random() < 0.25:
        case["bits"], case["clip"] = rng.choice([(3, 1.0), (4, 0.9), (4, 0.8), (3, 0.85)])
    if path == "w3a16":
        case["bits"] = 3
    if path == "weights":
        case["T"] = 0
    if path == "rotation":
        case["N"] = 0
        case["P"] = max(8, P)
    del case["name"]
    return case


def _activations(c, rows, gen):
    """fp16 [rows, K] on the GPU, by the benchmark's recipe."""
    K = c["n1"] * c["n2"]
    x = torch.randn(rows, K, device="cuda", generator=gen)
    if c["body"] == "student_t3":
        g = torch.zeros(rows, K, device="cuda")
        for _ in range(3):
            g += torch.randn(rows, K, device="cuda", generator=gen).square_()
        x /= (g / 3.0).sqrt_()
    channels = torch.randperm(K, device="cuda", generator=gen)[: c["massive"]]
    if c["frac"] > 0.0:
        hit = torch.rand(rows, K, device="cuda", generator=gen) < c["frac"]
        hit[:, channels] = False
        x = torch.where(hit, 20.0 * x, x)
    x[:, channels] *= c["scale"]
    return x.clamp_(-65504.0, 65504.0).half()


def _weight_codes(N, K, bits, gen):
    """Codes uint8 [N, K/2] and steps fp32 [N] of Gaussian weights, rounded to nearest per output channel."""
    top = float(2 ** (bits - 1) - 1)
    Q = torch.empty(N, K // 2, dtype=torch.uint8, device="cuda")
    sw = torch.empty(N, device="cuda")
    for a in range(0, N, 4096):
        w = 0.02 * torch.randn(min(4096, N - a), K, device="cuda", generator=gen)
        step = w.abs().amax(1) / top
        q = torch.floor(w / step[:, None] + 0.5).clamp_(-top - 1, top).to(torch.int32) & 15
        Q[a:a + 4096] = (q[:, 0::2] | (q[:, 1::2] << 4)).to(torch.uint8)
        sw[a:a + 4096] = step
    return Q, sw


def _factors(c, seed):
    rng = np.random.default_rng([seed, c["n1"], c["n2"]])
    return [torch.from_numpy(synth.random_orthogonal(n, rng).astype(np.float16)).cuda() for n in (c["n1"], c["n2"])]


def _givens(c, row):
    """The ART list on one calibration row (host arrays, as the online entry points take them)."""
    cfg = synth.LayerConfig("case", 1, c["n1"], c["n2"], 1, c["P"], c["body"], c["massive"], c["scale"], c["frac"], 20.0,
                            0.02, 0)
    return synth.art_pairs(cfg, row.float().cpu().numpy()[None])


def prepare(case, seed):
    c = dict(case)
    path, T, n1, n2, N, P, bits = (c[k] for k in ("path", "T", "n1", "n2", "N", "P", "bits"))
    K = n1 * n2
    gen = torch.Generator(device="cuda").manual_seed(seed)
    empty = lambda shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")   # noqa: E731
    if path == "rotation":
        c["X"] = _activations(c, T, gen)
        c["giv"] = (empty(P, torch.int32), empty(P, torch.int32), empty(P, torch.float32))
        c["R1"], c["R2"] = empty((n1, n1), torch.float16), empty((n2, n2), torch.float16)
        c["workspace"] = empty(sq.sq_build_rotation_workspace_bytes(T, n1, n2), torch.uint8)
        return c
    c["R1"], c["R2"] = _factors(c, seed)
    if path == "weights":
        c["giv"] = _givens(c, _activations(c, 1, gen)[0])
        c["W"] = (0.02 * torch.randn(K, N, device="cuda", generator=gen)).half()
        c["workspace"] = empty((N, K), torch.float16)
        c["Qw"], c["sw"] = empty((N, K // 2), torch.uint8), empty(N, torch.float32)
        return c
    c["X"] = _activations(c, T, gen)
    c["giv"] = _givens(c, c["X"][0])
    c["Qw"], c["sw"] = _weight_codes(N, K, bits if path == "w3a16" else 4, gen)
    c["Y"] = empty((T, N), torch.float16)
    if path in ("w4a16", "w3a16"):
        c["Xrot"] = empty((T, K), torch.float16)
        if path == "w3a16":
            Qw3 = empty((N, 3 * K // 8), torch.uint8)
            sq.sq_pack_w3(c["Qw"], Qw3)
            c["Qw"] = Qw3
        return c
    c["prepared"] = empty(sq.sq_prepared_rotation_bytes(n1, n2), torch.uint8)
    sq.sq_prepare_rotation(c["R1"], c["R2"], c["prepared"])
    if path == "single":
        c["workspace"] = torch.zeros(sq.sq_decode_layer_workspace_bytes(T, K), dtype=torch.uint8, device="cuda")
        return c
    c["Q"], c["s"] = empty((T, K // 2), torch.uint8), empty(T, torch.float32)
    if path == "w4a4_decode":
        tiled = empty(sq.sq_decode_weights_bytes(K, N), torch.uint8)
        sq.sq_tile_weights_decode(c["Qw"], tiled)
        c["Qw"] = tiled
    return c


def run(c):
    path = c["path"]
    if path == "rotation":
        sq.sq_build_rotation(c["X"], c["n1"], c["n2"], *c["giv"], c["R1"], c["R2"], c["workspace"])
        return {"i": c["giv"][0], "j": c["giv"][1], "theta": c["giv"][2], "R1": c["R1"], "R2": c["R2"]}
    plain = c["bits"] == 4 and c["clip"] == 1.0
    if path == "weights":
        if plain:
            sq.sq_prepare_weights(c["W"], *c["giv"], c["R1"], c["R2"], c["workspace"], c["Qw"], c["sw"])
        else:
            sq.sq_prepare_weights_variant(c["W"], *c["giv"], c["R1"], c["R2"], c["bits"], c["clip"], c["workspace"],
                                          c["Qw"], c["sw"])
        return {"Qw": c["Qw"], "sw": c["sw"]}
    if path == "single":
        sq.sq_decode_layer(c["X"], *c["giv"], c["prepared"], c["n1"], c["n2"], c["Qw"], c["sw"], c["Y"], c["workspace"])
        return {"Y": c["Y"]}
    if path in ("w4a16", "w3a16"):
        sq.sq_rotate_fp16(c["X"], *c["giv"], c["R1"], c["R2"], c["Xrot"])
        gemm = sq.sq_w4a16_gemm if path == "w4a16" else sq.sq_w3a16_gemm
        gemm(c["Xrot"], c["Qw"], c["sw"], c["Y"])
        return {"Xrot": c["Xrot"], "Y": c["Y"]}
    if plain:
        sq.sq_rotate_quantize_prepared(c["X"], *c["giv"], c["prepared"], c["n1"], c["n2"], c["Q"], c["s"])
    else:
        sq.sq_rotate_quantize_variant(c["X"], *c["giv"], c["R1"], c["R2"], c["bits"], c["clip"], c["Q"], c["s"])
    gemm = sq.sq_w4a4_gemm_decode if path == "w4a4_decode" else sq.sq_w4a4_gemm
    gemm(c["Q"], c["s"], c["Qw"], c["sw"], c["Y"])
    return {"Q": c["Q"], "s": c["s"], "Y": c["Y"]}


def work(case):
    path, T, n1, n2, N = (case[k] for k in ("path", "T", "n1", "n2", "N"))
    K = n1 * n2
    factors = 2 * (n1 * n1 + n2 * n2)
    if path == "rotation":
        return {"bytes": 2 * T * K + factors, "flops": 2 * (n1 ** 3 + n2 ** 3)}
    if path == "weights":
        return {"bytes": 2.5 * K * N + 4 * N + factors, "flops": 2 * N * K * (n1 + n2)}
    weight_bits = 3 if path == "w3a16" else 4
    between = {"single": 0, "w4a16": 2 * T * K, "w3a16": 2 * T * K}.get(path, T * K // 2 + 4 * T)
    return {"bytes": 2 * T * K + factors + between + K * N * weight_bits // 8 + 4 * N + 2 * T * N,
            "flops": 2 * T * K * (n1 + n2) + 2 * T * K * N}


def tolerance(case):
    """Four times what the paths differ by from the same computation in fp64 (rotation, quantizer and product)."""
    path, T, K = case["path"], case["T"], case["n1"] * case["n2"]
    if path == "rotation":           # fp64 throughout, one rounding to fp16: 2.2e-4 and 4.9e-4; the channels are the same
        return {"rel": 9e-4, "max": 2e-3}
    if path in ("w4a16", "w3a16"):   # one rounding to fp16 on the way and one at the end: 2.1e-4 and 5.8e-4
        return {"rel": 8.5e-4, "max": 2.5e-3}
    # a rotated value next to a rounding boundary takes the neighbouring code: up to 1.6e-6 of the code bytes, or a
    # single one of a small tensor, and with it every product of that row moves by one step
    codes = (case["N"] if path == "weights" else T) * K
    differ = max(7e-6, min(1e-2, 4.0 / codes))
    if path == "weights":            # steps in fp32: 1.3e-7 and 4.1e-7
        return {"rel": 6e-7, "max": 2e-6, "differ": differ}
    return {"rel": max(3e-3, min(3e-2, 1.0 / math.sqrt(codes))), "max": 0.6, "differ": differ}
