"""The work that a user of this library has it do, as cases for timing.

Sizes are those of the repository's own workloads (synth/configs.py: Llama2-7B
and GPT3-22B layers with their kept components L) and of bench.py, with token
counts from one decoded token over batched decode and short prompts to a whole
prefill.  Kinds:

  layer     the projected linear layer, Y = Wf·(Pt·X), bf16 or fp32
  mx        the MX-FP8 layer as it runs in a model: the bf16 activations are
            quantised, then projected and expanded (weights quantised once)
  train     one training step of a layer with a fixed P: fold the weight of
            this step, project, expand, both gradients
  autocorr  calibration: the autocorrelation of two batches of tokens
  gomse     calibration: the fp32 product C_X·C_W + C_W·C_X

The principal components are left out: that call's time is rocSOLVER's
eigensolver.
"""
import math

import torch

import paper_2410_05437_amd as espace

DEV = "cuda"
BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64


def listed():
    return [
        # a small fp32 layer: the repository's tiny workload, latency of the calls
        dict(name="layer_f32_small", kind="layer", dtype="f32", K=256, M=256, L=64, N=128, x="normed"),
        # interactive decoding, one sequence: Llama2-7B FFN up+gate
        dict(name="decode_upgate_n1", kind="layer", dtype="bf16", K=4096, M=22016, L=1536, N=1, x="normed"),
        # decoding a few sequences: Llama2-7B FFN down, odd count, deep projection
        dict(name="decode_down_n13", kind="layer", dtype="bf16", K=11008, M=4096, L=1536, N=13, x="gated"),
        # batched decoding on a server: Llama2-7B QKV
        dict(name="decode_qkv_n48", kind="layer", dtype="bf16", K=4096, M=12288, L=1536, N=48, x="normed"),
        # a short prompt, or one chunk of a chunked prefill: GPT3-22B FFN up, ragged L and N
        dict(name="prompt_up22b_n333", kind="layer", dtype="bf16", K=6144, M=24576, L=2458, N=333, x="normed"),
        # prefill of one full sequence: Llama2-7B QKV (the benchmark's layer)
        dict(name="prefill_qkv_n4096", kind="layer", dtype="bf16", K=4096, M=12288, L=1536, N=4096, x="normed"),
        # the largest layer: GPT3-22B FFN down, ragged L
        dict(name="prefill_down22b_n8192", kind="layer", dtype="bf16", K=24576, M=6144, L=2458, N=8192, x="gated"),
        # low-precision decoding: Llama2-7B FFN up+gate
        dict(name="mx_decode_upgate_n8", kind="mx", dtype="mxfp8", K=4096, M=22016, L=1536, N=8, x="normed"),
        # low-precision prefill: Llama2-7B FFN down
        dict(name="mx_prefill_down_n4096", kind="mx", dtype="mxfp8", K=11008, M=4096, L=1536, N=4096, x="gated"),
        # retraining with a fixed projection: Llama2-7B QKV, one sequence per step
        dict(name="train_qkv_n4096", kind="train", dtype="bf16", K=4096, M=12288, L=1536, N=4096, x="normed"),
        # calibration on normalised tokens: Llama2-7B width, two batches
        dict(name="autocorr_k4096", kind="autocorr", dtype="bf16", K=4096, M=0, L=0, N=16384, x="normed",
             normalize=True),
        # calibration with the weights: Llama2-7B width
        dict(name="gomse_k4096", kind="gomse", dtype="f32", K=4096, M=0, L=0, N=0, x="normed"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _size(rng, lo, hi):
    """A width between lo and hi: a multiple of 128, of 8, or any number."""
    v = _log(rng, lo, hi)
    step = rng.choice([128, 128, 8, 1])
    return min(hi, max(lo, int(round(v / step)) * step))


def draw(rng):
    kind = rng.choice(["layer"] * 6 + ["mx"] * 3 + ["train", "train", "autocorr", "gomse", "f32"])
    x = rng.choice(["normed", "gated"])
    if kind == "gomse":
        return dict(kind="gomse", dtype="f32", K=_size(rng, 256, 4096), M=0, L=0, N=0, x=x)
    if kind == "autocorr":
        dtype = rng.choice(["bf16", "bf16", "f32"])
        K = _size(rng, 512, 4096 if dtype == "bf16" else 2048)
        return dict(kind="autocorr", dtype=dtype, K=K, M=0, L=0,
                    N=int(_log(rng, 512, 16384 if dtype == "bf16" else 8192)), x=x,
                    normalize=rng.random() < 0.5)
    if kind == "f32":
        K, M = _size(rng, 128, 2048), _size(rng, 128, 4096)
        return dict(kind="layer", dtype="f32", K=K, M=M, L=max(8, int(K * rng.uniform(0.1, 0.5))),
                    N=int(_log(rng, 1, 2048)), x=x)
    while True:
        K, M = _size(rng, 1024, 24576), _size(rng, 1024, 24576)
        # what is kept of the dense layer's weights: 20 to 75% (the paper's tables)
        L = int(rng.uniform(0.2, 0.75) * K * M / (K + M))
        if rng.random() < 0.5:
            L = max(64, L // 64 * 64)
        N = int(_log(rng, 64 if kind == "train" else 1, 8192))
        c = dict(kind=kind, dtype="mxfp8" if kind == "mx" else "bf16", K=K, M=M, L=L, N=N, x=x)
        if work(c)["flops"] <= 1.2e12 and work(c)["bytes"] <= 1.2e9:
            return c


# ---- inputs --------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + 17)


def _normal(g, rows, cols):
    return torch.randn((rows, cols), generator=g, device=DEV, dtype=F32)


def _tokens(g, case, N=None):
    """Activations [N][K]: outputs of a norm layer (channels of unequal size, a
    few large ones), or a gated SiLU product."""
    N, K = case["N"] if N is None else N, case["K"]
    x = _normal(g, N, K)
    if case["x"] == "gated":
        return torch.nn.functional.silu(x) * _normal(g, N, K)
    s = torch.exp(0.5 * _normal(g, 1, K))
    s[:, :: 509] *= 8.0
    return x * s


def _weights(g, rows, cols, depth):
    """Entries of a weight, or of the rows of an orthonormal basis, of vectors of
    `depth` entries: N(0, 1/depth).  (P's columns are orthonormal in a model; a
    Haar-random one has these entries, and no step of the path asks for more.)"""
    return _normal(g, rows, cols) * depth ** -0.5


def _mat(t, dtype):
    """The matrix as the library takes it (rows padded to 16 bytes)."""
    out = espace.padded_empty(t.shape[0], t.shape[1], dtype, t.device, 8 if dtype == BF16 else 4)
    out.copy_(t)
    return out


def _inputs(case, seed):
    """The case's tensors, rounded to their type."""
    g = _gen(seed)
    kind, K, M, L, N = (case[k] for k in ("kind", "K", "M", "L", "N"))
    dt = F32 if case["dtype"] == "f32" else BF16
    if kind in ("layer", "mx"):
        # an iid N(0, 1/K) weight folded with orthonormal columns is iid N(0, 1/K)
        return dict(X=_mat(_tokens(g, case), dt), Pt=_mat(_weights(g, L, K, K), dt),
                    Wf=_mat(_weights(g, M, L, K), dt))
    if kind == "train":
        return dict(X=_mat(_tokens(g, case), dt), Pt=_mat(_weights(g, L, K, K), dt),
                    W=_mat(_weights(g, M, K, K), dt), dY=_mat(_normal(g, N, M) * 1e-3, dt))
    if kind == "autocorr":
        return dict(X=[_mat(_tokens(g, case, n), dt) for n in (N - N // 2, N // 2)])
    # two autocorrelations: symmetric, with a falling spectrum
    out = {}
    for name in ("A", "B"):
        t = _normal(g, K, K) * torch.arange(1, K + 1, device=DEV, dtype=F32).rsqrt()
        out[name] = _mat(torch.mm(t.t(), t).div_(K), F32)
    return out


def prepare(case, seed):
    """Inputs, weights and the buffers that a serving program keeps."""
    s = dict(case=case, **_inputs(case, seed))
    kind, K, M, L, N = (case[k] for k in ("kind", "K", "M", "L", "N"))
    if kind == "layer":
        s["ws"] = torch.empty(espace.espace_workspace_bytes(espace.OP_PROJECTED_LINEAR, M, K, L, N, s["X"].dtype),
                              dtype=torch.uint8, device=DEV)
        s["Y"] = espace.padded_empty(N, M, s["X"].dtype, DEV)
    elif kind == "mx":
        s["Pt"] = espace.espace_quantize_mxfp8(s["Pt"])
        s["Wf"] = espace.espace_quantize_mxfp8(s["Wf"])
        s["Xq"] = espace.mx_empty(N, K, DEV)
        s["ws"] = torch.empty(espace.espace_workspace_bytes(espace.OP_PROJECTED_LINEAR_MXFP8, M, K, L, N, BF16),
                              dtype=torch.uint8, device=DEV)
        s["Y"] = espace.padded_empty(N, M, BF16, DEV)
    return s


def run(s):
    kind = s["case"]["kind"]
    if kind == "layer":
        return espace.espace_projected_linear(s["X"], s["Pt"], s["Wf"], Y=s["Y"], workspace=s["ws"])
    if kind == "mx":
        espace.espace_quantize_mxfp8(s["X"], out=s["Xq"])
        return espace.espace_projected_linear_mxfp8(s["Xq"], s["Pt"], s["Wf"], Y=s["Y"], workspace=s["ws"])
    if kind == "train":
        Wf = espace.espace_fold_weights(s["W"], s["Pt"])
        Z = espace.espace_project(s["Pt"], s["X"])
        Y = espace.espace_expand(Z, Wf)
        dX, dW = espace.espace_projected_linear_backward(s["dY"], Z, s["Pt"], Wf)
        return dict(Y=Y, dX=dX, dW=dW)
    if kind == "autocorr":
        K = s["case"]["K"]
        C = espace.padded_empty(K, K, F32, DEV, 4).zero_()
        for X in s["X"]:
            espace.espace_autocorrelation_update(X, C, 1.0 / (len(s["X"]) * X.shape[0]),
                                                 normalize=s["case"]["normalize"])
        return C
    return espace.espace_symmetrized_product(s["A"], s["B"])


# ---- what a pass cannot do without, its tolerance and its exact result ------------


def work(case):
    kind, K, M, L, N = (case[k] for k in ("kind", "K", "M", "L", "N"))
    e = 4 if case["dtype"] == "f32" else 2
    if kind == "layer":
        return dict(flops=2 * L * N * (K + M), bytes=e * (N * K + L * K + M * L + N * M))
    if kind == "mx":   # bf16 activations in and out, weights of 8 bits and a scale byte per 32
        return dict(flops=2 * L * N * (K + M), bytes=2 * N * K + 2 * N * M + (L * K + M * L) * 33 // 32)
    if kind == "train":
        # fold, project, expand; dY·Wf, ·Pt; dYᵀ·Z, ·Pt
        return dict(flops=2 * L * (2 * M * K + 2 * N * K + 3 * N * M),
                    bytes=e * (N * K + L * K + M * K + N * M + N * M + N * K + M * K))
    if kind == "autocorr":
        return dict(flops=K * (K + 1) * N, bytes=e * N * K + 4 * K * K)
    return dict(flops=2 * K * K * K, bytes=4 * 3 * K * K)


def tolerance(case):
    """About four times the difference from `exact` measured on the listed cases
    and drawn ones (largest seen in brackets)."""
    kind = case["kind"]
    if kind == "gomse":
        return dict(rel=1e-5, max=1.6e-4)      # fp32 sums K deep (2.4e-6, 4.0e-5)
    if case["dtype"] == "f32" or (kind == "autocorr" and not case["normalize"]):
        return dict(rel=4e-6, max=1.6e-5)      # fp32 sums (8.5e-7, 3.8e-6); bf16 products are exact in fp32
    if kind == "autocorr":
        return dict(rel=2e-3, max=1e-1)        # unit tokens rounded to bf16 (4.4e-4, 2.4e-2)
    if kind == "mx":
        return dict(rel=9e-3, max=2e-1)        # Z's codes next to a rounding boundary, bf16 Y (2.3e-3, 4.9e-2)
    return dict(rel=1.1e-2, max=5.5e-2)        # Z, folded weight and results rounded to bf16 (2.8e-3, 1.4e-2)


def _mx_round(v):
    """v (float64) rounded to MX-FP8 along its rows: blocks of 32 share the scale
    2^(floor(log2 max) - 8), elements are E4M3."""
    rows, cols = v.shape
    b = torch.nn.functional.pad(v, (0, -cols % 32)).view(rows, -1, 32)
    amax = b.abs().amax(-1, keepdim=True)
    e = torch.where(amax > 0, torch.frexp(amax)[1] - 9, torch.full_like(amax, -127, dtype=torch.int32))
    scale = torch.ldexp(torch.ones_like(amax), e.clamp(-127, 127))
    q = (b / scale).clamp(-448, 448).to(F32).to(torch.float8_e4m3fn).to(F64)
    return (q * scale).reshape(rows, -1)[:, :cols]


def exact(case, seed):
    s = {k: [x.to(F64) for x in t] if isinstance(t, list) else t.to(F64) for k, t in _inputs(case, seed).items()}
    kind = case["kind"]
    if kind == "layer":
        return torch.mm(torch.mm(s["X"], s["Pt"].t()), s["Wf"].t())
    if kind == "mx":
        Z = _mx_round(torch.mm(_mx_round(s["X"]), _mx_round(s["Pt"]).t()))
        return torch.mm(Z, _mx_round(s["Wf"]).t())
    if kind == "train":
        Wf = torch.mm(s["W"], s["Pt"].t())
        Z = torch.mm(s["X"], s["Pt"].t())
        return dict(Y=torch.mm(Z, Wf.t()), dX=torch.mm(torch.mm(s["dY"], Wf), s["Pt"]),
                    dW=torch.mm(torch.mm(s["dY"].t(), Z), s["Pt"]))
    if kind == "autocorr":
        C = 0
        for X in s["X"]:
            n = X.shape[0]
            if case["normalize"]:
                X = X / X.norm(dim=1, keepdim=True)
            C = C + torch.mm(X.t(), X) / (len(s["X"]) * n)
        return C
    P = torch.mm(s["A"], s["B"].t())
    return P + P.t()
