"""The work this library is used for, as measurable cases.

Every case goes through the public entry points of `paper_2509_00404_amd.metis` the way a program that trains or
serves the split-FP4 linear layer calls them.  Seven kinds:

  serve     the weight was decomposed, split and quantized when the model was loaded; a call quantizes the
            activations of its tokens and multiplies (forward only).  Few tokens = decode, many = prefill.
  project   decompose + split a weight, quantize (or decompose + split) the activations, forward product: the first
            contact of a layer with the format.
  train     one linear layer in training: X, W and G decomposed in one batch, split in both orientations, forward,
            input-gradient and weight-gradient products.
  parts     the paper's own training step: the weight's factors and residual are stored variables and only
            quantized, X and G are decomposed and split, all rounding stochastic, weight gradient in fp32 and the
            gradients of the weight's factors.
  layer     all linears of one decoder layer in one step (the benchmark's default workload), the operands'
            preparation dealt over streams.
  quantize  a quantizer alone (nearest, stochastic, or random Hadamard + stochastic) over a tensor.
  mx        the MXFP4 variant of a forward product: both operands quantized, then multiplied.

Sizes are the linears of a LLaMA-3-8B layer and the token counts of the benchmark's configurations, the tests' ragged
shapes, and generic ones between.  Matrices have a planted power-law spectrum (weights, activations with outlier
channels, steep output gradients) as in `workloads.py`, drawn on the GPU from the seed.
"""
import math

import torch

from paper_2509_00404_amd import metis, workloads

FACTOR_SCALE = 2.0 ** -11            # tensor scale of the singular vectors (entries below 1)


def listed():
    return [
        # a decode step of a served model: 16 sequences, one token each, through an attention projection
        dict(name="decode", kind="serve", L=16, N=4096, K=4096, k=64, p=16, out="bf16"),
        # a prompt of 2048 tokens through an up projection
        dict(name="prefill", kind="serve", L=2048, N=14336, K=4096, k=64, p=16, out="bf16"),
        # the smallest configuration: latency and launches are all it costs
        dict(name="tiny", kind="project", L=128, N=256, K=512, k=8, p=8, rho_w=0.25, x_split=False, out="bf16"),
        # attention projection: weight decomposed over all its rows, activations quantized
        dict(name="attention", kind="project", L=8192, N=4096, K=4096, k=64, p=16, rho_w=1.0, x_split=False, out="bf16"),
        # training a narrow layer on a short batch of ragged sizes, whole sequences sampled, fp32 outputs
        dict(name="ragged", kind="train", L=1360, N=752, K=1232, k=20, p=12, rho_w=1.0, rho_x=0.125, group=16, out="f32"),
        # training a key / value projection on an ordinary batch
        dict(name="kv_step", kind="train", L=4096, N=1024, K=4096, k=64, p=16, rho_w=1.0, rho_x=0.0625, group=1, out="bf16"),
        # training the down projection on a large batch
        dict(name="down_step", kind="train", L=8192, N=4096, K=14336, k=64, p=16, rho_w=1.0, rho_x=0.0625, group=1,
             out="bf16"),
        # steady-state training of an attention projection from stored parts on a packed batch (no padding: the token
        # count is no round number), stochastic rounding
        dict(name="parts_step", kind="parts", L=6000, N=4096, K=4096, k=64, p=16, rho_x=0.0625),
        # one decoder layer (q, k, v, o, gate, up, down) at 16384 tokens
        dict(name="layer", kind="layer", L=16384, k=64, p=16, rho_w=1.0, rho_x=0.0625),
        # gradients into the stochastic quantizer, both orientations
        dict(name="quantize_sr", kind="quantize", M=8192, N=14336, rounding="sr", dtype="bf16", both=True),
        # the Hadamard recipe the paper compares with, on activations of an attention projection
        dict(name="quantize_rht", kind="quantize", M=8192, N=4096, rounding="rht", dtype="bf16", both=False),
        # the microscaling variant of an up projection
        dict(name="mx_linear", kind="mx", L=8192, N=14336, K=4096, out="bf16"),
    ]


def _log_uniform(rng, lo, hi, multiple):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(multiple * round(v / multiple), multiple * math.ceil(lo / multiple)), hi // multiple * multiple)


def draw(rng):
    kind = rng.choice(["serve", "serve", "project", "train", "train", "parts", "layer", "quantize", "mx"])
    k, p = rng.choice([(8, 8), (16, 16), (20, 12), (32, 16), (44, 12), (64, 16), (64, 16), (80, 16)])
    out = rng.choice(["bf16", "bf16", "f32"])
    if kind == "serve":
        return dict(kind=kind, L=_log_uniform(rng, 1, 8192, 1), N=_log_uniform(rng, 256, 14336, 16),
                    K=_log_uniform(rng, 256, 14336, 16), k=k, p=p, out=out)
    if kind == "project":
        return dict(kind=kind, L=_log_uniform(rng, 128, 16384, 16), N=_log_uniform(rng, 256, 14336, 16),
                    K=_log_uniform(rng, 512, 8192, 16), k=k, p=p, rho_w=rng.choice([0.25, 1.0]),
                    x_split=rng.random() < 0.5, out=out)
    if kind == "train":
        return dict(kind=kind, L=_log_uniform(rng, 512, 16384, 16), N=_log_uniform(rng, 256, 8192, 16),
                    K=_log_uniform(rng, 256, 8192, 16), k=k, p=p, rho_w=rng.choice([0.25, 1.0]),
                    rho_x=rng.choice([1 / 16, 1 / 8]), group=rng.choice([1, 1, 16]), out=out)
    if kind == "parts":
        return dict(kind=kind, L=_log_uniform(rng, 1024, 16384, 16), N=_log_uniform(rng, 512, 8192, 16),
                    K=_log_uniform(rng, 512, 8192, 16), k=k, p=p, rho_x=rng.choice([1 / 16, 1 / 8]))
    if kind == "layer":
        return dict(kind=kind, L=_log_uniform(rng, 1024, 6144, 16), k=64, p=16, rho_w=1.0, rho_x=0.0625)
    if kind == "quantize":
        rounding = rng.choice(["nearest", "sr", "rht"])
        dtype = rng.choice(["bf16", "f32"]) if rounding != "rht" else "bf16"
        return dict(kind=kind, M=_log_uniform(rng, 256, 16384, 16), N=_log_uniform(rng, 256, 14336, 16), rounding=rounding,
                    dtype=dtype, both=rounding != "rht" and rng.random() < 0.5)
    return dict(kind=kind, L=_log_uniform(rng, 256, 16384, 1), N=_log_uniform(rng, 256, 14336, 16),
                K=_log_uniform(rng, 512, 14336, 32), out=out)


# ---- inputs ---------------------------------------------------------------------------------------------------------

class _Draws:
    """Seeded matrices on the GPU: A = U0 diag(s) V0^T (+ noise) at a given RMS, as workloads.planted makes them."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1))

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, device="cuda", dtype=torch.float32)

    def planted(self, M, N, alpha, rms, head=0, noise=0.0, outliers=False):
        q = min(M, N, 192)
        s = torch.arange(1, q + 1, device="cuda", dtype=torch.float32) ** -alpha
        s[:head] *= 100.0
        A = (self.normal(M, q) * s) @ self.normal(N, q).t()
        A += (noise * float(s[0]) * math.sqrt(M * N) / (math.sqrt(M) + math.sqrt(N))) * self.normal(M, N)
        A *= rms / A.pow(2).mean().sqrt()
        if outliers:
            cols = torch.randperm(N, generator=self.g, device="cuda")[:max(1, round(N / 1000))]
            A[:, cols] *= 20.0
        return A.to(torch.bfloat16)

    # the trailing noise keeps every sketch well conditioned, as the full-rank tensors of a real model do
    def weight(self, N, K):
        return self.planted(N, K, alpha=1.0, rms=0.02, noise=0.01)

    def activation(self, L, K):
        return self.planted(L, K, alpha=1.2, rms=1.0, noise=0.003, outliers=True)

    def gradient(self, L, N):
        return self.planted(L, N, alpha=2.0, rms=1e-3, head=4, noise=0.0001)


def _tscale(A):
    return metis.tensor_scale(float(A.abs().max()))


class _Operand:
    """A matrix that is decomposed and split on every pass, with the buffers a program keeps for it."""

    def __init__(self, A, k, p, rho, seed, want_t=True, group=1):
        self.A, self.k, self.p, self.rho, self.seed, self.group = A, k, p, rho, seed, group
        M, N = A.shape
        if group > 1:                        # whole sequences: the rate that gives the same number of rows one by one
            rho = (metis.sample_count(M, k, p, rho, group) - 0.5) / M
        f32 = dict(dtype=torch.float32, device="cuda")
        self.U, self.S, self.V = torch.empty((M, k), **f32), torch.empty((k,), **f32), torch.empty((N, k), **f32)
        self.ws_dec = torch.empty((metis.decompose_workspace_bytes(M, N, k, p, rho),), dtype=torch.uint8, device="cuda")
        self.ws_split = torch.empty((metis.split_workspace_bytes(M, N, k),), dtype=torch.uint8, device="cuda")
        self.q = metis.SplitTensor(M, N, k, FACTOR_SCALE, FACTOR_SCALE, _tscale(A), want_t)

    def job(self):
        return dict(A=self.A, k=self.k, p=self.p, rho=self.rho, seed=self.seed, U=self.U, S=self.S, V=self.V,
                    workspace=self.ws_dec, group=self.group)

    def decompose(self):
        metis.decompose(self.A, self.k, self.p, self.rho, self.seed, workspace=self.ws_dec, out=(self.U, self.S, self.V))

    def split(self):
        metis.split_quantize(self.A, self.U, self.S, self.V, self.q, workspace=self.ws_split)

    def split_sr(self):
        metis.split_quantize_sr(self.A, self.U, self.S, self.V, self.seed, self.q, workspace=self.ws_split)


def _dtype(case):
    return torch.float32 if case.get("out") == "f32" or case.get("dtype") == "f32" else torch.bfloat16


def _empty(rows, cols, dtype):
    return torch.empty((rows, cols), dtype=dtype, device="cuda")


def _linear_ws(L, N, K, k):
    return torch.empty((max(metis.linear_workspace_bytes(L, N, K, k), 256),), dtype=torch.uint8, device="cuda")


def _plain(L, K, A):
    return metis.SplitTensor(L, K, 0, 1.0, 1.0, _tscale(A), want_t=False)


def prepare(case, seed):
    d = _Draws(seed)
    kind = case["kind"]
    s = dict(case=case)
    lib_seed = 7919 * (seed + 1)
    if kind == "serve":
        L, N, K, k, p = (case[x] for x in ("L", "N", "K", "k", "p"))
        w = _Operand(d.weight(N, K), k, p, 1.0, lib_seed, want_t=False)
        w.decompose()
        w.split()
        s["W"] = w.q
        s["x"] = d.activation(L, K)
        s["X"] = _plain(L, K, s["x"])
        s["Y"], s["ws"] = _empty(L, N, _dtype(case)), _linear_ws(L, N, K, k)
    elif kind == "project":
        L, N, K, k, p = (case[x] for x in ("L", "N", "K", "k", "p"))
        s["w"] = _Operand(d.weight(N, K), k, p, case["rho_w"], lib_seed, want_t=False)
        x = d.activation(L, K)
        if case["x_split"]:
            s["xo"] = _Operand(x, k, p, 0.0625, lib_seed + 1, want_t=False)
            s["batch"] = metis.DecomposeBatch([s["w"].job(), s["xo"].job()])
        else:
            s["x"], s["X"] = x, _plain(L, K, x)
        s["Y"], s["ws"] = _empty(L, N, _dtype(case)), _linear_ws(L, N, K, k)
    elif kind == "train":
        L, N, K, k, p, group = (case[x] for x in ("L", "N", "K", "k", "p", "group"))
        s["ops"] = [_Operand(d.weight(N, K), k, p, case["rho_w"], lib_seed),
                    _Operand(d.activation(L, K), k, p, case["rho_x"], lib_seed + 1, group=group),
                    _Operand(d.gradient(L, N), k, p, case["rho_x"], lib_seed + 2, group=group)]
        s["batch"] = metis.DecomposeBatch([o.job() for o in s["ops"]])
        s["out"] = _empty(L, N, _dtype(case)), _empty(L, K, _dtype(case)), _empty(N, K, _dtype(case))
        s["ws"] = _linear_ws(L, N, K, k)
    elif kind == "parts":
        L, N, K, k, p = (case[x] for x in ("L", "N", "K", "k", "p"))
        w = _Operand(d.weight(N, K), k, p, 1.0, lib_seed)
        w.decompose()                                       # once, when training starts
        w.residual = (w.A.float() - (w.U * w.S) @ w.V.t()).to(torch.bfloat16)
        w.A = w.ws_dec = w.ws_split = None
        s["w"] = w
        s["ops"] = [_Operand(d.activation(L, K), k, p, case["rho_x"], lib_seed + 1),
                    _Operand(d.gradient(L, N), k, p, case["rho_x"], lib_seed + 2)]
        s["batch"] = metis.DecomposeBatch([o.job() for o in s["ops"]])
        s["out"] = _empty(L, N, torch.bfloat16), _empty(L, K, torch.bfloat16), _empty(N, K, torch.float32)
        s["grads"] = _empty(N, k, torch.float32), _empty(k, k, torch.float32), _empty(K, k, torch.float32)
        s["ws"] = _linear_ws(L, N, K, k)
        s["ws_grads"] = torch.empty((metis.factor_grads_workspace_bytes(N, K, k),), dtype=torch.uint8, device="cuda")
    elif kind == "layer":
        L, k, p = case["L"], case["k"], case["p"]
        ops, products = [], []
        for i, (_, N, K) in enumerate(workloads.LAYER_LINEARS):
            W = _Operand(d.weight(N, K), k, p, case["rho_w"], lib_seed + 10 * i)
            X = _Operand(d.activation(L, K), k, p, case["rho_x"], lib_seed + 10 * i + 1)
            G = _Operand(d.gradient(L, N), k, p, case["rho_x"], lib_seed + 10 * i + 2)
            ops += [W, X, G]
            for product, a, b, rows, cols in ((metis.LINEAR_FWD, X, W, L, N), (metis.LINEAR_DGRAD, G, W, L, K),
                                              (metis.LINEAR_WGRAD, G, X, N, K)):
                products.append((product, a.q, b.q, _empty(rows, cols, torch.bfloat16), _linear_ws(L, N, K, k)))
        s["streams"] = [torch.cuda.Stream() for _ in range(3)]
        groups = [[] for _ in s["streams"]]
        for i, o in enumerate(sorted(ops, key=lambda o: -o.A.numel())):
            groups[i % len(groups)].append(o)
        s["groups"] = [(g, metis.DecomposeBatch([o.job() for o in g])) for g in groups]
        s["products"] = products
    elif kind == "quantize":
        M, N = case["M"], case["N"]
        s["A"] = d.gradient(M, N).to(_dtype(case))
        g = _tscale(s["A"])
        s["out"] = metis.Fp4Tensor(M, N, g)
        s["out_t"] = metis.Fp4Tensor(N, M, g) if case["both"] else None
        s["seed"] = lib_seed
    else:
        L, N, K = (case[x] for x in ("L", "N", "K"))
        s["x"], s["w"] = d.activation(L, K), d.weight(N, K)
        s["X"], s["W"], s["Y"] = metis.MxTensor(L, K), metis.MxTensor(N, K), _empty(L, N, _dtype(case))
    return s


# ---- one pass -------------------------------------------------------------------------------------------------------

def _run_serve(s):
    metis.quantize(s["x"], s["X"].R)
    return metis.fp4_linear_fwd(s["X"], s["W"], s["Y"], s["ws"])


def _run_project(s):
    w = s["w"]
    if "batch" in s:
        s["batch"].run()
        s["xo"].split()
        X = s["xo"].q
    else:
        w.decompose()
        metis.quantize(s["x"], s["X"].R)
        X = s["X"]
    w.split()
    return metis.fp4_linear_fwd(X, w.q, s["Y"], s["ws"]), w.S


def _run_train(s):
    W, X, G = s["ops"]
    s["batch"].run()
    for o in s["ops"]:
        o.split()
    Y, dX, dW = s["out"]
    metis.fp4_linear_fwd(X.q, W.q, Y, s["ws"])
    metis.fp4_linear_dgrad(G.q, W.q, dX, s["ws"])
    metis.fp4_linear_wgrad(G.q, X.q, dW, s["ws"])
    return Y, dX, dW, W.S, X.S, G.S


def _run_parts(s):
    w, (X, G) = s["w"], s["ops"]
    s["batch"].run()
    X.split_sr()
    G.split_sr()
    metis.split_from_parts(w.residual, w.U, w.S, w.V, w.q, seed=w.seed)
    Y, dX, dW = s["out"]
    metis.fp4_linear_fwd(X.q, w.q, Y, s["ws"])
    metis.fp4_linear_dgrad(G.q, w.q, dX, s["ws"])
    metis.fp4_linear_wgrad(G.q, X.q, dW, s["ws"])
    dU, dS, dV = metis.fp4_factor_grads(dW, w.q, *s["grads"], workspace=s["ws_grads"])
    return Y, dX, dW, dU, dS, dV


def _run_layer(s):
    main, streams = torch.cuda.current_stream(), s["streams"]
    # the operands are independent of one another: prepared side by side
    for st, (ops, batch) in zip(streams, s["groups"]):
        st.wait_stream(main)
        with torch.cuda.stream(st):
            batch.run()
            for o in ops:
                o.split()
    for st in streams:
        main.wait_stream(st)
    # the products' pre-passes side by side, then their main kernels back to back
    for i, st in enumerate(streams):
        st.wait_stream(main)
        with torch.cuda.stream(st):
            for product, a, b, _, ws in s["products"][i::len(streams)]:
                metis.fp4_linear_phase(product, metis.LINEAR_PREPARE, a, b, None, ws)
    for st in streams:
        main.wait_stream(st)
    return [metis.fp4_linear_phase(product, metis.LINEAR_APPLY, a, b, out, ws) for product, a, b, out, ws in s["products"]]


def _run_quantize(s):
    o, t = s["out"], s["out_t"]
    rounding = s["case"]["rounding"]
    if rounding == "nearest":
        metis.quantize(s["A"], o, t)
    elif rounding == "sr":
        metis.quantize_sr(s["A"], s["seed"], o, t)
    else:
        metis.quantize_rht_sr(s["A"], s["seed"], o)
    return (o.codes, o.scales) + ((t.codes, t.scales) if t is not None else ())


def _run_mx(s):
    metis.quantize_mx(s["x"], s["X"])
    metis.quantize_mx(s["w"], s["W"])
    return metis.mxfp4_gemm_nt(s["X"], s["W"], s["Y"])


_RUN = dict(serve=_run_serve, project=_run_project, train=_run_train, parts=_run_parts, layer=_run_layer,
            quantize=_run_quantize, mx=_run_mx)


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def _decompose_flops(M, N, k, p, rho):
    """Sketch and projection of the sampled rows, broadcast over all rows, low-rank product of the residual."""
    return 4.0 * min(M, max(k + p, math.ceil(rho * M))) * N * (k + p) + 4.0 * M * N * k


def _train_work(L, N, K, k, p, rho_w, rho_x):
    numel = L * N + L * K + N * K
    flops = (_decompose_flops(N, K, k, p, rho_w) + _decompose_flops(L, K, k, p, rho_x) + _decompose_flops(L, N, k, p, rho_x) +
             6.0 * L * N * K)
    return numel, flops


def work(case):
    kind = case["kind"]
    size = 4 if _dtype(case) == torch.float32 else 2
    if kind == "quantize":
        n = case["M"] * case["N"]
        return dict(bytes=n * (size + 0.5625 * (2 if case["both"] else 1)), flops=0.0)
    L, k, p = case["L"], case.get("k", 0), case.get("p", 0)
    if kind == "layer":
        total_bytes = total_flops = 0.0
        for _, N, K in workloads.LAYER_LINEARS:
            numel, flops = _train_work(L, N, K, k, p, case["rho_w"], case["rho_x"])
            total_bytes += 4.0 * numel                       # three bf16 inputs read, three bf16 results written
            total_flops += flops
        return dict(bytes=total_bytes, flops=total_flops)
    N, K = case["N"], case["K"]
    if kind == "serve":
        return dict(bytes=2.0 * L * K + 0.5625 * (N * K + k * (N + K)) + size * L * N, flops=2.0 * L * N * K)
    if kind == "project":
        flops = _decompose_flops(N, K, k, p, case["rho_w"]) + 2.0 * L * N * K
        if case["x_split"]:
            flops += _decompose_flops(L, K, k, p, 0.0625)
        return dict(bytes=2.0 * (L * K + N * K) + size * L * N, flops=flops)
    if kind == "train":
        numel, flops = _train_work(L, N, K, k, p, case["rho_w"], case["rho_x"])
        return dict(bytes=(2.0 + size) * numel, flops=flops)
    if kind == "parts":
        numel = L * N + L * K + N * K
        flops = (_decompose_flops(L, K, k, p, case["rho_x"]) + _decompose_flops(L, N, k, p, case["rho_x"]) + 6.0 * L * N * K +
                 4.0 * N * K * k)
        return dict(bytes=4.0 * numel + 2.0 * N * K + 8.0 * k * (N + K), flops=flops)
    return dict(bytes=2.0 * (L * K + N * K) + size * L * N, flops=2.0 * L * N * K)


def tolerance(case):
    """Quantized bytes are exact.  Products: the fused decompose + split call against the two calls (another rounding
    of the same residual, so codes differ at their thresholds) gives up to 2.1e-3, and the fp64 product of the quantized
    operands up to 2.3e-3 (bf16 outputs and the low-rank columns' bf16 rounding).  MXFP4 products have neither the split nor
    such columns: 1.7e-3 in bf16, and in fp32 only the order of the sums (1e-5)."""
    kind = case["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "mx":
        return dict(rel=4e-5) if _dtype(case) == torch.float32 else dict(rel=7e-3)
    return dict(rel=8e-3)
