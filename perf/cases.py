"""Performance cases of the routed any-precision linear layer: what a program that serves such a model has it do.

  block       a decode step: the seven routed linears of a decoder block as its four dependent stages {q, k, v}, {o},
              {gate, up}, {down}, one stage call each, replayed from a HIP graph that holds `layers` blocks (a serving
              loop captures its decode step once per batch size and replays it for every token).  Options that are
              served the same way: other slice widths (`slices`) and quantised activations (`abits`).
  stage       one stage call made eagerly, buffers left to the binding: a single routed linear at few tokens, where
              the launches and the host count as much as the kernels.
  mlp         a prompt: the gated MLP's two stages {gate, up}, {down} at hundreds to thousands of tokens, eager calls
              on buffers that the program keeps.
  mlp_router  a prompt routed by the two-layer router with a run-time threshold, then the linears that share its input.
  encode      packing a weight matrix, the offline direction (and what a weight update costs).

Shapes are those of the repository's workloads (Llama-2-7B, Llama-3-8B and Llama-70B shaped linears, the 2048 x 2048
single linear) and generic odd ones.  Weights are heavy-tailed (Student t times a log-normal row scale), tokens are
N(0, 1) in bf16 with outlier channels (decode) or outlier tokens (prompts), routers are N(0, 1 / K) with biases that
give the stated precision mix.
"""
import functools
import math

import numpy as np
import torch

import paper_2602_20191_amd as mbq

DEVICE = "cuda:0"
# tokens at 2, 4, 6, 8 bits
MIXES = {"uniform": (0.25, 0.25, 0.25, 0.25), "falling": (0.40, 0.30, 0.20, 0.10), "prompt": (0.50, 0.30, 0.15, 0.05),
         "skewed": (0.70, 0.20, 0.08, 0.02)}


def listed():
    return [
        # the smallest call a program makes: one token through one linear
        {"name": "stage_2048_1tok", "kind": "stage", "N": 2048, "K": 2048, "T": 1, "mix": "uniform"},
        # a single linear at a small batch
        {"name": "stage_2048_32tok", "kind": "stage", "N": 2048, "K": 2048, "T": 32, "mix": "falling"},
        # interactive decoding of one sequence
        {"name": "block_7b_1tok", "kind": "block", "hidden": 4096, "kv": 4096, "ffn": 11008, "T": 1, "layers": 2,
         "slices": "2222", "abits": 0, "mix": "uniform"},
        # batched decoding: the shape of the repository's main benchmark
        {"name": "block_7b_16tok", "kind": "block", "hidden": 4096, "kv": 4096, "ffn": 11008, "T": 16, "layers": 2,
         "slices": "2222", "abits": 0, "mix": "uniform"},
        # the same with slice widths whose precisions end inside a two-bit digit, at a small batch
        {"name": "block_7b_4tok_3122", "kind": "block", "hidden": 4096, "kv": 4096, "ffn": 11008, "T": 4, "layers": 2,
         "slices": "3122", "abits": 0, "mix": "uniform"},
        # the same with 4-bit activations
        {"name": "block_7b_16tok_a4", "kind": "block", "hidden": 4096, "kv": 4096, "ffn": 11008, "T": 16, "layers": 1,
         "slices": "2222", "abits": 4, "mix": "uniform"},
        # a loaded server: a grouped-query block at 64 tokens
        {"name": "block_8b_64tok", "kind": "block", "hidden": 4096, "kv": 1024, "ffn": 14336, "T": 64, "layers": 2,
         "slices": "2222", "abits": 0, "mix": "uniform"},
        # a large model's MLP at a large decode batch (or a short prompt)
        {"name": "mlp_70b_256tok", "kind": "mlp", "hidden": 8192, "ffn": 28672, "T": 256, "mix": "skewed"},
        # prompts
        {"name": "mlp_7b_2048tok", "kind": "mlp", "hidden": 4096, "ffn": 11008, "T": 2048, "mix": "prompt"},
        {"name": "mlp_70b_4096tok", "kind": "mlp", "hidden": 8192, "ffn": 28672, "T": 4096, "mix": "skewed"},
        # a ragged prompt on odd shapes, routed by the two-layer router
        {"name": "mlp_router_odd_777tok", "kind": "mlp_router", "N": 3000, "N2": 1000, "K": 2176, "H": 64, "T": 777},
        # packing a weight
        {"name": "encode_11008x4096", "kind": "encode", "N": 11008, "K": 4096},
    ]


def _spread(rng, lo, hi):
    """A whole number of lo .. hi, even over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choices(["block", "stage", "mlp", "mlp_router", "encode"], [40, 15, 30, 7, 8])[0]
    if kind == "block":
        hidden = 128 * _spread(rng, 8, 32)
        slices, abits = rng.choice([("2222", 0), ("2222", 0), ("2222", 0), ("422", 0), ("3122", 0), ("2222", 4), ("2222", 8)])
        tokens = _spread(rng, 1, 16 if slices == "3122" else 64)
        return {"kind": kind, "hidden": hidden, "kv": hidden // rng.choice([1, 4, 8]), "ffn": 128 * _spread(rng, 20, 112),
                "T": tokens, "layers": 1 if abits else 2, "slices": slices, "abits": abits,
                "mix": rng.choice(["uniform", "falling", "skewed"])}
    if kind == "stage":
        return {"kind": kind, "N": _spread(rng, 256, 8192), "K": 128 * _spread(rng, 4, 64), "T": _spread(rng, 1, 128),
                "mix": rng.choice(["uniform", "falling", "skewed"])}
    if kind == "mlp":
        hidden = 128 * _spread(rng, 16, 64)
        return {"kind": kind, "hidden": hidden, "ffn": 128 * max(16, min(224, int(hidden / 128 * rng.uniform(2.5, 3.6)))),
                "T": _spread(rng, 65, 4096), "mix": rng.choice(["uniform", "prompt", "skewed"])}
    if kind == "mlp_router":
        return {"kind": kind, "N": _spread(rng, 500, 8192), "N2": _spread(rng, 250, 4096), "K": 128 * _spread(rng, 8, 40),
                "H": rng.choice([32, 64, 96]), "T": _spread(rng, 16, 3000)}
    return {"kind": kind, "N": _spread(rng, 1000, 14336), "K": 128 * _spread(rng, 8, 64)}


# ---- inputs -------------------------------------------------------------------------------------------------------
def _weights(gen, N, K):
    """fp32 [N, K]: Student t with four degrees of freedom times 0.02 and a log-normal row scale."""
    z = torch.randn((N, K), generator=gen, device=DEVICE)
    u = torch.rand((N, K), generator=gen, device=DEVICE).mul_(torch.rand((N, K), generator=gen, device=DEVICE))
    z.div_(u.clamp_(min=1e-30).log_().mul_(-0.5).sqrt_())  # -2 log(u1 u2) is chi-squared with four degrees of freedom
    return z.mul_(0.02 * torch.exp(0.3 * torch.randn((N, 1), generator=gen, device=DEVICE)))


def _tokens(gen, T, K, outliers):
    """bf16 [T, K], N(0, 1); 1 % of the channels x 20 ("channels") or 2 % of the tokens with ten times the norm."""
    x = torch.randn((T, K), generator=gen, device=DEVICE)
    if outliers == "channels":
        x[:, torch.randperm(K, generator=gen, device=DEVICE)[: K // 100]] *= 20.0
    else:
        x[torch.rand((T,), generator=gen, device=DEVICE) < 0.02] *= 10.0
    return x.to(torch.bfloat16)


@functools.lru_cache(maxsize=None)
def _unit_bias(mix):
    """Biases that give the mix where the logits are independent N(0, 1) before them."""
    s = np.random.default_rng(7).standard_normal((20000, len(mix)))
    b = np.log(np.asarray(mix))
    for _ in range(200):
        got = np.bincount(np.argmax(s + b, axis=1), minlength=len(mix)) / len(s)
        b = b + 0.3 * np.log(np.asarray(mix) / np.maximum(got, 1e-6))
    return tuple(b - b.mean())


def _router(gen, K, mix, outliers, outputs=4):
    share = MIXES[mix]
    share = share if outputs == 4 else (share[0] + share[1], share[2], share[3])
    deviation = math.sqrt(0.99 + 0.01 * 400) if outliers == "channels" else 1.0
    Wr = torch.randn((outputs, K), generator=gen, device=DEVICE) / math.sqrt(K)
    return Wr, torch.tensor(np.asarray(_unit_bias(share)) * deviation, dtype=torch.float32, device=DEVICE)


def _routing(T, P=4):
    i32 = dict(dtype=torch.int32, device=DEVICE)
    return torch.zeros(T, **i32), torch.zeros(T, **i32), torch.zeros(P + 1, **i32)


class _Stage:
    """Projections that share their input, with the buffers a program keeps for them."""

    def __init__(self, gen, Ns, K, T, mix, outliers, slices="2222", abits=0):
        self.Ns, self.K, self.abits = list(Ns), K, abits
        self.cfg = None if slices == "2222" else mbq.Config([int(c) for c in slices])
        self.X = _tokens(gen, T, K, outliers)
        routers = [_router(gen, K, mix, outliers, len(slices)) for _ in Ns]
        self.Wr, self.br = [r[0] for r in routers], [r[1] for r in routers]
        self.blobs = [mbq.mbq_encode(_weights(gen, N, K)) for N in Ns]
        self.routing = [_routing(T) for _ in Ns]
        self.Y = [torch.zeros((T, N), dtype=torch.float32, device=DEVICE) for N in Ns]
        self.ws_route = mbq.route_workspace(T, K, DEVICE)
        self.ws_linear = mbq.linear_workspace(T, max(Ns), K, DEVICE)
        if abits:
            self.shift = 0.1 * torch.randn((K,), generator=gen, device=DEVICE)
            self.scale = torch.exp(0.3 * torch.randn((K,), generator=gen, device=DEVICE))
            self.act = (torch.zeros_like(self.X), torch.zeros((T,), dtype=torch.float32, device=DEVICE),
                        torch.zeros_like(self.X))

    def call(self):
        kept = dict(routing=self.routing, Y=self.Y, ws_route=self.ws_route, ws_linear=self.ws_linear)
        if self.abits:
            mbq.mbq_routed_linear_group_act(self.X, self.abits, self.shift, self.scale, self.Wr, self.br, self.blobs,
                                            self.Ns, act=self.act, **kept)
        elif self.cfg is not None:
            mbq.mbq_routed_linear_group_cfg(self.X, self.Wr, self.br, self.cfg, self.blobs, self.Ns, **kept)
        else:
            mbq.mbq_routed_linear_group(self.X, self.Wr, self.br, self.blobs, self.Ns, **kept)

    def outputs(self):
        return [list(r) + [y] for r, y in zip(self.routing, self.Y)] + ([list(self.act)] if self.abits else [])


def _block_stages(case):
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [((h, kv, kv), h), ((h,), h), ((f, f), h), ((h,), f)]


def _mlp_stages(case):
    return [((case["ffn"], case["ffn"]), case["hidden"]), ((case["hidden"],), case["ffn"])]


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    kind = case["kind"]
    state = {"kind": kind, "case": case}
    if kind == "block":
        stages = [_Stage(gen, Ns, K, case["T"], case["mix"], "channels", case["slices"], case["abits"])
                  for _ in range(case["layers"]) for Ns, K in _block_stages(case)]
        state["stages"] = stages
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            for s in stages:
                s.call()
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            for s in stages:
                s.call()
    elif kind == "mlp":
        state["stages"] = [_Stage(gen, Ns, K, case["T"], case["mix"], "tokens") for Ns, K in _mlp_stages(case)]
    elif kind == "stage":
        state["X"] = _tokens(gen, case["T"], case["K"], "channels")
        state["Wr"], state["br"] = _router(gen, case["K"], case["mix"], "channels")
        state["blob"] = mbq.mbq_encode(_weights(gen, case["N"], case["K"]))
    elif kind == "mlp_router":
        K, H = case["K"], case["H"]
        state["X"] = _tokens(gen, case["T"], K, "tokens")
        state["W1"] = torch.randn((H, K), generator=gen, device=DEVICE) / math.sqrt(K)
        state["b1"] = 0.1 * torch.randn((H,), generator=gen, device=DEVICE)
        state["W2"] = 2.0 * torch.randn((4, H), generator=gen, device=DEVICE) / math.sqrt(H)
        state["b2"] = 0.5 - 0.5 * torch.arange(4, dtype=torch.float32, device=DEVICE)
        state["Ns"] = [case["N"], case["N2"]]
        state["blobs"] = [mbq.mbq_encode(_weights(gen, N, K)) for N in state["Ns"]]
        state["ws_route"] = mbq.route_mlp_workspace(case["T"], K, H, DEVICE)
        state["ws_linear"] = mbq.linear_workspace(case["T"], max(state["Ns"]), K, DEVICE)
    else:
        state["W"] = _weights(gen, case["N"], case["K"])
        state["blob"] = torch.zeros(mbq.blob_bytes(case["N"], case["K"]), dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    kind = state["kind"]
    if kind == "block":
        state["graph"].replay()
        return [s.outputs() for s in state["stages"]]
    if kind == "mlp":
        for s in state["stages"]:
            s.call()
        return [s.outputs() for s in state["stages"]]
    if kind == "stage":
        return mbq.mbq_routed_linear_group(state["X"], [state["Wr"]], [state["br"]], [state["blob"]], [state["case"]["N"]])
    if kind == "mlp_router":
        routing = mbq.mbq_route_mlp(state["X"], state["W1"], state["b1"], state["W2"], state["b2"], 0.0,
                                    ws=state["ws_route"])
        Y = mbq.mbq_linear_group(state["X"], state["blobs"], state["Ns"], state["case"]["K"], [routing] * 2,
                                 ws=state["ws_linear"])
        return list(routing) + Y
    return mbq.mbq_encode(state["W"], state["blob"])


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def _average_bits(case):
    """(expected bits of the highest precision among the T tokens, of the average token) of a linear."""
    mix, bits = np.asarray(MIXES[case["mix"]]), np.asarray([2.0, 4.0, 6.0, 8.0])
    if case.get("slices", "2222") == "422":
        mix, bits = np.asarray([mix[0] + mix[1], mix[2], mix[3]]), bits[1:]
    below = np.cumsum(mix) ** case["T"]  # all tokens at or below
    return float(np.sum(np.diff(np.concatenate([[0.0], below])) * bits)), float(np.sum(mix * bits))


def work(case):
    kind = case["kind"]
    if kind == "encode":
        n = case["N"] * case["K"]
        return {"bytes": 4.0 * n + n + n / 16, "flops": 32.0 * n}  # four fp64 steps of about eight operations a weight
    T = case["T"]
    if kind == "mlp_router":
        K, N, H = case["K"], case["N"] + case["N2"], case["H"]
        return {"bytes": N * K * (1 + 1 / 16) + 2.0 * T * K + 4.0 * H * K + 4.0 * T * N,
                "flops": 2.0 * T * K * (N + H)}
    if kind == "stage":
        stages = [((case["N"],), case["K"])]
    else:
        stages = _mlp_stages(case) if kind == "mlp" else _block_stages(case) * case["layers"]
    top, _ = _average_bits(case)
    b = f = 0.0
    for Ns, K in stages:
        b += 2.0 * T * K * (3 if case.get("abits") else 1)  # activations (read; integers and rebuilt ones written)
        for N in Ns:
            b += N * K * (top / 8 + 1 / 16) + 16.0 * K + 4.0 * T * N  # slices and parameters, router, outputs
            f += 2.0 * T * K * (N + 4)
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Measured against products in 64 bits of the weights that mbq_dequant gives (seen in brackets); about four times
    that.  Up to 16 tokens activations reach the matrix cores in two 8-bit floating-point pieces under a block scale
    (off by up to 2^-21 of a block's largest element: 1.2e-4, at most 4.4e-3); quantised ones are exact there, and
    everywhere else only 32-bit sums round (1e-7 at 4-bit activations, up to 1.2e-5 and 5e-4 at large K and many
    tokens).  Routing and packed bytes are whole numbers."""
    if case["kind"] == "encode":
        return "exact"
    if case["T"] <= 16:
        return {"rel": 1e-5, "max": 1e-4} if case.get("abits") else {"rel": 5e-4, "max": 1.2e-2}
    return {"rel": 4e-5, "max": 2e-3}


# ---- the same results in 64 bits ------------------------------------------------------------------------------------
def _quantised(W):
    """Eight-bit codes (fp64 [N, G, 128]), group scales and zero points ([N, G, 1]) of fp32 weights: the recursion
    c = clamp(floor(R / s + z)), R -= s ((c - z) + 1/2), s /= 4 over four two-bit slices, step by step in 64 bits."""
    w = W.view(W.shape[0], -1, 128)
    lo, hi = w.amin(dim=2, keepdim=True), w.amax(dim=2, keepdim=True)
    span = torch.maximum(hi - lo, torch.maximum(lo.abs(), hi.abs()).mul(2.0 ** -16).clamp(min=2.0 ** -100))
    s0 = span * 0.25
    z0 = (-lo.double() / s0.double()).float().double()
    R, s, code = w.double(), s0.double(), 0.0
    for e in range(4):
        z = z0 if e == 0 else 2.0
        c = (R / s + z).floor_().clamp_(0.0, 3.0)
        code = code * 4.0 + c
        R = R - s * ((c - z) + 0.5)
        s = s * 0.25
    return code, s0.double(), z0


def _linear(X, W, bits):
    """X [T, K] times the weights rebuilt from the leading bits[i] bits of every code, fp64 [T, N]; W in row blocks."""
    Y = torch.zeros((X.shape[0], W.shape[0]), dtype=torch.float64, device=DEVICE)
    x, used = X.double(), torch.unique(bits).tolist()
    for n in range(0, W.shape[0], 2048):
        code, s0, z0 = _quantised(W[n:n + 2048])
        for b in used:
            rows = torch.nonzero(bits == b).flatten()
            rebuilt = s0 * (((code * 2.0 ** (b - 8)).floor_() + 0.5) * 2.0 ** (2 - b) - z0)
            Y[rows, n:n + 2048] = x[rows] @ rebuilt.view(rebuilt.shape[0], -1).T
    return Y


def _routed(choice, slices):
    """Precision array, tokens grouped by the two-bit slices that they need, where the groups begin; bits of a token.
    A precision is named by its slices less one, or, where a slice ends inside a two-bit digit, by its bits less one."""
    ends = np.cumsum([int(c) for c in slices])
    bits = torch.tensor(ends, device=DEVICE)[choice]
    digits = (bits + 1) // 2
    prec = bits - 1 if (ends % 2).any() else digits - 1
    offsets = torch.stack([(digits <= d).sum() for d in range(5)])
    return [prec, torch.sort(digits, stable=True)[1], offsets], bits


def _choice(X, Wr, br):
    return torch.argmax(X.double() @ Wr.double().T + br.double(), dim=1)


def _quantised_tokens(X, abits, shift, scale):
    """Per-token quantiser, one fp32 operation a step as it is defined: integers, row scales, the router's input."""
    t = (X.float() - shift) / scale
    top = float(2 ** abits - 1)
    lo, hi = t.amin(dim=1, keepdim=True).clamp(max=0.0), t.amax(dim=1, keepdim=True).clamp(min=0.0)
    step = (hi - lo).clamp(min=2.0 ** -100) / torch.full_like(lo, top)
    zero = torch.round(-lo / step).clamp(0.0, top)
    whole = (torch.round(t / step) + zero).clamp(0.0, top) - zero
    return whole, step.flatten(), ((whole * step) * scale + shift).to(torch.bfloat16)


def exact(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    kind = case["kind"]
    if kind == "encode":
        return None  # bytes
    if kind in ("block", "mlp"):
        slices, abits = case.get("slices", "2222"), case.get("abits", 0)
        stages = _mlp_stages(case) if kind == "mlp" else _block_stages(case) * case["layers"]
        out = []
        for Ns, K in stages:
            # drawn as _Stage draws them
            X = _tokens(gen, case["T"], K, "tokens" if kind == "mlp" else "channels")
            routers = [_router(gen, K, case["mix"], "tokens" if kind == "mlp" else "channels", len(slices)) for _ in Ns]
            W = [_weights(gen, N, K) for N in Ns]
            factor, seen, act = 1.0, X, []
            if abits:
                shift = 0.1 * torch.randn((K,), generator=gen, device=DEVICE)
                scale = torch.exp(0.3 * torch.randn((K,), generator=gen, device=DEVICE))
                whole, step, seen = _quantised_tokens(X, abits, shift, scale)
                X, factor, act = whole, step.double()[:, None], [[whole, step, seen]]
            for (Wr, br), w in zip(routers, W):
                routing, bits = _routed(_choice(seen, Wr, br), slices)
                out.append(routing + [factor * _linear(X, w, bits)])
            out += act
        # one list a stage, its projections first
        per, nested = [len(Ns) + (1 if abits else 0) for Ns, _ in stages], []
        for n in per:
            nested.append(out[:n])
            out = out[n:]
        return nested
    if kind == "stage":
        X = _tokens(gen, case["T"], case["K"], "channels")
        Wr, br = _router(gen, case["K"], case["mix"], "channels")
        routing, bits = _routed(_choice(X, Wr, br), "2222")
        return [routing], [_linear(X, _weights(gen, case["N"], case["K"]), bits)]
    K, H = case["K"], case["H"]
    X = _tokens(gen, case["T"], K, "tokens")
    W1 = torch.randn((H, K), generator=gen, device=DEVICE) / math.sqrt(K)
    b1 = 0.1 * torch.randn((H,), generator=gen, device=DEVICE)
    W2 = 2.0 * torch.randn((4, H), generator=gen, device=DEVICE) / math.sqrt(H)
    b2 = 0.5 - 0.5 * torch.arange(4, dtype=torch.float32, device=DEVICE)
    scores = (X.double() @ W1.double().T + b1.double()).clamp_(min=0.0) @ W2.double().T + b2.double()
    choice = torch.cumprod((scores[:, 1:] > 0.0).long(), dim=1).sum(dim=1)
    routing, bits = _routed(choice, "2222")
    return routing + [_linear(X, _weights(gen, N, K), bits) for N in (case["N"], case["N2"])]
