"""What a user of this package has it do, as measurable cases.

A case is a plain dict.  Five kinds cover the public entry points that a serving or training program calls:

    layer     one MeteoRA linear layer, linear_forward (weights packed once, or repacked on each call)
    group     layers that share their input (q/k/v, gate/up), linear_forward_group
    block     the seven linears of one decoder block as a decode step calls them, four grouped calls
    composed  the layer from its parts on a routing the caller holds: gate_topk, base_gemm, lora_forward
    train     a gate-training step of one module: linear_forward, then gate_backward with the input gradient

Sizes are those of the repository's seeded configurations and of its decode benchmark (Llama3-8B and Llama2-13B
layers, 28 adapters of rank 8 or 16, top-2) and of its tests (other adapter counts, ranks, top-1 to top-8, ragged
widths).  Values follow gen.inputs: Gaussian activations and weights scaled so that logits and outputs are of order
one, a Zipf-like gate bias where the routing is skewed.  A token whose logits are all but tied around its k-th choice
is drawn again, as the parity tests do: which adapter such a token takes is not defined beyond fp32 summation order.
"""
import math

import torch

import paper_2405_13053_amd as m

SCALE = 2.0
BETA = 0.25
D, KV, FFN = 4096, 1024, 14336   # decoder block: model, key/value and feed-forward widths
MARGIN = 1e-4                    # least gap between the logits of consecutive ranks, against about 1e-6 of fp32 noise


def _layer(name, T, d_in, d_out, N=28, r=8, k=2, dtype="bf16", routing="uniform", packed=True, kind="layer"):
    return {"name": name, "kind": kind, "T": T, "d_in": d_in, "d_out": d_out, "N": N, "r": r, "k": k, "dtype": dtype,
            "routing": routing, "packed": packed}


def listed():
    return [
        # the smallest layer: configuration 1, fp32 storage, 64 tokens; latency and launches only
        _layer("f32_64_tiny", 64, 256, 256, N=4, dtype="f32", packed=False),
        # one sequence generating: the q, k, v projections of one new token in one grouped call
        {"name": "decode_1_qkv", "kind": "group", "T": 1, "d_in": D, "d_out": "4096,1024,1024", "N": 28, "r": 8,
         "k": 2, "routing": "uniform"},
        # 64 sequences generating: every linear of one decoder block, the weights streamed from HBM
        {"name": "decode_64_block", "kind": "block", "T": 64, "N": 28, "r": 8, "k": 2, "routing": "uniform"},
        # configuration 4: 64 new tokens through a 13B-sized MLP layer on its own
        _layer("decode_64_mlp", 64, 5120, 13824),
        # a short prompt or a chunk of one: a few hundred tokens, ragged
        _layer("chunk_300_q", 300, D, D),
        # a prompt of odd length through a narrow layer with adapters that change from call to call (not packed),
        # rank 16, top-1 as in the paper's top-1 strategy
        _layer("prompt_1531_k_top1", 1531, D, KV, r=16, k=1, packed=False),
        # configuration 2, the headline: 4 prompts of 1024 tokens
        _layer("prefill_4096_q", 4096, D, D),
        # configuration 3: the widest MLP layer, skewed adapter load
        _layer("prefill_8192_up", 8192, D, FFN, routing="zipf"),
        # configuration 5: the largest layer, rank 16, skewed adapter load
        _layer("prefill_16384_down", 16384, FFN, D, r=16, routing="zipf"),
        # many adapters of high rank, four per token: beyond what the fused routing takes
        _layer("adapters64_2000_q", 2000, D, D, N=64, r=32, k=4, routing="zipf"),
        # a caller that routes once and applies base and adapters itself
        _layer("composed_3000", 3000, 5120, 5120, kind="composed"),
        # gate training of one module, with the gradient for the module in front of it
        _layer("train_4096_q", 4096, D, D, kind="train"),
    ]


_SHAPES = [(D, D), (D, KV), (D, FFN), (FFN, D), (5120, 5120), (5120, 13824)]
_ADAPTERS = [(28, 8, 2), (28, 8, 2), (28, 8, 1), (28, 16, 2), (28, 16, 1), (12, 16, 3), (7, 32, 3), (28, 12, 2),
             (64, 32, 4), (64, 32, 8), (28, 8, 8)]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["layer"] * 5 + ["group"] * 2 + ["block", "composed", "train"])
    N, r, k = rng.choice(_ADAPTERS)
    routing = rng.choice(["uniform", "zipf"])
    if kind == "block":
        N, r, k = rng.choice([(28, 8, 2), (28, 8, 1), (28, 16, 2)])
        return {"kind": kind, "T": _log_int(rng, 1, 128), "N": N, "r": r, "k": k, "routing": routing}
    if kind == "group":
        d_in, d_out = rng.choice([(D, "4096,1024,1024"), (D, "14336,14336"), (5120, "5120,5120,5120"),
                                  (5120, "13824,13824")])
        return {"kind": kind, "T": _log_int(rng, 1, 512), "d_in": d_in, "d_out": d_out, "N": N, "r": r, "k": k,
                "routing": routing}
    if kind == "layer" and rng.random() < 0.1:
        return {"kind": kind, "T": _log_int(rng, 8, 1024), "d_in": 8 * rng.randint(8, 96),
                "d_out": 8 * rng.randint(8, 96), "N": rng.choice([4, 7, 28]), "r": r, "k": min(k, 4), "dtype": "f32",
                "routing": routing, "packed": False}
    d_in, d_out = rng.choice(_SHAPES)
    if kind == "train":
        N, r, k = rng.choice([(28, 8, 2), (28, 8, 1), (28, 16, 2)])
    elif rng.random() < 0.3:   # ragged widths
        d_in, d_out = 8 * _log_int(rng, 32, 768), 8 * _log_int(rng, 32, 768)
    # at most about the work of half the largest layer (a training step is three such passes)
    most = int((8e10 if kind == "train" else 4.8e11) / (d_in * d_out))
    lo = {"layer": 1, "composed": 16, "train": 64}[kind]
    return {"kind": kind, "T": _log_int(rng, lo, max(lo, min(16384, most))), "d_in": d_in, "d_out": d_out, "N": N,
            "r": r, "k": k, "dtype": "bf16", "routing": routing,
            "packed": kind != "composed" and (kind == "train" or rng.random() < 0.75)}


def _widths(case):
    """Per call of one pass: (d_in, [d_out of each layer that shares the input])."""
    if case["kind"] == "block":
        return [(D, [D, KV, KV]), (D, [D]), (D, [FFN, FFN]), (FFN, [D])]
    if case["kind"] == "group":
        return [(case["d_in"], [int(v) for v in case["d_out"].split(",")])]
    return [(case["d_in"], [case["d_out"]])]


class _Inputs:
    def __init__(self, case, seed):
        self.case = case
        self.dtype = torch.float32 if case.get("dtype") == "f32" else torch.bfloat16
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def randn(self, shape, std=1.0, dtype=None):
        v = torch.randn(shape, generator=self.gen, device="cuda", dtype=torch.float32)
        return v.mul_(std).to(dtype or self.dtype)

    def bias(self):
        if self.case["routing"] != "zipf":
            return None
        j = torch.arange(self.case["N"], dtype=torch.float32, device="cuda")
        return -2.0 * torch.log(j + 1.0)

    def weights(self, d_in, d_out):
        N, r = self.case["N"], self.case["r"]
        return {"W": self.randn((d_out, d_in), d_in ** -0.5), "W_gate": self.randn((d_in, N), d_in ** -0.5, torch.float32),
                "gate_bias": self.bias(), "A": self.randn((N, d_in, r), d_in ** -0.5),
                "B": self.randn((N, r, d_out), r ** -0.5)}

    def tokens(self, d_in, members):
        """x[T, d_in], rows that are all but tied at any member's gate drawn again."""
        T, k, N = self.case["T"], self.case["k"], self.case["N"]
        x = self.randn((T, d_in))
        gate = torch.cat([mb["W_gate"] for mb in members], 1).double()
        left = torch.arange(T, device="cuda")
        for _ in range(20):
            near = torch.zeros(left.numel(), dtype=torch.bool, device="cuda")
            for at in range(0, left.numel(), 4096):
                g = x[left[at:at + 4096]].double() @ gate
                for i, mb in enumerate(members):
                    gi = g[:, i * N:(i + 1) * N]
                    gi = gi if mb["gate_bias"] is None else gi + mb["gate_bias"].double()
                    top = torch.topk(gi, min(k + 1, N), dim=1).values
                    if top.shape[1] > 1:
                        near[at:at + 4096] |= (top[:, :-1] - top[:, 1:]).amin(1) < MARGIN
            left = left[near]
            if left.numel() == 0:
                break
            x[left] = self.randn((left.numel(), d_in))
        return x


def prepare(case, seed):
    make = _Inputs(case, seed)
    T, N, r, k, dt = case["T"], case["N"], case["r"], case["k"], make.dtype
    state = {"case": case, "k": k, "calls": []}
    ws_bytes = 256
    for d_in, d_outs in _widths(case):
        members = [make.weights(d_in, d_out) for d_out in d_outs]
        x = make.tokens(d_in, members)
        for mb, d_out in zip(members, d_outs):
            mb["packed"] = m.pack_weights(mb["W_gate"], mb["A"], mb["B"]) if case.get("packed", True) else None
            mb["out"] = torch.empty((T, d_out), dtype=dt, device="cuda")
        if case["kind"] in ("group", "block"):
            need = m.group_workspace_bytes(d_outs, T, d_in, N, r, k, dt)
        else:
            need = m.workspace_bytes(T, d_in, d_outs[0], N, r, k, dt)
        ws_bytes = max(ws_bytes, need)
        state["calls"].append((x, members))
    state["ws"] = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")   # the calls of a pass follow each other
    if case["kind"] == "train":
        d_in, d_out = case["d_in"], case["d_out"]
        state["dy"] = make.randn((T, d_out), d_out ** -0.5)
        # runs of 16 tokens of one task, every 11th run without a label
        runs = torch.randint(0, N, ((T + 15) // 16,), generator=make.gen, device="cuda", dtype=torch.int32)
        runs[10::11] = -1
        state["labels"] = runs.repeat_interleave(16)[:T].contiguous()
        state["W_t"] = state["calls"][0][1][0]["W"].t().contiguous()
        state["ws_back"] = torch.empty(m.gate_backward_workspace_bytes(T, d_in, d_out, N, r, k, dt), dtype=torch.uint8,
                                       device="cuda")
    return state


def run(state):
    kind, k, ws = state["case"]["kind"], state["k"], state["ws"]
    if kind in ("group", "block"):
        return [m.linear_forward_group(x, members, k, SCALE, ws=ws) for x, members in state["calls"]]
    x, (mb,) = state["calls"][0]
    if kind == "layer":
        return m.linear_forward(x, mb["W"], mb["W_gate"], mb["gate_bias"], mb["A"], mb["B"], k, SCALE, out=mb["out"],
                                ws=ws, packed=mb["packed"])
    if kind == "composed":
        idx, w, _ = m.gate_topk(x, mb["W_gate"], mb["gate_bias"], k, ws=ws)
        m.base_gemm(x, mb["W"], out=mb["out"])
        m.lora_forward(x, mb["A"], mb["B"], idx, w, SCALE, out=mb["out"], accumulate=True, ws=ws)
        return {"out": mb["out"], "idx": idx, "w": w}
    out, idx, w = m.linear_forward(x, mb["W"], mb["W_gate"], mb["gate_bias"], mb["A"], mb["B"], k, SCALE,
                                   out=mb["out"], ws=ws, return_routing=True, packed=mb["packed"])
    dW, db, dl, dx = m.gate_backward(x, state["dy"], mb["gate_bias"], mb["B"], mb["packed"], k, SCALE,
                                     labels=state["labels"], beta=BETA, topk_idx=idx, topk_w=w, want_d_logits=True,
                                     ws=state["ws_back"], forward_ws=ws, A=mb["A"], W_gate=mb["W_gate"],
                                     W_t=state["W_t"], want_dx=True)
    return {"out": out, "dW_gate": dW, "dbias": db, "d_logits": dl, "dx": dx}


def work(case):
    """Each input read once and each output written once; of A and B what the selected adapters can be at most."""
    T, N, r, k = case["T"], case["N"], case["r"], case["k"]
    e = 4 if case.get("dtype") == "f32" else 2
    used = min(N, T * k)
    nbytes = flops = 0
    for d_in, d_outs in _widths(case):
        nbytes += T * d_in * e
        for d_out in d_outs:
            nbytes += d_out * d_in * e + d_in * N * 4 + used * r * (d_in + d_out) * e + T * d_out * e
            flops += 2 * T * d_in * (d_out + N) + 2 * T * k * r * (d_in + d_out)
            if case["kind"] == "train":
                # dy, W transposed, labels in; dx, dW_gate, dbias, d_logits out (x, A, B, W_gate counted above)
                nbytes += T * d_out * e + d_out * d_in * e + T * 4 + T * d_in * e + (d_in + 1 + T) * N * 4
                flops += 2 * T * d_in * (d_out + 2 * N) + 2 * T * k * r * (d_in + d_out)
    return {"bytes": float(nbytes), "flops": float(flops)}


def tolerance(case):
    """About four times the error of each kind against the same layer in float64: fp32 2e-7 (largest entry 1.3e-6), bf16
    2.4e-3 (largest 1.6e-2), of which the rounding of the output alone is 1.7e-3 (largest 3.9e-3)."""
    if case.get("dtype") == "f32":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 9e-3, "max": 6e-2, "differ": 1e-3}
