"""The calls whose speed this library is held to: causal forward, backward and decode.

(The conjugate-gradient mode is left out: its iterates beyond the second step are unstable under rounding, so that two
correct implementations return results that cannot be compared.)

A case is a dict of plain values:
  op      "forward" | "backward" | "decode"
  B, H    batch and heads
  n       sequence length, or the capacity of the key/value cache (decode)
  d       head dimension, one of 16, 32, 64, 128
  dtype   "bf16" | "f32", of the inputs; results are float32 unless "out" says otherwise
  values  "normal"      Q, K, V ~ N(0, 1)
          "unit"        the same with the rows of Q and K normalised to length 1
          "regression"  V = K A^T + 0.1 noise with one random d x d map per head
  train   forward only: a ridge per row is given, and the row statistics rho and delta are returned for a backward pass
  ragged  decode only: every sequence has a length of its own, between an eighth of the capacity and all of it
  out     "f32" | "bf16", type of the result (forward and decode)
Every call uses the ridge 1e-2 and the scale 1/sqrt(d).
"""
import math

import torch

import paper_2510_01450_amd as llla

LAMBDA = 1e-2
TYPES = {"f32": torch.float32, "bf16": torch.bfloat16}


def _case(op, B, H, n, d, dtype, values="normal", train=False, ragged=False, out="f32", name=None):
    case = {"op": op, "B": B, "H": H, "n": n, "d": d, "dtype": dtype, "values": values, "train": train, "ragged": ragged,
            "out": out}
    if name is not None:
        case["name"] = name
    return case


def listed():
    return [
        # one short sequence in fp32: an interactive call, all of it latency
        _case("forward", 1, 1, 128, 16, "f32", "unit", name="forward_tiny_f32"),
        # an fp32 model's attention layer at a usual context
        _case("forward", 2, 8, 1024, 64, "f32", "unit", name="forward_f32"),
        # prefill of a batch of prompts, the throughput configuration
        _case("forward", 4, 16, 4096, 64, "bf16", name="forward_prefill"),
        # prefill of one long prompt at the larger head dimension
        _case("forward", 1, 16, 8192, 128, "bf16", "regression", name="forward_long_d128"),
        # the forward half of a training step: many sequences of odd length, a learned ridge, statistics kept
        _case("forward", 8, 12, 1000, 64, "bf16", train=True, out="bf16", name="forward_train_odd"),
        # the backward half of a training step at the prefill shape
        _case("backward", 4, 16, 4096, 64, "bf16", name="backward_prefill"),
        # the backward of the fp32 layer above
        _case("backward", 2, 8, 1024, 64, "f32", "unit", name="backward_f32"),
        # one generated token of a single conversation
        _case("decode", 1, 16, 4096, 64, "bf16", name="decode_single"),
        # one generated token of a full serving batch, all caches full
        _case("decode", 32, 16, 32768, 64, "bf16", name="decode_batch"),
        # a serving batch of conversations of different lengths at the larger head dimension
        _case("decode", 16, 16, 16384, 128, "bf16", ragged=True, out="bf16", name="decode_ragged_d128"),
        # the same for an fp32 model
        _case("decode", 4, 16, 8192, 64, "f32", "unit", ragged=True, name="decode_ragged_f32"),
        # a model with many small heads
        _case("decode", 8, 32, 4096, 32, "bf16", name="decode_small_heads"),
    ]


def _between(rng, low, high):
    """A whole number, uniform in its logarithm."""
    return max(low, min(high, int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))))


def draw(rng):
    op = rng.choice(["forward", "forward", "backward", "decode", "decode"])
    dtype = rng.choice(["bf16", "bf16", "f32"])
    d = rng.choice([64, 64, 64, 128, 128, 32, 32, 16])
    H = rng.choice([1, 4, 8, 12, 16])
    if op == "decode":
        n = _between(rng, 100, 32768)
        # keys of all sequences and heads together: at most those of the largest listed decode, fewer in fp32
        most = (1 << 24 if dtype == "bf16" else 1 << 21) * 64 // max(d, 64)
        B = _between(rng, 1, max(1, min(64, most // (H * n))))
    else:
        # query-key pairs times d^2, at most those of the listed cases (fp32 at d = 128: a quarter of them)
        if dtype == "bf16":
            longest, most = (8192, 8.9e12) if op == "forward" else (4096, 2.2e12)
        else:
            longest, most = 2048, 3.4e10 if d <= 64 else 0.85e10
        per_row = H * max(d, 64) ** 2 / 2
        # a gradient with respect to the ridge means little before the rows see more keys than features
        n = _between(rng, 2 * d if op == "backward" else 33, min(longest, int(math.sqrt(most / per_row))))
        B = _between(rng, 1, max(1, min(32, int(most / (per_row * n * n)))))
    values = "unit" if dtype == "f32" else rng.choice(["normal", "normal", "regression"])
    return _case(op, B, H, n, d, dtype, values, train=op == "forward" and rng.random() < 0.4,
                 ragged=op == "decode" and rng.random() < 0.5,
                 out=rng.choice(["f32", "bf16"]) if op in ("forward", "decode") and dtype == "bf16" else "f32")


def _normal(gen, shape, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def prepare(case, seed):
    """The tensors a program holds before the call.  A serving loop also keeps its scratch and result buffers."""
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    dt = TYPES[case["dtype"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    decode = case["op"] == "decode"
    Q = _normal(gen, (B, H, d) if decode else (B, H, n, d), dt)
    K = _normal(gen, (B, H, n, d), dt)
    V = _normal(gen, (B, H, n, d), dt)
    if case["values"] == "unit":
        Q = Q / Q.norm(dim=-1, keepdim=True)
        K = K / K.norm(dim=-1, keepdim=True)
    elif case["values"] == "regression":
        for b in range(B):
            for h in range(H):
                A = _normal(gen, (d, d), torch.float32) / math.sqrt(d)
                V[b, h] = (torch.mm(K[b, h].float(), A) + 0.1 * V[b, h].float()).to(dt)
    s = {"case": case, "Q": Q, "K": K, "V": V, "scale": 1.0 / math.sqrt(d)}
    if decode:
        s["lens"] = None
        if case["ragged"]:
            lens = torch.randint(max(1, n // 8), n + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
            lens[B - 1] = n
            s["lens"] = lens
        s["ws"] = torch.empty(max(256, llla.decode_workspace_bytes(B, H, n, d, dt)), dtype=torch.uint8, device="cuda")
        s["O"] = torch.empty((B, H, d), dtype=TYPES[case["out"]], device="cuda")
    if case["op"] == "backward":
        s["dO"] = _normal(gen, (B, H, n, d), dt)
    if case["train"]:
        s["ridge"] = LAMBDA * torch.exp(0.5 * _normal(gen, (B, H, n), torch.float32))
    return s


def run(s):
    case = s["case"]
    if case["op"] == "decode":
        return llla.llla_decode(s["Q"], s["K"], s["V"], LAMBDA, s["scale"], seqlens=s["lens"], workspace=s["ws"], out=s["O"])
    if case["op"] == "backward":
        return llla.llla_backward(s["Q"], s["K"], s["V"], s["dO"], LAMBDA, s["scale"], return_dlambda=True)
    return llla.llla_forward(s["Q"], s["K"], s["V"], s["ridge"] if case["train"] else LAMBDA, s["scale"],
                             out_dtype=TYPES[case["out"]], return_stats=case["train"])


def work(case):
    """Bytes of the inputs and outputs; multiply-adds counted as two flops.  Per query-key pair the logit (2d), the symmetric
    half of the second moment (d^2 + d), the first moment (2d), the output weight and its product with the value (6d), as
    d^2 + 11d; per query the factorisation and the substitutions of its d x d system."""
    B, H, n, d = case["B"], case["H"], case["n"], case["d"]
    e = 2 if case["dtype"] == "bf16" else 4
    o = 2 if case["out"] == "bf16" else 4
    heads = B * H
    if case["op"] == "decode":
        keys = n * (9 / 16 if case["ragged"] else 1.0)             # mean length of a ragged batch
        return {"bytes": heads * (2 * keys * d * e + d * (e + o)), "flops": heads * (keys * (d * d + 11 * d) + d ** 3 / 3 + 4 * d * d)}
    rows, pairs = heads * n, heads * n * (n + 1) / 2
    if case["op"] == "backward":
        # the forward's moments with a second right-hand side, then the sums over pairs behind dQ, dK and dV
        return {"bytes": rows * (4 * d * e + 3 * d * 4 + 4), "flops": pairs * (d * d + 23 * d) + rows * (d ** 3 / 3 + 8 * d * d)}
    extra = rows * (4 * d + 8) if case["train"] else 0
    return {"bytes": rows * d * (3 * e + o) + extra, "flops": pairs * (d * d + 11 * d) + rows * (d ** 3 / 3 + 4 * d * d)}


def tolerance(case):
    """Four times the largest error seen against the fp64 oracle (one head per case, five dozen drawn cases).  Rows that see
    few keys have badly conditioned systems, so short sequences get more."""
    d, decode = case["d"], case["op"] == "decode"
    n = case["n"] // 8 if case["ragged"] else case["n"]            # the shortest sequence
    if case["op"] == "backward":
        # worst of the four gradients, that of the ridge; one more factor of the condition number than the forward
        # fp32 seen: 3.6e-5;  bf16 seen: 1.1e-2 below 16d rows and with values that are nearly a linear map, 1.8e-3 otherwise
        if case["dtype"] == "f32":
            return {"rel": 2e-4}
        return {"rel": 4e-2 if n < 16 * d or case["values"] == "regression" else 8e-3}
    if case["out"] == "bf16":
        return {"rel": 6e-3}                                       # seen: 1.75e-3, the rounding of the result
    if case["dtype"] == "f32" or (decode and d < 64):
        return {"rel": 5e-5 if n < 8 * d else 1e-5}                # seen: 1.1e-5 and 2.0e-6
    return {"rel": 4e-3 if n < 8 * d else 1.2e-3}                  # seen: 1.0e-3 and 2.8e-4 (weights as 16-bit floats)
