"""The calls whose speed counts: power attention as a program uses it, from one small float32 layer to the long
training step, through the public entry points of the package.

Inputs follow the recipe of paper_2507_04239_amd/inputs.py (q, k ~ N(0,1) d^-1/2; v, dY ~ N(0,1); log-gates
-0.02 Exp(1)), drawn on the GPU from the seed.  Sizes are the benchmark's configurations (inputs.WORKLOADS and
EXTRA_WORKLOADS) or generic ones beside them.

A case is a dict:
  kind      "fwd" forward pass, "train" forward + backward, "prompt" forward pass of a prompt and its hand-over into a
            decode state, "decode" one token for every sequence
  B, H, T, d, p, chunk (0: the library chooses), dtype, normalize, gated, keep (chunk states kept for the backward pass)
"""
import math

import torch

from paper_2507_04239_amd import binding, power_attn_bwd, power_attn_fwd

DECAY = 0.02      # mean log-gate
CONTEXT = 256     # tokens a decode state holds before the step


def _case(name, kind, B, H, T, d, p=2, chunk=0, dtype="bf16", normalize=True, gated=False, keep=False):
    c = dict(kind=kind, B=B, H=H, T=T, d=d, p=p, chunk=chunk, dtype=dtype, normalize=normalize, gated=gated, keep=keep)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # one small float32 layer: what a test or a first experiment calls; launches and latency
        _case("fwd_f32_T256_d16", "fwd", 1, 1, 256, 16, chunk=32, dtype="f32"),
        # a small model trained in float32
        _case("train_f32_T1024_d32", "train", 2, 4, 1024, 32, dtype="f32"),
        # scoring / prefill of a batch of documents in bf16
        _case("fwd_T8192_d64", "fwd", 4, 12, 8192, 64, chunk=128),
        # the long-context training step, the benchmark's headline
        _case("train_T65536_d64", "train", 1, 12, 65536, 64, chunk=128, keep=True),
        # the gated layer, states rebuilt in the backward pass (activation memory is what is short)
        _case("train_gated_T16384_d64", "train", 1, 12, 16384, 64, gated=True),
        # ordinary context lengths that are no round number: batches of padded text
        _case("train_T1000_d64", "train", 16, 12, 1000, 64),
        # degree 4, the large-state degree
        _case("train_p4_T16384_d32", "train", 2, 8, 16384, 32, p=4),
        # odd degree, un-normalised
        _case("train_p3_T16384_d64", "train", 1, 4, 16384, 64, p=3, normalize=False),
        # widest heads, the largest case (a quarter of the benchmark's batch, so that three sets of inputs fit)
        _case("train_T32768_d128", "train", 2, 16, 32768, 128, chunk=256, keep=True),
        # serving: prompts come in, of any length, and go on to be decoded
        _case("prompt_T3000_d64", "prompt", 4, 12, 3000, 64),
        # serving: one token for a batch of sequences, and for a single one
        _case("decode_B64_d64", "decode", 64, 12, 1, 64),
        _case("decode_B1_d64", "decode", 1, 12, 1, 64),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _length(rng, lo, hi):
    """Lengths over the whole range: round ones, multiples of 128 and odd ones alike."""
    t = _log(rng, lo, hi)
    r = rng.random()
    if r < 0.3:
        return max(lo, min(hi, 1 << round(math.log2(t))))
    if r < 0.6:
        return max(128, 128 * round(t / 128))
    return int(t)


def _heads(rng, T, most_tokens, most_heads=64):
    """(B, H) with B H T near what the range allows, or well below it."""
    bh = max(1, min(most_heads, int(most_tokens / T)))
    bh = max(1, int(_log(rng, max(1, bh / 8), bh)))
    H = rng.choice([h for h in (1, 2, 4, 8, 12, 16) if h <= bh])
    return max(1, bh // H), H


def draw(rng):
    kind = rng.choice(["fwd_f32", "train_f32", "fwd", "train", "train", "train_gated", "train_short", "train_degree",
                       "train_wide", "prompt", "decode", "decode"])
    if kind == "fwd_f32":
        T = 32 * round(_log(rng, 4, 128))
        B, H = _heads(rng, T, 16384, 16)
        return _case(None, "fwd", B, H, T, rng.choice([16, 32, 64]), chunk=rng.choice([0, 32]), dtype="f32")
    if kind == "train_f32":
        T = 32 * round(_log(rng, 4, 64))
        B, H = _heads(rng, T, 8192, 16)
        return _case(None, "train", B, H, T, rng.choice([16, 32, 64]), chunk=rng.choice([0, 32]), dtype="f32")
    if kind == "fwd":
        T = _length(rng, 512, 65536)
        B, H = _heads(rng, T, 786432)
        return _case(None, "fwd", B, H, T, 64, chunk=rng.choice([0, 128, 256]))
    if kind == "train":
        T = _length(rng, 4097, 131072)
        B, H = _heads(rng, T, 786432)
        return _case(None, "train", B, H, T, 64, chunk=rng.choice([0, 128, 256]), normalize=rng.random() < 0.8, keep=rng.random() < 0.5)
    if kind == "train_gated":
        T = _length(rng, 1024, 32768)
        B, H = _heads(rng, T, 393216)
        return _case(None, "train", B, H, T, 64, chunk=rng.choice([0, 0, 128]), gated=True, keep=rng.random() < 0.5)
    if kind == "train_short":
        T = _length(rng, 128, 4096)
        B, H = _heads(rng, T, 196608, 256)
        return _case(None, "train", B, H, T, rng.choice([32, 64, 64, 128]))
    if kind == "train_degree":
        T = _length(rng, 512, 16384)
        B, H = _heads(rng, T, 262144)
        p, d = rng.choice([(3, 32), (3, 64), (4, 32), (4, 32), (4, 64), (3, 128)])
        return _case(None, "train", B, H, T, d, p=p, normalize=p % 2 == 0)
    if kind == "train_wide":
        T = _length(rng, 2048, 32768)
        B, H = _heads(rng, T, 1048576)
        return _case(None, "train", B, H, T, 128, chunk=rng.choice([0, 128, 256]), keep=rng.random() < 0.5)
    if kind == "prompt":
        T = _length(rng, 100, 8192)
        B, H = _heads(rng, T, 262144)
        return _case(None, "prompt", B, H, T, 64, gated=rng.random() < 0.25)
    B = max(1, int(_log(rng, 1, 128)))
    d, p = rng.choice([(64, 2), (64, 2), (128, 2), (32, 4)])
    return _case(None, "decode", B if (d, p) == (64, 2) else max(1, B // 4), rng.choice([4, 8, 12]), 1, d, p=p, gated=rng.random() < 0.25)


class _Inputs:
    """q, k, v, dY and the log-gates of a case, made on the GPU from the seed alone."""

    def __init__(self, case, seed, T=None):
        dev = torch.device("cuda:0")
        gen = torch.Generator(device=dev)
        gen.manual_seed(int(seed))
        B, H, d = case["B"], case["H"], case["d"]
        T = case["T"] if T is None else T
        dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

        def normal(scale=1.0):
            return (torch.randn((B, H, T, d), device=dev, generator=gen) * scale).to(dt)

        self.q, self.k, self.v = normal(d ** -0.5), normal(d ** -0.5), normal()
        self.dO = normal() if case["kind"] == "train" else None
        self.log_g = None
        if case["gated"]:
            self.log_g = -DECAY * torch.empty((B, H, T), device=dev).exponential_(1.0, generator=gen)


def _problem(case, T, keep=False, chunk=1):
    return binding.make_problem(case["B"], case["H"], T, case["d"], case["d"], case["p"], chunk, case["normalize"], 1.0, case["dtype"],
                                "auto", keep, case["gated"])


def _state_views(case, state):
    """The float32 sums inside a decode state: the value part and the normaliser column (each padded to 256 bytes)."""
    n = case["B"] * case["H"] * math.comb(case["d"] + case["p"] - 1, case["p"])
    words, at = state.view(torch.float32), (n * case["d"] + 63) // 64 * 64
    return words[: n * case["d"]], words[at: at + n]


def prepare(case, seed):
    s = {"case": case}
    if case["kind"] == "decode":
        # a session that already holds CONTEXT tokens, and the next token's projections
        past = _Inputs(case, seed, CONTEXT)
        s["state"] = binding.power_attn_decode_init(_problem(case, 1))
        binding.power_attn_decode_absorb(_problem(case, CONTEXT), past.k, past.v, s["state"], past.log_g)
        now = _Inputs(case, seed + 7919, 1)
        s.update(prob=_problem(case, 1), q=now.q[:, :, 0].contiguous(), k=now.k[:, :, 0].contiguous(), v=now.v[:, :, 0].contiguous(),
                 log_g=None if now.log_g is None else now.log_g[:, :, 0].contiguous(), sums=_state_views(case, s["state"]))
        return s
    s["x"] = _Inputs(case, seed)
    if case["kind"] == "prompt":
        s.update(prob=_problem(case, case["T"]), prob1=_problem(case, 1))
        s["state"] = binding.power_attn_decode_init(s["prob1"])
        s["sums"] = _state_views(case, s["state"])
    s["ws"] = None
    if case["keep"]:
        need = binding.power_attn_workspace_bytes(_problem(case, case["T"], True, case["chunk"]), True)
        s["ws"] = torch.empty(max(need, 256), dtype=torch.uint8, device="cuda:0")
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "decode":
        o, z = binding.power_attn_decode_step(s["prob"], s["q"], s["k"], s["v"], s["state"], s["log_g"])
        return {"o": o, "z": z, "state": s["sums"]}
    x = s["x"]
    O, Z = power_attn_fwd(x.q, x.k, x.v, c["p"], c["chunk"], normalize=c["normalize"], workspace=s["ws"], keep_state=c["keep"], log_g=x.log_g)
    if c["kind"] == "fwd":
        return {"O": O, "Z": Z}
    if c["kind"] == "prompt":
        binding.power_attn_decode_init(s["prob1"], s["state"])
        binding.power_attn_decode_absorb(s["prob"], x.k, x.v, s["state"], x.log_g)
        return {"O": O, "Z": Z, "state": s["sums"]}
    grads = power_attn_bwd(x.q, x.k, x.v, O, Z, x.dO, c["p"], c["chunk"], normalize=c["normalize"], workspace=s["ws"], keep_state=c["keep"],
                           log_g=x.log_g)
    return {"O": O, "Z": Z, "grads": grads}


def _flops(case, backward):
    """Multiply-adds (x 2) of the cheaper evaluation per head: the attention form, or the chunked form at its best chunk
    with the symmetric state of C(d+p-1, p) rows."""
    T, d, p = case["T"], case["d"], case["p"]
    D = math.comb(d + p - 1, p)
    pair = 2 * (2 * d + 1) + (2 * 5 * d if backward else 0)        # S, PV, Z; then S, E, dQ, dK, dV
    state = 2 * D * (d + 1) * (6 if backward else 2)               # update and read-out; then R, dQ, dK, dV
    best = pair * T * (T + 1) / 2
    c = 16
    while c < T:
        best = min(best, pair * T * (c + 1) / 2 + state * (T - c))
        c *= 2
    return best


def work(case):
    B, H, T, d, p = case["B"], case["H"], case["T"], case["d"], case["p"]
    e = 2 if case["dtype"] == "bf16" else 4
    D = math.comb(d + p - 1, p)
    gate = 4 * B * H * T if case["gated"] else 0
    if case["kind"] == "decode":      # the state read and written once; q, k, v in, o, z out
        return {"bytes": B * H * (2 * D * (d + 1) * 4 + 4 * d * e + 4) + gate, "flops": B * H * 4 * D * (d + 1)}
    tok = B * H * T * d * e
    if case["kind"] == "train":       # q, k, v, dO in; O, Z, dQ, dK, dV out
        return {"bytes": 8 * tok + 4 * B * H * T + 2 * gate, "flops": B * H * _flops(case, True)}
    w = {"bytes": 4 * tok + 4 * B * H * T + gate, "flops": B * H * _flops(case, False)}
    if case["kind"] == "prompt":      # and the state written once, its sums formed once
        w["bytes"] += B * H * D * (d + 1) * 4
        w["flops"] += B * H * 2 * D * (d + 1) * T
    return w


def tolerance(case):
    # Measured against the definition in float64 on the GPU: float32 at most 8e-7; bf16 2e-3 .. 4e-3 per output, 5e-3 for
    # the gradient of the log-gates, 2.4e-3 for a state whose sums are rounded to bf16 once.  A decode step's float32 sums
    # are within 6e-8; its bf16 output may round to the other neighbour where two orders of summation meet a tie.
    if case["kind"] == "decode":
        return {"rel": 5e-4}
    return {"rel": 5e-6} if case["dtype"] == "f32" else {"rel": 1.5e-2}
