"""What a user of this library has it do: one MoE layer call after another, over the range of sizes it serves.

A pass is one `MoELayer.forward` (router logits where the layer has a router, top-k routing, permutation, grouped
expert FFN, shared experts, weighted sum), called eagerly or replayed from a HIP graph that the program captured once,
as decode loops do.  The layer shapes are those of the repository's benchmark; token counts run from a single
decode token to the largest prefill batch, most of them not multiples of any tile.
"""
import math

import numpy as np
import torch

import paper_2504_05897_amd as hm

# Layer shapes.  `shared` is the FFN width of the always-on shared experts together, `logits` where the routing comes
# from: "router" x . W_g inside the call, "zipf" / "hot" logits handed in (few popular experts / one expert that every
# tenth token visits).  `tokens` is the range of batch sizes the shape is served with.
SHAPES = {
    # fp32: the numerical check of a layer on a small model
    "toy": dict(dtype="f32", hidden=256, ffn=512, experts=8, top_k=2, slots=8, shared=0, logits="router", tokens=(1, 1024)),
    # few large experts
    "mixtral": dict(dtype="bf16", hidden=4096, ffn=14336, experts=8, top_k=2, slots=8, shared=0, logits="router", tokens=(1, 1024)),
    # the same with 4-bit expert weights
    "mixtral_w4": dict(dtype="w4", hidden=4096, ffn=14336, experts=8, top_k=2, slots=8, shared=0, logits="router", tokens=(1, 1024)),
    # many small experts, skewed routing
    "dsv2lite": dict(dtype="bf16", hidden=2048, ffn=1408, experts=64, top_k=6, slots=64, shared=2816, logits="zipf", tokens=(1, 4096)),
    # the same layer with room for half of its experts on the GPU, score-aware replacement
    "dsv2lite_cached": dict(dtype="bf16", hidden=2048, ffn=1408, experts=64, top_k=6, slots=32, shared=2816, logits="zipf",
                            tokens=(1, 5)),
    # many experts of medium size next to a wide shared expert
    "qwen2moe": dict(dtype="bf16", hidden=3584, ffn=2560, experts=64, top_k=8, slots=64, shared=20480, logits="hot", tokens=(1, 2048)),
    # balanced routing, for large prefill batches
    "stress": dict(dtype="bf16", hidden=2048, ffn=1408, experts=64, top_k=6, slots=64, shared=2816, logits="router",
                   tokens=(1024, 16384)),
}


def _case(shape, tokens, launch="eager", name=None):
    case = {k: v for k, v in SHAPES[shape].items() if k != "tokens"}
    case.update(tokens=tokens, launch=launch)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: a few tokens of an fp32 layer, nothing but launches and latency
        _case("toy", 16, name="toy_f32_16"),
        # one decode token, small experts: the inner step of single-stream decoding, replayed from a graph
        _case("dsv2lite", 1, "graph", name="dsv2lite_decode1"),
        # four sequences decoding with half of the experts resident: plan, staging of misses, scores for replacement
        _case("dsv2lite_cached", 4, name="dsv2lite_cached_decode4"),
        # eight sequences decoding, large experts: the weight stream is everything
        _case("mixtral", 8, "graph", name="mixtral_decode8"),
        # continuous batching at a batch size that is no power of two, called eagerly
        _case("qwen2moe", 21, name="qwen2moe_decode21"),
        # one token through 4-bit experts
        _case("mixtral_w4", 1, "graph", name="mixtral_w4_decode1"),
        # a short prompt: more rows than decode, far fewer than a full tile per expert
        _case("mixtral", 77, name="mixtral_prefill77"),
        # a medium prompt
        _case("mixtral", 512, name="mixtral_prefill512"),
        # a prompt through 4-bit experts
        _case("mixtral_w4", 301, name="mixtral_w4_prefill301"),
        # skewed routing: one expert with hundreds of rows, dozens with a handful
        _case("dsv2lite", 1003, name="dsv2lite_prefill1003"),
        # routed and shared experts of equal weight
        _case("qwen2moe", 2048, name="qwen2moe_prefill2048"),
        # the largest batch
        _case("stress", 16384, name="stress_prefill16384"),
    ]


def draw(rng):
    def between(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    shape = rng.choice(sorted(SHAPES) + ["other"])
    if shape != "other":
        case = _case(shape, between(*SHAPES[shape]["tokens"]))
    else:
        # a layer of some other model: sizes that no benchmark names
        hidden, ffn, top_k = 128 * between(8, 32), 64 * between(8, 64), rng.randint(1, 8)
        experts = min(rng.randint(top_k, 96), 4 * 10 ** 9 // (6 * hidden * ffn))
        case = dict(dtype="bf16", hidden=hidden, ffn=ffn, experts=experts, top_k=top_k, slots=experts,
                    shared=rng.choice([0, 0, ffn, 2 * ffn]), logits=rng.choice(["router", "zipf"]), tokens=between(1, 2048),
                    launch="eager")
    if case["tokens"] <= 32 and case["slots"] == case["experts"] and rng.random() < 0.5:
        case["launch"] = "graph"
    return case


_DTYPES = {"f32": (hm.HMOE_F32, torch.float32), "bf16": (hm.HMOE_BF16, torch.bfloat16), "w4": (hm.HMOE_BF16_W4, torch.bfloat16)}


def _logits(case, noise):
    """Router logits of the layers that get them from outside, out of N(0, 1) noise [tokens, experts] (numpy or torch)."""
    if case["logits"] == "zipf":
        p = [(e + 1) ** -1.1 for e in range(case["experts"])]
        for e in range(case["experts"]):
            noise[:, e] += math.log(case["experts"] * p[e] / sum(p))
    elif case["logits"] == "hot":
        noise[::10, 0] = noise[::10].max(1)[0] + 1.0 if isinstance(noise, torch.Tensor) else noise[::10].max(1) + 1.0
    return noise


def draw_weights(case, seed):
    """Expert, shared and router weights as the library takes them: numpy arrays, bfloat16 as bit patterns."""
    H, F, E, dt = case["hidden"], case["ffn"], case["experts"], _DTYPES[case["dtype"]][1]
    gen = torch.Generator(device="cuda").manual_seed(2 * seed + 1)

    def normal(n, std):
        host = torch.empty(n, dtype=dt, pin_memory=True)
        host.copy_(torch.empty(n, dtype=dt, device="cuda").normal_(0.0, std, generator=gen))
        return host.view(torch.int16).numpy().view(np.uint16) if dt == torch.bfloat16 else host.numpy()

    def swiglu(n, f):
        w = normal(n * 3 * f * H, 0.02).reshape(n, 3, f * H)
        return [(w[i, 0].reshape(f, H), w[i, 1].reshape(f, H), w[i, 2].reshape(H, f)) for i in range(n)]

    experts = swiglu(E, F)
    shared = swiglu(1, case["shared"]) if case["shared"] else []
    router = normal(E * H, H ** -0.5).reshape(E, H)
    return experts, shared, router


def draw_inputs(case, seed):
    """Token activations (normalised as a layer's input is) and, for layers that get them from outside, router logits."""
    T, H, dt = case["tokens"], case["hidden"], _DTYPES[case["dtype"]][1]
    gen = torch.Generator(device="cuda").manual_seed(2 * seed)
    x = torch.randn(T, H, device="cuda", generator=gen)
    x = (x / torch.sqrt(x.square().mean(1, keepdim=True) + 1e-5)).to(dt)
    logits = None
    if case["logits"] != "router":
        logits = _logits(case, torch.randn(T, case["experts"], device="cuda", generator=gen)).contiguous()
    return x, logits


def prepare(case, seed):
    experts, shared, router = draw_weights(case, seed)
    x, logits = draw_inputs(case, seed)
    cached = case["slots"] < case["experts"]
    desc = hm.make_desc(case["hidden"], case["ffn"], case["experts"], case["top_k"], case["slots"], _DTYPES[case["dtype"]][0])
    layer = hm.MoELayer(desc, experts, shared, router if logits is None else None, max_tokens=case["tokens"], host_copies=cached)
    state = {"layer": layer, "x": x, "logits": logits, "cached": cached, "graph": None}
    if cached:
        layer.set_policy(hm.HMOE_POLICY_MRS, 0.5)
    if case["launch"] == "graph":
        layer.forward(x, logits)
        torch.cuda.synchronize()
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            state["y"] = layer.forward(x, logits)
    torch.cuda.synchronize()
    return state


def run(state):
    if state["graph"] is not None:
        state["graph"].replay()
        return state["y"]
    y = state["layer"].forward(state["x"], state["logits"])
    if state["cached"]:
        return [y, state["layer"].update_scores(state["logits"])]
    return y


def work(case):
    T, H, F, E, K, shared = (case[k] for k in ("tokens", "hidden", "ffn", "experts", "top_k", "shared"))
    # experts that a batch of this size touches on average (each one's weights are read once)
    rng, batches = np.random.default_rng(0), 64 if T <= 256 else 4
    touched = 0.0
    for _ in range(batches):
        chosen = np.argpartition(-_logits(case, rng.standard_normal((min(T, 4096), E))), K - 1, axis=1)[:, :K]
        touched += len(np.unique(chosen)) / batches
    elem = 4 if case["dtype"] == "f32" else 2
    per_weight = 0.5 + 2 / 128 if case["dtype"] == "w4" else elem
    routing = E * H * elem if case["logits"] == "router" else T * E * 4
    return {"bytes": touched * 3 * H * F * per_weight + 3 * H * shared * per_weight + 2 * T * H * elem + routing,
            "flops": 6.0 * H * F * T * K + 6.0 * H * shared * T + (2.0 * T * H * E if case["logits"] == "router" else 0.0)}


def tolerance(case):
    # four times the error measured against an evaluation in 64 bits: 1.6e-7 in fp32, 2.84e-3 to 2.90e-3 with bfloat16
    # activations, intermediate and output (the same for every shape and for 4-bit weights, whose codes are exact)
    return {"rel": 7e-7 if case["dtype"] == "f32" else 1.15e-2}
