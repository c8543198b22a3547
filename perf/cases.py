"""The work that a user of this library has it do, as a list of measurable cases.

Three kinds of pass, all through the public entry points:
  layer   one sparse MoE feed-forward layer on T tokens (moe_forward, or moe_forward_static)
  stack   one step through a residual stack of layers (moe_stack_forward)
  stats   the routing-trace statistics of a whole sequence over all layers of a model
          (replacements, block-wise selection loss, offload counters, Delta Uniform)

listed() holds named cases over the real range; draw() gives further ones of the same ranges.
Inputs and weights are N(0, .) tensors drawn on the GPU from the seed, at the scales of
workloads/generate.py; their shapes are the benchmark's configurations, the model rows of the
paper's Table 1 and the sizes in between.
"""
import math

import torch

import paper_2503_00245_amd as moe
import workloads

DEV = "cuda:0"


def _layer(name, tokens, d, f, experts=8, top_k=2, rank=0, base=False, dtype="bf16", skew=False,
           static=False):
    c = {"kind": "layer", "tokens": tokens, "d_model": d, "d_ff": f, "experts": experts,
         "top_k": top_k, "rank": rank, "shared_base": base, "dtype": dtype, "skew": skew,
         "static": static}
    return c if name is None else dict(name=name, **c)


def _stack(name, layers, tokens, d, f, experts=8, top_k=2):
    c = {"kind": "stack", "layers": layers, "tokens": tokens, "d_model": d, "d_ff": f,
         "experts": experts, "top_k": top_k, "rank": 0, "shared_base": False, "dtype": "bf16",
         "skew": False}
    return c if name is None else dict(name=name, **c)


def _stats(name, layers, tokens, experts=8, top_k=2):
    c = {"kind": "stats", "layers": layers, "tokens": tokens, "experts": experts, "top_k": top_k}
    return c if name is None else dict(name=name, **c)


def listed():
    return [
        # the smallest call: the fp32 configuration, 32 tokens; launches and latency are all there is
        _layer("tiny_fp32_32", 32, 128, 256, experts=4, dtype="f32"),
        # one generated token through one layer of a wearables-sized model, in a serving loop that
        # owns no workspace
        _layer("wearables_decode_1", 1, 1024, 2816, static=True),
        # one generated token through one phone-sized layer: 138 MB of expert weights
        _layer("phone_decode_1", 1, 2048, 5632, skew=True),
        # a shared dense base plus rank-64 pairs, one generated token
        _layer("phone_wd_base_decode_1", 1, 2048, 5632, rank=64, base=True),
        # a token through the whole 24-layer model: what single-sample generation repeats
        _stack("phone_stack_decode_24", 24, 1, 2048, 5632),
        # a few sequences decoded together
        _layer("phone_batch_8", 8, 2048, 5632, skew=True),
        # a short prompt on a wearables-sized layer
        _layer("wearables_prefill_512", 512, 1024, 2816),
        # a prompt of odd length at the paper's own phone widths (no multiple of 64)
        _layer("paper_phone_prefill_777", 777, 1440, 3840),
        # the paper's sequence length on the phone-sized layer, loads skewed as trained routers' are
        _layer("phone_prefill_2048", 2048, 2048, 5632, skew=True),
        # the same with weight-decomposed experts (rank = half the hidden size)
        _layer("phone_wd_prefill_2048", 2048, 2048, 5632, rank=1024),
        # several prompts at once: the largest batch
        _layer("phone_prefill_16384", 16384, 2048, 5632, skew=True),
        # the routing statistics of a 2048-token sequence over the 24 layers of a model
        _stats("routing_stats_24x2048", 24, 2048),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mult8(v):
    return max(8, int(round(v / 8.0)) * 8)


def draw(rng):
    what = rng.choice(["decode", "decode", "few", "prefill", "prefill", "prefill", "fp32", "stack", "stats"])
    if what == "stats":
        experts = rng.choice([4, 8, 8, 16, 64])
        return _stats(None, rng.randint(1, 32), _log_int(rng, 64, 4096), experts,
                      min(experts, rng.choice([1, 2, 2, 4, 8])))
    if what == "fp32":
        experts = rng.choice([2, 4, 8])
        d = _mult8(_log_int(rng, 64, 512))
        return _layer(None, _log_int(rng, 1, 512), d, _mult8(d * rng.uniform(2.0, 2.75)), experts,
                      rng.choice([1, 2]), dtype="f32")
    # widths between Table 1's smallest row and the phone layer; the inner width is 8/3 to 11/4 of it
    d = _mult8(_log_int(rng, 400, 2048))
    f = _mult8(d * rng.uniform(8 / 3, 2.75))
    if what == "stack":
        return _stack(None, rng.randint(4, 24), rng.choice([1, 1, 1, 2]), d, f)
    # the ablation grid of active and total experts, mostly at the paper's 2 of 8
    experts = rng.choice([4, 8, 8, 8, 16])
    top_k = min(experts, rng.choice([1, 2, 2, 2, 4]))
    form = rng.choice(["dense", "dense", "dense", "wd", "base"])
    rank = {"dense": 0, "wd": _mult8(d / 2), "base": rng.choice([16, 64, 64, 128])}[form]
    tokens = {"decode": 1, "few": _log_int(rng, 2, 32), "prefill": _log_int(rng, 33, 8192)}[what]
    if tokens > 4096:
        top_k = min(top_k, 2)
    return _layer(None, tokens, d, f, experts, top_k, rank, form == "base",
                  skew=experts == 8 and rng.random() < 0.5, static=what == "decode" and rng.random() < 0.5)


class _Gen:
    """Tensors from one seed, made on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def normal(self, shape, std, dtype):
        return torch.empty(shape, dtype=dtype, device=DEV).normal_(0.0, std, generator=self.g)


def _weights(gen, case, down_std=0.02):
    d, f, e, r = case["d_model"], case["d_ff"], case["experts"], case["rank"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    w = {"router_w": gen.normal((e, d), 0.02, torch.float32), "router_b": None}
    if case["skew"]:  # expert loads of a Zipf(1.1) law, as the benchmark's phone layer has them
        w["router_b"] = torch.from_numpy(workloads.stored_zipf_bias("phone")).to(DEV)
    if r == 0 or case["shared_base"]:
        eb = 1 if case["shared_base"] else e
        w["w_gate"] = gen.normal((eb, f, d), 0.02, dt)
        w["w_up"] = gen.normal((eb, f, d), 0.02, dt)
        w["w_down"] = gen.normal((eb, d, f), down_std, dt)
    if r > 0:
        sigma = math.sqrt((0.005 if case["shared_base"] else 0.02) / math.sqrt(r))
        for name, shape in (("rg", (e, r, d)), ("ru", (e, r, d)), ("rd", (e, r, f)),
                            ("lg", (e, f, r)), ("lu", (e, f, r)), ("ld", (e, d, r))):
            w[name] = gen.normal(shape, sigma, dt)
    return w


def prepare(case, seed):
    gen = _Gen(seed)
    e, k, t = case["experts"], case["top_k"], case["tokens"]
    if case["kind"] == "stats":
        n = case["layers"]
        probs = torch.softmax(gen.normal((n, t, e), 1.0, torch.float32), dim=2)
        trace = torch.topk(probs, k, dim=2).indices.to(torch.int32).contiguous()
        i64 = dict(dtype=torch.int64, device=DEV)
        f64 = dict(dtype=torch.float64, device=DEV)
        return {"kind": "stats", "experts": e, "probs": probs, "trace": trace,
                "ws": torch.empty(moe.moe_bles_workspace_bytes(n, t, e), dtype=torch.uint8, device=DEV),
                "out": {"H_e": torch.empty(e, **i64), "H": torch.empty(1, **i64),
                        "bles": torch.empty(5, **f64), "changes": torch.empty(n, **i64),
                        "loads": torch.empty(n, **i64), "counts": torch.empty((n, e), **i64),
                        "delta": torch.empty(n, **f64), "mean": torch.empty(1, **f64)}}
    act = moe.MOE_F32 if case["dtype"] == "f32" else moe.MOE_BF16
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    x = gen.normal((t, case["d_model"]), 1.0, dt)
    if case["kind"] == "stack":
        n = case["layers"]
        tensors = [_weights(gen, case, 0.02 / math.sqrt(2 * n)) for _ in range(n)]
        shape = moe.shape_for(tensors[0], t, k, act)
        trace = torch.empty((n, t, k), dtype=torch.int32, device=DEV)
        return {"kind": "stack", "shape": shape, "tensors": tensors, "x": x,
                "layers": [moe.make_weights(w) for w in tensors],
                "ws": moe.alloc_workspace(shape, DEV), "out": {"y": torch.empty_like(x), "trace": trace}}
    tensors = _weights(gen, case)
    shape = moe.shape_for(tensors, t, k, act)
    return {"kind": "layer", "shape": shape, "tensors": tensors, "weights": moe.make_weights(tensors), "x": x,
            "ws": None if case["static"] else moe.alloc_workspace(shape, DEV),
            "out": {"y": torch.empty_like(x),
                    "topk_idx": torch.empty((t, k), dtype=torch.int32, device=DEV),
                    "topk_gate": torch.empty((t, k), dtype=torch.float32, device=DEV)}}


def run(state):
    out = state["out"]
    if state["kind"] == "stats":
        trace, e = state["trace"], state["experts"]
        moe.moe_expert_replacements(trace, e, out["H_e"], out["H"])
        moe.moe_bles_loss(state["probs"], trace, out["bles"], state["ws"])
        moe.moe_offload_counters(trace, e, out["changes"], out["loads"])
        moe.moe_delta_uniform(trace, e, out["counts"], out["delta"], out["mean"])
    elif state["kind"] == "stack":
        moe.moe_stack_forward(state["shape"], state["layers"], state["x"], out["y"], out["trace"], state["ws"])
    elif state["ws"] is None:
        moe.moe_forward_static(state["shape"], state["weights"], state["x"], out["y"], out["topk_idx"],
                               out["topk_gate"])
    else:
        moe.moe_forward(state["shape"], state["weights"], state["x"], out["y"], out["topk_idx"],
                        out["topk_gate"], state["ws"])
    return out


def work(case):
    """Bytes: every input once (of the experts only those that tokens select, in expectation for even
    routing), every output once.  Flops: the products of the selected experts; a shared base meets
    a token once, not once per selected expert."""
    e, k, t = case["experts"], case["top_k"], case["tokens"]
    if case["kind"] == "stats":
        n = case["layers"]
        return {"bytes": 4.0 * n * t * (k + e) + 8.0 * (e + 1 + 5 + 2 * n + n * e + n + 1), "flops": 2.0 * n * t * e}
    d, f, r, base = case["d_model"], case["d_ff"], case["rank"], case["shared_base"]
    es = 4 if case["dtype"] == "f32" else 2
    layers = case.get("layers", 1)
    hit = e * (1.0 - (1.0 - k / e) ** t)
    per_expert = 3.0 * r * (d + f) if r else 3.0 * d * f
    weights = hit * per_expert + (3.0 * d * f if base else 0.0)
    flops = 2.0 * t * k * per_expert + (6.0 * t * d * f if base else 0.0) + 2.0 * t * e * d
    byts = es * weights + 4.0 * e * d + (4.0 if case["kind"] == "stack" else 8.0) * t * k
    return {"bytes": layers * byts + 2.0 * es * t * d, "flops": layers * flops}


def tolerance(case):
    if case["kind"] == "stats":  # counts are whole; the soft part is a sum of 32-bit differences
        return {"rel": 1e-5, "max": 1e-5}
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    # bf16 storage of the hidden vectors and outputs; a token whose k-th and (k+1)-th logits differ by
    # less than the rounding of a 32-bit sum may pick either
    return {"rel": 1e-2, "max": 0.1, "differ": 0.002}
