"""The work a user has this library do, as a list of timed cases and a generator of more of them.

Every case is one pass of a BERT-shaped encoder layer's four linears (or of the embedding table, or of a whole model's
weights) through the public calls of `paper_1909_05840_amd`:

  infer    serving with weights quantized beforehand: per linear the activation quantizer and the integer forward
  ffn_q8   the feed-forward pair in an all-integer chain: the up projection leaves 8-bit codes (GELU inside), the down
           projection takes them
  dyn      serving without calibration: one activation range per token, asymmetric weight ranges
  train    one quantization-aware training step of a layer: weights re-quantized from fp32, forward, straight-through
           backward (dX and dW); `masked` keeps the clamp's derivative
  sweep    the headline benchmark's step: the four linears at every weight width, each stage as one batched call
  requant  all matrices of a model re-quantized from their fp32 masters in one call, a width per layer
  embed    the embedding table quantized, then a batch of token ids looked up

Sizes: `hidden` h gives the linears (3h, h), (h, h), (4h, h), (h, 4h); 768 and 1024 are BERT-base and BERT-large.
"""
import torch

import paper_1909_05840_amd as qb

CLIP = 6.0  # static activation range, six standard deviations of the synthetic activations


def listed():
    return [
        # a few tokens of one short request: launches and host work count
        {"name": "infer_8tok_4bit", "kind": "infer", "tokens": 8, "hidden": 768, "bits": 4},
        # one question-answering sequence of odd length
        {"name": "infer_390tok_8bit", "kind": "infer", "tokens": 390, "hidden": 768, "bits": 8},
        # a batch of 32 sequences of 128 tokens
        {"name": "infer_4096tok_4bit", "kind": "infer", "tokens": 4096, "hidden": 768, "bits": 4},
        # offline scoring with BERT-large: 64 sequences of 512 tokens
        {"name": "infer_32768tok_2bit_large", "kind": "infer", "tokens": 32768, "hidden": 1024, "bits": 2},
        # the same batch of 4096 tokens, activations kept in 8 bits between the two feed-forward linears
        {"name": "ffn_q8_4096tok_4bit", "kind": "ffn_q8", "tokens": 4096, "hidden": 768, "bits": 4},
        # a padding-free batch of ragged length, no calibrated ranges
        {"name": "dyn_1499tok_4bit", "kind": "dyn", "tokens": 1499, "hidden": 768, "bits": 4},
        # fine-tuning step, 32 x 128 tokens
        {"name": "train_4096tok_3bit", "kind": "train", "tokens": 4096, "hidden": 768, "bits": 3, "masked": False},
        # fine-tuning step, 32 x 384 tokens
        {"name": "train_12288tok_8bit", "kind": "train", "tokens": 12288, "hidden": 768, "bits": 8, "masked": False},
        # a narrow model with a width that is no multiple of a tile, a ragged batch, clamp-masked gradients
        {"name": "train_masked_1001tok_4bit", "kind": "train", "tokens": 1001, "hidden": 448, "bits": 4, "masked": True},
        # the headline benchmark: one layer, widths 2, 3, 4 and 8, batched calls
        {"name": "sweep_4096tok", "kind": "sweep", "tokens": 4096, "hidden": 768},
        # the weights of 12 layers at mixed widths
        {"name": "requant_12layers", "kind": "requant", "layers": 12, "hidden": 768},
        # BERT-large's 8-bit word embedding and a batch of 64 x 512 token ids
        {"name": "embed_30522x1024_8bit", "kind": "embed", "vocab": 30522, "hidden": 1024, "bits": 8, "ids": 32768},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["infer", "infer", "infer", "ffn_q8", "dyn", "train", "train", "sweep", "requant", "embed"])
    hidden = rng.choice([768, 768, 1024, 64 * rng.randint(4, 15)])
    bits = rng.choice([2, 3, 4, 8])
    if kind == "infer":
        return {"kind": kind, "tokens": _log_int(rng, 1, 32768), "hidden": hidden, "bits": bits}
    if kind == "ffn_q8":  # the 8-bit output takes input widths that are multiples of 128
        return {"kind": kind, "tokens": _log_int(rng, 64, 16384), "hidden": max(256, hidden // 128 * 128), "bits": bits}
    if kind == "dyn":
        return {"kind": kind, "tokens": _log_int(rng, 16, 16384), "hidden": hidden, "bits": bits}
    if kind == "train":
        most = int(12288 * (768 / max(hidden, 768)) ** 2)
        return {"kind": kind, "tokens": _log_int(rng, 256, most), "hidden": hidden, "bits": bits, "masked": rng.random() < 0.3}
    if kind == "sweep":
        return {"kind": kind, "tokens": _log_int(rng, 128, 6144), "hidden": min(hidden, 768)}
    if kind == "requant":
        return {"kind": kind, "layers": rng.randint(1, 12), "hidden": hidden}
    return {"kind": kind, "vocab": _log_int(rng, 512, 30522), "hidden": hidden, "bits": rng.choice([4, 8]), "ids": _log_int(rng, 128, 32768)}


def _linears(hidden):
    """(output neurons, input features) of QKV, attention output, feed-forward up and down"""
    return [(3 * hidden, hidden), (hidden, hidden), (4 * hidden, hidden), (hidden, 4 * hidden)]


def _groups(hidden):
    return 128 if hidden % 128 == 0 else 64


def _layer_bits(layers):
    """a fixed mixed-precision assignment: sensitive layers in the middle get more bits"""
    return [(2, 2, 3, 4, 8, 4, 3, 3, 4, 2, 3, 2)[i % 12] for i in range(layers)]


class _Draw:
    """tensors on the GPU from one seeded generator, with the distributions of the benchmark's synthetic inputs"""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32).mul_(std)

    def weight(self, n, k):  # 0.1 % outliers
        w = self.normal(n, k, std=0.04)
        return torch.where(torch.rand(n, k, generator=self.g, device="cuda") < 0.001, w * 10.0, w)


def prepare(case, seed):
    rnd = _Draw(seed)
    kind, hidden = case["kind"], case["hidden"]
    s = dict(case)
    if kind == "embed":
        s["E"] = rnd.normal(case["vocab"], hidden, std=0.02)
        s["token_ids"] = torch.randint(0, case["vocab"], (case["ids"],), generator=rnd.g, device="cuda", dtype=torch.int64)
        return s
    groups = s["groups"] = _groups(hidden)
    lin = _linears(hidden)
    if kind == "requant":  # the model's quantized weights live in flat buffers, allocated once
        jobs, at = [], {"packed": 0, "h": 0, "rs_w": 0}
        for b in _layer_bits(case["layers"]):
            for n, k in lin:
                jobs.append({"W": rnd.weight(n, k), "bits": b, "groups": groups, "at": dict(at), "size": (qb.qb_packed_nbytes(n, k, b), groups, n)})
                at["packed"] += qb.qb_packed_nbytes(n, k, b)
                at["h"] += groups
                at["rs_w"] += n
        flat = {"packed": torch.empty(at["packed"], dtype=torch.uint8, device="cuda"), "h": torch.empty(at["h"], device="cuda"),
                "m": torch.empty(at["h"], device="cuda"), "rs_w": torch.empty(at["rs_w"], dtype=torch.int32, device="cuda")}
        for j in jobs:
            where, (np_, ng, nn) = j.pop("at"), j.pop("size")
            j["packed"] = flat["packed"][where["packed"]:where["packed"] + np_]
            j["h"], j["m"] = (flat[f][where["h"]:where["h"] + ng] for f in ("h", "m"))
            j["rs_w"] = flat["rs_w"][where["rs_w"]:where["rs_w"] + nn]
        s["jobs"], s["flat"] = jobs, flat
        return s
    T = case["tokens"]
    if kind == "sweep":  # all buffers are kept from step to step
        s["act"] = [{"X": rnd.normal(T, k), "clip": CLIP, "Xq": torch.empty(T, k, dtype=torch.int8, device="cuda"),
                     "rs_x": torch.empty(T, dtype=torch.int32, device="cuda")} for _, k in lin]
        s["quant"], s["fwd"] = [], []
        for b in (2, 3, 4, 8):
            for i, (n, k) in enumerate(lin):
                q = {"W": rnd.weight(n, k), "bits": b, "groups": groups, "packed": torch.empty(qb.qb_packed_nbytes(n, k, b), dtype=torch.uint8, device="cuda"),
                     "h": torch.empty(groups, device="cuda"), "m": torch.empty(groups, device="cuda"), "rs_w": torch.empty(n, dtype=torch.int32, device="cuda")}
                a = s["act"][i]
                s["quant"].append(q)
                s["fwd"].append({"Xq": a["Xq"], "rs_x": a["rs_x"], "clip": CLIP, "packed": q["packed"], "h": q["h"], "rs_w": q["rs_w"], "bits": b,
                                 "groups": groups, "N": n, "Y": torch.empty(T, n, device="cuda")})
        return s
    s["N"] = [n for n, _ in lin]
    if kind == "ffn_q8":
        lin = lin[2:]
        s["N"] = s["N"][2:]
        s["X"] = rnd.normal(T, hidden)
    else:
        s["X"] = [rnd.normal(T, k) for _, k in lin]
    W = [rnd.weight(n, k) for n, k in lin]
    if kind == "train":
        s["W"] = W
        s["dY"] = [rnd.normal(T, n, std=1e-2).to(torch.bfloat16) for n, _ in lin]
        return s
    s["bias"] = [rnd.normal(n, std=0.1) for n, _ in lin]
    quantize = qb.qb_quantize_groupwise_asym if kind == "dyn" else qb.qb_quantize_groupwise
    s["weights"] = [quantize(w, case["bits"], groups) for w in W]
    return s


def run(s):
    kind = s["kind"]
    if kind == "infer":
        out = []
        for X, (packed, h, _, rs_w), n, bias in zip(s["X"], s["weights"], s["N"], s["bias"]):
            Xq, rs_x = qb.qb_quantize_act(X, CLIP)
            out.append(qb.qb_qlinear_fwd(Xq, rs_x, CLIP, packed, h, rs_w, s["bits"], s["groups"], n, bias=bias))
        return out
    if kind == "ffn_q8":
        (pu, hu, _, ru), (pd, hd, _, rd) = s["weights"]
        Xq, rs_x = qb.qb_quantize_act(s["X"], CLIP)
        Uq, rs_u = qb.qb_qlinear_fwd_q8(Xq, rs_x, CLIP, pu, hu, ru, s["bits"], s["groups"], s["N"][0], CLIP, bias=s["bias"][0], act=1)
        Y = qb.qb_qlinear_fwd(Uq, rs_u, CLIP, pd, hd, rd, s["bits"], s["groups"], s["N"][1], bias=s["bias"][1])
        return Uq, rs_u, Y
    if kind == "dyn":
        out = []
        for X, (packed, delta, q0, rs_w), n, bias in zip(s["X"], s["weights"], s["N"], s["bias"]):
            Xq, rs_x, hx = qb.qb_quantize_act_dyn(X)
            out.append(qb.qb_qlinear_fwd_asym_dyn(Xq, rs_x, hx, packed, delta, q0, rs_w, s["bits"], s["groups"], n, bias=bias))
        return out
    if kind == "train":
        bits, groups = s["bits"], s["groups"]
        weights = qb.qb_quantize_groupwise_batched([{"W": w, "bits": bits, "groups": groups} for w in s["W"]])
        Ys, codes, grads = [], [], []
        for X, (packed, h, _, rs_w), n in zip(s["X"], weights, s["N"]):
            Xq, rs_x = qb.qb_quantize_act(X, CLIP)
            Ys.append(qb.qb_qlinear_fwd(Xq, rs_x, CLIP, packed, h, rs_w, bits, groups, n))
            codes.append(Xq)
        for i in (3, 2, 1, 0):
            packed, h, m, _ = weights[i]
            if s["masked"]:
                grads.append(qb.qb_qlinear_bwd_ste_masked(s["dY"][i], codes[i], CLIP, packed, h, bits, groups, X=s["X"][i], W=s["W"][i], m=m))
            else:
                grads.append(qb.qb_qlinear_bwd_ste(s["dY"][i], codes[i], CLIP, packed, h, bits, groups))
        return Ys, grads
    if kind == "sweep":
        weights = qb.qb_quantize_groupwise_batched(s["quant"])
        acts = qb.qb_quantize_act_batched(s["act"])
        Ys = qb.qb_qlinear_fwd_batched(s["fwd"])
        return Ys, acts, [w[0] for w in weights], [w[1] for w in weights]
    if kind == "requant":
        qb.qb_quantize_groupwise_batched(s["jobs"])
        return s["flat"]
    codes, h, m = qb.qb_embedding_quantize_bits(s["E"], s["bits"], s["hidden"] // 64 * 8)
    return codes, h, m, qb.qb_embedding_gather_bits(codes, h, s["bits"], s["hidden"] // 64 * 8, s["token_ids"])


def work(case):
    kind, hidden = case["kind"], case["hidden"]
    if kind == "embed":
        d, width = hidden, case["bits"] / 8
        rows = min(case["ids"], case["vocab"])
        return {"bytes": case["vocab"] * d * (4 + width) + rows * d * width + case["ids"] * (8 + 4 * d), "flops": 0}
    lin = _linears(hidden)
    params = sum(n * k for n, k in lin)
    if kind == "requant":
        return {"bytes": sum(params * (4 + b / 8) for b in _layer_bits(case["layers"])), "flops": 0}
    T = case["tokens"]
    if kind == "sweep":  # the activations are quantized once and used by every width
        return {"bytes": sum(params * (4 + b / 8) for b in (2, 3, 4, 8)) + sum(5 * T * k for _, k in lin) + 4 * sum(4 * T * n for n, _ in lin), "flops": 8 * T * params}
    if kind == "ffn_q8":
        (nu, ku), (nd, kd) = lin[2:]
        return {"bytes": 4 * T * ku + T * nu + 4 * T * nd + (nu * ku + nd * kd) * case["bits"] / 8, "flops": 2 * T * (nu * ku + nd * kd)}
    if kind == "train":
        # (the clamp masks are taken from X and W, which are read anyway)
        return {"bytes": sum(T * (4 * k + 4 * n + 2 * n + 2 * k) for n, k in lin) + 8 * params, "flops": 6 * T * params}
    return {"bytes": sum(T * (4 * k + 4 * n) for n, k in lin) + params * case["bits"] / 8, "flops": 2 * T * params}


def tolerance(case):
    """Four times what a comparison with the same path in 64 bits showed (figures in the comments)."""
    kind = case["kind"]
    if kind in ("requant", "embed"):
        return "exact"  # codes, ranges, and one rounded product per looked-up value
    if kind == "ffn_q8":
        # the 32-bit error function moves a value across a rounding boundary now and then: 2.3e-6 of the codes, and with
        # them 0.7 % of the row sums; behind the down projection 6e-5 and at most 1.7e-2
        return {"rel": 2.5e-4, "max": 6e-2, "differ": 1e-2}
    if kind == "train":
        return {"rel": 9e-3, "max": 5e-2}  # bf16 weights and bf16 dX: 2.4e-3, 1.2e-2
    if kind == "dyn":
        return {"rel": 3e-6, "max": 4e-5}  # exact integer sums, two products that partly cancel: 7.9e-7, 1e-5
    return {"rel": 2e-7, "max": 7e-7}  # exact integer sums, then three 32-bit roundings: 4.4e-8, 1.7e-7
