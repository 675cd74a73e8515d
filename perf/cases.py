"""Workloads of the DP-SGD gradient step, measured through the package's entry points.

A case describes one pass of a training program: the captured activations and
output gradients of its linear layers are on the GPU, the pass forms the
per-example norms over all layers, the clip factors and the clipped sums, and,
where the case says so, the noise or the noisy optimizer step.

Fields of a case:

  work      "sums": norms, factors, clipped sums (up to the commit point of the
            protocol); "step": the same, then the noise in place;
            "adamw": noise + AdamW over given sums (what follows the commit)
  dtype     "f32" or "bf16", of activations and output gradients
  layers    "d_in>d_out" separated by blanks; "T:" in front gives that layer
            its own number of positions (convolutions), "=" in front lets the
            layer read the activations of the first layer of its group
  repeat    how often the list of layers is repeated
  B, T      examples and positions per example
  inputs    distribution of the activations: "normal" or "relu"
  mode      norm form: "auto", "ghost" or "materialize"
  fused     one call for norms and clipped sums instead of two
  micro     accumulated micro-batches of B examples each
"""

import math

import numpy as np
import torch

from paper_2609_20532_amd import dpsgd

MODES = {"auto": dpsgd.DPSGD_NORM_AUTO, "ghost": dpsgd.DPSGD_NORM_GHOST,
         "materialize": dpsgd.DPSGD_NORM_MATERIALIZE}

# Convolutions of WRN-16-4 as linear layers over positions (im2col).
CONV = " ".join(["1024:27>16", "1024:144>64", "1024:576>64", "1024:16>64", "1024:576>64",
                 "1024:576>64", "256:576>128", "256:1152>128", "256:64>128", "256:1152>128",
                 "256:1152>128", "64:1152>256", "64:2304>256", "64:128>256", "64:2304>256",
                 "64:2304>256", "1:256>10"])
BLOCK = "768>2304 768>768 768>3072 3072>768"


def _case(name, work, dtype, layers, B, T, repeat=1, inputs="normal", mode="auto", fused=False,
          micro=1):
    c = {"work": work, "dtype": dtype, "layers": layers, "repeat": repeat, "B": B, "T": T,
         "inputs": inputs, "mode": mode, "fused": fused, "micro": micro}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # One small linear layer without a sequence dimension: the smallest
        # step, all launches and host time.
        _case("linear_t1_f32", "step", "f32", "256>128", 32, 1),
        # A small MLP classifier (784 -> 512 -> 10) on a batch of images.
        _case("mlp_t1_f32", "step", "f32", "784>512 512>10", 256, 1, inputs="relu"),
        # The pooled classification head of a 768-wide encoder: one position
        # per example, the large batches that private training uses.
        _case("head_t1_bf16", "sums", "bf16", "768>768 768>10", 2048, 1),
        # Low-rank adapters (r = 4) on the fused QKV of a 12-block 768-wide
        # language model, float32 as captured, all 24 matrices in one call.
        _case("lora_r4_f32", "sums", "f32", "768>4 4>2304", 64, 128, repeat=12, fused=True),
        # Low-rank adapters (r = 8) on query and value in bfloat16, sentences
        # padded to the longest of the batch.
        _case("lora_r8_ragged_bf16", "sums", "bf16", "768>8 8>768 =768>8 8>768", 48, 203,
              repeat=12, fused=True),
        # A WRN-16-4 micro-batch in float32: convolutions as linear layers
        # over 1024, 256 and 64 positions, and the classifier.
        _case("conv_f32", "sums", "f32", CONV, 256, 1, inputs="relu"),
        # One MLP up-projection at T = 512.
        _case("mlp_up_t512_bf16", "sums", "bf16", "768>3072", 64, 512),
        # A large linear layer at T = 1024 together with a rank-16 adapter
        # pair, one call for norms and sums.
        _case("large_linear_lora_bf16", "sums", "bf16", "4096>11008 =4096>16 16>4096", 16, 1024,
              fused=True),
        # All 48 linear layers of a 12-block transformer under one global
        # clip: the largest pass.
        _case("transformer_bf16", "sums", "bf16", BLOCK, 128, 256, repeat=12),
        # Two blocks of it on sentences padded to an odd length, the batch
        # taken as two accumulated micro-batches.
        _case("transformer_ragged_bf16", "sums", "bf16", BLOCK, 32, 183, repeat=2, micro=2),
        # The output head of a language model: a vocabulary that no tile
        # divides, few examples.
        _case("vocab_head_bf16", "sums", "bf16", "768>50257", 4, 128),
        # After the commit: noise and the AdamW step over the parameters of
        # the 12-block transformer (85 M).
        _case("noise_adamw", "adamw", "f32", BLOCK, 1, 1, repeat=12),
    ]


# ------------------------------------------------------------------ drawn cases


def _log(rng, lo, hi, step=1):
    """A multiple of step, spread over the logarithm of [lo, hi]."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(step, int(round(v / step)) * step)


def _width(rng, lo, hi):
    """A layer width: most are multiples of 64 or 8, some are odd."""
    step = rng.choice([256, 64, 64, 8, 8, 1])
    return min(hi, max(lo, _log(rng, lo, hi, step)))


_LIMIT = None


def _cost(case):
    w = work(case)
    return w["bytes"] / 4e12 + w["flops"] / (1e15 if case["dtype"] == "bf16" else 9e13)


def draw(rng):
    global _LIMIT
    if _LIMIT is None:
        _LIMIT = max(_cost(c) for c in listed())
    while True:
        c = _draw(rng)
        if _cost(c) <= _LIMIT / 2:
            return c


def _draw(rng):
    kind = rng.choice(["rows", "adapter", "dense", "dense", "conv", "noise"])
    dtype = rng.choice(["f32", "bf16"])
    if kind == "rows":
        # Layers without a sequence dimension, from a handful of examples to
        # the batches of private training.
        n = rng.randint(1, 3)
        dims = [_width(rng, 16, 4096) for _ in range(n)] + [_log(rng, 2, 1024)]
        layers = " ".join("%d>%d" % (a, b) for a, b in zip(dims, dims[1:]))
        return _case("", rng.choice(["step", "sums"]), dtype, layers, _log(rng, 16, 4096), 1,
                     inputs=rng.choice(["normal", "relu"]))
    if kind == "adapter":
        d = _log(rng, 256, 4096, 64)
        r = rng.choice([1, 2, 4, 8, 12, 16])
        T = _log(rng, 32, 1024)
        B = max(2, min(256, _log(rng, 2 ** 11, 2 ** 14) // T))
        return _case("", "sums", dtype, "%d>%d %d>%d" % (d, r, r, d * rng.choice([1, 1, 3])), B, T,
                     repeat=rng.randint(1, 12), fused=rng.random() < 0.8)
    if kind == "dense":
        # Linear layers over sequences: tiled, eighths and odd widths, any T.
        n = rng.randint(1, 3)
        dims = [_width(rng, 64, 4096) for _ in range(n + 1)]
        layers = " ".join("%d>%d" % (a, b) for a, b in zip(dims, dims[1:]))
        T = rng.choice([_log(rng, 16, 1024), _log(rng, 16, 1024, 64)])
        B = max(2, min(256, _log(rng, 2 ** 10, 2 ** 14) // T))
        return _case("", rng.choice(["sums", "sums", "step"]), dtype, layers, B, T,
                     repeat=rng.randint(1, 2),
                     mode=rng.choice(["auto", "auto", "auto", "ghost", "materialize"]),
                     fused=rng.random() < 0.3, micro=rng.choice([1, 1, 2]))
    if kind == "conv":
        layers, side = [], rng.choice([32, 28, 16, 14, 8, 7])
        c = rng.choice([3, 16, 32, 64])
        for _ in range(rng.randint(2, 4)):
            k = rng.choice([1, 9, 9])
            o = rng.choice([16, 32, 48, 64, 96, 128, 256])
            layers.append("%d:%d>%d" % (side * side, c * k, o))
            c = o
            if side >= 14 and rng.random() < 0.4:
                side //= 2
        return _case("", "sums", dtype, " ".join(layers), _log(rng, 16, 512), 1, inputs="relu")
    dims = [_width(rng, 16, 4096) for _ in range(2)]
    return _case("", "adamw", "f32", "%d>%d" % tuple(dims), 1, 1, repeat=rng.randint(1, 12))


# ------------------------------------------------------------- inputs and passes


def _layers(case):
    """(T, d_in, d_out, layer whose activations it reads) of every layer."""
    out = []
    group = case["layers"].split()
    for _ in range(case["repeat"]):
        first = len(out)
        for text in group:
            share = text.startswith("=")
            text = text.lstrip("=")
            T = case["T"]
            if ":" in text:
                T, text = text.split(":")
            d_in, d_out = text.split(">")
            out.append((int(T), int(d_in), int(d_out), first if share else len(out)))
    return out


def _clip(case):
    # Every layer adds about 1 to the squared norm of an example of scale 1.
    return math.sqrt(len(_layers(case)))


def _noise_args(case, seed):
    return {"sigma": 0.8, "C": _clip(case), "seed": 1000003 * (int(seed) + 1) + 17,
            "step": 3, "scale": 1.0 / (case["B"] * case["micro"])}


def _inputs(case, seed, micro):
    """Activations and output gradients of every layer on the GPU. The
    examples' gradients differ in scale, so that about half are clipped."""
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    B = case["B"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7919 * int(seed) + 31 * micro + 5)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)

    scale = torch.exp(0.5 * randn(B)).view(B, 1, 1)
    As, Gs = [], []
    for l, (T, d_in, d_out, src) in enumerate(_layers(case)):
        if src != l:
            A = As[src]
        else:
            A = randn(B, T, d_in)
            if case["inputs"] == "relu":
                A.clamp_(min=0.0).mul_(math.sqrt(2.0))
            A = A.to(dt)
        G = randn(B, T, d_out)
        G.mul_(scale).mul_(1.0 / math.sqrt(float(T) * d_in * d_out))
        As.append(A)
        Gs.append(G.to(dt))
    return As, Gs


def _flat(case, gen, fill):
    """One buffer for a quantity of all parameters, and its per-layer views
    (each 16-byte aligned)."""
    dims = [(d_out, d_in) for _, d_in, d_out, _ in _layers(case)]
    offs, n = [], 0
    for r, c in dims:
        offs.append(n)
        n += -(-r * c // 4) * 4
    buf = fill(torch.randn(n, generator=gen, device="cuda", dtype=torch.float32))
    return buf, [buf[o:o + r * c].view(r, c) for o, (r, c) in zip(offs, dims)]


def _adamw_state(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(104729 * int(seed) + 11)
    numel = sum(d_in * d_out for _, d_in, d_out, _ in _layers(case))
    s = {}
    s["sum"], s["sums"] = _flat(case, gen, lambda x: x.mul_(_clip(case) * 8.0 / math.sqrt(numel)))
    s["param"], s["params"] = _flat(case, gen, lambda x: x.mul_(0.03))
    s["m"], s["ms"] = _flat(case, gen, lambda x: x.mul_(0.1))
    s["v"], s["vs"] = _flat(case, gen, lambda x: x.mul_(0.1).square_())
    return s


OPT = {"lr": 1e-3, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8, "weight_decay": 0.01, "t": 5}


def prepare(case, seed):
    s = {"case": case, "noise": _noise_args(case, seed), "C": _clip(case)}
    if case["work"] == "adamw":
        s.update(_adamw_state(case, seed))
        s["layers"] = [dpsgd.shape_layer(1, 1, d_in, d_out, dpsgd.DPSGD_F32, l)
                       for l, (_, d_in, d_out, _) in enumerate(_layers(case))]
        s["opt"] = dpsgd.make_adamw(**OPT)
        return s
    s["mode"] = MODES[case["mode"]]
    s["tensors"], s["micro"], s["bufs"] = [], [], []
    for k in range(case["micro"]):
        As, Gs = _inputs(case, seed, k)
        s["tensors"].append((As, Gs))
        s["micro"].append([dpsgd.make_layer(A, G, l) for l, (A, G) in enumerate(zip(As, Gs))])
        buf = dpsgd.alloc_step(s["micro"][0], s["mode"], fused=case["fused"])
        if k:
            buf.grads = s["bufs"][0].grads   # the micro-batches add up in one set of sums
        s["bufs"].append(buf)
    return s


def run(s):
    case = s["case"]
    if case["work"] == "adamw":
        n = s["noise"]
        dpsgd.dpsgd_noise_adamw_multi(s["layers"], s["sums"], s["params"], s["ms"], s["vs"],
                                      n["sigma"], n["C"], n["seed"], n["step"], n["scale"],
                                      s["opt"])
        return {"param": s["param"], "m": s["m"], "v": s["v"]}
    mode, C = s["mode"], s["C"]
    for k, (layers, buf) in enumerate(zip(s["micro"], s["bufs"])):
        if k == 0:
            dpsgd.run_clipped_sum(layers, buf, C, mode, fused=case["fused"])
        elif case["fused"]:
            dpsgd.dpsgd_clipped_sum_multi(layers, mode, C, buf.grads, buf.norms_sq,
                                          accumulate=True, factors_out=buf.factors,
                                          mask_out=buf.mask, workspace=buf.fused_ws)
        else:
            dpsgd.dpsgd_per_example_norms_multi(layers, mode, buf.norms_sq,
                                                workspace=buf.norms_ws)
            dpsgd.dpsgd_clip_accumulate_multi(layers, buf.norms_sq, C, buf.grads, accumulate=True,
                                              factors_out=buf.factors, mask_out=buf.mask,
                                              workspace=buf.clip_ws)
    if case["work"] == "step":
        n = s["noise"]
        dpsgd.dpsgd_add_noise_multi(s["micro"][0], s["bufs"][0].grads, n["sigma"], n["C"],
                                    n["seed"], n["step"], n["scale"])
    return {"norms_sq": [b.norms_sq for b in s["bufs"]], "factors": [b.factors for b in s["bufs"]],
            "mask": [b.mask for b in s["bufs"]], "grads": s["bufs"][0].grads}


# ------------------------------------------------------- work, tolerance, exact


def work(case):
    """Bytes: inputs read once, results written once. Operations: the clipped
    sum's products and the cheaper form of the norm."""
    layers = _layers(case)
    numel = sum(d_in * d_out for _, d_in, d_out, _ in layers)
    if case["work"] == "adamw":
        return {"bytes": 28.0 * numel, "flops": 60.0 * numel}
    B, esz = float(case["B"]), 2.0 if case["dtype"] == "bf16" else 4.0
    nbytes = flops = 0.0
    for l, (T, d_in, d_out, src) in enumerate(layers):
        nbytes += B * T * (d_out + (d_in if src == l else 0)) * esz
        product = 2.0 * B * T * d_in * d_out
        gram = B * T * (T + 1.0) * (d_in + d_out)
        flops += product + min(product, gram)
    nbytes, flops = nbytes * case["micro"], flops * case["micro"]
    return {"bytes": nbytes + 4.0 * numel, "flops": flops}


def tolerance(case):
    # About four times the largest error against float64 that the cases show:
    # 1.2e-6 for float32 sums over 32768 rows, 1.4e-3 where a bfloat16 layer's
    # clip weight is rounded into the bfloat16 operand, 1.1e-7 for the
    # optimizer step. "differ" covers examples whose norm lies within rounding
    # of the bound.
    if case["work"] == "adamw":
        return {"rel": 5e-7, "max": 1e-4}
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "differ": 0.002}
    return {"rel": 6e-3, "differ": 0.002}


def _philox_normals(numel, seed, tensor_id, step):
    """Standard normals of the noise stream in float64: Philox4x32-10 words
    and the Box-Muller transform, as the header documents them."""
    out = torch.empty(-(-numel // 4) * 4, dtype=torch.float64, device="cuda")
    mask = 0xFFFFFFFF
    blocks, chunk = out.numel() // 4, 1 << 23

    def mul(x, m):
        # 32 x 32 -> 64 bits from 16-bit halves (int64 is signed).
        lo, hi = x & 0xFFFF, x >> 16
        a, b = lo * m, hi * m
        low = (a + ((b & 0xFFFF) << 16))
        return ((b >> 16) + (low >> 32)) & mask, low & mask

    for b0 in range(0, blocks, chunk):
        j = torch.arange(b0, min(b0 + chunk, blocks), device="cuda", dtype=torch.int64)
        x = [j & mask, j >> 32, torch.full_like(j, tensor_id), torch.full_like(j, step)]
        k0, k1 = seed & mask, (seed >> 32) & mask
        for _ in range(10):
            h0, l0 = mul(x[0], 0xD2511F53)
            h1, l1 = mul(x[2], 0xCD9E8D57)
            x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
            k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
        u = [((w >> 8) + 1).double() * 2.0 ** -24 for w in (x[0], x[2])]
        v = [(w >> 8).double() * 2.0 ** -24 for w in (x[1], x[3])]
        z = []
        for a, t in zip(u, v):
            r = torch.sqrt(-2.0 * torch.log(a))
            z += [r * torch.cos(2.0 * math.pi * t), r * torch.sin(2.0 * math.pi * t)]
        out[4 * b0:4 * (b0 + j.numel())] = torch.stack(z, dim=1).reshape(-1)
    return out[:numel]


def _exact_sums(case, seed, micro):
    As, Gs = _inputs(case, seed, micro)
    B = case["B"]
    nsq = torch.zeros(B, dtype=torch.float64, device="cuda")
    layers = _layers(case)
    for l, (T, d_in, d_out, _) in enumerate(layers):
        per = max(d_in * d_out, T * (d_in + d_out), T * T) * 8
        step = max(1, min(B, (1 << 31) // per))
        for b in range(0, B, step):
            A, G = As[l][b:b + step].double(), Gs[l][b:b + step].double()
            if T == 1:
                nsq[b:b + step] += A.square().sum((1, 2)) * G.square().sum((1, 2))
            elif T * (d_in + d_out) <= 2 * d_in * d_out:
                ga = torch.bmm(A, A.transpose(1, 2).contiguous())
                gg = torch.bmm(G, G.transpose(1, 2).contiguous())
                nsq[b:b + step] += (ga * gg).sum((1, 2))
            else:
                nsq[b:b + step] += torch.bmm(G.transpose(1, 2).contiguous(), A).square().sum((1, 2))
    n = torch.sqrt(nsq)
    C = _clip(case)
    clipped = n > C
    c = torch.where(clipped, C / n, torch.ones_like(n))
    sums = []
    for l, (T, d_in, d_out, _) in enumerate(layers):
        S = torch.zeros(d_out, d_in, dtype=torch.float64, device="cuda")
        step = max(1, min(B, (1 << 30) // (T * (d_in + d_out))))
        for b in range(0, B, step):
            A = As[l][b:b + step].double().reshape(-1, d_in)
            G = (Gs[l][b:b + step].double() * c[b:b + step].view(-1, 1, 1)).reshape(-1, d_out)
            S += torch.mm(G.t().contiguous(), A)
        sums.append(S)
    return nsq, c, clipped.to(torch.uint8), sums


def exact(case, seed):
    n = _noise_args(case, seed)
    if case["work"] == "adamw":
        s = _adamw_state(case, seed)
        o = {k: float(np.float32(v)) for k, v in OPT.items()}
        res = {k: s[k].double() for k in ("param", "m", "v")}
        sigma_c = float(np.float32(np.float32(n["sigma"]) * np.float32(n["C"])))
        off = 0
        for l, (_, d_in, d_out, _) in enumerate(_layers(case)):
            num = d_in * d_out
            at = slice(off, off + num)
            z = _philox_normals(num, n["seed"], l, n["step"])
            g = float(np.float32(n["scale"])) * (s["sum"][at].double() + sigma_c * z)
            m = o["beta1"] * res["m"][at] + (1.0 - o["beta1"]) * g
            v = o["beta2"] * res["v"][at] + (1.0 - o["beta2"]) * g * g
            mh, vh = m / (1.0 - o["beta1"] ** OPT["t"]), v / (1.0 - o["beta2"] ** OPT["t"])
            p = res["param"][at]
            res["param"][at] = p - o["lr"] * (mh / (torch.sqrt(vh) + o["eps"]) +
                                              o["weight_decay"] * p)
            res["m"][at], res["v"][at] = m, v
            off += -(-num // 4) * 4
        return res
    out = {"norms_sq": [], "factors": [], "mask": [], "grads": None}
    for k in range(case["micro"]):
        nsq, c, mask, sums = _exact_sums(case, seed, k)
        out["norms_sq"].append(nsq)
        out["factors"].append(c)
        out["mask"].append(mask)
        out["grads"] = sums if k == 0 else [a + b for a, b in zip(out["grads"], sums)]
    if case["work"] == "step":
        for l, S in enumerate(out["grads"]):
            z = _philox_normals(S.numel(), n["seed"], l, n["step"]).view_as(S)
            out["grads"][l] = n["scale"] * (S + n["sigma"] * n["C"] * z)
    return out
