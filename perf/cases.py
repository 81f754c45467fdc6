"""The work that a program hands to this library, as cases that can be timed and compared.

A case is a dict of plain values:
  path    which calls one pass makes (see `run`)
  kind    data type: 0 dynamic tree, 1 linear, 2 static tree, 3 mantissa
  n       elements
  block   elements per scale (0: one scale for the whole array)
  values  distribution of the inputs: "normal", "laplace", "student", "relu" or "uniform"
and, where the path has them,
  K       worker buffers that are averaged
  local   whether the caller's own fp32 array is one more term of the average
  layout  tensors of a set: the number of a configuration of `workloads.SHAPES`, or 0 with `tensors` and `cut` for a
          set of that many tensors of unequal sizes
  offset  elements between an aligned address and the first element (a tensor that is a view into a flat buffer)
  given   whether the scale of the error statistics is handed in (a decade) instead of taken from the sample
"""
import math
import random

import torch

from paper_1511_04561_amd import dq8, workloads

#: elements of the AlexNet-shaped gradient bucket
BUCKET = workloads.C3_NUMEL


def listed():
    return [
        # The smallest call a training loop makes: one bias gradient of a fully connected layer with its own maximum,
        # compressed before it is sent and expanded where it arrives.  Latency and launches count here.
        {"name": "bias_tensor", "path": "tensors", "kind": 0, "n": 4096, "block": 0, "layout": 0, "tensors": 1, "cut": 0,
         "offset": 0, "values": "normal"},
        # The gradients of the 784-1024-1024-10 perceptron layer by layer, as backpropagation finishes them: six tensors
        # of 10 to 1 048 576 elements, one maximum and one pair of calls each.
        {"name": "mlp_layer_by_layer", "path": "tensors", "kind": 0, "n": workloads.config_numel(1), "block": 0, "layout": 1,
         "tensors": 6, "cut": 0, "offset": 0, "values": "normal"},
        # The small convnet's ten gradients back to back, one maximum each: the own set is compressed in one call, and
        # seven received sets are averaged with the own fp32 gradients.
        {"name": "convnet_exchange", "path": "set_exchange", "kind": 1, "n": workloads.config_numel(2), "block": 0, "layout": 2,
         "tensors": 10, "cut": 0, "K": 7, "local": True, "values": "laplace"},
        # The AlexNet-shaped gradients as sixteen matrices with one maximum each (the paper's normalisation),
        # compressed and expanded in one call each.
        {"name": "alexnet_matrices", "path": "set", "kind": 0, "n": BUCKET, "block": 0, "layout": 3, "tensors": 16, "cut": 0,
         "values": "student"},
        # One large fully connected layer (9216 x 4096) by itself, normalised by the matrix's maximum.
        {"name": "fc_matrix", "path": "tensors", "kind": 0, "n": 9216 * 4096, "block": 0, "layout": 0, "tensors": 1, "cut": 0,
         "offset": 0, "values": "student"},
        # Activations of a batch of 1024 behind a rectifier, half of them zero, one maximum per sample: the forward
        # pass of model parallelism.
        {"name": "activation_rows", "path": "rows", "kind": 0, "n": 1024 * 4096, "block": 4096, "values": "relu"},
        # The same for a layer whose width is not a multiple of anything (1001 outputs), static type: rows start at
        # every alignment.
        {"name": "odd_rows", "path": "rows", "kind": 2, "n": 2048 * 1001, "block": 1001, "values": "relu"},
        # The AlexNet-shaped gradient bucket, 4096 elements per scale: what a worker compresses and sends,
        {"name": "bucket_compress", "path": "compress", "kind": 0, "n": BUCKET, "block": 4096, "values": "student"},
        # what it expands after the last exchange,
        {"name": "bucket_expand", "path": "expand", "kind": 0, "n": BUCKET, "block": 4096, "values": "student"},
        # the average of eight workers' buckets into fp32,
        {"name": "bucket_average", "path": "average", "kind": 0, "n": BUCKET, "block": 4096, "K": 8, "local": False,
         "values": "student"},
        # and the second round of the exchange on an eight-GPU node: seven received buckets and the own fp32 gradients
        # averaged and compressed again.
        {"name": "bucket_second_round", "path": "average_compress", "kind": 0, "n": BUCKET, "block": 4096, "K": 7, "local": True,
         "values": "student"},
        # Choosing a data type: mean and relative error of a sample of 25 million values (Table 2 of the paper).
        {"name": "sample_error", "path": "error", "kind": 1, "n": 25_000_000, "block": 0, "given": False, "values": "normal"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["tensors", "set", "set_exchange", "rows", "compress", "expand", "average", "average_compress", "error"])
    kind = rng.choice([0, 0, 1, 2, 3])
    values = rng.choice(["normal", "laplace", "student"])
    if path in ("tensors", "set", "set_exchange"):
        # tensors with one maximum each, from a bias to the largest fully connected layer, any number of elements
        count = 1 if path == "tensors" and rng.random() < 0.5 else rng.randint(2, 12 if path == "tensors" else 64)
        n = _log(rng, 1024, 9216 * 4096 if path == "tensors" else BUCKET)
        if path == "set_exchange":
            n = min(n, BUCKET // 2)
        case = {"path": path, "kind": kind, "n": max(n, 64 * count), "block": 0, "layout": 0, "tensors": count, "cut": rng.randrange(1 << 30),
                "values": values}
        if path == "tensors":
            case["offset"] = rng.choice([0, 0, 0, 1, 2, 3])
        if path == "set_exchange":
            case["K"] = rng.choice([1, 2, 3, 4, 7, 8])
            case["local"] = rng.random() < 0.5
        return case
    if path == "rows":
        # 16 to 2048 samples of 100 to 9216 activations, odd widths among them
        width = rng.choice([1000, 1001, 4096, 4096, 9216, _log(rng, 100, 9216), _log(rng, 100, 9216)])
        rows = min(_log(rng, 16, 2048), 8_000_000 // width)
        return {"path": path, "kind": kind, "n": rows * width, "block": width, "values": "relu"}
    if path == "error":
        given = kind in (2, 3)
        block = 0 if given else rng.choice([0, 0, 4096, 1024])
        return {"path": path, "kind": kind, "n": _log(rng, 100_000, 25_000_000), "block": block, "given": given,
                "values": rng.choice(["uniform", "normal", "normal"])}
    # a flat bucket, from a few thousand gradients to the whole network's, any number of elements
    block = rng.choice([64, 256, 1024, 2048, 4096, 4096, 4096, 8192, 16384, 1000, 3000])
    case = {"path": path, "kind": kind, "n": _log(rng, 4096, BUCKET), "block": block, "values": values}
    if path in ("average", "average_compress"):
        case["K"] = rng.choice([1, 2, 3, 4, 5, 7, 8, 8, 16])
        case["local"] = rng.random() < 0.4
        # the bytes of a call do not exceed those of the largest bucket with eight workers
        case["n"] = min(case["n"], BUCKET * 12 // (case["K"] + 8))
    return case


def _sizes(case):
    """Elements of the tensors of a set."""
    if case["layout"]:
        return [workloads.numel(shape) for _, shape in workloads.SHAPES[case["layout"]]]
    r = random.Random(case["cut"])
    count, n = case["tensors"], case["n"]
    weight = [math.exp(r.uniform(0.0, 7.0)) for _ in range(count)]  # as unequal as biases and weights
    sizes = [max(1, int(n * w / sum(weight))) for w in weight]
    sizes[sizes.index(max(sizes))] += n - sum(sizes)
    return sizes


def _values(case, n, gen):
    """n values as the case's tensors hold them."""
    v = case["values"]
    if v == "uniform":
        return torch.rand(n, device="cuda", generator=gen)
    z = torch.randn(n, device="cuda", generator=gen)
    if v == "normal":
        return z if case["path"] == "error" else z.mul_(1e-3)
    if v == "relu":  # Exp(1), about half exact zeros
        e = torch.rand(n, device="cuda", generator=gen).mul_(-1.0).log1p_().neg_()
        return torch.where(z > 0, e, torch.zeros_like(e))
    if v == "laplace":  # Laplace(0, 5e-4), one value in a hundred fifty times as large
        u = torch.rand(n, device="cuda", generator=gen)
        x = u.mul(-0.999999).log1p_().neg_().mul_(5e-4) * z.sign()
        return torch.where(torch.rand(n, device="cuda", generator=gen) < 0.01, x * 50.0, x)
    chi = torch.zeros_like(z)  # Student-t with three degrees of freedom
    for _ in range(3):
        chi += torch.randn(n, device="cuda", generator=gen).square_()
    return z.mul_(1e-3).mul_(chi.div_(3.0).rsqrt_())


def _empty(n, dtype):
    return torch.empty(n, dtype=dtype, device="cuda")


def prepare(case, seed):
    dq8.init()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    path, kind, n, block = case["path"], case["kind"], case["n"], case["block"]
    s = {"path": path, "kind": kind, "block": block}
    if path == "tensors":
        s["tensors"] = []
        for m in _sizes(case):
            off = case["offset"]
            x = _empty(off + m, torch.float32)[off:]
            x.copy_(_values(case, m, gen))
            s["tensors"].append((x, _empty(1, torch.float32), _empty(off + m, torch.uint8)[off:], _empty(off + m, torch.float32)[off:]))
    elif path in ("set", "set_exchange"):
        sizes = _sizes(case)
        s["bounds"] = torch.tensor([0] + sizes, dtype=torch.int64).cumsum(0).cuda()
        s["x"] = _values(case, n, gen)
        s["codes"], s["scales"], s["out"] = _empty(n, torch.uint8), _empty(len(sizes), torch.float32), _empty(n, torch.float32)
        if path == "set_exchange":
            received = [dq8.encode_segments(kind, _values(case, n, gen), s["bounds"]) for _ in range(case["K"])]
            s["worker_codes"], s["worker_scales"] = [c for c, _ in received], [a for _, a in received]
            s["local"] = s["x"] if case["local"] else None
    elif path == "rows":
        s["x"] = _values(case, n, gen)
    elif path == "error":
        s["x"] = _values(case, n, gen)
        nb = dq8.n_blocks(n, block)
        s["scales"] = torch.full((nb,), 10.0, device="cuda") if case["given"] else _empty(nb, torch.float32)
        s["given"] = case["given"]
        s["stats"], s["means"] = _empty((nb, 4), torch.float64), _empty(2, torch.float64)
    else:
        nb = dq8.n_blocks(n, block)
        if path == "compress":
            s["x"] = _values(case, n, gen)
            s["codes"], s["scales"] = _empty(n, torch.uint8), _empty(nb, torch.float32)
        elif path == "expand":
            s["codes"], s["scales"] = dq8.encode(kind, _values(case, n, gen), block)
            s["out"] = _empty(n, torch.float32)
        else:
            received = [dq8.encode(kind, _values(case, n, gen), block) for _ in range(case["K"])]
            s["worker_codes"], s["worker_scales"] = [c for c, _ in received], [a for _, a in received]
            s["local"] = _values(case, n, gen) if case["local"] else None
            if path == "average":
                s["out"] = _empty(n, torch.float32)
            else:
                s["codes"], s["scales"] = _empty(n, torch.uint8), _empty(nb, torch.float32)
    return s


def run(s):
    path, kind, block = s["path"], s["kind"], s["block"]
    if path == "tensors":
        done = []
        for x, scale, codes, out in s["tensors"]:
            dq8.encode(kind, x, block, scales=scale, codes=codes)
            dq8.decode(kind, codes, scale, block, out=out)
            done.append((codes, scale, out))
        return done
    if path == "set":
        dq8.encode_segments(kind, s["x"], s["bounds"], scales=s["scales"], codes=s["codes"])
        dq8.decode_segments(kind, s["codes"], s["scales"], s["bounds"], out=s["out"])
        return s["codes"], s["scales"], s["out"]
    if path == "set_exchange":
        dq8.encode_segments(kind, s["x"], s["bounds"], scales=s["scales"], codes=s["codes"])
        dq8.decode_accumulate_avg_segments(kind, s["worker_codes"], s["worker_scales"], s["bounds"], out=s["out"], local=s["local"])
        return s["codes"], s["scales"], s["out"]
    if path == "rows":
        codes, scales = dq8.encode(kind, s["x"], block)
        return codes, scales, dq8.decode(kind, codes, scales, block)
    if path == "compress":
        return dq8.encode(kind, s["x"], block, scales=s["scales"], codes=s["codes"])
    if path == "expand":
        return dq8.decode(kind, s["codes"], s["scales"], block, out=s["out"])
    if path == "average":
        return dq8.decode_accumulate_avg(kind, s["worker_codes"], s["worker_scales"], block, out=s["out"], local=s["local"])
    if path == "average_compress":
        return dq8.decode_avg_encode(kind, s["worker_codes"], s["worker_scales"], block, local=s["local"], scales=s["scales"],
                                     codes=s["codes"])
    stats, means = dq8.error_stats(kind, s["x"], block, scales=s["scales"], scales_given=s["given"], stats=s["stats"], means=s["means"])
    return stats, means, s["scales"]


def work(case):
    """Bytes with every input read once and every output written once (fp32 values 4, codes 1, scales 4 each), and the
    arithmetic of the definition per element: a product to expand a code, a comparison for the maximum and a quotient to
    compress a value, a sum per averaged term and a quotient for the mean."""
    path, n = case["path"], case["n"]
    if path in ("tensors", "set", "set_exchange"):
        nb = case["tensors"]
    else:
        nb = dq8.n_blocks(n, case["block"])
    compress, expand = 5 * n + 4 * nb, 5 * n + 4 * nb
    if path in ("tensors", "set", "rows"):
        return {"bytes": compress + expand, "flops": 3 * n}
    if path == "compress":
        return {"bytes": compress, "flops": 2 * n}
    if path == "expand":
        return {"bytes": expand, "flops": n}
    if path == "error":
        return {"bytes": 4 * n + 4 * nb + 32 * nb + 16, "flops": 6 * n}
    K, local = case["K"], 4 * n if case["local"] else 0
    received = K * (n + 4 * nb)
    if path == "average":
        return {"bytes": received + local + 4 * n, "flops": (2 * K + 1) * n}
    if path == "average_compress":
        return {"bytes": received + local + n + 4 * nb, "flops": (2 * K + 3) * n}
    # set_exchange: the own values are read once for the compression, and again as a term of the average
    return {"bytes": compress + received + local + 4 * n, "flops": (2 * K + 3) * n}


def tolerance(case):
    """Codes, scales, expanded and averaged values are exact functions of the input: every operation is a single rounding in a
    stated order.  The error statistics hold binary64 sums of up to 25 million terms of one sign whose order is free: two
    launches, and the same sums in another order, differ by up to 2.4e-15 (relative)."""
    if case["path"] == "error":
        return {"rel": 1e-14, "max": 1e-14}
    return "exact"
