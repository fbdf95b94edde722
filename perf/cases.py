"""Performance cases of the library: what a program that trains with it calls, through the Python binding.

A case names a kind of work and its sizes; `run` makes one pass of that work on the state that `prepare`
made.  Every state holds what such a program keeps between iterations (gradient, stream and parameter
buffers), and every pass draws from the random stream of one iteration.

kinds
  step             the whole iteration on one GPU: W workers' gradients quantized one call each, then the fused
                   server update (what bench.py times)
  worker           a worker's Quantize(g, K) of one flat gradient; `scale` selects max |g| or the L2 norm
  server           the fused server update of W streams that arrived from elsewhere
  exchange         the paper's full exchange: this worker quantizes, the server re-quantizes the sum of W streams,
                   the worker updates its parameters from the mean
  exchange_minmax  the same with the deterministic [min, max] encoder, one range per bucket
  exchange_tensor  the same with one [min, max] range per tensor, as the paper prints it
  layers           a model's layer tensors, a few launches for all: this worker quantizes, the server updates
  layers_minmax    the paper's arrangement: the layers named in `encoded` travel over one [min, max] range each, the
                   others as fp32
  norms            the sums of squares of W workers' gradients (the Adaptive baseline's rule needs them)
"""
import math

import torch

from paper_1804_08066_amd import mqgrad as mq
from paper_1804_08066_amd import workloads

DEV = "cuda"
LR = 0.1
SEED = 20180806          # of the quantizer's random stream
ITERATION = 3

CNN = ",".join(str(n) for _, n in workloads.SMALL_CNN_SHAPES)   # ten layers, 1.07 M values


def listed():
    return [
        # the first thing a new user runs, and any small model: two launches, latency counts
        dict(name="step_small", kind="step", n=65_536, W=1, bits=4, bucket=512, values="normal"),
        # the small CNN, every layer quantized, two batched launches
        dict(name="layers_cnn", kind="layers", sizes=CNN, W=4, bits=2, bucket=512, values="laplace"),
        # the small CNN as the paper sends it: the two large fully connected layers encoded, the rest as fp32
        dict(name="layers_cnn_paper", kind="layers_minmax", sizes=CNN, encoded="4,6", W=4, bits=4, values="laplace"),
        # a ResNet-50-sized gradient with outliers on a worker; the straddling widths are the training schedule's middle
        dict(name="worker_resnet", kind="worker", n=25_600_000, bits=3, bucket=2048, scale="max", values="outliers"),
        # norm scaling of the QSGD family at its usual bucket, a ragged flat gradient
        dict(name="worker_norm", kind="worker", n=10_000_019, bits=4, bucket=512, scale="l2", values="student"),
        # the server of the same model
        dict(name="server_resnet", kind="server", n=25_600_000, W=8, bits=5, bucket=512, values="outliers"),
        # a large server late in the schedule: sixteen streams at eight bits, over the network
        dict(name="server_large", kind="server", n=100_000_000, W=16, bits=8, bucket=1024, values="normal"),
        # Algorithm 1 with per-bucket stochastic quantization: both directions of the exchange
        dict(name="exchange_resnet", kind="exchange", n=25_600_000, W=8, bits=4, bucket=1024, values="outliers"),
        # a fully connected layer (3136 x 2304), one range per row of the matrix
        dict(name="exchange_rows", kind="exchange_minmax", n=3136 * 2304, W=4, bits=6, bucket=2304, values="laplace"),
        # the paper's own iteration on its larger layer (2304 x 3840) and its twelve nodes
        dict(name="exchange_paper", kind="exchange_tensor", n=2304 * 3840, W=12, bits=4, values="laplace"),
        # the Adaptive baseline's norms of eight workers
        dict(name="norms_resnet", kind="norms", n=25_600_000, W=8, values="outliers"),
        # the benchmark's step, the largest call: 100 M elements, eight workers
        dict(name="step_large", kind="step", n=100_000_000, W=8, bits=4, bucket=1024, values="normal"),
    ]


def _draw_bucket(rng):
    if rng.random() < 0.65:
        return 1 << rng.randint(5, 14)                       # 32 .. 16384
    return 32 * int(round(math.exp(rng.uniform(math.log(2), math.log(512)))))


def draw(rng):
    """One more case.  n spreads over its logarithm from 4096 up to what keeps the pass below the largest listed one."""
    kind = rng.choice(["step", "worker", "worker", "server", "server", "exchange", "exchange_minmax", "exchange_tensor",
                       "layers", "layers_minmax", "norms"])
    values = rng.choice(["normal", "laplace", "outliers", "student"])
    bits = rng.randint(1, 8)
    W = int(round(math.exp(rng.uniform(0.0, math.log(24)))))  # 1 .. 24
    if kind in ("layers", "layers_minmax"):
        count = rng.randint(2, 12)
        sizes = [int(math.exp(rng.uniform(math.log(10), math.log(3_000_000)))) for _ in range(count)]
        W = min(W, 10)                                        # 2 W pointers per layer, 256 in a launch
        case = dict(kind=kind, sizes=",".join(str(n) for n in sizes), W=W, bits=bits, values=values)
        if kind == "layers":
            case["bucket"] = _draw_bucket(rng)
        else:
            large = sorted(range(count), key=lambda i: -sizes[i])[:rng.randint(1, 3)]
            case["encoded"] = ",".join(str(i) for i in sorted(large))
        return case
    per_element = {"step": 5.0 * W, "worker": 5.0, "server": W + 8.0, "norms": 4.0 * W, "exchange": 2.0 * W + 15.0,
                   "exchange_minmax": 2.0 * W + 15.0, "exchange_tensor": 3.0 * W + 15.0}[kind]
    most = min(100_000_000, int(1.2e9 / per_element))
    n = int(math.exp(rng.uniform(math.log(4096), math.log(most))))
    case = dict(kind=kind, n=n, values=values)
    if kind != "worker":
        case["W"] = W
    if kind != "norms":
        case["bits"] = bits
    if kind in ("step", "worker", "server", "exchange", "exchange_minmax"):
        case["bucket"] = _draw_bucket(rng)
    if kind == "worker":
        case["scale"] = "l2" if rng.random() < 0.25 else "max"
    return case


def _gradient(case, n, seed):
    kind = case["values"]
    if kind == "normal":
        return workloads.normal(n, 1e-2, seed, DEV)
    if kind == "laplace":
        return workloads.laplace(n, 2e-3, seed, DEV)
    if kind == "outliers":
        return workloads.normal_with_outliers(n, 1e-3, 1e-3, 100.0, seed, DEV)
    return workloads.student_t(n, 3, 1e-3, seed, DEV)


def _words(n, bits):
    return torch.zeros(mq.mqg_packed_words(n, bits), dtype=torch.int32, device=DEV)


def _floats(n):
    return torch.zeros(n, dtype=torch.float32, device=DEV)


def _params(n, seed):
    return workloads.uniform(n, -0.05, 0.05, seed, DEV)


def _bases(sizes, bucket):
    out, run = [], 0
    for n in sizes:
        out.append(run)
        run += -(-n // bucket) * bucket
    return out


def prepare(case, seed):
    kind, base = case["kind"], 1_000_003 * int(seed)
    s = dict(case=case)
    if kind in ("layers", "layers_minmax"):
        sizes = [int(x) for x in case["sizes"].split(",")]
        W, bits = case["W"], case["bits"]
        encoded = range(len(sizes)) if kind == "layers" else [int(i) for i in case["encoded"].split(",")]
        bucket = case.get("bucket", 0)
        grads = [[_gradient(case, n, base + 101 * w + 7919 * i) for i, n in enumerate(sizes)] for w in range(W)]
        outs = []                                             # per worker: (words, scales or ranges) per encoded layer
        for w in range(W):
            mine = [grads[w][i] for i in encoded]
            if kind == "layers":
                s["bases"] = _bases(sizes, bucket)
                outs.append(mq.mqg_quantize_tensors(mine, bits, bucket, SEED, ITERATION, w, s["bases"]))
            else:
                outs.append(mq.mqg_quantize_minmax_tensors(mine, bits, 0))
        params = [_params(n, base + 555 + i) for i, n in enumerate(sizes)]
        layers, at = [], {layer: k for k, layer in enumerate(encoded)}
        for i in range(len(sizes)):
            if i in at:
                layers.append({"params": params[i], "packed": [o[at[i]][0] for o in outs], "scales": [o[at[i]][1] for o in outs]})
            else:
                layers.append({"params": params[i], "raw": [grads[w][i] for w in range(W)]})
        s.update(mine=[grads[0][i] for i in encoded], outs=outs[0], layers=layers, params=params)
        return s

    n, W, bits, bucket = case["n"], case.get("W", 1), case.get("bits", 0), case.get("bucket", 0)
    keep_all = kind in ("step", "norms")
    s["grads"], s["packed"], s["scales"] = [], [], []
    for w in range(W):
        g = _gradient(case, n, base + w)
        if keep_all or w == 0 and kind != "server":
            s["grads"].append(g)
        if kind == "norms":
            continue
        if kind == "exchange_minmax":
            p, r = mq.mqg_quantize_minmax(g, bits, bucket)
        elif kind == "exchange_tensor":
            p, r = mq.mqg_quantize_minmax_tensor(g, bits)
        else:
            p, r = mq.mqg_quantize(g, bits, bucket, SEED, ITERATION, w)
        s["packed"].append(p)
        s["scales"].append(r)
    if kind == "norms":
        s["workspace"] = torch.zeros(mq.mqg_sum_squares_workspace_bytes(W) // 8, dtype=torch.float64, device=DEV)
        s["out"] = torch.zeros(W, dtype=torch.float64, device=DEV)
        return s
    if kind != "worker":
        s["params"] = _params(n, base + 555)
    if kind.startswith("exchange"):
        s["mean_packed"] = _words(n, bits)
        s["mean_scales"] = torch.zeros_like(s["scales"][0])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "layers":
        W, bits, bucket = case["W"], case["bits"], case["bucket"]
        mq.mqg_quantize_tensors(s["mine"], bits, bucket, SEED, ITERATION, 0, s["bases"], outputs=s["outs"])
        mq.mqg_aggregate_update_tensors(s["layers"], W, bits, bucket, LR)
        return s["outs"], s["params"]
    if kind == "layers_minmax":
        W, bits = case["W"], case["bits"]
        mq.mqg_quantize_minmax_tensors(s["mine"], bits, 0, outputs=s["outs"])
        mq.mqg_aggregate_update_minmax_tensors(s["layers"], W, bits, 0, LR)
        return s["outs"], s["params"]
    if kind == "norms":
        return mq.mqg_sum_squares_batch(s["grads"], workspace=s["workspace"], out=s["out"])

    n, bits, bucket = case["n"], case["bits"], case.get("bucket", 0)
    packed, scales, grads = s["packed"], s["scales"], s["grads"]
    if kind == "worker":
        if case["scale"] == "l2":
            return mq.mqg_quantize(grads[0], bits, bucket, SEED, ITERATION, 0, packed_out=packed[0], scales_out=scales[0],
                                   mode=mq.MQG_SCALE_L2)
        return mq.mqg_quantize(grads[0], bits, bucket, SEED, ITERATION, 0, packed_out=packed[0], scales_out=scales[0])
    params = s["params"]
    if kind == "step":
        for w, g in enumerate(grads):
            mq.mqg_quantize(g, bits, bucket, SEED, ITERATION, w, packed_out=packed[w], scales_out=scales[w])
        mq.mqg_aggregate_update(packed, scales, n, bits, bucket, LR, params)
        return packed, scales, params
    if kind == "server":
        mq.mqg_aggregate_update(packed, scales, n, bits, bucket, LR, params, origin=mq.MQG_CODES_FROM_MEMORY)
        return params
    mean_packed, mean_scales = s["mean_packed"], s["mean_scales"]
    if kind == "exchange":
        mq.mqg_quantize(grads[0], bits, bucket, SEED, ITERATION, 0, packed_out=packed[0], scales_out=scales[0])
        mq.mqg_aggregate_requantize(packed, scales, n, bits, bucket, SEED, ITERATION, len(packed),
                                    packed_out=mean_packed, scales_out=mean_scales)
        mq.mqg_dequantize_update(mean_packed, mean_scales, n, bits, bucket, LR, params)
    elif kind == "exchange_minmax":
        mq.mqg_quantize_minmax(grads[0], bits, bucket, packed_out=packed[0], ranges_out=scales[0])
        mq.mqg_aggregate_requantize_minmax(packed, scales, n, bits, bucket, packed_out=mean_packed, ranges_out=mean_scales)
        mq.mqg_aggregate_update_minmax([mean_packed], [mean_scales], n, bits, bucket, LR, params)
    else:
        mq.mqg_quantize_minmax_tensor(grads[0], bits, packed_out=packed[0], range_out=scales[0])
        mq.mqg_aggregate_requantize_minmax_tensor(packed, scales, n, bits, packed_out=mean_packed, range_out=mean_scales)
        mq.mqg_aggregate_update_minmax_tensor([mean_packed], [mean_scales], n, bits, LR, params)
    return packed[0], scales[0], mean_packed, mean_scales, params


def work(case):
    """Every input read once and every output written once.  flops: what the arithmetic of the method needs per
    value (range, position and rounding: about 6 to encode; one fused multiply-add to decode and add), not counting
    the random numbers."""
    kind, W = case["kind"], case.get("W", 1)
    if kind in ("layers", "layers_minmax"):
        sizes = [int(x) for x in case["sizes"].split(",")]
        encoded = set(range(len(sizes))) if kind == "layers" else {int(i) for i in case["encoded"].split(",")}
        by = fl = 0.0
        for i, n in enumerate(sizes):
            ranges = 4.0 * -(-n // case["bucket"]) if kind == "layers" else 8.0
            code = n * case["bits"] / 8.0 + ranges
            if i in encoded:
                by += 4.0 * n + code + W * code + 8.0 * n
                fl += n * (6.0 + 2.0 * W + 2.0)
            else:
                by += 4.0 * n * W + 8.0 * n
                fl += n * (W + 2.0)
        return {"bytes": by, "flops": fl}
    n = case["n"]
    if kind == "norms":
        return {"bytes": W * (4.0 * n + 8.0), "flops": 2.0 * W * n}
    bucket = case.get("bucket", 0)
    ranges = {"exchange_minmax": 8.0, "exchange_tensor": 8.0}.get(kind, 4.0) * (-(-n // bucket) if bucket else 1)
    code = n * case["bits"] / 8.0 + ranges
    encode, update = 4.0 * n + code, 8.0 * n
    if kind == "worker":
        return {"bytes": encode, "flops": 6.0 * n}
    if kind == "step":
        return {"bytes": W * encode + W * code + update, "flops": n * (8.0 * W + 2.0)}
    if kind == "server":
        return {"bytes": W * code + update, "flops": n * (2.0 * W + 2.0)}
    return {"bytes": encode + (W + 1) * code + code + update, "flops": n * (6.0 + 2.0 * W + 6.0 + 4.0)}


def tolerance(case):
    """Every result is defined to the bit (ordered fp32 chains, integer codes), except sums of squares, whose order
    is free: the fp64 norms (within 7e-16 of fp64 sums in two other orders), the L2 scale (fp32 quads, fp64 above:
    3e-8, largest 1.2e-7, of the fp64 norm) and the codes that follow from it (none of 1.2 M words changed with the
    fp64 norm's scales; a scale 1 ulp off moves a code with probability of about 6e-8 times its level)."""
    if case["kind"] == "norms":
        return {"rel": 3e-15, "max": 3e-15}
    if case.get("scale") == "l2":
        return {"rel": 1.2e-7, "max": 5e-7, "differ": 4e-6}
    return "exact"
