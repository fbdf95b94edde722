"""GPU parity for the multi-tensor entry points: several layers per launch, uncompressed layers."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import to_u32, ulp_distance

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("bucket", [96, 512, 1184, 1376, 1760, 2048, 8192, 16384])
def test_batched_quantize_equals_per_tensor_and_oracle(bucket):
    sizes = [n for _, n in workloads.SMALL_CNN_SHAPES] + [0, 1, 40000 + 3]
    bases, run = [], 0
    for n in sizes:
        bases.append(run)
        run += (n + bucket - 1) // bucket * bucket
    assert all(b % 8 == 0 for b in bases)
    grads = [workloads.laplace(n, 2e-3, 70 + i, DEV) if n else torch.empty(0, device=DEV) for i, n in enumerate(sizes)]
    for bits in (1, 3, 8):
        outs = mqgrad.mqg_quantize_tensors(grads, bits, bucket, seed=4, iteration=7, worker=2, elem_bases=bases)
        torch.cuda.synchronize()
        for i, g in enumerate(grads):
            if sizes[i] == 0:
                continue
            pk_o, sc_o = ref.quantize(g.cpu().numpy(), bits, bucket, 4, 7, 2, bases[i])
            assert np.array_equal(to_u32(outs[i][0]), pk_o), "layer %d b=%d" % (i, bits)
            assert np.array_equal(outs[i][1].cpu().numpy(), sc_o), "layer %d b=%d" % (i, bits)


@pytest.mark.parametrize("bucket", [96, 512, 4096])
def test_batched_quantize_with_l2_scales_and_injected_scales(bucket):
    # the bucket's L2 norm as the range, and layers whose scales are given: bit-identical to the per-layer
    # calls; codes equal the oracle's once the oracle's L2 scales are injected (its norms are summed in fp64)
    sizes = [4800, 102400, 64, 40000 + 3, 7]
    bases, run = [], 0
    for n in sizes:
        bases.append(run)
        run += (n + bucket - 1) // bucket * bucket
    grads = [workloads.laplace(n, 3e-3, 170 + i, DEV) for i, n in enumerate(sizes)]
    bits = 3
    outs = mqgrad.mqg_quantize_tensors(grads, bits, bucket, seed=6, iteration=1, worker=3, elem_bases=bases,
                                       scale_mode=mqgrad.MQG_SCALE_L2)
    torch.cuda.synchronize()
    for i, g in enumerate(grads):
        pk1, sc1 = mqgrad.mqg_quantize(g, bits, bucket, 6, 1, 3, bases[i], mode=mqgrad.MQG_SCALE_L2)
        torch.cuda.synchronize()
        assert torch.equal(outs[i][0], pk1) and torch.equal(outs[i][1], sc1), "layer %d" % i
        sc_o = ref.bucket_scales(g.cpu().numpy(), bucket, ref.SCALE_L2)
        assert np.all(np.abs(sc1.cpu().numpy() - sc_o) <= 1e-6 * sc_o)
    # scales of the oracle injected into layers 0, 1 and 3; layers 2 and 4 compute their own (max-abs)
    inject = [torch.from_numpy(ref.bucket_scales(g.cpu().numpy(), bucket, ref.SCALE_L2)).to(DEV) if i in (0, 1, 3) else None
              for i, g in enumerate(grads)]
    outs = mqgrad.mqg_quantize_tensors(grads, bits, bucket, seed=6, iteration=1, worker=3, elem_bases=bases, scales_in=inject)
    torch.cuda.synchronize()
    for i, g in enumerate(grads):
        gh = g.cpu().numpy()
        if inject[i] is not None:
            pk_o, sc_o = ref.quantize(gh, bits, bucket, 6, 1, 3, bases[i], scales_in=inject[i].cpu().numpy())
        else:
            pk_o, sc_o = ref.quantize(gh, bits, bucket, 6, 1, 3, bases[i])
        assert np.array_equal(to_u32(outs[i][0]), pk_o), "layer %d" % i
        assert np.array_equal(outs[i][1].cpu().numpy(), sc_o), "layer %d" % i


def test_unaligned_layer_views_in_a_batch():
    base = workloads.normal(30000, 0.01, 5, DEV)
    grads = [base[1:5001], base[6000:6000 + 7000], base[14003:14003 + 999]]
    outs = mqgrad.mqg_quantize_tensors(grads, 5, 512, seed=1, elem_bases=[0, 8192, 16384])
    torch.cuda.synchronize()
    for g, (pk, sc), eb in zip(grads, outs, [0, 8192, 16384]):
        pk_o, sc_o = ref.quantize(g.cpu().numpy(), 5, 512, 1, 0, 0, eb)
        assert np.array_equal(to_u32(pk), pk_o) and np.array_equal(sc.cpu().numpy(), sc_o)


def test_config2_iterations_with_batched_calls_and_raw_small_layers():
    # the paper's selective quantization: the large layers are quantized, biases and the small last
    # layer travel uncompressed; one quantize launch per worker and one update launch per iteration
    W, bucket, lr, iters, seed = 4, 512, 0.1, 12, 0
    shapes = workloads.SMALL_CNN_SHAPES
    quantized = [n >= 4096 for _, n in shapes]
    bases = workloads.config2_elem_bases(bucket)
    bits_seq = workloads.config2_bits_sequence(iters, seed)
    params = workloads.config2_params(seed, DEV)
    p_ref = [p.cpu().numpy().copy() for p in params]
    q_idx = [i for i, q in enumerate(quantized) if q]
    for it in range(iters):
        bits = bits_seq[it]
        grads = [workloads.config2_grads(it, w, seed, DEV) for w in range(W)]
        outs = [mqgrad.mqg_quantize_tensors([grads[w][i] for i in q_idx], bits, bucket, seed=seed + w, iteration=it,
                                            worker=w, elem_bases=[bases[i] for i in q_idx]) for w in range(W)]
        layers = []
        for i in range(len(shapes)):
            if quantized[i]:
                k = q_idx.index(i)
                layers.append({"params": params[i], "packed": [outs[w][k][0] for w in range(W)],
                               "scales": [outs[w][k][1] for w in range(W)]})
            else:
                layers.append({"params": params[i], "raw": [grads[w][i] for w in range(W)]})
        mqgrad.mqg_aggregate_update_tensors(layers, W, bits, bucket, lr)
        torch.cuda.synchronize()
        for i, (_, n) in enumerate(shapes):
            if quantized[i]:
                want = [ref.quantize(grads[w][i].cpu().numpy(), bits, bucket, seed + w, it, w, bases[i]) for w in range(W)]
                p_ref[i] = ref.aggregate_update([x[0] for x in want], [x[1] for x in want], n, bits, bucket, lr, p_ref[i])
            else:
                p_ref[i] = ref.average_update_raw([grads[w][i].cpu().numpy() for w in range(W)], lr, p_ref[i])
            assert ulp_distance(params[i].cpu().numpy(), p_ref[i]).max() == 0, "iteration %d layer %d" % (it, i)


def test_batch_limits_are_reported():
    g = [workloads.normal(64, 0.01, i, DEV) for i in range(33)]
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_quantize_tensors(g, 4, 32, seed=0)
    W = 8
    layers = [{"params": torch.zeros(64, device=DEV), "raw": [g[0]] * W} for _ in range(32)]   # 256 pointers: fits
    mqgrad.mqg_aggregate_update_tensors(layers, W, 4, 32, 0.1)
    outs = mqgrad.mqg_quantize_tensors(g[:1], 4, 32, seed=0)
    layers.append({"params": torch.zeros(64, device=DEV), "packed": [outs[0][0]] * W, "scales": [outs[0][1]] * W})
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_aggregate_update_tensors(layers, W, 4, 32, 0.1)
    torch.cuda.synchronize()


# ---- the [min, max] encoding (Section 3.2 footnote) with several layers per launch -------------------

MINMAX_SIZES = [n for _, n in workloads.SMALL_CNN_SHAPES] + [0, 1, 40000 + 3, 3 * 16384 + 4096 + 37]


@pytest.mark.parametrize("bucket", [96, 512, 2048, 4096, 6144, 8192, 12288, 16384, 0])
def test_batched_minmax_encode_equals_the_oracle_per_layer(bucket):
    # bucket 0: one range per layer, as the paper encodes (the oracle with one bucket that covers the layer)
    grads = [workloads.normal_with_outliers(n, 0.01, 1e-3, 25.0, 90 + i, DEV) + 1e-3 * i if n else torch.empty(0, device=DEV)
             for i, n in enumerate(MINMAX_SIZES)]
    for bits in (1, 3, 4, 8):
        outs = mqgrad.mqg_quantize_minmax_tensors(grads, bits, bucket)
        torch.cuda.synchronize()
        for i, g in enumerate(grads):
            n = MINMAX_SIZES[i]
            if n == 0:
                continue
            pk_o, rg_o = ref.quantize_minmax(g.cpu().numpy(), bits, bucket if bucket else n)
            assert outs[i][1].cpu().numpy().tobytes() == rg_o.tobytes(), "ranges of layer %d b=%d" % (i, bits)
            assert np.array_equal(to_u32(outs[i][0]), pk_o), "layer %d b=%d" % (i, bits)


@pytest.mark.parametrize("bucket", [160, 1024, 0])
@pytest.mark.parametrize("bits", [2, 3, 5, 8])
def test_batched_minmax_server_step_with_raw_small_layers(bits, bucket):
    # the paper's selective quantization with the footnote's encoder: large layers encoded, small ones raw;
    # one encode call per worker and one update launch
    W, lr = 3, 0.1
    shapes = workloads.SMALL_CNN_SHAPES
    encoded = [n >= 4096 for _, n in shapes]
    e_idx = [i for i, e in enumerate(encoded) if e]
    grads = [[workloads.laplace(n, 2e-3, 1000 * w + i, DEV) + 5e-4 * w for i, (_, n) in enumerate(shapes)] for w in range(W)]
    params = [workloads.uniform(n, -0.05, 0.05, 40 + i, DEV) for i, (_, n) in enumerate(shapes)]
    p0 = [p.cpu().numpy().copy() for p in params]
    outs = [mqgrad.mqg_quantize_minmax_tensors([grads[w][i] for i in e_idx], bits, bucket) for w in range(W)]
    layers = []
    for i in range(len(shapes)):
        if encoded[i]:
            k = e_idx.index(i)
            layers.append({"params": params[i], "packed": [outs[w][k][0] for w in range(W)],
                           "scales": [outs[w][k][1] for w in range(W)]})
        else:
            layers.append({"params": params[i], "raw": [grads[w][i] for w in range(W)]})
    mqgrad.mqg_aggregate_update_minmax_tensors(layers, W, bits, bucket, lr)
    torch.cuda.synchronize()
    for i, (_, n) in enumerate(shapes):
        if encoded[i]:
            B = bucket if bucket else n
            want = [ref.quantize_minmax(grads[w][i].cpu().numpy(), bits, B) for w in range(W)]
            p1 = ref.aggregate_update_minmax([x[0] for x in want], [x[1] for x in want], n, bits, B, lr, p0[i])
        else:
            p1 = ref.average_update_raw([grads[w][i].cpu().numpy() for w in range(W)], lr, p0[i])
        assert ulp_distance(params[i].cpu().numpy(), p1).max() == 0, "layer %d" % i


def test_batched_minmax_calls_report_bad_arguments():
    g = [workloads.normal(64, 0.01, i, DEV) for i in range(33)]
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_quantize_minmax_tensors(g, 4, 32)            # more than MQG_MAX_TENSORS layers
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_quantize_minmax_tensors(g[:2], 9, 32)        # bits outside 1..8
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_quantize_minmax_tensors(g[:2], 4, 48)        # bucket not a multiple of 32
    outs = mqgrad.mqg_quantize_minmax_tensors(g[:1], 4, 0)
    layers = [{"params": torch.zeros(64, device=DEV), "packed": [outs[0][0]] * 8, "scales": [outs[0][1]] * 8}] * 17
    with pytest.raises(mqgrad.MqgError):
        mqgrad.mqg_aggregate_update_minmax_tensors(layers, 8, 4, 0, 0.1)   # 272 pointers
    mqgrad.mqg_aggregate_update_minmax_tensors(layers[:16], 8, 4, 0, 0.1)
    torch.cuda.synchronize()


# (layers, encoded ones among them, workers): the largest batch that travels in the small form of the kernels' arguments (12
# layers, 96 pointers), one more layer, more pointers, and the most of both
@pytest.mark.parametrize("count,encoded,W", [(12, 4, 6), (13, 4, 1), (12, 4, 7), (12, 12, 5), (32, 32, 4), (20, 5, 10)])
@pytest.mark.parametrize("kind,bits,bucket", [("centred", 2, 512), ("centred", 3, 64), ("centred", 4, 96), ("centred", 5, 1024), ("centred", 8, 32),
                                              ("minmax", 2, 160), ("minmax", 7, 2048), ("minmax", 3, 1024), ("minmax", 8, 512), ("minmax", 4, 0)])
def test_batched_server_steps_of_many_layers_and_workers(kind, bits, bucket, count, encoded, W):
    lr = 0.1
    sizes = [(i * 7919 + 613) % 9000 + 1 for i in range(count)]
    sizes[1] = 0
    grads = [[workloads.laplace(n, 2e-3, 100 * w + i, DEV) + 5e-4 * w if n else torch.empty(0, device=DEV) for i, n in enumerate(sizes)] for w in range(W)]
    params = [workloads.uniform(max(n, 1), -0.05, 0.05, 40 + i, DEV)[:n] for i, n in enumerate(sizes)]
    p0 = [p.cpu().numpy().copy() for p in params]
    if kind == "centred":
        outs = [mqgrad.mqg_quantize_tensors(grads[w][:encoded], bits, bucket, seed=w, iteration=1, worker=w) for w in range(W)]
    else:
        outs = [mqgrad.mqg_quantize_minmax_tensors(grads[w][:encoded], bits, bucket) for w in range(W)]
    layers = [{"params": params[i], "packed": [outs[w][i][0] for w in range(W)], "scales": [outs[w][i][1] for w in range(W)]} if i < encoded
              else {"params": params[i], "raw": [grads[w][i] for w in range(W)]} for i in range(count)]
    (mqgrad.mqg_aggregate_update_tensors if kind == "centred" else mqgrad.mqg_aggregate_update_minmax_tensors)(layers, W, bits, bucket, lr)
    torch.cuda.synchronize()
    for i, n in enumerate(sizes):
        if n == 0:
            continue
        if i >= encoded:
            p1 = ref.average_update_raw([grads[w][i].cpu().numpy() for w in range(W)], lr, p0[i])
        else:
            pk, sc = [to_u32(outs[w][i][0]) for w in range(W)], [outs[w][i][1].cpu().numpy() for w in range(W)]
            step = ref.aggregate_update if kind == "centred" else ref.aggregate_update_minmax
            p1 = step(pk, sc, n, bits, bucket if bucket else n, lr, p0[i])
        assert ulp_distance(params[i].cpu().numpy(), p1).max() == 0, "layer %d" % i


# (kind, bits, bucket, elements of the first tensor): each encoder's shapes, in batches of 12 tensors and of 13
@pytest.mark.parametrize("count", [12, 13])
@pytest.mark.parametrize("kind,bits,bucket,first", [
    ("maxabs", 2, 512, (1 << 24) + 5), ("maxabs", 5, 512, (1 << 24) + 5), ("maxabs", 4, 4096, 9001), ("maxabs", 2, 1184, 9001), ("maxabs", 8, 1184, 9001),
    ("maxabs", 2, 1376, 9001), ("maxabs", 8, 1376, 9001), ("maxabs", 2, 1760, 9001), ("maxabs", 8, 1760, 9001), ("maxabs", 5, 6176, 20001),
    ("maxabs", 6, 12320, 30001), ("l2", 3, 96, 9001), ("minmax", 4, 832, 9001), ("minmax", 3, 1088, 9001), ("minmax", 5, 1760, 9001),
    ("minmax", 2, 7200, 20001), ("minmax", 7, 14400, 40001)])
def test_batched_encoders_equal_the_single_ones_at_either_size_of_batch(kind, bits, bucket, first, count):
    sizes = [first] + [(i * 7919 + 613) % 9000 + 1 for i in range(1, count)]
    grads = [workloads.normal(n, 0.01, 60 + i, DEV) for i, n in enumerate(sizes)]
    if kind == "minmax":
        batch = mqgrad.mqg_quantize_minmax_tensors(grads, bits, bucket)
        alone = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
    else:
        mode = mqgrad.MQG_SCALE_L2 if kind == "l2" else mqgrad.MQG_SCALE_MAXABS
        bases = [(1 << 25) * i for i in range(count)]
        batch = mqgrad.mqg_quantize_tensors(grads, bits, bucket, seed=4, iteration=7, worker=2, elem_bases=bases, scale_mode=mode)
        alone = [mqgrad.mqg_quantize(g, bits, bucket, 4, 7, 2, bases[i], mode=mode) for i, g in enumerate(grads)]
    torch.cuda.synchronize()
    for i, (b, a) in enumerate(zip(batch, alone)):
        assert torch.equal(b[0], a[0]) and torch.equal(b[1], a[1]), "tensor %d" % i
