"""The [min, max] encoders' workgroup sizes: four to seven waves for whole buckets up to 4096 elements, one bucket
per workgroup above, with ends that are whole quads or single elements."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import to_u32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("W,bits", [(3, 3), (2, 4), (50, 8)])
@pytest.mark.parametrize("bucket", [96, 4064, 2304, 2752, 1792, 4128, 6176, 8224, 12320, 16352, 32, 1024, 4096, 8192, 16384])
def test_minmax_tiles_match_the_oracle(bucket, W, bits):
    tile = max(7168, bucket)
    for n in (bucket - 1, 2 * tile, 2 * tile + 36, 2 * tile + bucket // 2 + 3):
        grads = [workloads.laplace(n + 1, 1e-3, 31 * w + bits, DEV)[1:] + 2e-4 * (w % 3 - 1) for w in range(W)]
        q = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
        mean = mqgrad.mqg_aggregate_requantize_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket)
        batch = mqgrad.mqg_quantize_minmax_tensors(grads[:2], bits, bucket)
        torch.cuda.synchronize()
        want = [ref.quantize_minmax(g.cpu().numpy(), bits, bucket) for g in grads]
        for got in (q, batch):
            for (pk, rg), (pk_o, rg_o) in zip(got, want):
                assert rg.cpu().numpy().tobytes() == rg_o.tobytes(), n
                assert np.array_equal(to_u32(pk), pk_o), n
        pk_o, rg_o = ref.aggregate_requantize_minmax([w[0] for w in want], [w[1] for w in want], n, bits, bucket)
        assert mean[1].cpu().numpy().tobytes() == rg_o.tobytes(), n
        assert np.array_equal(to_u32(mean[0]), pk_o), n


# The re-encoding step keeps eight workers' words in flight in short launches and four in longer ones; up to four workers
# take no loop.  Where a compute unit gets at most one workgroup (256 of them), it has four waves whatever the bucket.
@pytest.mark.parametrize("bucket,tile,tiles", [(1024, 4096, 512), (96, 42 * 96, 512), (2304, 4608, 256), (2304, 2304, 256), (2752, 5504, 256),
                                               (2752, 2752, 256), (1792, 7168, 256), (1792, 3584, 256), (4128, 4128, 256), (8192, 8192, 256),
                                               (12320, 12320, 256)])
@pytest.mark.parametrize("W,bits", [(4, 1), (4, 3), (4, 4), (4, 5), (5, 1), (5, 3), (5, 4), (5, 5), (9, 8)])
def test_reencoding_at_the_edges_of_a_short_launch(bucket, tile, tiles, W, bits):
    base = workloads.laplace(tiles * tile + 1, 1e-3, W, DEV)
    grads = [(base.roll(977 * w) * (1 + w)) for w in range(W)]
    for n in (tiles * tile, tiles * tile + 1):
        q = [mqgrad.mqg_quantize_minmax(g[:n], bits, bucket) for g in grads]
        got = mqgrad.mqg_aggregate_requantize_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket)
        torch.cuda.synchronize()
        pk_o, rg_o = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, bucket)
        assert got[1].cpu().numpy().tobytes() == rg_o.tobytes()
        assert np.array_equal(to_u32(got[0]), pk_o)
