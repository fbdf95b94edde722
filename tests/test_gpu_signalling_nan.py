"""A signalling NaN in a gradient takes no part in a range, and no finite value beside it is lost with it."""
import numpy as np
import pytest
import torch

from paper_1804_08066_amd import mqgrad, workloads

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SIGNALLING = [0x7F800001, 0xFF800001, 0x7FBFFFFF, 0xFFA00000]


def poisoned(n, bucket, seed):
    """A gradient with one signalling NaN per bucket, at every place of a quad beside the bucket's smallest and largest
    value, and the gradient with zeros (a value inside every range) in their place."""
    g = workloads.normal(n, 1e-2, seed, DEV).cpu().numpy()
    with_nan = g.copy()
    for k in range(0, n, bucket):
        quads = min(n - k, bucket) // 4
        if quads == 0:
            continue
        quad = k + 4 * (k // bucket % quads)
        at = np.random.default_rng(k).permutation(4)
        g[quad + at[0]], g[quad + at[1]] = 0.5 + k / n, -0.75 - k / n
        g[quad + at[2]] = 0.0
        with_nan[quad:quad + 4] = g[quad:quad + 4]
        with_nan.view(np.uint32)[quad + at[2]] = SIGNALLING[k // bucket % 4]
    return torch.from_numpy(with_nan).to(DEV), torch.from_numpy(g).to(DEV)


def same_ranges_and_numbers(got, want, bits, bad):
    assert got[1].cpu().numpy().tobytes() == want[1].cpu().numpy().tobytes()
    differing = (got[0] ^ want[0]).cpu().numpy().view(np.uint32)
    bit = np.nonzero(np.unpackbits(differing.view(np.uint8), bitorder="little"))[0]
    assert np.isin(bit // bits, bad).all()        # only codes of the NaN themselves may differ


@pytest.mark.parametrize("bits", [1, 4, 7])
@pytest.mark.parametrize("bucket", [32, 512, 1024, 2048, 8192, 16384, 96, 2304, 4128, 8224])
@pytest.mark.parametrize("n", [5003, 70001])
def test_bucket_ranges_keep_what_stands_beside_a_signalling_nan(n, bucket, bits):
    g, finite = poisoned(n, bucket, 3 + bits)
    bad = np.nonzero(np.isnan(g.cpu().numpy()))[0]
    results = [(mqgrad.mqg_quantize(x, bits, bucket, 5), mqgrad.mqg_quantize_tensors([x], bits, bucket, 5)[0],
                mqgrad.mqg_quantize_minmax(x, bits, bucket), mqgrad.mqg_quantize_minmax_tensors([x], bits, bucket)[0]) for x in (g, finite)]
    torch.cuda.synchronize()
    for got, want in zip(*results):
        same_ranges_and_numbers(got, want, bits, bad)


@pytest.mark.parametrize("n", [5003, 16384, 70001, 1 << 21])
def test_tensor_ranges_keep_what_stands_beside_a_signalling_nan(n):
    g, finite = poisoned(n, 1 << (n.bit_length() - 3), 7)
    bad = np.nonzero(np.isnan(g.cpu().numpy()))[0]
    results = [(mqgrad.mqg_quantize_minmax_tensor(x, 4), mqgrad.mqg_quantize_minmax_tensors([x, x[:n // 2]], 4, 0)[0], mqgrad.mqg_tensor_range(x))
               for x in (g, finite)]
    torch.cuda.synchronize()
    for got, want in zip(*(r[:2] for r in results)):
        same_ranges_and_numbers(got, want, 4, bad)
    assert results[0][2].tolist() == results[1][2].tolist()
