"""The re-encoding steps with one 32-element cell per lane, at the sizes from which they take over: every width, buckets
inside a wave, across waves and one per workgroup, worker counts around the words in flight, ragged ends at every offset
in a cell, streams too large for the last-level cache, ranges that are not finite."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import first_mismatch, to_u32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
M = 1 << 20


def gradients(n, W, seed):
    return [workloads.laplace(n, 1e-3, 31 * seed + w, DEV) + 1e-4 * w for w in range(W)]


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("n,W", [(3 * M // 2 + 1, 3), (3 * M // 2 + 2048, 1), (2 * M + 4, 9), (2 * M + 8192 + 33, 4), (2 * M + 77 * 32, 2)])
def test_whole_tensor_steps_match_the_oracle(n, W, bits):
    grads = gradients(n, W, bits)
    grads[0][n - 1] = 0.5            # the largest value is the tensor's last
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, n)
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
    assert np.array_equal(to_u32(pk), want_pk), first_mismatch(to_u32(pk), want_pk)
    mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits, packed_out=q[0][0])   # over a stream it reads
    torch.cuda.synchronize()
    assert np.array_equal(to_u32(q[0][0]), want_pk)


def test_whole_tensor_streams_larger_than_the_last_level_cache():
    bits, W = 8, 64
    n = (256 << 20) // W + 32 * 100 + 13
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in gradients(n, 2, bits)]
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([q[w % 2][0] for w in range(W)], [q[w % 2][1] for w in range(W)], n, bits)
    torch.cuda.synchronize()
    want = ref.aggregate_requantize_minmax([to_u32(q[w % 2][0]) for w in range(W)], [q[w % 2][1].cpu().numpy() for w in range(W)], n, bits, n)
    assert rg.cpu().numpy().tobytes() == want[1].tobytes()
    assert np.array_equal(to_u32(pk), want[0]), first_mismatch(to_u32(pk), want[0])


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
def test_a_tensors_range_that_is_not_finite(bad):
    bits, W, n = 4, 3, 3 * M // 2 + 9
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in gradients(n, W, 3)]
    q[1][1][:] = bad
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    assert rg.tolist() == [float("inf"), float("-inf")]
    assert not to_u32(pk).any()
