"""One [min, max] range per tensor, at the sizes where its launches change: the largest tensor of one
workgroup, tails of the server's tiles with fewer than two words, several workgroups per tensor."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import to_u32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TILE = 4096      # elements per workgroup of the server's two passes


def encode(grads, bits):
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    torch.cuda.synchronize()
    for g, (pk, rg) in zip(grads, q):
        pk_o, rg_o = ref.quantize_minmax(g.cpu().numpy(), bits, g.numel())
        assert rg.cpu().numpy().tobytes() == rg_o.tobytes()
        assert np.array_equal(to_u32(pk), pk_o)
    return q


@pytest.mark.parametrize("bits", [1, 3, 4, 8])
@pytest.mark.parametrize("n", [4095, 8193, 16384, 16385, 5 * TILE + 1, 5 * TILE + 4, 5 * TILE + 32, 5 * TILE + 33,
                               6 * TILE, 9 * 8192 - 1, 1030 * 8192 + 2049])
def test_tensor_range_exchange_at_the_edges(n, bits):
    W = 3
    grads = [workloads.laplace(n + 1, 1e-3, 5 * w + bits, DEV)[1:] + 1e-4 * w for w in range(W)]   # off a 16-byte boundary
    grads[0][n - 1] = 0.5            # the largest value is the tensor's last, the smallest its first
    grads[1][0] = -0.75
    q = encode(grads, bits)
    want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, n)
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
    assert np.array_equal(to_u32(pk), want_pk)
    # the mean's codes in the place of a worker's
    mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits, packed_out=q[1][0])
    torch.cuda.synchronize()
    assert np.array_equal(to_u32(q[1][0]), want_pk)


@pytest.mark.parametrize("extra", [0, 1])
def test_the_largest_folded_step_and_the_first_with_atomics(extra):
    n, bits, W = 16384 * TILE + extra, 2, 2
    grads = [workloads.normal(n, 1e-2, 3 + w, DEV) for w in range(W)]
    grads[1][n - 1] = 0.5
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, n)
    assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
    assert np.array_equal(to_u32(pk), want_pk)


@pytest.mark.parametrize("W,bits", [(1, 1), (64, 1), (24, 4)])
@pytest.mark.parametrize("tail", [1, 4, 8, 9, 32, 33])
def test_tails_without_two_words_of_their_own(tail, W, bits):
    for tiles in (4, 5, 41):
        n = tiles * TILE + tail
        grads = [workloads.laplace(n, 1e-3, 5 * w + bits, DEV) + 1e-4 * w for w in range(W)]
        q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
        pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
        torch.cuda.synchronize()
        want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, n)
        assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
        assert np.array_equal(to_u32(pk), want_pk)


@pytest.mark.parametrize("sizes", [[1, 5, 8191], [16384, 3, 70001], [8 * 8192, 1, 33, 2 * 8192 - 1, 2 * 8192]])
def test_batched_tensor_ranges_mix_one_and_several_workgroups(sizes):
    grads = [workloads.normal(n, 1e-2, 3 + n, DEV) for n in sizes]
    for bits in (1, 5):
        outs = mqgrad.mqg_quantize_minmax_tensors(grads, bits, 0)
        torch.cuda.synchronize()
        for g, (pk, rg) in zip(grads, outs):
            pk_o, rg_o = ref.quantize_minmax(g.cpu().numpy(), bits, g.numel())
            assert rg.cpu().numpy().tobytes() == rg_o.tobytes()
            assert np.array_equal(to_u32(pk), pk_o)


@pytest.mark.parametrize("n", [3, 2047, 8191, 8192, 8195, 4 * 8192 + 2052, 512 * 8192 - 1, 512 * 8192 + 1, 513 * 8192 + 2051])
def test_ranges_at_the_edges_of_pieces_and_grids(n):
    g = workloads.normal(n + 1, 1e-2, 5, DEV)[1:]      # off a 16-byte boundary
    for at in (0, n // 2, n - 1):                      # the extremes where the share of a workgroup begins or ends
        g[at] = 0.5 + at
        g[n - 1 - at] = -0.5 - at
        rg = mqgrad.mqg_tensor_range(g)
        pk, rt = mqgrad.mqg_quantize_minmax_tensor(g, 3)
        torch.cuda.synchronize()
        assert rg.tolist() == rt.tolist() == [g.min().item(), g.max().item()]
    assert np.array_equal(to_u32(pk), ref.quantize_minmax(g.cpu().numpy(), 3, n)[0])


@pytest.mark.parametrize("n", [5000, 16384, 70001])
def test_values_that_are_not_numbers_take_no_part_in_a_tensors_range(n):
    g = workloads.normal(n, 1e-2, 9, DEV)
    g[8:12] = float("nan")           # all that one lane holds
    rest = torch.cat([g[:8], g[12:]])
    _, rg = mqgrad.mqg_quantize_minmax_tensor(g, 4)
    torch.cuda.synchronize()
    assert rg.tolist() == [rest.min().item(), rest.max().item()]
