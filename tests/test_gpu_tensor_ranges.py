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


def codes(pk, n, bits):
    return ref.unpack(to_u32(pk), n, bits)


@pytest.mark.parametrize("n", [5000, 16384, 70001])
def test_values_that_are_not_numbers_take_no_part_in_a_tensors_range(n):
    bits = 4
    g = workloads.normal(n, 1e-2, 9, DEV)
    g[8:12] = float("nan")           # all that one lane holds
    g[n - 7] = float("nan")
    numbers = ~torch.isnan(g)
    mn, mx = g[numbers].min().item(), g[numbers].max().item()
    filled = torch.where(numbers, g, torch.full_like(g, mn))       # the oracle's codes over the same range
    want = codes(torch.from_numpy(ref.quantize_minmax(filled.cpu().numpy(), bits, n)[0].view(np.int32)), n, bits)
    batch = mqgrad.mqg_quantize_minmax_tensors([filled, g, g[:33]], bits, 0)[1]
    for pk, rg in (mqgrad.mqg_quantize_minmax_tensor(g, bits), batch):
        torch.cuda.synchronize()
        assert rg.tolist() == [mn, mx]
        assert np.array_equal(codes(pk, n, bits), want)            # a NaN's own code is 0, which is the smallest value's
    assert mqgrad.mqg_tensor_range(g).tolist() == [mn, mx]


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf")])
@pytest.mark.parametrize("n", [5000, 16384, 16385, 70001])
def test_one_workers_range_that_is_not_finite(n, bad):
    """The sum has no number in it, or infinities of one sign: small tensors (one workgroup) and larger ones agree on
    the rule, and on the codes."""
    bits, W = 4, 3
    grads = [workloads.normal(n, 1e-2, 9 + w, DEV) for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    q[1][1][:] = bad
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    # a step of inf - inf or NaN makes every value of that worker NaN: the empty range, and code 0 throughout
    assert rg.tolist() == [float("inf"), float("-inf")]
    assert not codes(pk, n, bits).any()


@pytest.mark.parametrize("bucket", [32, 1024, 96, 2304, 4128, 8192])
def test_infinities_and_zeros_of_both_signs_in_a_bucket(bucket):
    """A bucket with infinities has them as its range and code 0 throughout; a bucket of values from 0 up with zeros of both
    signs has the range from +0 and code 0 for either zero.  Its neighbours are as ever."""
    bits, n = 3, 6 * bucket
    g = workloads.normal(n, 1e-2, 4, DEV)
    g[bucket + 5] = float("inf")
    g[2 * bucket + 7] = float("-inf")
    g[3 * bucket + 1], g[3 * bucket + 2] = float("inf"), float("-inf")
    g[4 * bucket:5 * bucket] = g[4 * bucket:5 * bucket].abs()
    g[4 * bucket:5 * bucket:3] = 0.0
    g[4 * bucket + 1:5 * bucket:3] = -0.0
    host = g.cpu().numpy()
    batch = mqgrad.mqg_quantize_minmax_tensors([g], bits, bucket)[0]
    for pk, rg in (mqgrad.mqg_quantize_minmax(g, bits, bucket), batch):
        torch.cuda.synchronize()
        rg, code = rg.cpu().numpy().reshape(-1, 2), codes(pk, n, bits)
        for k in range(6):
            part = host[k * bucket:(k + 1) * bucket]
            assert rg[k].tolist() == [part.min(), part.max()]
            if k in (1, 2, 3):
                assert not code[k * bucket:(k + 1) * bucket].any()
            else:
                assert np.array_equal(code[k * bucket:(k + 1) * bucket], codes(torch.from_numpy(ref.quantize_minmax(part, bits, bucket)[0].view(np.int32)), bucket, bits))
        assert not np.signbit(rg[4, 0])
        assert not code[4 * bucket:5 * bucket:3].any() and not code[4 * bucket + 1:5 * bucket:3].any()


def most_parts(bits):
    return min(32 * bits, 128)          # pairs of keys that two tiles' words hold


@pytest.mark.parametrize("bits", range(1, 9))
@pytest.mark.parametrize("tail", [1, 33, 64 * 4 + 1, TILE // 2, TILE - 1, TILE])
def test_ranges_that_travel_in_the_output(bits, tail):
    """Small tensors, where every workgroup of the encoder and of the server's second pass folds the range itself: the most
    workgroups that may find it, one more, and two, with every kind of last tile."""
    W = 2
    for find, per in ((8192, "encoder"), (TILE, "server")):
        for parts in (2, most_parts(bits), most_parts(bits) + 1):
            n = (parts - 1) * TILE + tail if per == "server" else parts * 8192 - 8192 % TILE + tail % 8192
            if n <= 16384:
                continue
            grads = [workloads.laplace(n + 1, 1e-3, 7 * w + bits, DEV)[1:] + 1e-4 * w for w in range(W)]
            grads[0][n - 1], grads[1][0], grads[1][n // 2] = 0.5, -0.75, 0.25
            q = encode(grads, bits)
            want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, n)
            pk, rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
            torch.cuda.synchronize()
            assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
            assert np.array_equal(to_u32(pk), want_pk)


@pytest.mark.parametrize("bits", [1, 3, 4])
@pytest.mark.parametrize("sizes", [(20000, 17, 100_000, 8191), (0, 16384, 40_961, 5), (33_000, 2_000_000, 70_001), tuple(16385 + 77 * i for i in range(14))])
def test_ranges_of_several_layers(sizes, bits):
    """All layers' ranges in the output, some layers of one workgroup, one layer too large (none in the output), more layers
    than the small form of the arguments takes."""
    grads = [workloads.laplace(n, 1e-3, i + bits, DEV) + 1e-4 * i for i, n in enumerate(sizes)]
    for g in grads:
        if g.numel() > 3:
            g[-1], g[g.numel() // 2] = 0.5, -0.25
    out = mqgrad.mqg_quantize_minmax_tensors(grads, bits, 0)
    torch.cuda.synchronize()
    for g, (pk, rg) in zip(grads, out):
        if g.numel() == 0:
            continue
        want_pk, want_rg = ref.quantize_minmax(g.cpu().numpy(), bits, g.numel())
        assert rg.cpu().numpy().tobytes() == want_rg.tobytes(), g.numel()
        assert np.array_equal(to_u32(pk), want_pk), g.numel()
