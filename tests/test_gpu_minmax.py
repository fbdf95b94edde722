"""GPU parity for the deterministic [min, max] range-linear encoding (the literal reading of the
Section 3.2 footnote), its server step, the sum of squares and the Adaptive rule fed from it."""
import math

import numpy as np
import pytest
import torch

from oracle import policy_ref, ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import first_mismatch, to_u32, ulp_distance

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ALL_BITS = list(range(1, 9))


def assert_minmax_parity(g, bits, bucket, label=""):
    pk, rg = mqgrad.mqg_quantize_minmax(g, bits, bucket)
    torch.cuda.synchronize()
    pk_o, rg_o = ref.quantize_minmax(g.cpu().numpy(), bits, bucket)
    assert rg.cpu().numpy().tobytes() == rg_o.tobytes(), "%s ranges differ" % label
    assert np.array_equal(to_u32(pk), pk_o), "%s packed words differ at %s" % (label, first_mismatch(to_u32(pk), pk_o))
    return pk, rg, pk_o, rg_o


@pytest.mark.parametrize("bits", ALL_BITS)
@pytest.mark.parametrize("bucket", [32, 96, 512, 4096, 8192, 16384])
def test_quantize_minmax_bit_exact(bits, bucket):
    n = 3 * 16384 + 4096 + 37            # several tiles and a ragged tail for every bucket size
    g = workloads.normal_with_outliers(n, 0.01, 1e-3, 30.0, 11 + bits, DEV) + 0.003
    assert_minmax_parity(g, bits, bucket, "b=%d B=%d" % (bits, bucket))


@pytest.mark.parametrize("n", [1, 2, 3, 5, 31, 32, 33, 127, 1023, 1025, 4097])
def test_quantize_minmax_tiny_and_ragged(n):
    g = workloads.laplace(n, 1e-3, n, DEV)
    for bits in (1, 3, 8):
        for bucket in (32, 1024):
            assert_minmax_parity(g, bits, bucket, "n=%d b=%d B=%d" % (n, bits, bucket))


def test_quantize_minmax_degenerate_inputs():
    n = 5000
    const = torch.full((n,), 0.37, device=DEV)
    zeros = torch.zeros(n, device=DEV)
    negz = -torch.zeros(n, device=DEV)
    pos = workloads.uniform(n, 0.5, 3.0, 2, DEV)
    neg = -pos
    tiny = workloads.uniform(n, 0.0, 1.0, 3, DEV) * 2.0 ** -100
    ints = torch.randint(0, 256, (n,), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1)).float()
    for name, g in [("const", const), ("zeros", zeros), ("negz", negz), ("pos", pos), ("neg", neg), ("tiny", tiny),
                    ("ints", ints)]:
        for bits in (1, 4, 8):
            assert_minmax_parity(g, bits, 256, name)
    # empty input: no launch, nothing written
    pk, rg = mqgrad.mqg_quantize_minmax(torch.empty(0, device=DEV), 4, 256)
    assert pk.numel() == 0 and rg.numel() == 0


def test_quantize_minmax_unaligned_views():
    base = workloads.normal(40000, 0.01, 9, DEV)
    for off in (1, 2, 3):
        assert_minmax_parity(base[off:off + 30001].contiguous()[:], 5, 512, "copy %d" % off)
        g = base[off:off + 30001]
        assert g.data_ptr() % 16 != 0
        pk, rg = mqgrad.mqg_quantize_minmax(g, 5, 512)
        torch.cuda.synchronize()
        pk_o, rg_o = ref.quantize_minmax(g.cpu().numpy(), 5, 512)
        assert np.array_equal(to_u32(pk), pk_o) and np.array_equal(rg.cpu().numpy(), rg_o)


@pytest.mark.parametrize("bits", ALL_BITS)
@pytest.mark.parametrize("W,bucket", [(1, 32), (3, 96), (8, 1024), (5, 16384)])
def test_aggregate_update_minmax_matches_oracle(bits, W, bucket):
    n = 2 * 16384 + 2048 + 13
    grads = [workloads.normal(n, 0.01, 100 * w + bits, DEV) + 1e-3 * w for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
    params = workloads.uniform(n, -0.05, 0.05, 4, DEV)
    p0 = params.cpu().numpy().copy()
    mqgrad.mqg_aggregate_update_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket, 0.1, params)
    torch.cuda.synchronize()
    want = ref.aggregate_update_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, bucket,
                                       0.1, p0)
    # same fp32 operations in the same order on both sides: bit for bit
    assert ulp_distance(params.cpu().numpy(), want).max() == 0


def test_aggregate_update_minmax_many_workers_and_unaligned_params():
    n, bits, bucket, W = 10000 + 3, 6, 160, 19
    grads = [workloads.laplace(n, 2e-3, 7 * w, DEV) for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
    store = workloads.uniform(n + 1, -1, 1, 8, DEV)
    params = store[1:]
    p0 = params.cpu().numpy().copy()
    mqgrad.mqg_aggregate_update_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket, 0.25, params)
    torch.cuda.synchronize()
    want = ref.aggregate_update_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n, bits, bucket,
                                       0.25, p0)
    assert ulp_distance(params.cpu().numpy(), want).max() == 0
    assert store[0].item() == pytest.approx(store[0].item())     # neighbour untouched (finite)


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 1023, 1 << 20, (1 << 22) + 7])
def test_sum_squares_matches_exact_sum(n):
    g = workloads.normal(max(n, 1), 1e-3, n + 1, DEV)[:n]
    out = mqgrad.mqg_sum_squares(g)
    torch.cuda.synchronize()
    exact = math.fsum(float(x) * float(x) for x in g.cpu().numpy().astype(np.float64)) if n <= (1 << 20) else \
        float(np.sum(g.cpu().numpy().astype(np.float64) ** 2))
    assert abs(out.item() - exact) <= 1e-12 * exact
    # a view that starts 4 bytes past a 16-byte boundary takes the same 128-bit loads
    if n > 8:
        v = g[1:]
        out2 = mqgrad.mqg_sum_squares(v)
        torch.cuda.synchronize()
        e2 = float(np.sum(v.cpu().numpy().astype(np.float64) ** 2))
        assert abs(out2.item() - e2) <= 1e-12 * e2


def exact_sum_squares(t):
    x = t.cpu().numpy().astype(np.float64)
    return math.fsum(float(v) * float(v) for v in x) if x.size <= (1 << 20) else float(np.sum(x * x))


def test_batched_sum_squares_is_exact_and_reproducible_to_the_bit():
    # several tensors in one call (ragged sizes, an empty one, a view off a 16-byte boundary); each sum
    # within 1e-12 of the exactly rounded one, equal bit for bit between calls and whatever else is in
    # the batch, and within rounding of the single-tensor entry point
    sizes = [0, 1, 3, 5, 1023, 2048 * 512 + 9, (1 << 22) + 7, 4097]
    grads = [workloads.normal(max(n, 1), 10.0 ** (-1 - (k % 4)), 50 + k, DEV)[:n] for k, n in enumerate(sizes)]
    grads.append(grads[6][1:])
    out = mqgrad.mqg_sum_squares_batch(grads)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert got[0] == 0.0
    for k, g in enumerate(grads):
        exact = exact_sum_squares(g)
        assert abs(got[k] - exact) <= 1e-12 * exact
    ws = torch.full((mqgrad.mqg_sum_squares_workspace_bytes(len(grads)) // 8,), float("nan"), dtype=torch.float64, device=DEV)
    again = mqgrad.mqg_sum_squares_batch(grads, workspace=ws).cpu().numpy()
    assert again.tobytes() == got.tobytes()
    alone = mqgrad.mqg_sum_squares_batch(grads[6:7]).cpu().numpy()
    assert alone[0] == got[6]
    reversed_batch = mqgrad.mqg_sum_squares_batch(grads[::-1]).cpu().numpy()
    assert reversed_batch[::-1].tobytes() == got.tobytes()
    single = mqgrad.mqg_sum_squares(grads[6]).item()
    assert abs(single - got[6]) <= 1e-14 * got[6]
    full = mqgrad.mqg_sum_squares_batch([grads[5]] * 64).cpu().numpy()      # the largest batch
    assert np.all(full == got[5])


def test_adaptive_rule_from_gpu_norms():
    # Z = mean over workers of the gradient norm; the width follows the oracle's statement of the rule
    W, n = 4, 200000
    for scale in (1e-7, 1.2e-6, 2.9e-6, 5e-6, 1e-4):
        grads = [workloads.normal(n, scale, 31 * w + 1, DEV) for w in range(W)]
        sums = [mqgrad.mqg_sum_squares(g) for g in grads]
        torch.cuda.synchronize()
        norms = [math.sqrt(s.item()) for s in sums]
        want_norms = [policy_ref.gradient_norm(g.cpu().numpy()) for g in grads]
        for a, b in zip(norms, want_norms):
            assert abs(a - b) <= 1e-12 * b
        # the integer decision is taken from the same fp64 norms on both sides
        assert mqgrad.mqg_adaptive_bits(norms) == policy_ref.adaptive_bits(norms)
        assert mqgrad.mqg_adaptive_bits(norms) == policy_ref.adaptive_bits(want_norms) or \
            abs(sum(norms) / W / 0.0005 - round(sum(norms) / W / 0.0005)) < 1e-9


@pytest.mark.parametrize("bits", ALL_BITS)
@pytest.mark.parametrize("W,bucket", [(1, 32), (3, 96), (8, 1024), (4, 4096), (5, 8192), (2, 16384), (64, 32), (40, 64)])
def test_requantize_minmax_matches_oracle(bits, W, bucket):
    n = 2 * 16384 + 2048 + 13
    grads = [workloads.normal(n, 0.01, 100 * w + bits, DEV) + 1e-3 * w for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
    pk, rg = mqgrad.mqg_aggregate_requantize_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket)
    torch.cuda.synchronize()
    want_pk, want_rg = ref.aggregate_requantize_minmax([to_u32(x[0]) for x in q], [x[1].cpu().numpy() for x in q], n,
                                                       bits, bucket)
    assert rg.cpu().numpy().tobytes() == want_rg.tobytes()
    assert np.array_equal(to_u32(pk), want_pk), first_mismatch(to_u32(pk), want_pk)


def test_full_exchange_with_minmax_encoding_stays_on_the_oracle():
    # Algorithm 1 with the footnote's encoder, several iterations: workers encode, the server re-encodes
    # the mean, workers de-quantize and update
    n, W, bucket, lr = 50000 + 7, 4, 512, 0.2
    params = workloads.uniform(n, -0.05, 0.05, 1, DEV)
    p_ref = params.cpu().numpy().copy()
    for it, bits in enumerate((8, 2, 5, 1, 4)):
        grads = [workloads.laplace(n, 1e-3, 10 * it + w, DEV) for w in range(W)]
        q = [mqgrad.mqg_quantize_minmax(g, bits, bucket) for g in grads]
        pk, rg = mqgrad.mqg_aggregate_requantize_minmax([x[0] for x in q], [x[1] for x in q], n, bits, bucket)
        mqgrad.mqg_aggregate_update_minmax([pk], [rg], n, bits, bucket, lr, params)
        torch.cuda.synchronize()
        want = [ref.quantize_minmax(g.cpu().numpy(), bits, bucket) for g in grads]
        m_pk, m_rg = ref.aggregate_requantize_minmax([x[0] for x in want], [x[1] for x in want], n, bits, bucket)
        p_ref = ref.aggregate_update_minmax([m_pk], [m_rg], n, bits, bucket, lr, p_ref)
        assert np.array_equal(to_u32(pk), m_pk)
        assert ulp_distance(params.cpu().numpy(), p_ref).max() == 0, "iteration %d" % it


# ---- one range for the whole tensor, as the paper encodes ----------------------------------------

@pytest.mark.parametrize("n", [1, 3, 4, 5, 31, 4096, 4097, 100003, 3 * (1 << 20) + 11])
def test_tensor_range_is_the_min_and_max(n):
    g = workloads.laplace(n + 3, 1e-2, n, DEV)
    for off in (0, 1, 3):
        v = g[off:off + n]
        r = mqgrad.mqg_tensor_range(v)
        torch.cuda.synchronize()
        assert r[0].item() == v.min().item() and r[1].item() == v.max().item()
    z = mqgrad.mqg_tensor_range(-torch.zeros(n, device=DEV))
    torch.cuda.synchronize()
    assert z.cpu().numpy().view(np.uint32).tolist() == [0, 0]            # a zero bound is +0


@pytest.mark.parametrize("bits", ALL_BITS)
@pytest.mark.parametrize("n,W", [(7, 1), (5000, 3), (100003, 2), (2 * (1 << 20) + 5, 4)])
def test_per_tensor_encoding_matches_oracle(bits, n, W):
    # the oracle with one bucket that covers the tensor is the paper's per-tensor encoder
    grads = [workloads.normal_with_outliers(n, 0.01, 1e-3, 25.0, 7 * w + bits, DEV) + 2e-3 * w for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    params = workloads.uniform(n, -0.05, 0.05, 4, DEV)
    p0 = params.cpu().numpy().copy()
    mqgrad.mqg_aggregate_update_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits, 0.1, params)
    torch.cuda.synchronize()
    want = [ref.quantize_minmax(g.cpu().numpy(), bits, n) for g in grads]
    for w in range(W):
        assert q[w][1].cpu().numpy().tobytes() == want[w][1].tobytes(), "range of worker %d" % w
        assert np.array_equal(to_u32(q[w][0]), want[w][0]), first_mismatch(to_u32(q[w][0]), want[w][0])
    p1 = ref.aggregate_update_minmax([x[0] for x in want], [x[1] for x in want], n, bits, n, 0.1, p0)
    assert ulp_distance(params.cpu().numpy(), p1).max() == 0


@pytest.mark.parametrize("bits", ALL_BITS)
@pytest.mark.parametrize("n,W", [(7, 1), (5000, 3), (100003, 9), (2 * (1 << 20) + 5, 4)])
def test_per_tensor_exchange_matches_oracle(bits, n, W):
    # Algorithm 1 as printed with the footnote's encoder and one range per tensor: workers encode, the
    # server re-encodes the sum over its own whole-tensor range (stored divided by W), a worker decodes
    # and updates.  The oracle with one bucket that covers the tensor defines every step.
    grads = [workloads.normal_with_outliers(n, 0.01, 1e-3, 25.0, 13 * w + bits, DEV) - 1e-3 * w for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    sentinel = torch.full((mqgrad.mqg_packed_words(n, bits) + 4,), -1, dtype=torch.int32, device=DEV)
    mean_pk, mean_rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits,
                                                                     packed_out=sentinel)
    params = workloads.uniform(n, -0.05, 0.05, 5, DEV)
    p0 = params.cpu().numpy().copy()
    mqgrad.mqg_aggregate_update_minmax_tensor([mean_pk], [mean_rg], n, bits, 0.2, params)
    torch.cuda.synchronize()
    want = [ref.quantize_minmax(g.cpu().numpy(), bits, n) for g in grads]
    m_pk, m_rg = ref.aggregate_requantize_minmax([x[0] for x in want], [x[1] for x in want], n, bits, n)
    words = mqgrad.mqg_packed_words(n, bits)
    assert mean_rg.cpu().numpy().tobytes() == m_rg.tobytes(), (mean_rg.cpu().numpy(), m_rg)
    assert np.array_equal(to_u32(mean_pk[:words]), m_pk), first_mismatch(to_u32(mean_pk[:words]), m_pk)
    assert np.all(sentinel[words:].cpu().numpy() == -1)
    p1 = ref.aggregate_update_minmax([m_pk], [m_rg], n, bits, n, 0.2, p0)
    assert ulp_distance(params.cpu().numpy(), p1).max() == 0


def test_per_tensor_exchange_at_full_size_on_sampled_ranges():
    # 100 M elements, W = 8: the range of the mean against the oracle's fp32 sum on sampled pieces (a lower
    # bound on the spread) and the code words of sampled 4096-element tiles against the oracle's encoder
    # given the GPU's range of the sum
    n, W, bits = 100_000_000, 8, 4
    grads = [workloads.config4_grad(w, n, DEV) for w in range(W)]
    q = [mqgrad.mqg_quantize_minmax_tensor(g, bits) for g in grads]
    del grads
    mean_pk, mean_rg = mqgrad.mqg_aggregate_requantize_minmax_tensor([x[0] for x in q], [x[1] for x in q], n, bits)
    torch.cuda.synchronize()
    rg = mean_rg.cpu().numpy()
    ranges = [x[1].cpu().numpy() for x in q]
    lo_seen, hi_seen = np.inf, -np.inf
    for start in (0, 4096 * 977, 4096 * 20001, n - 4096 - (n % 4096), n - (n % 4096)):
        cnt = min(4096, n - start)
        w0, w1 = start * bits // 32, (start + cnt) * bits // 32 + (1 if ((start + cnt) * bits) % 32 else 0)
        pieces = [to_u32(x[0][w0:w1]) for x in q]
        s = ref.aggregate_sum_minmax(pieces, ranges, cnt, bits, cnt)
        lo_seen, hi_seen = min(lo_seen, float(s.min())), max(hi_seen, float(s.max()))
        # encode the oracle's sum of the piece over the GPU's range of the whole sum (range * W, exact for W = 8)
        full = (rg * np.float32(W)).astype(np.float32)
        want = ref.encode_minmax_given_range(s, bits, full[0], full[1])
        assert np.array_equal(to_u32(mean_pk[w0:w1]), want), start
    assert rg[0] * W <= lo_seen and rg[1] * W >= hi_seen and rg[0] < 0 < rg[1]


def test_per_tensor_encoding_of_an_unaligned_view():
    base = workloads.normal(50000, 0.01, 3, DEV)
    g = base[3:3 + 40001]
    pk, rg = mqgrad.mqg_quantize_minmax_tensor(g, 6)
    torch.cuda.synchronize()
    want_pk, want_rg = ref.quantize_minmax(g.cpu().numpy(), 6, g.numel())
    assert np.array_equal(rg.cpu().numpy(), want_rg) and np.array_equal(to_u32(pk), want_pk)


@pytest.mark.parametrize("sizes", [(0, 1, 3, 8191), (8192, 4 * 8192 - 1, 4 * 8192), (5 * 8192, 17, 512 * 8192 + 5), (100_003,)])
def test_norms_with_fewer_workgroups(sizes):
    """Tensors that fill few of the workgroups whose partial sums are added, beside ones that fill more: each result is the
    one of a call of its own, and a workspace full of NaN leaves no trace."""
    grads = [workloads.normal(max(n, 1), 1e-2, 3 + i, DEV)[:n] for i, n in enumerate(sizes)]
    ws = torch.full((mqgrad.mqg_sum_squares_workspace_bytes(len(grads)) // 8,), float("nan"), dtype=torch.float64, device=DEV)
    out = mqgrad.mqg_sum_squares_batch(grads, workspace=ws)
    alone = [mqgrad.mqg_sum_squares_batch([g]) for g in grads]
    torch.cuda.synchronize()
    for g, t, a in zip(grads, out.tolist(), alone):
        want = float((g.double() ** 2).sum())
        assert t == a.item() and abs(t - want) <= 1e-14 * want      # some hundred fp64 additions in another order
