"""The quantizer's wave shapes by the size of the launch: 512 elements per wave up to 2^21 elements, 1024 up to 2^24,
then 2048 -- for single tensors and for the layers of a batch together."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_1804_08066_amd import mqgrad, workloads
from helpers import to_u32

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TINY, SHORT = 1 << 21, 1 << 24


def check(got, g, bits, bucket, worker, base):
    pk_o, sc_o = ref.quantize(g.cpu().numpy(), bits, bucket, 11, 2, worker, base)
    assert np.array_equal(to_u32(got[0]), pk_o)
    assert np.array_equal(got[1].cpu().numpy(), sc_o)


@pytest.mark.parametrize("bits,bucket", [(1, 32), (3, 512), (5, 256), (8, 512), (4, 1024), (7, 128)])
@pytest.mark.parametrize("n", [3, 511, 513, 4 * 512 + 5, TINY, TINY + 1])
def test_single_tensors_at_the_edges(n, bits, bucket):
    g = workloads.student_t(n + 1, 3, 1e-3, n % 97 + bits, DEV)[1:]   # off a 16-byte boundary
    got = mqgrad.mqg_quantize(g, bits, bucket, 11, 2, 5, elem_base=1024)
    torch.cuda.synchronize()
    check(got, g, bits, bucket, 5, 1024)


@pytest.mark.parametrize("n", [SHORT, SHORT + 4])
def test_single_tensors_at_the_larger_edge(n):
    g = workloads.normal(n, 1e-2, 3, DEV)
    got = mqgrad.mqg_quantize(g, 4, 512, 11, 2, 5)
    torch.cuda.synchronize()
    check(got, g, 4, 512, 5, 0)


@pytest.mark.parametrize("total,bits", [(TINY, 6), (TINY + 1, 6), (SHORT, 6), (SHORT + 1, 6), (SHORT + 1, 3)])
def test_layers_together_choose_the_shape(total, bits):
    sizes = [5, 0, 1000003, 4096, total - 1000003 - 4096 - 5 - 700, 700]
    grads = [workloads.laplace(max(n, 1), 1e-3, i, DEV)[:n] for i, n in enumerate(sizes)]
    bases = [8 * 1024 * i for i in range(len(sizes))]
    got = mqgrad.mqg_quantize_tensors(grads, bits, 64, 11, 2, 5, bases)
    torch.cuda.synchronize()
    for g, q, base in zip(grads, got, bases):
        if g.numel():
            check(q, g, bits, 64, 5, base)


@pytest.mark.parametrize("bucket", [32, 64, 128, 256, 512, 1024])
def test_l2_norms_do_not_depend_on_the_shape(bucket):
    g = workloads.normal(SHORT + 4096, 1e-2, 9, DEV)
    whole = mqgrad.mqg_quantize(g, 4, bucket, 11, mode=mqgrad.MQG_SCALE_L2)
    for n in (TINY, SHORT):
        part = mqgrad.mqg_quantize(g[:n], 4, bucket, 11, mode=mqgrad.MQG_SCALE_L2)
        assert torch.equal(part[1], whole[1][:n // bucket]) and torch.equal(part[0], whole[0][:n // 8])
