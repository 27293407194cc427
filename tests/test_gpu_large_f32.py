"""fp32 products over blocks of 2 GiB and more, which the contraction kernels'
32-bit byte offsets do not reach: the vector-ALU kernel, against torch's fp64
product on the rows at both ends and past each 2 GiB bound.

Tolerance: sums of 16400 fp32 products of N(0,1) data in ascending order, each
within about sqrt(K) * 2^-24 of its norm: 1e-5.
"""
import pytest
import torch

from helpers import describe
from paper_2609_03905_amd import ea

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kmajor", [False, True])
def test_operand_block_beyond_2_gib(kmajor):
    m, k, n = 33000, 16400, 40
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    a = torch.randn((m, k), generator=g, device="cuda")
    b = torch.randn((n, k) if kmajor else (k, n), generator=g, device="cuda")
    spec, pb = ("ij,kj->ik", [[0, n], [0, k]]) if kmajor else ("ij,jk->ik", [[0, k], [0, n]])
    ops = [((m, k), "f32", [[0, m], [0, k]]), (tuple(b.shape), "f32", pb), ((m, n), "f32", [[0, m], [0, n]])]
    assert describe(spec, ea.JOIN_MUL, ea.AGG_SUM, ops)["kind"] == "gemm32"
    A, B = (ea.Relation(s, d, p, data=x.view(torch.uint8).reshape(-1)) for (s, d, p), x in zip(ops, (a, b)))
    C = ea.Relation((m, n), "f32", ops[2][2])
    C.data.fill_(0xFF)
    ea.joinagg(spec, ea.JOIN_MUL, ea.AGG_SUM, [A, B], C)
    torch.cuda.synchronize()
    got = C.bytes().view(torch.float32).reshape(m, n)
    edge = (1 << 31) // (4 * k)  # the row that crosses 2 GiB
    rows = torch.tensor([0, 1, edge - 1, edge, edge + 1, m - 1], device="cuda")
    ref = a[rows].double() @ (b.T if kmajor else b).double()
    assert float((got[rows].double() - ref).norm() / ref.norm()) < 1e-5
    assert bool(torch.isfinite(got).all())
