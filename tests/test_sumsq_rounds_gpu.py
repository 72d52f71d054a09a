"""GPU test of the gradient's sum of squares at lengths around the rounds in which its workgroups read (1024 of them, 4096 values
each at a time): shorter than one, whole ones, remainders that end inside a workgroup's part and inside a 16-byte load.
Against float64.  A thread sums at most 4 (n / 2^22 + 4) squares in fp32 beside each other in eight chains, all terms
positive: relative error below that count times 2^-24, 2e-6 for the lengths here."""
import pytest
import torch

pytestmark = pytest.mark.gpu
ROUND = 1024 * 4096


@pytest.mark.parametrize("n", [1, 3, 1023, 4097, ROUND - 1, ROUND, ROUND + 3, ROUND + 1024, 2 * ROUND - 4, 3 * ROUND + 262147])
def test_sum_of_squares_in_rounds(n):
    from paper_2601_02609_amd import binding as B
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(n, device="cuda", generator=g)
    print(f"[sumsq] n={n}", flush=True)
    got = float(B.cce_grad_sumsq(x))
    want = float(x.double().square().sum())
    assert abs(got - want) <= 2e-6 * want
