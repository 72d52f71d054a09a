"""GPU test of the gradient's sum of squares at lengths around the rounds in which its workgroups read (1024 of them, 1024 values
each at a time): shorter than one, whole ones, remainders that end inside a workgroup's part and inside a 16-byte load.
Against float64.  A thread sums at most n / 2^21 + 1 squares in fp32 in each of eight chains, all terms positive: relative error
below that count and the few sums behind it times 2^-24, 2e-6 for the lengths here."""
import pytest
import torch

pytestmark = pytest.mark.gpu
ONE, ROUND = 1024 * 1024, 4 * 1024 * 1024             # one round, four of them


@pytest.mark.parametrize("n", [1, 3, 1023, 4097, ONE - 4, ONE + 4, 2 * ONE + 1023, ROUND - 1, ROUND, ROUND + 3, ROUND + 1024, 2 * ROUND - 4, 3 * ROUND + 262147])
def test_sum_of_squares_in_rounds(n):
    from paper_2601_02609_amd import binding as B
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(n, device="cuda", generator=g)
    print(f"[sumsq] n={n}", flush=True)
    got = float(B.cce_grad_sumsq(x))
    want = float(x.double().square().sum())
    assert abs(got - want) <= 2e-6 * want
