"""The bias sum on both sides of the line between one workgroup and several (4,096 hills of capacity), at the edges of
a thread's rounds, against the FP64 oracle at the bar of the other bias tests."""
import pytest

from tests.test_gpu_bias_blocks import test_bias_and_deposit as bias_and_deposit

pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [0, 1, 1023, 1025, 4095, 4096])
@pytest.mark.parametrize("capacity", [4096, 4097])
@pytest.mark.parametrize("dims,period", [(1, 0.0), (1, 6.0), (2, 0.0), (2, 6.0)])
def test_both_sides_of_the_line(orc, K, capacity, dims, period):
    bias_and_deposit(orc, K, capacity, dims, period)
