"""GPU parity of the approximate Wasserstein distance over the sizes and distributions at which its sort takes another
path: one bucket, several, more than the sample sort takes; shared values, one value, a few intervals crowded."""
import numpy as np
import pytest
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd.api import Codec
from parity import oracle_compressed

pytestmark = pytest.mark.gpu

VALUES = {
    "smooth": lambda g, n: g.standard_normal(n),
    "wide": lambda g, n: np.exp(20.0 * g.standard_normal(n)) * g.choice([-1.0, 1.0], n),         # exponents everywhere
    "mostly zero": lambda g, n: np.where(g.random(n) < 0.9, 0.0, g.standard_normal(n)),
    "few values": lambda g, n: g.integers(-3, 4, n).astype(np.float64),
    "one value": lambda g, n: np.full(n, 0.7),
    "rising": lambda g, n: np.linspace(-1.0, 2.0, n),
    # two thirds within 1e-9 of one value, which is none of the splitters': an interval far more crowded than the others
    "crowded": lambda g, n: np.where(g.random(n) < 0.67, 0.5 + 1e-9 * g.standard_normal(n), 40.0 * g.standard_normal(n)),
    # every 64th far away, the others one period after the other
    "periodic": lambda g, n: np.where(np.arange(n) % 64 == 5, 1e6, np.sin(np.arange(n) * (2 * np.pi / 64))),
}
SIZES = [1, 2, 255, 4095, 4096, 4097, 8193, 70001, 524288, 1 << 20]


@pytest.mark.parametrize("values", list(VALUES))
@pytest.mark.parametrize("n", SIZES)
def test_distance_at_every_path_of_the_sort(n, values):
    g = np.random.Generator(np.random.PCG64(n + len(values)))
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    ops = []
    for scale in (1.0, 1.5):
        v = VALUES[values](g, n) * scale
        N = torch.from_numpy(np.abs(v)).cuda()
        F = torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
        ops.append((N, F))
    for p in (1.0, 68.0):
        got = float(codec.approximate_wasserstein(*ops[0], *ops[1], p).item())
        oc = [oracle_compressed(N, F, (2 * n,), (2,), 8, "f64", np.array([True, False]), "dct") for N, F in ops]
        want = po.approximate_wasserstein(oc[0], oc[1], p)
        # the bar of the other tests of this distance: exp and pow differ between the libraries, softmax outputs cancel
        assert abs(got - want) <= 1e-9 * abs(want) + 1e-300, (n, values, p, got, want)
    assert float(codec.approximate_wasserstein(*ops[0], *ops[0], 3.0).item()) == 0.0


def test_more_blocks_than_the_sample_sort_takes():
    n = (1 << 22) + 1
    test_distance_at_every_path_of_the_sort(n, "smooth")
    test_distance_at_every_path_of_the_sort(n - 1, "mostly zero")
