"""The order that the approximate Wasserstein distance brings up to 65536 block means into, bit for bit, at the sizes where one kernel hands
over to the next and with more means in a range than a workgroup sorts at once; the distance itself at the same sizes."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd import api
from paper_2406_11209_amd.api import Codec
from parity import oracle_compressed
from test_gpu_wasserstein_sort import ORDERS, keys, scattered

pytestmark = pytest.mark.gpu

RUN = 32        # of which one mean is a sample


def unsampled(n):
    run = np.arange(-(-n // RUN), dtype=np.int64)
    length = np.minimum(n - run * RUN, RUN)
    return np.setdiff1d(np.arange(n), run * RUN + ((scattered(run) * length) >> 32))


def missed_cluster(g, n):
    """Half of the means that are no samples within 1e-6 of each other: thirty and more times what a workgroup takes, in one range."""
    v = g.random(n)
    free = unsampled(n)
    take = free[g.random(free.size) < 0.5]
    v[take] = 0.5 + 1e-6 * g.random(take.size)
    return v


def missed_value(g, n):
    """The same with one value, which is no splitter, and some beside it."""
    v = g.random(n)
    free = unsampled(n)
    take = free[g.random(free.size) < 0.7]
    v[take] = np.where(g.random(take.size) < 0.9, 0.5, 0.5 + 1e-9 * g.standard_normal(take.size))
    return v


CASES = {"missed cluster": missed_cluster, "missed value": missed_value, **{k: ORDERS[k] for k in ("smooth", "one value", "few values", "rarely NaN", "NaN", "infinite")}}


@pytest.mark.parametrize("values", list(CASES))
@pytest.mark.parametrize("n", [1, 2, 3, 33, 63, 64, 65, 1023, 1024, 1025, 4096, 4097, 4128, 5000, 32769, 65535, 65536, 65537])
def test_few_block_means_come_out_in_order(n, values):
    g = np.random.Generator(np.random.PCG64(n + len(values)))
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    operands, means, oc = [], [], []
    for scale in (1.0, -1.5):
        v = CASES[values](g, n) * scale
        F = np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)
        N = np.where(np.isnan(v), v, np.abs(v))
        operands += [torch.from_numpy(N).cuda(), torch.from_numpy(F).cuda()]
        means.append(N * F[:, 0].astype(np.float64) * (1.0 / (127.0 * np.sqrt(2.0))))
        if np.isfinite(v).all():
            oc.append(oracle_compressed(operands[-2], operands[-1], (2 * n,), (2,), 8, "f64", np.array([True, False]), "dct"))
    need = ctypes.c_size_t()
    api.check(codec._lib.pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)))
    workspace = torch.full((need.value,), 255, dtype=torch.uint8, device="cuda")
    got = float(codec.approximate_wasserstein(*operands, 2.0, workspace=workspace).item())
    first = 256 + 2 * 1024 * 2 * 8
    out = workspace[first:first + 16 * n].cpu().numpy().view(np.uint64).reshape(2, n)
    for have, mean in zip(out, means):
        value = np.where(have >> np.uint64(63), have & np.uint64((1 << 63) - 1), ~have).view(np.float64)
        assert np.all(have[:-1] <= have[1:]) and np.isnan(value).sum() == np.isnan(mean).sum()
        assert np.array_equal(have[~np.isnan(value)], np.sort(keys(mean[~np.isnan(mean)])))
    if len(oc) == 2:
        want = po.approximate_wasserstein(*oc, 2.0)
        assert abs(got - want) <= 1e-9 * abs(want) + 1e-300, (got, want)      # the bar of the other tests of this distance


@pytest.mark.parametrize("m", [1023, 1024, 1025, 1500, 2047, 2048, 2049, 4100])
@pytest.mark.parametrize("n", [16384, 65536])
def test_ranges_about_what_a_workgroup_sorts_at_once(n, m):
    """A range of m means: one to a thread, two to a thread, and more than are held at once."""
    g = np.random.Generator(np.random.PCG64(n + m))
    free = unsampled(n)
    drawn = np.setdiff1d(np.arange(n), free)
    # all others at most 0 or at least 1, and enough samples 0 and 1 for both to be splitters: the range is what lies between
    v = np.where(g.random(n) < 0.5, -g.random(n), 1.0 + g.random(n))
    v[drawn[::8]], v[drawn[4::8]] = 0.0, 1.0
    v[g.choice(free, m, replace=False)] = 0.01 + 0.98 * g.random(m)
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    N, F = torch.from_numpy(np.abs(v)).cuda(), torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
    need = ctypes.c_size_t()
    api.check(codec._lib.pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)))
    workspace = torch.full((need.value,), 255, dtype=torch.uint8, device="cuda")
    assert float(codec.approximate_wasserstein(N, F, N, F, 2.0, workspace=workspace).item()) == 0.0
    first = 256 + 2 * 1024 * 2 * 8
    out = workspace[first:first + 16 * n].cpu().numpy().view(np.uint64).reshape(2, n)
    want = np.sort(keys(np.abs(v) * np.where(v < 0, -127.0, 127.0) * (1.0 / (127.0 * np.sqrt(2.0)))))
    assert np.array_equal(out[0], want) and np.array_equal(out[1], want)
