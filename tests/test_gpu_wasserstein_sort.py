"""GPU parity of the approximate Wasserstein distance over the sizes and distributions at which its sort takes another
path: one bucket, several, more than the sample sort takes; shared values, one value, a few intervals crowded."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd import api
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
# 70001, 300001 and 524288: four, eight and sixteen samples a bucket; 2^20: four again, of which the sort takes as many as it can hold
SIZES = [1, 2, 255, 4095, 4096, 4097, 8193, 70001, 300001, 524288, 1 << 20]


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


def buckets_of_sort(n):
    buckets = 1
    while n > 4096 and buckets * 2048 < n:
        buckets *= 2
    return buckets


def scattered(i):
    """The kernels' 32 bits of a run's number."""
    x = i.astype(np.uint64)
    for factor, shift in ((2654435761, 15), (1779033703, 13), (3144134277, 16)):
        x = (x * np.uint64(factor)) & np.uint64(0xFFFFFFFF)
        x ^= x >> np.uint64(shift)
    return x.astype(np.int64)


def sampled(n):
    """The places in the input from which the splitters of the sample sort are drawn: more of them a bucket where buckets are large, and at most
    2048 of few buckets (sample_place of the kernels, and the rule where they are launched)."""
    buckets = buckets_of_sort(n)
    per_bucket, most = (16 if n > 1400 * buckets else 8 if n > 1100 * buckets else 4, 2048) if buckets <= 256 else (4, 4096)
    shift = (min(per_bucket * buckets, most) - 1).bit_length()
    i = np.arange(1 << shift, dtype=np.int64)
    lo, hi = (n * i) >> shift, (n * (i + 1)) >> shift
    return lo + ((scattered(i) * (hi - lo)) >> 32)


def keys_of_buckets(v):
    """How many of the values lie between neighbouring splitters, which are left out."""
    n = len(v)
    drawn, buckets = np.sort(v[sampled(n)]), buckets_of_sort(n)
    split = drawn[(np.arange(1, buckets) * len(drawn)) // buckets - 1]
    ends = np.sort(v)
    above = np.append(np.searchsorted(ends, split, "left"), n)
    return above - np.append(0, np.searchsorted(ends, split, "right"))


def hidden_cluster(g, n):
    """Two fifths of the keys within 1e-6 of each other, between two splitters 1e-3 or more apart, none of them sampled: an interval with more
    keys than LDS takes, by value and by key."""
    v = g.random(n)
    free = np.setdiff1d(np.arange(n), sampled(n))
    take = free[g.random(free.size) < 0.4]
    v[take] = 0.5 + 1e-6 * g.random(take.size)
    if 65536 < n <= 1 << 22:                                         # that the sample sort takes: one bucket with all of the cluster
        assert keys_of_buckets(v).max() >= take.size > 8192
    return v


def not_finite(bits):
    def values(g, n):
        v = np.where(g.random(n) < 0.5, g.standard_normal(n), np.exp(20.0 * g.standard_normal(n)))
        at = g.random(n) < 0.3
        v[at] = g.choice(np.array(bits, dtype=np.uint64), int(at.sum())).view(np.float64)
        return v
    return values


INFINITY, MINUS = 0x7FF0 << 48, 1 << 63
ORDERS = {
    **VALUES,
    "small and large": lambda g, n: np.exp(g.uniform(-27.6, 0.0, n)) * g.choice([-1.0, 1.0], n),
    "hidden cluster": hidden_cluster,
    "infinite": not_finite([INFINITY, INFINITY | MINUS]),
    "rarely NaN": lambda g, n: np.where(np.arange(n) % 4099 == 7, np.nan, g.standard_normal(n)),
    "NaN": not_finite([INFINITY, INFINITY | MINUS, 0x7FF8 << 48, 0xFFF8 << 48, 0x7FFFFFFFFFFFFFFF, 0xFFFFFFFFFFFFFFFF]),
}


def keys(v):
    """Unsigned numbers in the order of the doubles, NaN by its sign at either end."""
    u = v.view(np.uint64)
    return np.where(u >> np.uint64(63), ~u, u | np.uint64(1 << 63))


@pytest.mark.parametrize("values", list(ORDERS))
@pytest.mark.parametrize("n", SIZES + [(1 << 22) + 1])
def test_block_means_come_out_in_order(n, values):
    """The keys that the workspace is left with (behind the parameters and the partial sums) are the block means in order, bit for bit: what the
    softmax hides of a wrong order shows here.  A NaN's bits may change, its place in the order is by its sign."""
    g = np.random.Generator(np.random.PCG64(n + len(values)))
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    operands, means = [], []
    for scale in (1.0, -1.5):
        v = ORDERS[values](g, n) * scale
        F = np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)
        N = np.where(np.isnan(v), v, np.abs(v))
        operands += [torch.from_numpy(N).cuda(), torch.from_numpy(F).cuda()]
        means.append(N * F[:, 0].astype(np.float64) * (1.0 / (127.0 * np.sqrt(2.0))))
    need = ctypes.c_size_t()
    api.check(codec._lib.pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)))
    workspace = torch.zeros(need.value, dtype=torch.uint8, device="cuda")
    codec.approximate_wasserstein(*operands, 2.0, workspace=workspace)
    first = 256 + 2 * 1024 * 2 * 8
    got = workspace[first:first + 16 * n].cpu().numpy().view(np.uint64).reshape(2, n)
    for have, mean in zip(got, means):
        assert np.all(have[:-1] <= have[1:])
        value = np.where(have >> np.uint64(63), have & np.uint64((1 << 63) - 1), ~have).view(np.float64)
        assert np.isnan(value).sum() == np.isnan(mean).sum()
        want = np.sort(keys(mean[~np.isnan(mean)]))
        assert np.array_equal(have[~np.isnan(value)], want)


@pytest.mark.parametrize("seed", range(3))
@pytest.mark.parametrize("n,width", [(524288, 725), (131072, 363), (262144, 512), (400000, 1000), (99000, 330)])
def test_buckets_of_an_image_are_even(n, width, seed):
    """Means in the rows of a smooth image with a little noise: no bucket of its 4 to 16 samples has more keys than a workgroup holds, whatever the rows'
    length is to the runs of which one key each is a sample (a bucket of 4 samples has 4 times the average once in 10^4)."""
    g = np.random.Generator(np.random.PCG64(n + seed))
    rows = -(-n // width)
    y, x = np.arange(rows)[:, None] / rows, np.arange(width)[None, :] / width
    v = 1e-3 * g.standard_normal((rows, width))
    for _ in range(12):
        cy, cx, size = g.random(), g.random(), g.uniform(0.02, 0.1)
        v += g.uniform(-1, 1) * np.exp(-((y - cy) ** 2 + (x - cx) ** 2) / (2 * size * size))
    v = v.reshape(-1)[:n]
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    N = torch.from_numpy(np.abs(v)).cuda()
    F = torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
    need = ctypes.c_size_t()
    api.check(codec._lib.pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)))
    workspace = torch.zeros(need.value, dtype=torch.uint8, device="cuda")
    codec.approximate_wasserstein(N, F, N, F, 2.0, workspace=workspace)
    buckets, tiles = buckets_of_sort(n), min(-(-n // 2048), 256)
    up = lambda size: (size + 255) // 256 * 256  # noqa: E731
    totals = 256 + 2 * 1024 * 2 * 8 + 2 * up(16 * n) + up(4 * 2 * tiles * 2 * buckets)
    got = workspace[totals:totals + 16 * buckets].cpu().numpy().view(np.uint32).reshape(2, buckets, 2)
    assert got[0].sum() == n and np.array_equal(got[0][:, 0], keys_of_buckets(v))
    assert got[0][:, 0].max() <= 8192


@pytest.mark.parametrize("m", [1024, 1025, 2049, 4095, 4096])
@pytest.mark.parametrize("n", [1 << 18, 300001, 1 << 20])
def test_bucket_that_is_crowded_between_its_own_splitters(n, m):
    """A bucket of m keys, 150 of them next to each other in the order and none where the bucket draws its own 256 splitters: too many in one
    interval, by value and between those.  Such a bucket is left to k_bucket_sort_rest, which sorts it in registers, four keys a thread.  Tiles
    of the input come into a bucket one after the other, so runs of keys that are drawn and runs that are not lie in a tile each."""
    g = np.random.Generator(np.random.PCG64(n + m))
    buckets, tiles = buckets_of_sort(n), min(-(-n // 2048), 256)
    tile_keys = -(-n // tiles)
    # all other keys at most 0 or at least 1, some of them 0 and 1: these two are splitters, and the bucket is what lies between
    v = np.where(g.random(n) < 0.5, -1.0, 2.0) + g.random(n) * np.where(g.random(n) < 0.1, 0.0, 1e-3)
    places = sampled(n)
    v[places[::16]], v[places[8::16]] = 0.0, 1.0
    v[(v > 0.0) & (v < 1.0)] = 0.0
    group = np.ones(m, dtype=bool)
    group[(np.arange(256) * m) // 256] = False
    group &= np.cumsum(group) <= 150
    assert group.sum() == 150
    values = 0.05 + 0.9 * g.random(m)
    values[np.abs(values - 0.5) < 1e-4] = 0.4
    values[group] = 0.5 + 1e-9 * g.permutation(150)
    free = np.setdiff1d(np.arange(n), places)
    starts = np.flatnonzero(np.diff(group.astype(int), prepend=2))   # of runs
    ends = np.append(starts[1:], m)
    tile = 0
    for a, b in zip(starts, ends):
        while a < b:
            room = free[(free >= tile * tile_keys) & (free < min((tile + 1) * tile_keys, n))]
            take = min(b - a, room.size)
            v[g.choice(room, take, replace=False)] = values[a:a + take]
            a, tile = a + take, tile + 1
    assert tile <= tiles and ((v > 0.0) & (v < 1.0)).sum() == m
    drawn = np.sort(v[places])
    split = drawn[(np.arange(1, buckets) * len(drawn)) // buckets - 1]
    bucket = int(np.searchsorted(split, 1.0))
    assert split[bucket - 1] == 0.0 and split[bucket] == 1.0 and keys_of_buckets(v)[bucket] == m
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    N = torch.from_numpy(np.abs(v)).cuda()
    F = torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
    need = ctypes.c_size_t()
    api.check(codec._lib.pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)))
    workspace = torch.zeros(need.value, dtype=torch.uint8, device="cuda")
    assert float(codec.approximate_wasserstein(N, F, N, F, 2.0, workspace=workspace).item()) == 0.0
    up = lambda size: (size + 255) // 256 * 256  # noqa: E731
    first = 256 + 2 * 1024 * 2 * 8
    # behind the two operands' keys, twice: the counts, the totals and the splitters; then the list of what was left over
    rest = first + 2 * up(16 * n) + up(4 * 2 * tiles * 2 * buckets) + up(4 * 2 * 2 * buckets) + up(8 * 2 * buckets)
    listed = workspace[rest:rest + 8 + 8 * buckets].cpu().numpy().view(np.uint32)
    assert {2 * bucket, 2 * bucket + 1} <= set(listed[2:2 + int(listed[0])])        # of either operand
    got = workspace[first:first + 16 * n].cpu().numpy().view(np.uint64).reshape(2, n)
    want = np.sort(keys(np.abs(v) * np.where(v < 0, -127.0, 127.0) * (1.0 / (127.0 * np.sqrt(2.0)))))
    assert np.array_equal(got[0], want) and np.array_equal(got[1], want)


@pytest.mark.parametrize("ftype,low", [("f64", -np.inf), ("f64", -1.7e308), ("f16", -np.inf)])
@pytest.mark.parametrize("n", [3, 300, 4097, 66001, (1 << 22) + 1])
def test_means_below_all_numbers_have_no_weight(n, ftype, low):
    """A block mean of minus infinity (N that has overflowed, or its product with the index) is a probability of zero, be it all that a
    thread or a workgroup meets."""
    g = np.random.Generator(np.random.PCG64(n))
    codec = Codec((2,), ftype, "i8", np.array([True, False]))
    for where in (g.random(n) < 0.01, np.arange(n) < n // 2, np.arange(n) > 0):
        where[n // 2] = True
        ops, oc = [], []
        for k in range(2):
            v = g.standard_normal(n)
            if k == 0:
                v[where] = low
            N = torch.from_numpy(np.abs(v)).cuda().to(torch.float64 if ftype == "f64" else torch.float16)
            F = torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
            ops.append((N, F))
            oc.append(oracle_compressed(N, F, (2 * n,), (2,), 8, ftype, np.array([True, False]), "dct"))
        for p in (1.0, 68.0):
            got = float(codec.approximate_wasserstein(*ops[0], *ops[1], p).item())
            with np.errstate(over="ignore"):
                want = po.approximate_wasserstein(oc[0], oc[1], p)
            assert want > 0.0 and abs(got - want) <= 1e-9 * want, (n, p, got, want)


def near(g, n):
    """Two sequences as close as two roundings of one: every bucket matters."""
    v = g.standard_normal(n)
    return v, v * (1.0 + 1e-7 * g.standard_normal(n))


def tails(g, n):
    """Equal but for a few of the largest, the smallest, or values in the middle: nearly all buckets can be left out, at either end or at both."""
    v = g.standard_normal(n)
    w = v + np.where(g.random(n) < 20.0 / n, 2.0, 0.0) - np.where(g.random(n) < 20.0 / n, 3.0, 0.0)
    return v, w


def sums_to_one(g, n):
    """No softmax: the means are the probabilities, zeros and equal ones among them."""
    a, b = g.exponential(1.0, n) ** 3, np.where(g.random(n) < 0.3, 0.0, g.exponential(1.0, n) ** 3)
    b[g.random(n) < 0.1] = b.max()
    return a / a.sum(), b / b.sum()


def few_against_many(g, n):
    """One operand of three values, the other of as many as there are blocks: its buckets meet one of the other's."""
    return g.integers(0, 3, n).astype(np.float64), g.standard_normal(n)


@pytest.mark.parametrize("values", [near, tails, sums_to_one, few_against_many], ids=lambda f: f.__name__)
@pytest.mark.parametrize("n", [65535, 65537, 131073, 262145, (1 << 20) + 1, (1 << 21) + 1])
def test_distance_where_buckets_are_left_out(n, values):
    """The sizes from which buckets that cannot matter are neither scattered nor sorted, and at which more of them come to a thread."""
    g = np.random.Generator(np.random.PCG64(n))
    codec = Codec((2,), "f64", "i8", np.array([True, False]))
    factor = np.sqrt(2.0) if values is sums_to_one else 1.0        # a mean is N F0 / (r sqrt(2))
    ops, oc = [], []
    for v in values(g, n):
        v = v * factor
        N, F = torch.from_numpy(np.abs(v)).cuda(), torch.from_numpy(np.where(v < 0, -127, 127).astype(np.int8).reshape(n, 1)).cuda()
        ops.append((N, F))
        oc.append(oracle_compressed(N, F, (2 * n,), (2,), 8, "f64", np.array([True, False]), "dct"))
    for p in (2.0, 68.0, 80.0):
        got = float(codec.approximate_wasserstein(*ops[0], *ops[1], p).item())
        want = po.approximate_wasserstein(oc[0], oc[1], p)
        # 1e-9 as above; differences of nearly equal probabilities are off by the rounding of these, too: 2^-51 of the largest, which is
        # exp(largest of n normal numbers) / (n exp(1/2)), below exp(5) / (1.6 n) = 90 / n
        assert abs(got - want) <= 1e-9 * abs(want) + (90.0 * 2.0 ** -51 / n if values is near else 1e-300), (n, p, got, want)
    # NaN in an operand whose means are the probabilities comes through, wherever it is in the order
    if values is sums_to_one:
        for where in (0, n // 2):
            ops[0][0][where] = float("nan")
            assert np.isnan(codec.approximate_wasserstein(*ops[0], *ops[1], 68.0).item())
