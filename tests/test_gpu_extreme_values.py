"""GPU parity on arrays whose blocks are near the ends of the working type's range: maxima for which r / N, 1 / N or r C leave
the range although N and the indices are ordinary numbers."""
import numpy as np
import pytest
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd import synth
from parity import SHAPE, Case, route, take_wherever_possible
from test_gpu_any_mask import kind

pytestmark = pytest.mark.gpu

# factors on a field of magnitude one.  FP32 work: 127 / N overflows below 3.7e-37; 127 C overflows above 2.7e36.  FP64 work: r / N
# overflows below 1.8e-304 (int16), 1.2e-299 (int32) and 7e-307 (int8); r C above 5e303 and 8e298.
NARROW, WIDE = (1e-37, 2e36), (1e-305, 1e-307, 1e304)
# block, array, working and index type of every masked family's kernels ...
MASKED_ROWS = [((8, 8), "f32", "f32", 8), ((8, 8), "f64", "f64", 16), ((8, 8), "f64", "f32", 8), ((8, 8), "f64", "f64", 32),
               ((4, 4, 4), "f32", "f32", 8), ((4, 4, 4), "f64", "f64", 16), ((16, 16), "f32", "f32", 8), ((16, 16), "f64", "f64", 16),
               ((16, 16), "f64", "f64", 32), ((4, 16, 16), "f32", "f32", 8), ((4, 16, 16), "f64", "f64", 16), ((8, 8, 8), "f32", "f32", 8),
               ((8, 8, 8), "bf16", "f32", 8), ((8, 8, 8), "f64", "f64", 16), ((8, 8, 8), "f64", "f64", 32),
               ((16, 16, 16), "f32", "f32", 8), ((16, 16, 16), "f64", "f64", 16)]
# ... and of the kernels per block shape
SHAPES = [((16,), "f32", "f32", 8), ((64,), "f32", "f32", 8), ((8, 16), "f32", "f32", 8), ((4, 4), "f32", "f32", 8),
          ((32, 32), "f32", "f32", 8), ((32, 32), "f64", "f64", 16), ((4, 8, 8), "f32", "f32", 8), ((2, 8, 8), "f64", "f64", 16),
          ((4, 4, 4, 4), "f64", "f64", 32), ((2, 4, 8, 8), "f32", "f32", 8)]
EXTENTS = {1: (65536,), 2: (1024, 1040), 3: (64, 96, 520), 4: (16, 16, 32, 64)}


@pytest.mark.parametrize("masked,block,dtype,ftype,bits", [(True,) + s for s in MASKED_ROWS] + [(False,) + s for s in SHAPES],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_blocks_at_the_ends_of_the_range(masked, block, dtype, ftype, bits):
    g = np.random.Generator(np.random.PCG64(len(block) + bits))
    vol = int(np.prod(block))
    mask = None
    if masked:
        mask = np.zeros(vol, dtype=bool)
        mask[g.permutation(vol)[:vol // 3]] = True
        mask[0] = True
        mask = mask.reshape(block)
    shape = EXTENTS[len(block)]
    field = synth.bump_field(shape, 6, g, (2.0, 8.0)) + 0.2 + 0.01 * g.standard_normal(shape)
    cast = {"f64": lambda a: a, "f32": lambda a: a.astype(np.float32), "bf16": synth.to_bf16_bits}[dtype]
    for factor in (WIDE if ftype == "f64" else NARROW):
        if bits == 32 and factor > 1.0:
            factor = 1e297                                       # the oracle forms r C in 64 bits, too
        largest = {1: 8.0, 2: 32.0, 3: 64.0, 4: 32.0}[len(block)] if factor > 1.0 else 1.0      # keeps coefficients finite
        case = Case(cast(field * (factor / largest)), None, dtype, block, bits, ftype, mask)
        want = kind(block, dtype, ftype, bits) if masked else SHAPE
        take_wherever_possible(case.codec, want)
        assert route(case.codec, "compress", shape, dtype) == want
        N, F, ref, _ = case.check_compress("A")
        assert np.abs(ref.F).max() > 100                         # ordinary indices: nothing vanished
        y = case.codec.decompress(N, F, shape, case.xA.dtype)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(y.float() if dtype == "bf16" else y).all())
        case.check_decompress(N, F)


def test_lines_of_64_keep_their_digits_below_the_normal_numbers():
    """N F / r is a normal number, N / r is not."""
    g = np.random.Generator(np.random.PCG64(3))
    x = (g.standard_normal(64 * 1024) * 4e-39).astype(np.float32)
    case = Case(x, None, "f32", (64,), 8, "f32")
    assert route(case.codec, "decompress", x.shape, "f32") == SHAPE
    N, F = case.codec.compress(case.xA)
    y = case.codec.decompress(N, F, x.shape, torch.float32)
    ref = po.decompress(case.oc(N, F))
    # Everything is a multiple of u = 2^-149 here.  A coefficient is off by u / 2, a value by that times the sum of the basis, 64 x 0.18:
    # 6 u; the transform's passes round some twelve times, up to as much again each: 18 u.  N / 127 is 1e-40: rounded to a
    # multiple of u it is off by 7e-6 of itself, and the maxima of 1.7e-38 by some 90 u
    assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() <= 24 * 2.0 ** -149 + 2e-7 * np.abs(ref).max()


def operand(n_blocks, kept, bits, N, seed):
    """Random indices with a full range in every block, and the given N."""
    g = np.random.Generator(np.random.PCG64(seed))
    r = 2 ** (bits - 1) - 1
    F = g.integers(-r, r + 1, (n_blocks, kept)).astype({8: np.int8, 16: np.int16, 32: np.int32}[bits])
    F[:, 0] = r
    return torch.from_numpy(np.asarray(N)).cuda(), torch.from_numpy(F).cuda()


@pytest.mark.parametrize("bits", [8, 16, 32])
@pytest.mark.parametrize("kept", [5, 19, 33])
@pytest.mark.parametrize("times", [1, 100])                  # few blocks: element by element from memory; more: through LDS
def test_rebinning_of_blocks_at_the_ends_of_the_range(times, kept, bits):
    """Sum, difference and shift of blocks whose kept counts make no whole vectors, N from the smallest subnormal numbers up."""
    mask = np.zeros(64, dtype=bool)
    mask[:kept] = True
    case = Case(np.zeros((8 * 24 * times, 8)), None, "f64", (8, 8), bits, "f64", mask.reshape(8, 8))
    scales = np.array([5e-324, 3e-322, 1e-320, 1e-310, 1e-308, 1e-305, 1e-300, 1.0, 1e150, 1e290, 1e298, 0.0])
    N1, F1 = operand(24 * times, kept, bits, np.tile(scales, 2 * times), kept)
    N2, F2 = operand(24 * times, kept, bits, np.tile(np.tile(scales, 2) * np.repeat([0.5, 3.0], 12), times), kept + 1)
    for got, want in ((case.codec.add(N1, F1, N2, F2), po.add(case.oc(N1, F1), case.oc(N2, F2))),
                      (case.codec.subtract(N1, F1, N2, F2), po.add(case.oc(N1, F1), po.negate(case.oc(N2, F2)))),
                      (case.codec.add_scalar(N1, F1, 0.0), po.add_scalar(case.oc(N1, F1), 0.0))):
        n, f = got[0].cpu().numpy(), got[1].cpu().numpy().astype(np.int64)
        assert np.array_equal(n, want.N.reshape(-1))
        r = 2 ** (bits - 1) - 1
        # where N is subnormal its rounding can put a quotient beyond r: the index is then r
        assert np.array_equal(f, np.clip(np.nan_to_num(want.t, nan=0.0).round(), -r, r).astype(np.int64))


@pytest.mark.parametrize("kept", [5, 19, 33])
@pytest.mark.parametrize("times", [1, 400])
def test_rebinning_keeps_infinities(times, kept):
    """A block whose N has overflowed (FP16) stays infinite through the operations, and its neighbours stay what they are."""
    mask = np.zeros(64, dtype=bool)
    mask[:kept] = True
    case = Case(np.zeros((8 * 6 * times, 8)), None, "f64", (8, 8), 8, "f16", mask.reshape(8, 8))
    N1, F1 = operand(6 * times, kept, 8, np.tile(np.array([1.0, np.inf, 2.0, np.inf, 0.5, 0.0], dtype=np.float16), times), kept)
    N2, F2 = operand(6 * times, kept, 8, np.tile(np.array([1.0, 1.0, 2.0, 0.0, 0.5, 3.0], dtype=np.float16), times), kept + 1)
    at = torch.arange(6 * times, device="cuda")
    fine, infinite = at[(at % 6 != 1) & (at % 6 != 3)], at[(at % 6 == 1) | (at % 6 == 3)]
    for got, plain in ((case.codec.add(N1, F1, N2, F2), case.codec.add(N1[fine], F1[fine], N2[fine], F2[fine])),
                       (case.codec.add_scalar(N1, F1, 0.75), case.codec.add_scalar(N1[fine], F1[fine], 0.75))):
        assert bool(torch.isinf(got[0][infinite]).all())
        assert torch.equal(got[0][fine], plain[0]) and torch.equal(got[1][fine], plain[1])


@pytest.mark.parametrize("ftype,bits", [("f64", 8), ("f64", 16), ("f64", 32), ("f16", 8), ("f16", 16), ("f32", 32)])
@pytest.mark.parametrize("kept", [1, 5, 16, 19, 33, 64])
@pytest.mark.parametrize("n", [24, 2407])
def test_rebinning_in_place_at_the_ends_of_the_range(n, kept, ftype, bits):
    """Sum, difference and shift into the buffers of an operand are what they are in buffers of their own, also where blocks whose N is
    infinite or near the ends of the range are among the others: few of them, and many."""
    mask = np.zeros(64, dtype=bool)
    mask[:kept] = True
    case = Case(np.zeros((8, 8)), None, "f64", (8, 8), bits, ftype, mask.reshape(8, 8))
    ends = {"f64": [1e-320, 1e-300, 1e298, np.inf, 5e-324], "f32": [1e-44, np.inf, 3e38], "f16": [np.inf, 6e-8, 6e4]}[ftype]
    g = np.random.Generator(np.random.PCG64(kept))
    dtype = {"f64": np.float64, "f32": np.float32, "f16": np.float16}[ftype]
    for share in (0.01, 0.3):
        N = [g.uniform(0.5, 2.0, n) for _ in range(2)]
        for k in range(2):
            where = np.flatnonzero(g.uniform(size=n) < share)
            where = np.union1d(where, [n - 1 - k])
            N[k][where] = np.resize(ends, where.size)
        (N1, F1), (N2, F2) = (operand(n, kept, bits, N[k].astype(dtype), kept + k) for k in range(2))
        codec = case.codec
        calls = [(lambda a, out: codec.add(*a, *out), 2), (lambda a, out: codec.subtract(*a, *out), 2),
                 (lambda a, out: codec.add_scalar(*a, 0.75, *out), 1)]
        for call, operands in calls:
            args = [N1, F1, N2, F2][:2 * operands]
            want = call(args, ())
            for over in range(operands):
                mine = [t.clone() for t in args]
                got = call(mine, mine[2 * over:2 * over + 2])
                assert got[0].data_ptr() == mine[2 * over].data_ptr()
                assert torch.equal(got[0].nan_to_num(nan=-1.0), want[0].nan_to_num(nan=-1.0)) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("bits,kept", [(8, 5), (8, 19), (8, 33), (8, 63), (16, 5), (16, 19), (16, 63), (32, 19)])
@pytest.mark.parametrize("n", [40, 2400])
def test_reductions_keep_infinities(n, bits, kept):
    """A block whose N has overflowed (FP16) makes norms, distances and products infinite, not NaN: not where its last indices
    are padding, and not where most of them are zero."""
    mask = np.zeros(64, dtype=bool)
    mask[:kept] = True
    case = Case(np.zeros((8 * n, 8)), None, "f64", (8, 8), bits, "f16", mask.reshape(8, 8))
    N1, F1 = operand(n, kept, bits, np.full(n, 1.5, dtype=np.float16), kept)
    N2, F2 = operand(n, kept, bits, np.full(n, 0.5, dtype=np.float16), kept + 1)
    N1[17] = float("inf")
    F1[F1 == 0] = 1                              # infinity times a zero index is no number, and neither is a distance of it
    assert case.codec.difference_norm2(N1, F1, N2, F2).item() == np.inf
    F1[17, 1:] = 0
    assert case.codec.norm2(N1, F1).item() == np.inf
    assert case.codec.dot(N1, F1, N2, F2).item() == np.inf
    assert case.codec.segmented("norm2", 4, n // 4, N1, F1).tolist()[17 // (n // 4)] == np.inf
    assert np.isfinite(case.codec.segmented("norm2", 4, n // 4, N1, F1).cpu().numpy()[2:]).all()
