"""GPU parity of the matrix-core kernels for lines of 64 elements in FP64 work: tiles of sixteen blocks and shares of sixteen elements at
their ends, every type, masks, rows that are no whole blocks, the ends of the range; against the oracle and the general kernels."""
import numpy as np
import pytest
import torch

from paper_2406_11209_amd import synth
from paper_2406_11209_amd.api import PBZ_PATH_GENERIC
from parity import DENSE, LINES, Case, route

pytestmark = pytest.mark.gpu

# one element; a share less one, a share, one more; a block less one; the sixteenth block and the next; rows of one block, of several, ragged
SHAPES = [((64,), (n,)) for n in (1, 15, 16, 17, 63, 64, 65, 1023, 1024, 1025, 64 * 64 * 16 + 7)] + \
         [((1, 64), s) for s in ((1, 64), (17, 64), (5, 1000), (33, 129), (300, 1))] + [((1, 1, 64), (3, 5, 200))]


def make(block, shape, dtype, bits, ftype, mask, transform="dct", scale=1.0):
    g = np.random.Generator(np.random.PCG64(int(np.prod(shape)) + bits))
    cast = {"f64": lambda a: a, "f32": lambda a: a.astype(np.float32), "bf16": synth.to_bf16_bits, "f16": lambda a: a.astype(np.float16)}[dtype]
    field = synth.bump_field(shape, 6, g, (2.0, 16.0)) + 0.3 + 0.05 * g.standard_normal(shape)
    return Case(cast(field * scale), None, dtype, block, bits, ftype, mask, transform=transform)


def masked(block, kept):
    if kept is None:
        return None
    m = np.zeros(64, dtype=bool)
    m[np.random.Generator(np.random.PCG64(kept)).permutation(64)[:kept]] = True
    m[0] = True
    return m.reshape(block)


@pytest.mark.parametrize("block,shape", SHAPES, ids=lambda v: "x".join(map(str, v)))
@pytest.mark.parametrize("dtype,ftype,bits,kept,transform", [("f64", "f64", 16, None, "dct"), ("f32", "f32", 16, 19, "dct"), ("f64", "f64", 8, 33, "haar"),
                                                             ("bf16", "bf16", 32, None, "dct"), ("f16", "f32", 16, 1, "dct"), ("f32", "f64", 32, 7, "haar")])
def test_lines(block, shape, dtype, ftype, bits, kept, transform):
    case = make(block, shape, dtype, bits, ftype, masked(block, kept), transform)
    N, F, _, _ = case.check_compress("A")
    case.check_decompress(N, F)
    check_against_the_dense_kernels(case, N, F, shape, dtype, ftype)


def check_against_the_dense_kernels(case, N, F, shape, dtype, ftype):
    """Which these calls went to before: equal up to the order of the sums."""
    assert route(case.codec, "compress", shape, dtype) == route(case.codec, "decompress", shape, dtype) == LINES
    case.codec.set_kernel_path(PBZ_PATH_GENERIC)
    assert route(case.codec, "compress", shape, dtype) == DENSE
    Ng, Fg = case.codec.compress(case.xA)
    y = case.codec.decompress(N, F, shape, case.xA.dtype)
    case.codec.set_kernel_path(0)
    z = case.codec.decompress(N, F, shape, case.xA.dtype)
    # 64 products of rounding 2^-53 each, of at most |C| <= N
    assert bool(((N.double() - Ng.double()).abs() <= (64 * 2.0 ** -53 + {"f64": 0.0, "f32": 2.0 ** -23, "bf16": 2.0 ** -7}[ftype]) * Ng.double()).all())
    assert int((F.to(torch.int64) - Fg.to(torch.int64)).abs().max()) <= 1
    steps = {"f64": 2.0 ** -46, "f32": 2.0 ** -23, "bf16": 2.0 ** -7, "f16": 2.0 ** -10}[dtype]
    assert bool(((y.double() - z.double()).abs() <= steps * y.double().abs().max()).all())


# 4096 tiles of sixteen blocks are 4 Mi elements: from there on eight waves share a table when compressing; 3072 tiles, and 4096 with eight
# waves, stand at once, so that waves take a second tile.  The last tile is not full, nor is its last block.
@pytest.mark.parametrize("block,shape", [((64,), ((4 << 20) - 1025,)), ((64,), ((4 << 20) + 7,)), ((1, 64), (4099, 1030)), ((64,), ((9 << 20) + 999,))],
                         ids=["below", "above", "rows", "two_turns"])
@pytest.mark.parametrize("dtype,ftype,bits,kept", [("f64", "f64", 32, None), ("f32", "f32", 16, 19), ("bf16", "bf16", 16, 63), ("f32", "f64", 8, 33)])
def test_more_lines_than_stand_at_once(block, shape, dtype, ftype, bits, kept):
    case = make(block, (1,) * len(shape), dtype, bits, ftype, masked(block, kept))
    g = torch.Generator("cuda").manual_seed(bits)
    x = torch.rand(shape, generator=g, device="cuda").to(case.xA.dtype) + 0.25
    case.xA = x
    N, F = case.codec.compress(x)
    check_against_the_dense_kernels(case, N, F, shape, dtype, ftype)


@pytest.mark.parametrize("scale", [1e-305, 1e-307, 1e300])
def test_lines_at_the_ends_of_the_range(scale):
    case = make((64,), (64 * 40 + 3,), "f64", 16, "f64", None, scale=scale)
    N, F, ref, _ = case.check_compress("A")
    assert np.abs(ref.F).max() == 32767
    case.check_decompress(N, F)


@pytest.mark.parametrize("power", [1019, -1000])
@pytest.mark.parametrize("bits,kept", [(8, None), (16, 19), (32, None)])
def test_lines_come_out_the_same_times_a_power_of_two(bits, kept, power):
    """N is that much larger and the indices are what they were, also where r times a coefficient (2^1019 2^3 2^31) leaves the range."""
    case = make((64,), (64 * 300 + 5,), "f64", bits, "f64", masked((64,), kept))
    x = case.xA / (8.0 * case.xA.abs().max())                   # coefficients below 1
    N, F = case.codec.compress(x)
    far_N, far_F = case.codec.compress(x * 2.0 ** power)
    assert torch.equal(far_N, N * 2.0 ** power) and torch.equal(far_F, F)
    far_y = case.codec.decompress(far_N, far_F, x.shape)
    if power < 0:                                               # (N F is formed first: beyond the range with N this large)
        assert torch.equal(far_y, case.codec.decompress(N, F, x.shape) * 2.0 ** power)


def test_not_finite_blocks_keep_to_themselves():
    """NaN makes a block N = 0 and zeros, infinity N = infinity and the index -r, as on the general kernels; the blocks beside it stay."""
    case = make((64,), (64 * 40,), "f32", 16, "f32", None)
    plain = case.codec.compress(case.xA)
    x = case.xA.clone()
    x[64 * 5 + 3], x[64 * 20] = float("nan"), float("inf")
    N, F = case.codec.compress(x)
    case.codec.set_kernel_path(PBZ_PATH_GENERIC)
    Ng, Fg = case.codec.compress(x)
    assert torch.equal(N[[5, 20]], Ng[[5, 20]]) and torch.equal(F[[5, 20]], Fg[[5, 20]])
    others = [k for k in range(40) if k not in (5, 20)]
    assert torch.equal(N[others], plain[0][others]) and torch.equal(F[others], plain[1][others])
