"""GPU parity on arrays whose blocks are near the ends of the working type's range: maxima for which r / N, 1 / N or r C leave
the range although N and the indices are ordinary numbers."""
import numpy as np
import pytest
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd import synth
from parity import Case

pytestmark = pytest.mark.gpu

# factors on a field of magnitude one.  FP32 work: 127 / N overflows below 3.7e-37; 127 C overflows above 2.7e36.  FP64 work: r / N
# overflows below 1.8e-304 (int16), 1.2e-299 (int32) and 7e-307 (int8); r C above 5e303 and 8e298.
NARROW, WIDE = (1e-37, 2e36), (1e-305, 1e-307, 1e304)
# block, array, working and index type of every masked family's kernels ...
MASKED = [((8, 8), "f32", "f32", 8), ((8, 8), "f64", "f64", 16), ((8, 8), "f64", "f32", 8), ((8, 8), "f64", "f64", 32),
          ((4, 4, 4), "f32", "f32", 8), ((4, 4, 4), "f64", "f64", 16), ((16, 16), "f32", "f32", 8), ((16, 16), "f64", "f64", 16),
          ((16, 16), "f64", "f64", 32), ((4, 16, 16), "f32", "f32", 8), ((4, 16, 16), "f64", "f64", 16), ((8, 8, 8), "f32", "f32", 8),
          ((8, 8, 8), "bf16", "f32", 8), ((8, 8, 8), "f64", "f64", 16), ((8, 8, 8), "f64", "f64", 32),
          ((16, 16, 16), "f32", "f32", 8), ((16, 16, 16), "f64", "f64", 16)]
# ... and of the kernels per block shape
SHAPES = [((16,), "f32", "f32", 8), ((64,), "f32", "f32", 8), ((8, 16), "f32", "f32", 8), ((4, 4), "f32", "f32", 8),
          ((32, 32), "f32", "f32", 8), ((32, 32), "f64", "f64", 16), ((4, 8, 8), "f32", "f32", 8), ((2, 8, 8), "f64", "f64", 16),
          ((4, 4, 4, 4), "f64", "f64", 32), ((2, 4, 8, 8), "f32", "f32", 8)]
EXTENTS = {1: (65536,), 2: (1024, 1040), 3: (64, 96, 520), 4: (16, 16, 32, 64)}


@pytest.mark.parametrize("masked,block,dtype,ftype,bits", [(True,) + s for s in MASKED] + [(False,) + s for s in SHAPES],
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
    N, F = case.codec.compress(case.xA)
    y = case.codec.decompress(N, F, x.shape, torch.float32)
    ref = po.decompress(case.oc(N, F))
    # Everything is a multiple of u = 2^-149 here.  A coefficient is off by u / 2, a value by that times the sum of the basis, 64 x 0.18:
    # 6 u; the transform's passes round some twelve times, up to as much again each: 18 u.  N / 127 is 1e-40: rounded to a
    # multiple of u it is off by 7e-6 of itself, and the maxima of 1.7e-38 by some 90 u
    assert np.abs(y.cpu().numpy().astype(np.float64) - ref).max() <= 24 * 2.0 ** -149 + 2e-7 * np.abs(ref).max()
