"""Calls that the kernels for exactly one setting would take and that go to those per block shape: small arrays, and those whose rows have few blocks, or
are no whole blocks.  Against the oracle, at sizes where the rule first applies; where it must not, and without device tables (first call under capture)."""
import numpy as np
import pytest
import torch

from paper_2406_11209_amd import api, synth
from paper_2406_11209_amd.api import Codec
from parity import EXACT, MASKED, SHAPE, TORCH_DTYPE, Case, route, take_wherever_possible

CAST = {"f64": lambda a: a, "f32": lambda a: a.astype(np.float32), "bf16": synth.to_bf16_bits, "f16": lambda a: a.astype(np.float16)}

# shape, block, array, work, index bits, directions that go to the kernels per block shape
ROWS = [((20000, 8), (8, 8), "f32", "f32", 8, "cd"),                  # small arrays, of any row width
        ((23000, 8), (8, 8), "f32", "f32", 8, "cd"),
        ((400000, 8), (8, 8), "f32", "f32", 8, "cd"),
        ((2300, 10, 12), (1, 8, 8), "f32", "f32", 8, "cd"),           # a partial block in each row and column
        ((513, 258), (8, 8), "f64", "f64", 16, "cd"),
        ((263, 510), (8, 8), "f64", "f64", 8, "cd"),
        ((1200, 123), (8, 8), "f32", "f32", 8, "d"),
        ((300, 258), (8, 8), "bf16", "f32", 8, "d"),
        ((300, 258), (8, 8), "f16", "f16", 8, "d"),
        ((16001, 10), (8, 8), "f32", "f32", 16, "cd"),
        ((65, 66, 21), (4, 4, 4), "f64", "f64", 16, "cd"),
        ((161, 161, 6), (4, 4, 4), "f32", "f32", 8, "cd"),
        ((200, 200, 8), (4, 4, 4), "f32", "f32", 32, "cd"),
        ((200, 204, 4), (4, 4, 4), "f64", "f32", 8, "cd"),
        ((2001, 16, 16), (1, 16, 16), "f32", "f32", 16, "cd"),
        ((6200, 32, 16), (1, 16, 16), "f32", "f32", 16, "cd"),
        ((130, 40, 50), (1, 16, 16), "f32", "f32", 16, "d"),
        ((130, 33, 51), (1, 16, 16), "f64", "f64", 32, "d"),
        ((2000, 17, 30), (1, 16, 16), "bf16", "f32", 8, "cd"),
        ((96, 181, 190), (8, 8, 8), "f64", "f64", 16, "cd"),
        ((40, 41, 43), (8, 8, 8), "f64", "f32", 8, ""),
        ((512, 264), (8, 8), "f32", "f32", 8, "d"),                   # just above the least size
        ((90000, 56), (8, 8), "f32", "f32", 16, "cd"),                # larger ones: few blocks a row, whole and not
        ((41000, 126), (8, 8), "f64", "f64", 8, "cd"),
        ((700, 700, 12), (4, 4, 4), "f32", "f32", 32, "cd"),
        ((400, 404, 38), (4, 4, 4), "f64", "f64", 16, "cd"),
        ((22000, 16, 16), (1, 16, 16), "f32", "f32", 16, "cd"),
        ((2048, 2048), (8, 8), "f32", "f32", 8, ""),                  # whole waves of them keep their kernels
        ((256, 128, 128), (4, 4, 4), "f32", "f32", 16, ""),
        ((256, 256), (8, 8), "f32", "f32", 8, "")]                    # and so do the smallest


@pytest.mark.parametrize("row", ROWS, ids=[f"{r[0]}-{r[1]}-{r[2]}-{r[3]}-{r[4]}" for r in ROWS])
def test_where_calls_go(row):
    """Decided on the host.  The Haar transform as the DCT, or not at all; a shape below the rule's least size, and one of whole waves above its largest, as before."""
    shape, block, dtype, ftype, bits, directions = row
    c, haar = Codec(block, ftype, bits), Codec(block, ftype, bits, None, "haar")
    for op, letter in (("compress", "c"), ("decompress", "d")):
        want = SHAPE if letter in directions else EXACT
        assert route(c, op, shape, dtype) == want, op
        assert route(haar, op, shape, dtype) in (want, EXACT), op
        assert (c.kernel_name(op, shape, dtype) == "generic") == (want == SHAPE)
        few = tuple(min(s, 4 * b + s % b) for s, b in zip(shape, block))
        assert route(c, op, few, dtype) == EXACT
    wide = tuple(2 * b for b in block[:-1]) + (block[-1] * 64 * 1024,)        # whole waves of large arrays keep their kernels
    assert route(c, "compress", wide, dtype) == route(c, "decompress", wide, dtype) == EXACT


@pytest.mark.gpu
@pytest.mark.parametrize("row", ROWS, ids=[f"{r[0]}-{r[1]}-{r[2]}-{r[3]}-{r[4]}" for r in ROWS])
def test_against_the_oracle(row):
    shape, block, dtype, ftype, bits, directions = row
    g = np.random.Generator(np.random.PCG64(sum(shape) + bits))
    field = synth.bump_field(shape, 6, g, (2.0, 8.0)) + 0.2 + 0.01 * g.standard_normal(shape)
    case = Case(CAST[dtype](field), None, dtype, block, bits, ftype, None, api.PBZ_PATH_AUTO)
    N, F, _, _ = case.check_compress("A")
    case.check_decompress(N, F)
    case.check_compress_statistics(N, F)                         # of the same {N, F}, bit for bit, on whatever route


@pytest.mark.gpu
@pytest.mark.parametrize("row", [r for r in ROWS if r[5] == "cd"], ids=lambda r: f"{r[0]}-{r[1]}")
def test_first_call_under_capture(row):
    """These kernels make no tables here: a codec's first call may be a captured one, as with the kernels they stand in for.  Three replays, with
    eager work in between; and F that is not on 16 bytes, which they leave to the general path."""
    shape, block, dtype, ftype, bits, _ = row
    gen = torch.Generator("cuda").manual_seed(3)
    x = torch.empty(shape, dtype=TORCH_DTYPE[dtype], device="cuda")
    fresh, eager = Codec(block, ftype, bits), Codec(block, ftype, bits)
    N, F = fresh.empty_compressed(shape)
    y = torch.empty_like(x)
    x.normal_(generator=gen)
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=side):
        fresh.compress(x, N, F)
        fresh.decompress(N, F, shape, out=y)
    for _ in range(3):
        x.normal_(generator=gen)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        N2, F2 = eager.compress(x)
        y2 = eager.decompress(N2, F2, shape, x.dtype)
        torch.cuda.synchronize()
        assert torch.equal(N, N2) and torch.equal(F, F2) and torch.equal(y, y2)
    far = torch.zeros(F.numel() + 8, dtype=F.dtype, device="cuda")[1:1 + F.numel()].view(F.shape)
    far_N, _ = eager.compress(x, torch.empty_like(N), far)
    torch.cuda.synchronize()
    # another kernel's rounding: an index at a tie may be the next one
    assert torch.allclose(far_N.double(), N.double(), rtol=1e-6, atol=0)
    assert int((far.long() - F.long()).abs().max()) <= 1 and float((far != F).double().mean()) <= 1e-3
    assert torch.allclose(eager.decompress(far_N, far, shape, x.dtype).double(), y.double(), rtol=0, atol=0.1)


# block, array, work, index bits of the specialised families under a mask
MASKED_ROWS = [((8, 8), "f32", "f32", 8), ((8, 8), "f64", "f32", 8), ((8, 8), "f16", "f16", 8), ((4, 4, 4), "f32", "f32", 8),
               ((16, 16), "f32", "f32", 8), ((16, 16), "f64", "f64", 16), ((16, 16), "bf16", "f32", 8), ((16, 16), "f32", "f32", 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("row", MASKED_ROWS, ids=lambda r: "-".join(map(str, r)))
def test_small_arrays_under_a_mask(row):
    """Small calls under a mask go to the kernels per block shape, large ones to the family's: whole and ragged, against the oracle, and both against
    each other where they meet."""
    block, dtype, ftype, bits = row
    g = np.random.Generator(np.random.PCG64(bits + block[0]))
    mask = np.zeros(block, dtype=bool)
    mask.flat[g.permutation(mask.size)[:mask.size // 2]] = True
    mask.flat[0] = True
    for odd in (0, 2):
        shape = tuple(block[:-1][:-1]) + (5 * block[-2] - odd // 2, 37 * block[-1] - odd)
        field = synth.bump_field(shape, 6, g, (2.0, 8.0)) + 0.2 + 0.01 * g.standard_normal(shape)
        case = Case(CAST[dtype](field), None, dtype, block, bits, ftype, mask, api.PBZ_PATH_AUTO)
        assert route(case.codec, "compress", shape, dtype) == route(case.codec, "decompress", shape, dtype) == SHAPE
        N, F, _, _ = case.check_compress("A")
        case.check_decompress(N, F)
        shape = tuple(block[:-2]) + (64 * block[-2], block[-1] * 256 - odd)
        x = torch.randn(shape, generator=torch.Generator("cuda").manual_seed(1), device="cuda", dtype=torch.float32).to(TORCH_DTYPE[dtype])
        here, family = Codec(block, ftype, bits, mask), Codec(block, ftype, bits, mask)
        take_wherever_possible(family, MASKED)
        N, F = here.compress(x)
        N2, F2 = family.compress(x)
        y, y2 = here.decompress(N, F, shape, x.dtype), family.decompress(N, F, shape, x.dtype)
        torch.cuda.synchronize()
        assert torch.allclose(N.double(), N2.double(), rtol=1e-3 if ftype == "f16" else 1e-6, atol=0)
        # 32 bits: 2^31 steps of FP64 rounding each.  Indices are taken before N is rounded to 16 bits, so FP16's are no further apart
        assert int((F.long() - F2.long()).abs().max()) <= (2 ** 10 if bits == 32 else 1)
        assert torch.allclose(y.double(), y2.double(), rtol=1e-2 if dtype in ("f16", "bf16") else 0, atol=1e-5 * float(y.double().abs().max()))
