"""GPU parity of the compressed-space operations on blocks whose indices are no power-of-two number of 16-byte vectors and
on pointers that are not 16-byte aligned: at the edges of the lane teams, of the dwords and of a wave's span."""
import numpy as np
import pytest
import torch

import parity
from paper_2406_11209_amd import synth
from paper_2406_11209_amd.api import Codec
from parity import Case

pytestmark = pytest.mark.gpu

# (block extent, kept): one index; below, at and above one dword and one 16-byte vector; 19 of 64; team sizes 2 .. 64;
# more than 256 dwords per block (a lane's dwords no longer stay in registers); whole blocks of 4096 indices
KEPT = [(8, 1), (8, 3), (16, 5), (64, 17), (64, 19), (128, 65), (256, 129), (256, 255), (64 * 32, 1025), (4096, 4095)]


def make(extent, kept, bits, ftype, n_blocks, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    block = (extent,) if extent <= 256 else (64, extent // 64)
    shape = (n_blocks * extent,) if extent <= 256 else (n_blocks * 64, extent // 64)
    mask = np.zeros(extent, dtype=bool)
    mask[0] = True
    mask[1 + g.permutation(extent - 1)[:kept - 1]] = True
    dtype = "f64" if ftype == "f64" else "f32"
    cast = np.float64 if dtype == "f64" else np.float32
    mk = lambda: (synth.bump_field(shape, 6, g, (2.0, 16.0)) + 0.5 + 0.05 * g.standard_normal(shape)).astype(cast)
    return Case(mk(), mk(), dtype, block, bits, ftype, mask.reshape(block))


def check_everything(case, N1, F1, N2, F2):
    case.check_add(N1, F1, N2, F2)
    case.check_subtract(N1, F1, N2, F2)
    case.check_add_scalar(N1, F1, 0.75)
    case.check_mul_scalar(N1, F1, -2.5)
    case.check_negate(N1, F1)
    case.check_reductions(N1, F1, N2, F2)
    case.check_pair_statistics(N1, F1, N2, F2)
    case.check_blockwise(N1, F1, N2, F2)


@pytest.mark.parametrize("extent,kept", KEPT, ids=["%d_of_%d" % (k, e) for e, k in KEPT])
@pytest.mark.parametrize("bits,ftype", [(8, "f32"), (16, "f64"), (32, "f32"), (16, "f16"), (8, "f64"), (32, "f64")])
def test_any_kept_count_and_alignment(extent, kept, bits, ftype):
    n_blocks = 5 if extent > 256 else (300 if kept > 64 else 1031)
    check_kept_count(extent, kept, bits, ftype, n_blocks)


@pytest.mark.parametrize("extent,kept", KEPT[:-2], ids=["%d_of_%d" % (k, e) for e, k in KEPT[:-2]])
@pytest.mark.parametrize("bits,ftype", [(8, "f32"), (16, "f64"), (32, "f32"), (16, "f16"), (8, "f64"), (32, "f64")])
def test_any_kept_count_of_more_blocks(extent, kept, bits, ftype):
    """So many that small ones go through LDS, too: fewer are taken element by element from memory."""
    check_kept_count(extent, kept, bits, ftype, 2300 if kept > 64 else 2531)


def check_kept_count(extent, kept, bits, ftype, n_blocks):
    case = make(extent, kept, bits, ftype, n_blocks, 1000 * kept + bits)
    N1, F1 = case.codec.compress(case.xA)
    N2, F2 = case.codec.compress(case.xB)
    check_everything(case, N1, F1, N2, F2)
    # runs of blocks from the middle: the two operands at two different phases
    n = n_blocks - 3
    case.shape = (n * case.block[0],) + tuple(case.shape[1:])
    check_everything(case, N1[1:1 + n], F1[1:1 + n], N2[2:2 + n], F2[2:2 + n])
    # the same runs with results that replace an operand, or go to a third phase, leaving their surroundings alone
    want = case.codec.add(N1[1:1 + n].clone(), F1[1:1 + n].clone(), N2[2:2 + n].clone(), F2[2:2 + n].clone())
    big_N, big_F = torch.zeros_like(N1), torch.full_like(F1, 77)
    case.codec.add(N1[1:1 + n], F1[1:1 + n], N2[2:2 + n], F2[2:2 + n], big_N[3:], big_F[3:])
    before = F1.clone()
    case.codec.add(N1[1:1 + n], F1[1:1 + n], N2[2:2 + n], F2[2:2 + n], N1[1:1 + n], F1[1:1 + n])
    torch.cuda.synchronize()
    assert torch.equal(big_F[3:], want[1]) and torch.equal(big_N[3:], want[0]) and bool((big_F[:3] == 77).all())
    assert torch.equal(F1[1:1 + n], want[1]) and torch.equal(N1[1:1 + n], want[0])
    assert torch.equal(F1[:1], before[:1]) and torch.equal(F1[1 + n:], before[1 + n:])


def test_segments_at_every_phase():
    """Steps of 37 blocks of 10 int8 indices: every step starts at another address modulo 16."""
    case = make(64, 10, 8, "f32", 37 * 21, 5)
    N, F = case.codec.compress(case.xA)
    run, steps = 37, 21
    got = case.codec.segmented("variance", steps, run, N, F)
    cov = case.codec.segmented("covariance", steps - 1, run, N, F, N[run:], F[run:])
    dist = case.codec.segmented("difference_norm2", steps - 1, run, N, F, N[run:], F[run:])
    one = lambda op, t, *rest: getattr(case.codec, op)(N[t * run:(t + 1) * run], F[t * run:(t + 1) * run], *rest).item()
    for t in range(steps):
        assert got[t].item() == pytest.approx(one("variance", t), rel=1e-13)
        if t + 1 < steps:
            nxt = (N[(t + 1) * run:(t + 2) * run], F[(t + 1) * run:(t + 2) * run])
            assert dist[t].item() == pytest.approx(one("difference_norm2", t, *nxt), rel=1e-13)
            assert abs(cov[t].item() - one("covariance", t, *nxt)) <= 1e-13 * abs(got[t].item())


@pytest.mark.parametrize("run", [70, 230, 700])                # 9, 30 and 92 KB a segment
@pytest.mark.parametrize("segments", [341, 342, 400, 410, 682, 683, 1025, 2049])
def test_many_segments_by_one_workgroup_each_or_a_few(segments, run):
    g = torch.Generator("cuda").manual_seed(segments + run)
    mask = np.zeros(64, dtype=bool)
    mask[:33] = True
    codec = Codec((8, 8), "f64", 32, mask.reshape(8, 8))
    n, r = segments * run, 2 ** 31 - 1
    (N1, F1), (N2, F2) = [(torch.rand(n, generator=g, device="cuda", dtype=torch.float64) + 0.1,
                           torch.randint(-r, r + 1, (n, 33), generator=g, device="cuda").to(torch.int32)) for _ in range(2)]
    C1, C2 = [(F.double() * (N / r)[:, None]).view(segments, run, 33) for N, F in ((N1, F1), (N2, F2))]
    sums = lambda x: x.sum(dim=(1, 2))
    size = sums(C1 * C1 + C2 * C2)
    mean = C1[:, :, 0].sum(dim=1) / (8 * run)                  # a first coefficient is 8 times its block's mean
    for got, want in ((codec.segmented("norm2", segments, run, N1, F1) ** 2, sums(C1 * C1)),
                      (codec.segmented("variance", segments, run, N1, F1) * (64 * run), sums(C1 * C1) - mean * mean * (64 * run)),
                      (codec.segmented("dot", segments, run, N1, F1, N2, F2), sums(C1 * C2)),
                      (codec.segmented("difference_norm2", segments, run, N1, F1, N2, F2) ** 2, sums((C1 - C2) ** 2))):
        assert bool(((got - want).abs() <= 1e-12 * size).all())      # 2^-53 a term, 23000 terms at most


# kept counts and block counts around which a call changes from one kernel to another: element by element or through LDS
HALVES = [(8, 1, 8, 16385), (8, 3, 16, 16385), (64, 19, 8, 2049), (128, 128, 32, 2049), (128, 100, 32, 16385), (256, 160, 32, 16385),
          (256, 192, 16, 2049), (64, 20, 32, 257), (16, 5, 16, 257), (4096, 2049, 32, 2049), (4096, 4096, 32, 2049), (4096, 4096, 16, 2049),
          (64, 19, 8, 1025), (256, 192, 16, 1025), (128, 65, 16, 513), (8, 3, 16, 257), (8, 1, 32, 513), (4096, 2500, 32, 3073), (4096, 3000, 32, 3073),
          (4096, 3601, 32, 4097), (256, 144, 32, 5121), (256, 160, 8, 1025), (8, 2, 16, 32769), (128, 66, 16, 513),
          (64, 18, 16, 1025), (64, 19, 16, 1025), (64, 63, 32, 1025), (128, 65, 32, 1025), (64, 56, 8, 1025), (64, 57, 8, 1025)]


@pytest.mark.parametrize("extent,kept,bits,n", HALVES, ids=["%d_of_%d_i%d_x%d" % (k, e, b, n) for e, k, b, n in HALVES])
def test_a_call_agrees_with_the_calls_on_its_halves(extent, kept, bits, n):
    g = torch.Generator("cuda").manual_seed(kept + n)
    block = (extent,) if extent <= 256 else (64, extent // 64)
    mask = np.zeros(extent, dtype=bool)
    mask[:kept] = True
    codec = Codec(block, "f32", bits, mask.reshape(block))
    r = 2 ** (bits - 1) - 1
    ops = []
    for _ in range(2):
        F = torch.randint(-r, r + 1, (n + 1, kept), generator=g, device="cuda").to({8: torch.int8, 16: torch.int16, 32: torch.int32}[bits])
        ops.append((torch.rand(n + 1, generator=g, device="cuda") + 0.1, F))
    # one block on, so that aligned blocks of whole vectors come this way, too
    (N1, F1), (N2, F2) = [(N[1:], F[1:]) for N, F in ops]
    h = n // 2
    parts = [slice(0, h), slice(h, n)]
    for whole, halves in ((codec.add(N1, F1, N2, F2), [codec.add(N1[p], F1[p], N2[p], F2[p]) for p in parts]),
                          (codec.add_scalar(N1, F1, 0.75), [codec.add_scalar(N1[p], F1[p], 0.75) for p in parts])):
        assert torch.equal(whole[0], torch.cat([p[0] for p in halves]))
        # both quotients are rounded correctly, up to double rounding within 2^-53 of a tie
        assert int((whole[1] != torch.cat([p[1] for p in halves])).sum()) <= (2 if bits == 32 else 0)
    for op, args in (("blockwise_variance", (N1, F1)), ("blockwise_covariance", (N1, F1, N2, F2))):
        whole = getattr(codec, op)(*args)
        split = torch.cat([getattr(codec, op)(*[a[p] for a in args]) for p in parts])
        scale = codec.blockwise_variance(N1, F1).abs() + codec.blockwise_variance(N2, F2).abs()
        assert bool(((whole - split).abs() <= 1e-13 * scale).all())
    for op, args, power in (("norm2", (N1, F1), 2), ("difference_norm2", (N1, F1, N2, F2), 2), ("dot", (N1, F1, N2, F2), 1)):
        whole = getattr(codec, op)(*args).item() ** power
        split = sum(getattr(codec, op)(*[a[p] for a in args]).item() ** power for p in parts)
        size = codec.norm2(N1, F1).item() ** 2 + codec.norm2(N2, F2).item() ** 2
        assert abs(whole - split) <= 1e-12 * size, op
    for op in ("variance", "norm2"):
        halves = codec.segmented(op, 2, h, N1[:2 * h], F1[:2 * h])
        for half, p in zip(halves.tolist(), (slice(0, h), slice(h, 2 * h))):
            assert half == pytest.approx(getattr(codec, op)(N1[p], F1[p]).item(), rel=1e-12)


# Around the most dwords that a lane holds (5 or 6, 10 or 12, 12), with every remainder of a dword, as many blocks as it takes to have a lane hold
# that many; then the largest blocks that a team of 64 lanes holds, and the next
HELD = ([(8, k, 64 * 4096 + 37) for k in (1, 3, 15, 19, 20, 21, 22, 24, 25)] + [(16, k, 64 * 4096 + 37) for k in (1, 3, 19, 20, 21, 23, 24, 25)] +
        [(32, k, 64 * 4096 + 37) for k in (1, 11, 12, 13)] +
        [(8, k, 70) for k in (1279, 1280, 1281, 1536, 1537)] + [(16, k, 70) for k in (1280, 1281, 1536, 1537)] + [(32, k, 70) for k in (768, 769, 1024, 2047, 4095)])


@pytest.mark.parametrize("ftype", ["f32", "f64"])
@pytest.mark.parametrize("bits,kept,n", HELD, ids=["i%d_%d_x%d" % h for h in HELD])
def test_rebinning_of_blocks_held_in_registers(bits, kept, n, ftype):
    g = torch.Generator("cuda").manual_seed(100 * kept + bits)
    mask = np.zeros(64 if kept <= 64 else 4096, dtype=bool)
    mask[:kept] = True
    codec = Codec((64,) if kept <= 64 else (64, 64), ftype, bits, mask if kept <= 64 else mask.reshape(64, 64))
    r = 2 ** (bits - 1) - 1
    divisor = torch.tensor(float(r), dtype=torch.float64, device="cuda")      # torch multiplies by the reciprocal of a plain number
    itype, ntype = {8: torch.int8, 16: torch.int16, 32: torch.int32}[bits], {"f32": torch.float32, "f64": torch.float64}[ftype]
    make = lambda: (torch.rand(n + 1, generator=g, device="cuda", dtype=torch.float64).to(ntype) + 0.1,
                    torch.randint(-r, r + 1, (n + 1, kept), generator=g, device="cuda").to(itype))
    operands = [make(), make()]
    operands[0][1][5] = 0
    operands[1][1][5] = 0                                       # a block of zeros in both
    for first, second in ((0, 0), (1, 0), (0, 1)):              # equal and different phases of the two operands
        (N1, F1), (N2, F2) = [(N[p:p + n], F[p:p + n]) for (N, F), p in zip(operands, (first, second))]
        # the three roundings of a coefficient as the kernels have them; |quotient| <= r
        add = F1.double() * N1.double()[:, None] + F2.double() * N2.double()[:, None]
        shift = N1.double()[:, None] * F1.double() / divisor
        shift[:, 0] += 0.375 * np.sqrt(64.0 if kept <= 64 else 4096.0)
        for c, scale, got in ((add, add.abs().amax(1) / divisor, codec.add(N1, F1, N2, F2)),
                              (shift, shift.abs().amax(1), codec.add_scalar(N1, F1, 0.375))):
            quotient = (c if c is add else c * r) / scale[:, None]
            want = torch.where(scale[:, None] > 0, quotient, torch.zeros_like(c)).round()
            # the sum's N is rounded correctly; N F / r before the shift is, too, up to double rounding: a unit in the last place
            assert bool(((got[0] - scale.to(ntype)).abs() <= (2.0 ** -52 * scale if c is shift and ftype == "f64" else 0)).all())
            # both quotients are rounded correctly, up to double rounding within 2^-53 of a tie
            assert int((got[1] != want.to(itype)).sum()) <= (2 if bits == 32 else 0)
        # the result in an operand's place, with its neighbours as they were
        N, F = operands[0][0].clone(), operands[0][1].clone()
        codec.add(N[first:first + n], F[first:first + n], N2, F2, N[first:first + n], F[first:first + n])
        want = codec.add(N1, F1, N2, F2)
        assert torch.equal(F[first:first + n], want[1]) and torch.equal(N[first:first + n], want[0])
        assert torch.equal(F[:first], operands[0][1][:first]) and torch.equal(F[first + n:], operands[0][1][first + n:])
