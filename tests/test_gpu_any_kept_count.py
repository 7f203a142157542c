"""GPU parity of the compressed-space operations on blocks whose indices are no power-of-two number of 16-byte vectors and
on pointers that are not 16-byte aligned: at the edges of the lane teams, of the dwords and of a wave's span."""
import numpy as np
import pytest
import torch

import parity
from paper_2406_11209_amd import synth
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
