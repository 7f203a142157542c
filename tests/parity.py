"""Helpers of the GPU parity tests: run one workload through the HIP path and through the oracle, and
compare to the stated tolerances.

Tolerances
----------
* Indices: bit-exact, except that an entry whose pre-rounding value t (as the oracle computes it in FP64)
  lies within TAU of a rounding boundary k + 1/2 may differ by one; at most 1e-4 of the entries may
  differ at all.  TAU = r * u * (2 + sum(i)) with u the unit round-off of the precision the binning
  decision is taken in (2^-24 when the kernels bin in FP32: working type FP32/16-bit with int8 indices;
  2^-53 otherwise), the bound on how far a transform in that precision can move t.
* N: relative 1e-6 (FP32 and 16-bit working types; one rounding of a value whose FP32 computation is
  accurate to a few ulp) / 1e-13 (FP64).
* Decompressed arrays and scalars: relative 1e-5 when the working type is FP32 or narrower, 1e-12 when
  it is FP64; arrays relative to the array's largest magnitude, scalars relative to their own magnitude
  plus a floor at the natural scale of a sum that cancels (||A|| ||B|| for dot and covariance, ...).
* Decompress and every operation are compared on identical (N, F): the oracle is run on the compressed
  arrays the GPU produced (a legitimately flipped tie moves a decoded coefficient by N/r, which would
  swamp 1e-5 otherwise).
"""
from __future__ import annotations

import ctypes
import math
from dataclasses import dataclass
from typing import Optional, Sequence

import numpy as np
import torch

from oracle import pbz_oracle as po
from paper_2406_11209_amd import api
from paper_2406_11209_amd.api import Codec

TORCH_DTYPE = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
MAX_MISMATCH_FRACTION = 1e-4
# Haar coefficients of the smooth synthetic fields crowd near half-integers after scaling (the oracle's own
# pre-rounding values lie inside the tie band four times as often as for the DCT: 1.9e-3 against 4e-4 of them on
# the 16 x 16 case), so FP32 arithmetic of any order flips more of them; every flip must still be a tie and +-1.
MAX_MISMATCH_FRACTION_HAAR = 1e-3
EXACT_TIE = 1e-9     # |frac(t) - 1/2| below this: a tie in exact arithmetic


# Which kernels take a compress or decompress call (the library's internal numbering, in the order in which it asks them): those for
# exactly this setting, the same families under any mask, those per block shape, those for lines of 64, the tiled and the dense ones.
EXACT, MASKED, SHAPE, LINES, TILED, DENSE = range(6)


def route(codec: Codec, op: str, shape, dtype: str, array: int = 256) -> int:
    """Where a call would go; `array`: the array's address (its alignment counts)."""
    fn = codec._lib.pbz_internal_route
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.POINTER(ctypes.c_int64), ctypes.c_int, ctypes.c_uint64]
    got = fn(codec._h, int(op == "decompress"), (ctypes.c_int64 * len(shape))(*shape), api.FTYPES[dtype], array)
    assert got >= 0
    return got


def take_wherever_possible(codec: Codec, kind: int) -> None:
    """MASKED or SHAPE: that kind of kernels for every call they can take, whatever the rules on sizes say."""
    fn = codec._lib.pbz_internal_set_route
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int]
    assert fn(codec._h, kind) == 0


def value_tol(ftype: str) -> float:
    return 1e-12 if ftype == "f64" else 1e-5


def n_tol(ftype: str) -> float:
    return {"f64": 1e-13, "f32": 1e-6, "f16": 1e-3, "bf16": 8e-3}[ftype]


def bins_in_f32(ftype: str, index_bits: int) -> bool:
    return ftype != "f64" and index_bits == 8


def tie_band(block: Sequence[int], ftype: str, index_bits: int) -> float:
    u = 2.0 ** -24 if bins_in_f32(ftype, index_bits) else 2.0 ** -53
    return po.index_radius(index_bits) * u * (2 + sum(block))


def to_device(x: np.ndarray, dtype: str) -> torch.Tensor:
    if dtype == "bf16":
        return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(x)).cuda()


def to_host_f64(t: torch.Tensor) -> np.ndarray:
    return t.detach().to(torch.float64).cpu().numpy()


def oracle_compressed(N: torch.Tensor, F: torch.Tensor, shape, block, index_bits, ftype, mask,
                      transform: str = "dct") -> po.Compressed:
    """The oracle's view of a compressed array that lives on the GPU (same bits)."""
    P = np.ones(tuple(block), dtype=bool) if mask is None else np.asarray(mask, dtype=bool).reshape(tuple(block))
    grid = po.block_grid(shape, block)
    return po.Compressed(s=tuple(shape), i=tuple(block), N=to_host_f64(N).reshape(grid), F=F.cpu().numpy(), P=P,
                         index_bits=index_bits, ftype=ftype, transform=transform)


STRICT_FROM = 100_000   # arrays of at least this many indices are held to the target's rule with no allowance


@dataclass
class IndexCounts:
    """What check_indices saw: every differing index, how many of them lie inside the tie band, and how many sit on
    a value that is a half-integer in exact arithmetic (both neighbours equally correct)."""
    size: int = 0
    total: int = 0
    in_band: int = 0
    exact_tie: int = 0

    def __int__(self):
        return self.total

    def __eq__(self, other):
        return self.total == other if isinstance(other, int) else NotImplemented

    def __iadd__(self, other):
        self.size += other.size; self.total += other.total; self.in_band += other.in_band; self.exact_tie += other.exact_tie
        return self

    def __str__(self):
        rate = self.total / self.size if self.size else 0.0
        return (f"{self.total} of {self.size} indices differ ({rate:.2e}); in the tie band {self.in_band}, "
                f"at exact ties {self.exact_tie}")


def check_cap(counts: IndexCounts, what: str, max_fraction: float = MAX_MISMATCH_FRACTION, strict=None):
    """The cap on the number of differing indices.  Strict form (the target's own rule, arrays of STRICT_FROM indices
    and more, so every full-size workload): every differing index counts, exact ties included, and the count may not
    exceed max_fraction of the entries.  Small-array form (the unit-test shapes, where the expected count is below
    ten and one unlucky draw would decide): exact ties are not counted and the count gets three standard deviations
    of counting noise, at least one."""
    strict = counts.size >= STRICT_FROM if strict is None else strict
    if strict:
        assert counts.total <= max_fraction * counts.size, f"{what}: {counts} (cap {max_fraction:.0e}, strict)"
        return
    expected = max_fraction * counts.size
    allowed = max(1, int(math.ceil(expected + 3.0 * math.sqrt(expected))))
    counted = counts.total - counts.exact_tie
    assert counted <= allowed, f"{what}: {counts} (cap {max_fraction:.0e} allows {allowed} at inexact ties)"


def check_indices(F_gpu: np.ndarray, F_ref: np.ndarray, t_ref: np.ndarray, tau: float, what: str = "F",
                  max_fraction: float = MAX_MISMATCH_FRACTION, strict=None, cap: bool = True) -> IndexCounts:
    """Indices bit-exact except at rounding ties: every differing index differs by one and its exact pre-rounding
    value lies within tau of a half-integer; the number of differing indices is capped (check_cap).  cap=False leaves
    the cap to the caller, who adds up the counts of several pieces of one array first."""
    assert F_gpu.shape == F_ref.shape, (F_gpu.shape, F_ref.shape)
    bad = F_gpu != F_ref
    counts = IndexCounts(size=int(F_ref.size), total=int(np.count_nonzero(bad)))
    if counts.total:
        diff = F_gpu[bad].astype(np.int64) - F_ref[bad].astype(np.int64)
        assert np.max(np.abs(diff)) <= 1, f"{what}: an index differs by more than 1"
        tb = t_ref[bad]
        dist = np.abs(np.abs(tb - np.floor(tb)) - 0.5)
        counts.in_band = int((dist <= tau).sum())
        assert counts.in_band == counts.total, (f"{what}: {counts.total - counts.in_band} mismatches are not rounding "
                                                f"ties (worst distance {dist.max():.3e} > band {tau:.3e})")
        # A value that is a half-integer in exact arithmetic has two equally correct indices.  "Exact" is to the
        # resolution of the oracle's own t: with 32-bit indices |t| reaches 2^31, where FP64 resolves only 2^-22, so
        # a half-integer in exact arithmetic can sit a few 1e-7 from one in the oracle's t.
        exact = np.maximum(EXACT_TIE, 4.0 * np.abs(tb) * 2.0 ** -52)
        counts.exact_tie = int((dist <= exact).sum())
    if cap:
        check_cap(counts, what, max_fraction, strict)
    return counts


def check_N(N_gpu: np.ndarray, N_ref: np.ndarray, ftype: str, what: str = "N"):
    N_gpu = N_gpu.reshape(-1)
    N_ref = N_ref.reshape(-1)
    assert np.all(np.isfinite(N_gpu))
    assert np.all(np.abs(N_gpu - N_ref) <= n_tol(ftype) * np.abs(N_ref)), \
        f"{what}: worst relative error {np.max(np.abs(N_gpu - N_ref) / np.maximum(np.abs(N_ref), 1e-300)):.3e}"


def check_array(y_gpu: np.ndarray, y_ref: np.ndarray, tol: float, what: str = "array"):
    scale = float(np.max(np.abs(y_ref))) if y_ref.size else 0.0
    err = float(np.max(np.abs(y_gpu - y_ref))) if y_ref.size else 0.0
    assert err <= tol * scale + 1e-300, f"{what}: max error {err:.3e} > {tol:.0e} * {scale:.3e}"


def check_scalar(got: float, want: float, tol: float, floor: float, what: str):
    assert math.isfinite(got), what
    assert abs(got - want) <= tol * abs(want) + tol * floor, \
        f"{what}: got {got!r}, oracle {want!r}, |diff| {abs(got - want):.3e}"


class Case:
    """One array pair + settings, run through both implementations."""

    transform = "dct"

    def __init__(self, A: np.ndarray, B: Optional[np.ndarray], dtype: str, block, index_bits: int, ftype: str,
                 mask: Optional[np.ndarray] = None, path: int = 0, transform: str = "dct"):
        self.dtype, self.block, self.bits, self.ftype, self.mask = dtype, tuple(block), index_bits, ftype, mask
        self.shape = tuple(A.shape)
        self.transform = transform
        self.codec = Codec(self.block, ftype, index_bits, mask, transform)
        if path:
            self.codec.set_kernel_path(path)
        self.hostA, self.hostB = A, B
        self.xA = to_device(A, dtype)
        self.xB = None if B is None else to_device(B, dtype)
        self.tau = tie_band(self.block, ftype, index_bits)
        self.tol = value_tol(ftype)

    def host_f64(self, x: np.ndarray) -> np.ndarray:
        if self.dtype == "bf16":
            return po.bf16_bits_to_f64(x)
        return np.asarray(x, dtype=np.float64)

    # --- codec -------------------------------------------------------------------------------
    def check_compress(self, which="A"):
        x_dev = self.xA if which == "A" else self.xB
        x_host = self.hostA if which == "A" else self.hostB
        N, F = self.codec.compress(x_dev)
        torch.cuda.synchronize()
        ref = po.compress(self.host_f64(x_host), self.block, self.bits, self.ftype, self.mask, self.transform)
        check_N(to_host_f64(N), ref.N, self.ftype)
        n_bad = check_indices(F.cpu().numpy(), ref.F, ref.t, self.tau,
                              max_fraction=MAX_MISMATCH_FRACTION_HAAR if self.transform == "haar" else MAX_MISMATCH_FRACTION)
        self.__dict__.setdefault("last_counts", {})[which] = n_bad
        return N, F, ref, n_bad

    def check_wasserstein(self, N1, F1, N2, F2, p: float):
        """Algorithm 13 against the oracle.  exp and pow come from different libraries on the two sides and every
        difference of two softmax outputs loses digits to cancellation, so the bar is 1e-9 relative, not 1e-12."""
        got = self.codec.approximate_wasserstein(N1, F1, N2, F2, p)
        torch.cuda.synchronize()
        want = po.approximate_wasserstein(self.oc(N1, F1), self.oc(N2, F2), p)
        got = float(got.item())
        assert math.isfinite(got)
        assert abs(got - want) <= 1e-9 * abs(want) + 1e-300, f"wasserstein(p={p}): got {got!r}, oracle {want!r}"
        return got

    def check_compress_statistics(self, N, F, which="A"):
        """The fused entry point writes the same {N, F} as pbz_compress, and its statistics (and those of the
        one-pass pbz_statistics) are the oracle's mean / variance / norm2 of that compressed array."""
        x_dev = self.xA if which == "A" else self.xB
        Ns, Fs, st = self.codec.compress_statistics(x_dev)
        one_pass = self.codec.statistics(N, F)
        torch.cuda.synchronize()
        assert torch.equal(Fs, F) and torch.equal(Ns, N), "fused compress differs from pbz_compress"
        A = self.oc(N, F)
        na = po.norm2(A)
        n_el = float(A.n_blocks) * float(np.prod(self.block))
        want = (po.mean(A), po.variance(A), na)
        floors = (na / math.sqrt(n_el), na * na / n_el, 0.0)
        for got in (st.cpu().numpy(), one_pass.cpu().numpy()):
            for g, w, f, name in zip(got, want, floors, ("mean", "variance", "norm2")):
                check_scalar(float(g), w, self.tol, f, "statistics." + name)
        # one triple per block index along dimension 0: the oracle's statistics of each run of blocks
        _, _, rows = self.codec.compress_statistics(x_dev, per_step=True)
        rows = rows.cpu().numpy()
        per = A.n_blocks // A.b[0]
        assert rows.shape == (A.b[0], 3)
        for t in range(A.b[0]):
            run = po.Compressed(s=(A.i[0],) + tuple(A.s[1:]), i=A.i, N=A.N.reshape(A.b)[t:t + 1],
                                F=A.F[t * per:(t + 1) * per], P=A.P, index_bits=A.index_bits, ftype=A.ftype,
                                transform=A.transform)
            nr = po.norm2(run)
            n_run = float(per) * float(np.prod(self.block))
            for g, w, f, name in zip(rows[t], (po.mean(run), po.variance(run), nr),
                                     (nr / math.sqrt(n_run), nr * nr / n_run, 0.0), ("mean", "variance", "norm2")):
                check_scalar(float(g), w, self.tol, f, f"statistics[{t}].{name}")
        return st

    def check_pair_statistics(self, N1, F1, N2, F2):
        """The nine statistics of one pass over both operands, each against the oracle's own function."""
        got = self.codec.pair_statistics(N1, F1, N2, F2)
        torch.cuda.synchronize()
        got = got.cpu().numpy()
        A, B = self.oc(N1, F1), self.oc(N2, F2)
        na, nb = po.norm2(A), po.norm2(B)
        n_el = float(A.n_blocks) * float(np.prod(self.block))
        want = [(po.dot(A, B), na * nb), (po.cosine_similarity(A, B), 1.0), (po.covariance(A, B), na * nb / n_el),
                (po.mean(A), na / math.sqrt(n_el)), (po.mean(B), nb / math.sqrt(n_el)),
                (po.variance(A), na * na / n_el), (po.variance(B), nb * nb / n_el), (na, 0.0), (nb, 0.0)]
        for name, g, (w, floor) in zip(self.codec.PAIR_STATISTICS, got, want):
            check_scalar(float(g), w, self.tol, floor, "pair_statistics." + name)
        return got

    def oc(self, N, F) -> po.Compressed:
        return oracle_compressed(N, F, self.shape, self.block, self.bits, self.ftype, self.mask, self.transform)

    def check_decompress(self, N, F, out_dtype: Optional[str] = None):
        out_dtype = out_dtype or self.dtype
        y = self.codec.decompress(N, F, self.shape, TORCH_DTYPE[out_dtype])
        torch.cuda.synchronize()
        ref = po.decompress(self.oc(N, F))
        tol = self.tol
        # the output cast dominates: half an ulp of the output type (an FP32 array only when the arithmetic and N are FP64)
        if out_dtype in ("bf16", "f16") or (out_dtype == "f32" and self.tol < 2.0 ** -24):
            tol = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11, "f32": 2.0 ** -24}[out_dtype] * 1.01
            err = np.abs(to_host_f64(y) - ref)
            assert np.all(err <= tol * np.abs(ref) + self.tol * np.max(np.abs(ref)) + 1e-30), \
                f"decompress[{out_dtype}]: worst {np.max(err):.3e}"
        else:
            check_array(to_host_f64(y), ref, tol, f"decompress[{out_dtype}]")
        return y

    # --- element-wise ops ------------------------------------------------------------------------
    def check_negate(self, N, F):
        G = self.codec.negate(F)
        torch.cuda.synchronize()
        assert np.array_equal(G.cpu().numpy(), po.negate(self.oc(N, F)).F)
        return G

    def check_mul_scalar(self, N, F, x: float):
        N2, F2 = self.codec.mul_scalar(N, F, x)
        torch.cuda.synchronize()
        ref = po.multiply_scalar(self.oc(N, F), x)
        assert np.array_equal(F2.cpu().numpy(), ref.F)
        assert np.array_equal(to_host_f64(N2), ref.N.reshape(-1)), "mul_scalar: N must match bit for bit"
        return N2, F2

    def check_add(self, N1, F1, N2, F2):
        N3, F3 = self.codec.add(N1, F1, N2, F2)
        torch.cuda.synchronize()
        ref = po.add(self.oc(N1, F1), self.oc(N2, F2))
        # the kernel takes the printed operation order in FP64, like the oracle: ties included, exact
        check_N(to_host_f64(N3), ref.N, self.ftype, "add.N")
        check_indices(F3.cpu().numpy(), ref.F, ref.t, po.index_radius(self.bits) * 2.0 ** -50, "add.F")
        return N3, F3

    def check_subtract(self, N1, F1, N2, F2):
        """The one-pass difference: the oracle's add(A, negate(B)), and bit for bit the two-call route."""
        N3, F3 = self.codec.subtract(N1, F1, N2, F2)
        N4, F4 = self.codec.add(N1, F1, N2, self.codec.negate(F2))
        torch.cuda.synchronize()
        ref = po.add(self.oc(N1, F1), po.negate(self.oc(N2, F2)))
        check_N(to_host_f64(N3), ref.N, self.ftype, "subtract.N")
        check_indices(F3.cpu().numpy(), ref.F, ref.t, po.index_radius(self.bits) * 2.0 ** -50, "subtract.F")
        assert torch.equal(N3, N4) and torch.equal(F3, F4), "subtract differs from negate + add"
        return N3, F3

    def check_add_scalar(self, N, F, x: float):
        N2, F2 = self.codec.add_scalar(N, F, x)
        torch.cuda.synchronize()
        ref = po.add_scalar(self.oc(N, F), x)
        # FP64 on both sides; the kernel multiplies by 1/r and r/N where the oracle divides: a few ulp on t
        check_N(to_host_f64(N2), ref.N, self.ftype, "add_scalar.N")
        check_indices(F2.cpu().numpy(), ref.F, ref.t, po.index_radius(self.bits) * 2.0 ** -48, "add_scalar.F")
        return N2, F2

    def check_blockwise(self, N1, F1, N2, F2):
        A, B = self.oc(N1, F1), self.oc(N2, F2)
        pairs = [("blockwise_mean", self.codec.blockwise_mean(N1, F1), po.blockwise_mean(A)),
                 ("blockwise_variance", self.codec.blockwise_variance(N1, F1), po.blockwise_variance(A)),
                 ("blockwise_std", self.codec.blockwise_std(N1, F1), po.blockwise_std(A)),
                 ("blockwise_covariance", self.codec.blockwise_covariance(N1, F1, N2, F2), po.blockwise_covariance(A, B))]
        torch.cuda.synchronize()
        for name, got, want in pairs:
            tol = self.tol
            if name == "blockwise_std":      # sqrt of a difference that can cancel to ~0: compare the squares' scale
                tol = math.sqrt(self.tol) if self.ftype != "f64" else 1e-9
            check_array(to_host_f64(got), want.reshape(-1), tol, name)

    def check_ssim(self, N1, F1, N2, F2, **kw):
        A, B = self.oc(N1, F1), self.oc(N2, F2)
        got = float(self.codec.ssim(N1, F1, N2, F2, **kw).item())
        want = po.ssim(A, B, **kw)
        # Variance and covariance come out of the one pass as S - D1 D2 / n, whose rounding (a few units in the
        # last place of S) is relative to the mean square of the arrays, not to the variance; Algorithm 12 takes
        # roots of the variances and divides by sums that can be as small as its stabilisers.  Both sides work in
        # FP64 from the same {N, F}: the bar adds what that rounding can do to the three factors.
        n_el = float(A.n_blocks) * float(np.prod(self.block))
        s_l, s_c = kw.get("s_l", 1e-4), kw.get("s_c", 9e-4)
        da, db = (16 * 2.0 ** -52 * po.norm2(X) ** 2 / n_el for X in (A, B))         # on var_a, var_b (and cov)
        va, vb = max(po.variance(A), 0.0), max(po.variance(B), 0.0)
        root_err = lambda v, d: min(math.sqrt(d), d / (2.0 * math.sqrt(v))) if v > 0.0 else math.sqrt(d)
        ea, eb = root_err(va, da), root_err(vb, db)
        d_sd = ea * math.sqrt(vb) + eb * math.sqrt(va) + ea * eb
        d_cov = math.sqrt(da * db)
        weight = max(1.0, kw.get("w_c", 1.0), kw.get("w_s", 1.0), kw.get("w_l", 1.0))
        slack = weight * ((2.0 * d_sd + da + db) / max(s_c, 1e-300) + (d_cov + d_sd) / max(0.5 * s_c, 1e-300)
                          + (da + db) / max(s_l, 1e-300))
        floor = 1.0 + slack / self.tol
        check_scalar(got, want, self.tol, floor, "ssim")
        return got

    # --- reductions ------------------------------------------------------------------------------
    def check_reductions(self, N1, F1, N2, F2, ops=("dot", "norm2", "cosine_similarity", "mean", "covariance", "variance",
                                                      "difference_norm2")):
        A, B = self.oc(N1, F1), self.oc(N2, F2)
        na, nb = po.norm2(A), po.norm2(B)
        n_el = float(A.n_blocks) * float(np.prod(self.block))
        out = {}
        for op in ops:
            if op == "dot":
                got, want, floor = self.codec.dot(N1, F1, N2, F2), po.dot(A, B), na * nb
            elif op == "norm2":
                got, want, floor = self.codec.norm2(N1, F1), na, 0.0
            elif op == "cosine_similarity":
                got, want, floor = self.codec.cosine_similarity(N1, F1, N2, F2), po.cosine_similarity(A, B), 1.0
            elif op == "mean":
                got, want, floor = self.codec.mean(N1, F1), po.mean(A), na / math.sqrt(n_el)
            elif op == "covariance":
                got, want, floor = self.codec.covariance(N1, F1, N2, F2), po.covariance(A, B), na * nb / n_el
            elif op == "variance":
                got, want, floor = self.codec.variance(N1, F1), po.variance(A), na * na / n_el
            elif op == "difference_norm2":    # each difference carries a rounding relative to its operands
                got, want, floor = self.codec.difference_norm2(N1, F1, N2, F2), po.difference_norm2(A, B), na + nb
            else:
                raise ValueError(op)
            torch.cuda.synchronize()
            got = float(got.item())
            check_scalar(got, want, self.tol, floor, op)
            out[op] = got
        return out
