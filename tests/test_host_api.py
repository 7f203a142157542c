"""Host-only checks of the C ABI: the library loads without a GPU, exports every symbol the header
declares, validates arguments before touching a device, and does the layout / storage arithmetic of
Sec. III-B and Sec. IV-C.  No compute call is made here."""
import ctypes
import os
import re
import types

import numpy as np
import pytest

from paper_2406_11209_amd import api
from paper_2406_11209_amd.api import Codec, PbzError

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    text = open(os.path.join(ROOT, "include", "pbz.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pbz_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = api.load_library()
    names = header_functions()
    assert len(names) == 36
    for name in names:
        assert hasattr(lib, name), name
    assert sorted(api.SIGNATURES) == names        # the binding covers exactly the header


def test_status_strings():
    for code in range(0, -14, -1):
        assert api.status_string(code) not in ("", "unknown status")
    assert api.status_string(-99) == "unknown status"


def _create(ndim, block, ftype=api.PBZ_F32, itype=api.PBZ_I8, mask=None):
    lib = api.load_library()
    h = ctypes.c_void_p()
    arr = (ctypes.c_int64 * max(1, len(block)))(*block)
    m = None if mask is None else (ctypes.c_uint8 * len(mask))(*mask)
    st = lib.pbz_codec_create(ctypes.byref(h), ndim, arr, ftype, itype, m)
    if st == 0:
        lib.pbz_codec_destroy(h)
    return st


def test_codec_create_validation():
    assert _create(2, [8, 8]) == 0
    assert _create(0, [8]) == -2
    assert _create(9, [2] * 9) == -2
    assert _create(2, [8, 6]) == -3              # not a power of two
    assert _create(2, [0, 8]) == -3
    assert _create(1, [512]) == -3               # extent limit
    assert _create(2, [128, 64]) == -3           # volume limit
    assert _create(2, [8, 8], ftype=7) == -4
    assert _create(2, [8, 8], itype=api.PBZ_I64) == -4
    assert _create(2, [2, 2], mask=[0, 0, 0, 0]) == -5
    assert _create(2, [2, 2], mask=[0, 1, 0, 0]) == 0
    lib = api.load_library()
    assert lib.pbz_codec_create(None, 2, (ctypes.c_int64 * 2)(8, 8), 1, 0, None) == -1
    lib.pbz_codec_destroy(None)                  # tolerated


def test_layout_of_the_five_workloads():
    rows = [((256, 256), (8, 8), "f32", "i8", None, 1024, 64, 4096, 65536),
            ((4096, 4096), (8, 8), "f32", "i16", (4, 4), 262144, 16, 1048576, 8388608),
            ((64, 1024, 1024), (1, 16, 16), "f32", "i8", None, 262144, 256, 1048576, 67108864),
            ((512, 512, 512), (4, 4, 4), "f64", "i16", None, 2097152, 64, 16777216, 268435456),
            ((1024, 1024, 512), (8, 8, 8), "f32", "i8", (4, 4, 4), 1048576, 64, 4194304, 67108864)]
    for shape, block, ft, it, keep, nb, kept, nbytes, fbytes in rows:
        mask = None
        if keep:
            mask = np.zeros(block, dtype=bool)
            mask[tuple(slice(0, k) for k in keep)] = True
        lay = Codec(block, ft, it, mask).layout(shape)
        assert (lay.n_blocks, lay.kept_per_block, lay.n_bytes, lay.f_bytes) == (nb, kept, nbytes, fbytes)
        assert lay.workspace_bytes >= 8 * 5


def test_layout_takes_extents_of_any_kind_of_number():
    codec = Codec((8, 8), "f32", "i8")
    want = codec.layout([20, 16])
    for shape in ((20, 16), (np.int64(20), np.int32(16)), (np.array(20), np.array(16)), (20.0, 16), np.array([20, 16])):
        assert codec.layout(shape) == want


def test_layout_ragged_and_errors():
    c = Codec((2, 4), "f32", "i16")
    lay = c.layout((3, 5))
    assert (lay.n_blocks, lay.kept_per_block, lay.n_bytes, lay.f_bytes) == (4, 8, 16, 64)
    with pytest.raises(PbzError) as e:
        c.layout((3, 0))
    assert e.value.status == -7
    with pytest.raises(PbzError):
        c.layout((2**40, 2**40))


def test_compressed_bits_follow_the_papers_component_list(golden):
    # Sec. IV-C example: (3,224,224), block 4^3, FP32 N, int16, no pruning -> ratio ~2.91; int8 + half pruned -> ~10.66
    for s, u, i, f, ib, kept, want, stored in golden("paper_compression_ratios.txt"):
        s = tuple(int(v) for v in s.split(","))
        i = tuple(int(v) for v in i.split(","))
        mask = np.zeros(int(np.prod(i)), dtype=bool)
        mask[: int(kept)] = True
        c = Codec(i, {32: "f32", 64: "f64"}[int(f)], int(ib), mask)
        bits = c.compressed_bits(s)
        d, nb = len(s), 3136
        assert bits == 4 + 64 * d + 64 + 64 * d + int(np.prod(i)) + int(f) * nb + int(ib) * int(kept) * nb
        assert bits == int(stored)                 # the count added up by hand from the paper's component list
        assert abs(int(u) * int(np.prod(s)) / bits - float(want)) < 0.01


def test_entry_points_reject_bad_arguments_before_any_launch():
    lib = api.load_library()
    c = Codec((8, 8), "f32", "i8")
    h = c._h
    shape = (ctypes.c_int64 * 2)(16, 16)
    bad_shape = (ctypes.c_int64 * 2)(16, -1)
    p = ctypes.c_void_p(256)   # never dereferenced: every call below fails validation first
    need = ctypes.c_size_t()
    assert lib.pbz_compress(h, None, 1, shape, p, p, None) == -1
    assert lib.pbz_compress(h, p, 9, shape, p, p, None) == -4
    assert lib.pbz_compress(h, p, 1, bad_shape, p, p, None) == -7
    assert lib.pbz_decompress(h, p, None, shape, p, 1, None) == -1
    assert lib.pbz_decompress(h, p, p, shape, p, -1, None) == -4
    assert lib.pbz_negate(h, 0, p, p, None) == -7
    assert lib.pbz_negate(h, 4, None, p, None) == -1
    assert lib.pbz_mul_scalar(h, 4, p, p, float("nan"), p, p, None) == -9
    assert lib.pbz_mul_scalar(h, 4, p, p, float("inf"), p, p, None) == -9
    assert lib.pbz_add(h, 4, p, p, p, None, p, p, None) == -1
    assert lib.pbz_dot(h, 4, p, p, p, p, p, p, 16, None) == -8          # workspace too small
    assert lib.pbz_dot(h, 4, p, p, p, p, p, ctypes.c_void_p(257), 1 << 20, None) == -8   # misaligned
    assert lib.pbz_norm2(h, 4, p, p, None, p, 1 << 20, None) == -1
    assert lib.pbz_dot(h, -3, p, p, p, p, p, p, 1 << 20, None) == -7
    mask = np.ones((8, 8), dtype=bool)
    mask[0, 0] = False
    nodc = Codec((8, 8), "f32", "i8", mask)
    for fn in (lib.pbz_mean, lib.pbz_variance):
        assert fn(nodc._h, 4, p, p, p, p, 1 << 20, None) == -6
    assert lib.pbz_covariance(nodc._h, 4, p, p, p, p, p, p, 1 << 20, None) == -6
    assert lib.pbz_add_scalar(nodc._h, 4, p, p, 1.0, p, p, None) == -6
    assert lib.pbz_ssim(nodc._h, 4, p, p, p, p, 0.0, 0.0, 1.0, 1.0, 1.0, p, p, 1 << 20, None) == -6
    for fn in (lib.pbz_blockwise_mean, lib.pbz_blockwise_variance, lib.pbz_blockwise_std):
        assert fn(nodc._h, 4, p, p, p, None) == -6
        assert fn(h, 4, p, None, p, None) == -1
    assert lib.pbz_blockwise_covariance(h, 4, p, p, None, p, p, None) == -1
    assert lib.pbz_segmented(h, 9, 2, 4, p, p, p, p, p, p, 1 << 20, None) == -4
    assert lib.pbz_segmented(h, 0, 2, 4, p, p, None, p, p, p, 1 << 20, None) == -1      # dot needs both operands
    assert lib.pbz_segmented(h, 1, 0, 4, p, p, None, None, p, p, 1 << 20, None) == -7
    assert lib.pbz_segmented(nodc._h, 3, 2, 4, p, p, None, None, p, p, 1 << 20, None) == -6
    # the variant on the library's fixed scratch array: the same checks, and its own capacity limits
    assert lib.pbz_segmented_static(h, 9, 2, 4, p, p, p, p, p, None) == -4
    assert lib.pbz_segmented_static(h, 0, 2, 4, p, p, None, p, p, None) == -1
    assert lib.pbz_segmented_static(h, 1, 0, 4, p, p, None, None, p, None) == -7
    assert lib.pbz_segmented_static(h, 1, 2, 0, p, p, None, None, p, None) == -7
    assert lib.pbz_segmented_static(nodc._h, 3, 2, 4, p, p, None, None, p, None) == -6
    assert lib.pbz_segmented_static(h, 1, 4097, 4, p, p, None, None, p, None) == -13
    assert lib.pbz_segmented_static(h, 1, 2, (1 << 40) // 64 // 2 + 1, p, p, None, None, p, None) == -13
    assert lib.pbz_stream_copy(None, p, 64, None) == -1
    assert lib.pbz_stream_copy(p, p, 0, None) == -7
    assert lib.pbz_stream_copy(p, ctypes.c_void_p(264), 64, None) == -8
    assert lib.pbz_add_scalar(h, 4, p, p, float("nan"), p, p, None) == -9
    assert lib.pbz_difference_norm2(h, 4, p, p, p, None, p, p, 1 << 20, None) == -1
    assert lib.pbz_approximate_wasserstein_workspace(h, 1000, ctypes.byref(need)) == 0 and need.value >= 32 * 1000
    assert lib.pbz_approximate_wasserstein_workspace(h, 1 << 31, ctypes.byref(need)) == -7
    assert lib.pbz_approximate_wasserstein(h, 4, p, p, p, p, 0.5, p, p, 1 << 20, None) == -9
    assert lib.pbz_approximate_wasserstein(h, 4, p, p, p, p, float("nan"), p, p, 1 << 20, None) == -9
    assert lib.pbz_approximate_wasserstein(h, 4, p, p, p, p, 2.0, p, p, 64, None) == -8
    assert lib.pbz_approximate_wasserstein(h, 4, p, p, None, p, 2.0, p, p, 1 << 20, None) == -1
    assert lib.pbz_approximate_wasserstein(nodc._h, 4, p, p, p, p, 2.0, p, p, 1 << 20, None) == -6
    assert lib.pbz_pair_statistics(nodc._h, 4, p, p, p, p, p, p, 1 << 20, None) == -6
    assert lib.pbz_pair_statistics(h, 4, p, p, p, None, p, p, 1 << 20, None) == -1
    assert lib.pbz_pair_statistics(h, 4, p, p, p, p, p, p, 64, None) == -8
    assert lib.pbz_statistics(nodc._h, 4, p, p, p, p, 1 << 20, None) == -6
    assert lib.pbz_statistics(h, 4, p, p, p, p, 64, None) == -8
    assert lib.pbz_compress_statistics_workspace(h, shape, 1, ctypes.byref(need)) == 0
    assert need.value == c.layout((16, 16)).workspace_bytes + 2 * 32      # two block rows, one wave each, four FP64 values per wave
    assert lib.pbz_compress_statistics_workspace(h, bad_shape, 1, ctypes.byref(need)) == -7
    assert lib.pbz_compress_statistics(h, p, 1, shape, p, p, 0, None, p, 1 << 20, None) == -1
    assert lib.pbz_compress_statistics(nodc._h, p, 1, shape, p, p, 0, p, p, 1 << 20, None) == -6
    assert lib.pbz_compress_statistics(h, p, 1, shape, p, p, 1, p, p, 64, None) == -8
    assert lib.pbz_compress_statistics(h, p, 1, shape, p, p, 0, p, p, c.layout((16, 16)).workspace_bytes, None) == -8
    assert lib.pbz_ssim(h, 4, p, p, p, p, float("inf"), 0.0, 1.0, 1.0, 1.0, p, p, 1 << 20, None) == -9
    assert lib.pbz_ssim(h, 4, p, p, p, p, 0.0, 0.0, 1.0, 1.0, 1.0, p, p, 64, None) == -8


def test_wasserstein_workspace_never_shrinks_with_more_blocks():
    """A workspace for the largest array serves every smaller one: around each size at which the sort's plan changes, and between."""
    codec = Codec((8, 8), "f32", "i8")
    need = ctypes.c_size_t()

    def bytes_for(n):
        assert api.load_library().pbz_approximate_wasserstein_workspace(codec._h, n, ctypes.byref(need)) == 0
        return need.value

    edges = [4096, 8192, 1 << 22] + [2048 << k for k in range(12)] + [8192 * k for k in (2, 3, 100, 255, 256, 257)]
    sizes = sorted({max(1, e + d) for e in edges for d in (-2, -1, 0, 1, 2)} | set(range(1, 30000, 7)) | {int(1.03 ** k) for k in range(720)})
    needs = [bytes_for(n) for n in sizes]
    for n, a, b in zip(sizes, needs, needs[1:]):
        assert a <= b, (n, a, b)


def test_transform_switch():
    lib = api.load_library()
    c = Codec((8, 8), "f32", "i8", transform="haar")
    assert c.kernel_name("compress", (64, 64), "f32") == "lane_f32_8x8_i8_haar"
    assert Codec((8, 8), "f32", "i8").kernel_name("compress", (64, 64), "f32") == "lane_f32_8x8_i8"
    assert lib.pbz_codec_set_transform(c._h, 0) == 0        # nothing compressed yet: may still change
    assert c.kernel_name("compress", (64, 64), "f32") == "lane_f32_8x8_i8"
    assert lib.pbz_codec_set_transform(c._h, 7) == -4
    assert lib.pbz_codec_set_transform(None, 1) == -1
    with pytest.raises(KeyError):
        Codec((8, 8), "f32", "i8", transform="walsh")


def test_kernel_name_and_path_switch():
    c = Codec((8, 8), "f32", "i8")
    assert c.kernel_name("compress", (64, 64), "f32") is not None
    assert c.kernel_name("nonsense", (64, 64), "f32") is None
    c.set_kernel_path(api.PBZ_PATH_GENERIC)
    assert c.kernel_name("compress", (64, 64), "f32") == "generic"
    assert c.kernel_name("decompress", (64, 64), "f32") == "generic"
    with pytest.raises(PbzError):
        c.set_kernel_path(5)


# which kernel the dispatch picks (decided on the host from shapes and types alone, so testable without a GPU)
DISPATCH = [
    # block, work type, index type, keep, array shape, array type -> kernel
    ((8, 8), "f32", "i8", None, (256, 256), "f32", "lane_f32_8x8_i8"),
    ((8, 8), "f32", "i16", (4, 4), (4096, 4096), "f32", "lane_f32_8x8_i16_box4x4"),
    ((8, 8), "f32", "i16", None, (64, 72), "f32", "lane_f32_8x8_i16"),
    ((8, 8), "f64", "i8", None, (64, 72), "f64", "lane_f64_8x8_i8"),
    ((8, 8), "f64", "i16", None, (61, 75), "f64", "lane_f64_8x8_i16"),
    ((8, 8), "f32", "i8", None, (64, 72), "bf16", "lane_bf16_8x8_i8"),
    ((8, 8), "f16", "i8", None, (64, 72), "f16", "lane_f16_8x8_i8"),
    ((8, 8), "f32", "i8", None, (64, 72), "f64", "lane_f64_w32_8x8_i8"),
    ((8, 8), "bf16", "i16", None, (64, 72), "f64", "lane_f64_w32_8x8_i16"),
    ((4, 4, 4), "f32", "i8", None, (9, 13, 22), "f64", "lane_f64_w32_4x4x4_i8"),
    ((4, 4, 4), "f32", "i16", None, (9, 13, 22), "f64", "lane_f64_w32_4x4x4_i16"),
    ((4, 4, 4), "f64", "i16", None, (512, 512, 512), "f64", "lane_f64_4x4x4_i16"),
    ((4, 4, 4), "f64", "i8", None, (9, 13, 22), "f64", "lane_f64_4x4x4_i8"),
    ((4, 4, 4), "f32", "i8", None, (9, 13, 24), "f32", "lane_f32_4x4x4_i8"),
    ((4, 4, 4), "f32", "i16", None, (9, 13, 24), "f32", "lane_f32_4x4x4_i16"),
    ((1, 16, 16), "f32", "i8", None, (64, 1024, 1024), "f32", "quad16_f32_16x16_i8"),
    ((16, 16), "f32", "i8", None, (33, 50), "f16", "quad16_f16_16x16_i8"),
    ((16, 16), "bf16", "i8", None, (33, 50), "bf16", "quad16_bf16_16x16_i8"),
    ((4, 16, 16), "f32", "i8", None, (250, 1024, 1024), "f32", "quad16_f32_4x16x16_i8"),
    ((4, 16, 16), "f32", "i8", None, (9, 20, 38), "f16", "quad16_f16_4x16x16_i8"),
    ((8, 8, 8), "f32", "i8", (4, 4, 4), (1024, 1024, 512), "bf16", "oct8_bf16_8x8x8_i8_box4x4x4"),
    ((8, 8, 8), "f32", "i8", None, (17, 9, 24), "bf16", "oct8_bf16_8x8x8_i8"),
    ((8, 8, 8), "f32", "i8", (4, 4, 4), (17, 9, 21), "f32", "oct8_f32_8x8x8_i8_box4x4x4"),
    ((8, 8, 8), "f32", "i8", None, (17, 9, 24), "f16", "oct8_f16_8x8x8_i8"),
    ((8, 8, 8), "f32", "i16", None, (17, 9, 21), "f32", "oct8_f32_8x8x8_i16"),
    ((8, 8, 8), "f16", "i16", None, (16, 16, 64), "f32", "oct8_f32_8x8x8_i16"),
    ((8, 8, 8), "f32", "i32", None, (17, 9, 21), "f32", "oct8_f32_8x8x8_i32"),
    ((8, 8, 8), "f64", "i8", None, (16, 16, 16), "f64", "oct8_f64_8x8x8_i8"),
    ((8, 8, 8), "f64", "i16", None, (512, 512, 256), "f64", "oct8_f64_8x8x8_i16"),
    ((8, 8, 8), "f32", "i16", None, (17, 9, 23), "f64", "oct8_f64_8x8x8_i16"),             # FP64 array, FP32 N
    ((8, 8, 8), "f64", "i32", None, (17, 9, 23), "f64", "oct8_f64_8x8x8_i32"),
    ((16, 16), "f32", "i16", None, (64, 64), "f32", "quad16_f32_16x16_i16"),
    ((1, 16, 16), "f16", "i16", None, (5, 33, 50), "f32", "quad16_f32_16x16_i16"),
    ((4, 16, 16), "f32", "i16", None, (9, 20, 38), "f32", "quad16_f32_4x16x16_i16"),
    ((16, 16, 16), "f32", "i16", None, (40, 40, 66), "f32", "cube16_f32_16x16x16_i16"),
    ((16, 16, 16), "bf16", "i16", None, (32, 32, 64), "f32", "cube16_f32_16x16x16_i16"),
    ((16, 16, 16), "f32", "i8", None, (100, 500, 500), "f32", "cube16_f32_16x16x16_i8"),
    ((16, 16), "f32", "i32", None, (64, 64), "f32", "quad16_f32_16x16_i32"),
    ((4, 16, 16), "f16", "i32", None, (9, 20, 38), "f32", "quad16_f32_4x16x16_i32"),
    ((16, 16), "f64", "i8", None, (33, 50), "f64", "quad16_f64_16x16_i8"),
    ((16, 16), "f64", "i16", None, (4096, 4096), "f64", "quad16_f64_16x16_i16"),
    ((1, 16, 16), "f32", "i16", None, (3, 33, 51), "f64", "quad16_f64_16x16_i16"),         # FP64 array, FP32 N
    ((16, 16), "f64", "i32", None, (33, 50), "f64", "quad16_f64_16x16_i32"),
    ((4, 16, 16), "f64", "i16", None, (9, 20, 38), "f64", "quad16_f64_4x16x16_i16"),
    ((16, 16, 16), "f32", "i32", None, (40, 40, 66), "f32", "cube16_f32_16x16x16_i32"),
    ((16, 16, 16), "f64", "i16", None, (40, 40, 66), "f32", "cube16_f32_16x16x16_i16"),    # FP32 array, FP64 N
    ((8, 8, 8), "f64", "i16", None, (16, 16, 16), "f32", "oct8_f32_8x8x8_i16"),
    ((16, 16), "f64", "i32", None, (64, 64), "f32", "quad16_f32_16x16_i32"),
    ((4, 16, 16), "f64", "i16", None, (8, 32, 32), "f32", "quad16_f32_4x16x16_i16"),
    ((16, 16, 16), "f64", "i8", None, (40, 40, 66), "f64", "cube16_f64_16x16x16_i8"),
    ((16, 16, 16), "f64", "i16", None, (512, 512, 512), "f64", "cube16_f64_16x16x16_i16"),
    ((16, 16, 16), "f64", "i32", None, (17, 16, 71), "f64", "cube16_f64_16x16x16_i32"),
    ((4, 16, 16), "f64", "i32", None, (8, 32, 32), "f64", "quad16_f64_4x16x16_i32"),
    ((4, 16, 16), "f64", "i8", None, (8, 32, 32), "f64", "quad16_f64_4x16x16_i8"),
    # FP64 arrays with an FP32 / 16-bit working type and int8: FP32 arithmetic
    ((16, 16), "f32", "i8", None, (64, 64), "f64", "quad16_f64_w32_16x16_i8"),
    ((4, 16, 16), "bf16", "i8", None, (9, 20, 38), "f64", "quad16_f64_w32_4x16x16_i8"),
    ((8, 8, 8), "f32", "i8", None, (16, 16, 16), "f64", "oct8_f64_w32_8x8x8_i8"),
    ((8, 8, 8), "f16", "i8", (4, 4, 4), (17, 9, 21), "f64", "oct8_f64_w32_8x8x8_i8_box4x4x4"),
    ((16, 16, 16), "f32", "i8", None, (40, 40, 66), "f64", "cube16_f64_w32_16x16x16_i8"),
    ((1, 1, 8, 8), "f32", "i8", None, (3, 2, 40, 64), "f32", "lane_f32_8x8_i8"),          # leading unit-block dimensions fold
    ((8, 8), "f32", "i32", None, (64, 64), "f32", "lane_f32_8x8_i32"),
    ((8, 8), "f64", "i32", None, (37, 67), "f64", "lane_f64_8x8_i32"),
    ((4, 4, 4), "bf16", "i32", None, (9, 14, 24), "f32", "lane_f32_4x4x4_i32"),
    ((4, 4, 4), "f64", "i32", None, (512, 512, 512), "f64", "lane_f64_4x4x4_i32"),
    # no specialised kernel: the general ones
    ((2, 16, 16), "f32", "i8", None, (8, 64, 64), "f64", "generic"),
    ((8, 8), "f32", "i32", (4, 4), (64, 64), "f32", "generic"),                            # int32 with a box
    ((8, 8), "f64", "i16", None, (64, 64), "f32", "generic"),                              # FP32 array, FP64 N
    ((16, 16), "f32", "i16", None, (64, 64), "f16", "generic"),                            # 16-bit array, int16
    ((8, 8, 8), "f32", "i8", (2, 2, 2), (16, 16, 16), "f32", "generic"),                   # another mask
    ((8, 8, 8), "f64", "i8", None, (16, 16, 16), "f32", "generic"),                        # FP32 array, FP64 N, int8
    ((8, 8, 8), "f32", "i16", (4, 4, 4), (16, 16, 16), "f32", "generic"),                  # int16 with a box
    ((8, 8, 8), "f32", "i16", None, (16, 16, 16), "bf16", "generic"),                      # int16, 16-bit array
    ((16, 16, 16), "f32", "i16", (8, 8, 8), (32, 32, 64), "f32", "generic"),
    ((2, 8, 8), "f32", "i8", None, (4, 64, 64), "f32", "generic"),
    ((8, 8), "f32", "i8", None, (6, 3), "f32", "generic"),                                 # rows shorter than a 16-byte piece
    ((8, 8, 8), "f32", "i8", None, (17, 9, 23), "bf16", "generic"),                        # odd 16-bit rows
    ((2, 2, 8, 8), "f32", "i8", None, (4, 4, 64, 64), "f32", "generic"),                   # four blocked dimensions
]


@pytest.mark.parametrize("row", DISPATCH, ids=[f"{r[0]}-{r[1]}-{r[2]}-{r[5]}-{r[6]}" for r in DISPATCH])
def test_dispatch_table(row):
    block, ftype, itype, keep, shape, dtype, kernel = row
    mask = None
    if keep is not None:
        mask = np.zeros(block, dtype=bool)
        mask[tuple(slice(0, k) for k in keep)] = True
    c = Codec(block, ftype, itype, mask)
    assert c.kernel_name("compress", shape, dtype) == kernel
    assert c.kernel_name("decompress", shape, dtype) == kernel
    h = Codec(block, ftype, itype, mask, "haar")
    assert h.kernel_name("compress", shape, dtype) == (kernel if kernel == "generic" else kernel + "_haar")


def test_binding_checks_compressed_buffers_before_the_call():
    """The C side trusts the pointers it is given, so the binding compares N, F and the output with the layout of the
    shape it passes: wrong dimensionality, size or dtype never reaches the library."""
    import torch
    c = Codec((8, 8), "f32", "i8")
    x = torch.zeros((16, 16))
    N, F = torch.zeros(4), torch.zeros((4, 64), dtype=torch.int8)
    with pytest.raises(ValueError, match="dimensionality"):
        c.decompress(N, F, (16,))
    with pytest.raises(ValueError, match="size"):
        c.decompress(N[:3], F, (16, 16))
    with pytest.raises(ValueError, match="size"):
        c.decompress(N, F, (16, 24))
    with pytest.raises(ValueError, match="dtype"):
        c.compress(x, N.double(), F)
    with pytest.raises(ValueError, match="dtype"):
        c.compress(x, N, F.to(torch.int16))
    with pytest.raises(ValueError, match="array's size"):
        c.decompress(N, F, (16, 16), out=torch.zeros((16, 8)))


def test_every_specialised_kernel_has_a_gpu_parity_row():
    """The dispatch is walked over block shapes, array / working / index types, masks and both transforms (on the host:
    no kernel runs); every specialised kernel it can name must be named by a row of the GPU parity tables, so that a
    kernel cannot be added without a test that runs it against the oracle."""
    import itertools

    import test_gpu_parity as gpu_rows
    covered = {row[6] for row in gpu_rows.FAST_RAGGED} | {row[6] for row in gpu_rows.HAAR}
    boxes = {(8, 8): [(4, 4)], (8, 8, 8): [(4, 4, 4)]}
    reachable = {}
    for block in [(8, 8), (16, 16), (4, 4, 4), (8, 8, 8), (4, 16, 16), (16, 16, 16)]:
        shape = tuple(2 * b for b in block[:-1]) + (6 * block[-1],)
        for dtype, ftype, itype, keep, transform in itertools.product(
                ("f32", "f64", "f16", "bf16"), ("f32", "f64", "f16", "bf16"), ("i8", "i16", "i32"),
                [None] + boxes.get(block, []), ("dct", "haar")):
            mask = None
            if keep is not None:
                mask = np.zeros(block, dtype=bool)
                mask[tuple(slice(0, k) for k in keep)] = True
            c = Codec(block, ftype, itype, mask, transform)
            name = c.kernel_name("compress", shape, dtype)
            assert c.kernel_name("decompress", shape, dtype) == name
            if name != "generic":
                reachable.setdefault(name, (block, dtype, ftype, itype, keep))
    assert len(reachable) > 100
    missing = {name: how for name, how in reachable.items() if name not in covered}
    assert not missing, f"specialised kernels without a GPU parity row: {missing}"


def test_every_general_kernel_has_a_gpu_parity_row():
    """The same for the kernels that pbz_kernel_name calls "generic": every one of the families' kernels under any mask that the
    dispatch can reach is run by a row of test_gpu_any_mask, and every block shape with kernels of its own by test_gpu_block_shapes
    (their types are run-time arguments; FP32 and FP64 work and both transforms are separate kernels)."""
    import itertools

    import test_gpu_any_mask as masks
    import test_gpu_block_shapes as shapes
    from parity import MASKED, SHAPE, route, take_wherever_possible
    def kernel(block, dtype, ftype, bits):       # whether N is FP64 is the kernel's own in one family, whether the work is in the others
        lane = block in ((8, 8), (4, 4, 4))
        return block, dtype, ftype == "f64" or (bits > 8 and not lane), bits

    run = {kernel(block, dtype, ftype, int(bits)) for block, dtype, ftype, bits in masks.ROWS
           if masks.kind(block, dtype, ftype, int(bits)) == MASKED}
    reachable = set()
    blocks = list(masks.SHAPES) + [(4, 8), (16, 8), (8, 16), (32, 32), (2, 8, 8), (4, 8, 8), (8, 4, 4), (4, 4, 8), (16,), (4, 4, 4, 4)]
    for block, dtype, ftype, bits in itertools.product(blocks, api.FTYPES, api.FTYPES, (8, 16, 32)):
        mask = np.ones(block, dtype=bool)
        mask.reshape(-1)[-1] = False
        c = Codec(block, ftype, bits, mask)
        take_wherever_possible(c, MASKED)
        for shape in (tuple(8 * b for b in block), tuple(3 * b + 1 for b in block[:-1]) + (8 * block[-1] + 4,)):
            if MASKED in (route(c, "compress", shape, dtype), route(c, "decompress", shape, dtype)):
                reachable.add(kernel(block, dtype, ftype, bits))
    assert len(reachable) >= 43
    assert reachable <= run, f"kernels for any mask without a GPU parity row: {sorted(reachable - run)}"
    works = {ftype == "f64" or bits > 8 for _, ftype, bits in shapes.TYPES}
    assert works == {False, True}
    for extents in itertools.chain.from_iterable(itertools.product((1, 2, 4, 8, 16, 32, 64), repeat=nd) for nd in (1, 2, 3, 4)):
        if extents[0] == 1 or np.prod(extents) > 4096:
            continue                                       # leading extents of one fold away
        for ftype in ("f32", "f64"):
            c = Codec(extents, ftype, "i8", None)
            take_wherever_possible(c, SHAPE)
            got = route(c, "compress", tuple(4 * e for e in extents), "bf16" if ftype == "f32" else "f16")
            if got == SHAPE:
                assert extents in shapes.SHAPES, extents


def test_kernels_for_any_mask_and_per_block_shape_take_their_rows():
    """What the GPU rows force is what they get: also without a GPU, so that a shape that drops out of a list is seen here."""
    import test_gpu_any_mask as masks
    import test_gpu_block_shapes as shapes
    from parity import LINES, MASKED, SHAPE, TILED, route, take_wherever_possible
    for block, dtype, ftype, bits in masks.ROWS:
        mask = np.ones(block, dtype=bool)
        mask.reshape(-1)[-1] = False
        c = Codec(block, ftype, int(bits), mask)
        want = masks.kind(block, dtype, ftype, int(bits))
        take_wherever_possible(c, want)
        for shape in masks.SHAPES[block]:
            assert route(c, "compress", shape, dtype) == route(c, "decompress", shape, dtype) == want, (block, dtype, bits, shape)
            assert route(c, "compress", shape, dtype, 264) == TILED
    for block in shapes.SHAPES:
        for dtype, ftype, bits in shapes.TYPES:
            mask = np.ones(block, dtype=bool)
            mask.reshape(-1)[-1] = False
            c = Codec(block, ftype, bits, mask)
            take_wherever_possible(c, SHAPE)
            want = SHAPE if shapes.taken(block, ftype, bits) else LINES
            shape = tuple(3 * b + 1 for b in block)
            assert route(c, "compress", shape, dtype) == route(c, "decompress", shape, dtype) == want, (block, dtype, ftype, bits)


def test_host_only_calls_do_without_the_native_binding():
    """A library without _binding.so beside it still loads; the first device call says what is missing."""
    import subprocess
    import sys
    code = """
import sys
sys.modules["paper_2406_11209_amd._binding"] = None
import torch
from paper_2406_11209_amd import api
api.load_library(api.LIB_PATH)
codec = api.Codec((8, 8), "f32", "i8")
assert codec.layout((16, 24)).n_blocks == 6 and codec.kernel_name("compress", (16, 24), "f32")
try:
    codec.negate(torch.zeros(4, 64, dtype=torch.int8))
except RuntimeError as e:
    assert "_binding.so is missing" in str(e)
else:
    raise AssertionError("no error")
"""
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT, timeout=300)


def test_a_reduction_keeps_its_workspace_while_others_come_and_go(monkeypatch):
    """The table of workspaces' addresses is cleared when it is large, by any thread: the call that has just made its entry goes on."""
    torch = pytest.importorskip("torch")
    codec = Codec((8, 8), "f32", "i8")
    space = torch.zeros(64, dtype=torch.uint8)
    monkeypatch.setattr(codec, "workspace", lambda device: space)
    monkeypatch.setattr(api, "_stream", lambda: 7)
    calls = []

    def entry(at, handle, spaces, *rest):
        codec._spaces.clear()                          # as another thread might, between any two steps
        calls.append(spaces.get((-1, 7)))
        return None if calls[-1] is None else 0

    codec._spaces.update({(0, s): (1, 1) for s in range(300)})
    monkeypatch.setattr(api, "_binding", types.SimpleNamespace(reduce=entry))
    for _ in range(2):
        codec.norm2(torch.zeros(1), torch.zeros(1, 64, dtype=torch.int8), torch.zeros(1, dtype=torch.float64))
    assert calls == [None, (space.data_ptr(), 64)] * 2


def test_native_calls_refuse_what_the_device_could_not_read():
    """Tensors in host memory, no tensors at all and wrong counts end in Python errors before an entry point is called."""
    torch = pytest.importorskip("torch")
    codec = Codec((8, 8), "f32", "i8")
    N, F, x = torch.zeros(4), torch.zeros(4, 64, dtype=torch.int8), torch.zeros(16, 16)
    one = torch.zeros(1, dtype=torch.float64)
    for call in (lambda: codec.negate(F, F), lambda: codec.add(N, F, N, F, N, F), lambda: codec.mul_scalar(N, F, 2.0, N, F),
                 lambda: codec.mean(N, F, one), lambda: codec.dot(N, F, N, F, one), lambda: codec.compress(x, N, F),
                 lambda: codec.decompress(N, F, (16, 16), out=x), lambda: codec.blockwise_mean(N, F, torch.zeros(4, dtype=torch.float64)),
                 lambda: codec.segmented("variance", 2, 2, N, F, out=torch.zeros(2, dtype=torch.float64))):
        with pytest.raises(ValueError, match="contiguous device tensors"):
            call()
    with pytest.raises(AttributeError):
        codec.negate(None, F)
    from paper_2406_11209_amd import _binding
    for name in ("blocks", "reduce", "scalar", "compress", "decompress", "segmented"):
        with pytest.raises(TypeError):
            getattr(_binding, name)(1, 2)
