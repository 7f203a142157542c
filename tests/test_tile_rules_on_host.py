"""What the kernels per block shape decide before a launch (csrc/pbz_brick.h), compiled for the host: the values that a lane holds, at the shapes,
types and masks whose best choice is not their neighbours', on both sides of the sizes where it changes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MI = 1 << 20
FP32, FP64, COMPRESS, DECOMPRESS, FULL, MASK = 0, 1, 1, 0, 0, 1

# work, direction, bytes of an array's element and of an index, mask, block, [(elements, values)]
TILES = [(FP32, COMPRESS, 2, 1, FULL, (1, 2, 8, 8), [(MI, 16), (16 * MI, 16)]),           # single rows: 32 makes runs of two indices, 1.2-1.45 of the time
         (FP32, COMPRESS, 4, 1, FULL, (1, 1, 16, 8), [(MI, 16), (16 * MI, 16)]),
         (FP32, COMPRESS, 4, 1, FULL, (1, 1, 16, 16), [(16 * MI, 16)]),
         (FP32, COMPRESS, 4, 1, MASK, (1, 2, 8, 8), [(4 * MI, 16), (4 * MI + 1, 64)]),
         (FP32, COMPRESS, 8, 1, MASK, (1, 2, 8, 8), [(8 * MI, 16), (8 * MI + 1, 64)]),
         (FP32, COMPRESS, 4, 1, MASK, (1, 1, 16, 8), [(4 * MI, 16), (4 * MI + 1, 32)]),
         (FP32, COMPRESS, 4, 1, FULL, (4, 4, 4, 4), [(16 * MI, 16), (16 * MI + 1, 64)]),
         (FP32, COMPRESS, 4, 1, MASK, (4, 4, 4, 4), [(4 * MI, 16), (16 * MI, 32)]),
         (FP32, COMPRESS, 4, 1, FULL, (1, 4, 8, 8), [(4 * MI, 32), (4 * MI + 1, 64)]),
         (FP32, COMPRESS, 8, 1, FULL, (1, 4, 8, 8), [(8 * MI, 32), (8 * MI + 1, 64)]),
         (FP32, COMPRESS, 2, 1, MASK, (1, 4, 8, 8), [(2 * MI, 32), (2 * MI + 1, 64)]),
         (FP64, COMPRESS, 4, 2, MASK, (1, 4, 8, 8), [(2 * MI, 32), (2 * MI + 1, 64)]),
         (FP64, COMPRESS, 8, 2, MASK, (1, 4, 4, 8), [(MI, 16), (MI + 1, 32)]),
         (FP64, COMPRESS, 8, 2, FULL, (1, 4, 4, 8), [(4 * MI, 16), (4 * MI + 1, 32)]),
         (FP64, COMPRESS, 2, 2, MASK, (1, 1, 8, 16), [(16 * MI, 16), (16 * MI + 1, 32)]),
         (FP64, COMPRESS, 8, 1, FULL, (1, 1, 8, 4), [(MI, 8), (2 * MI, 32)]),
         (FP32, DECOMPRESS, 2, 1, FULL, (4, 4, 4, 4), [(16 * MI, 64)]),
         (FP32, DECOMPRESS, 4, 1, FULL, (4, 4, 4, 4), [(16 * MI, 32)]),
         (FP32, DECOMPRESS, 4, 1, MASK, (1, 2, 8, 8), [(4 * MI, 16), (4 * MI + 1, 64)]),
         (FP32, DECOMPRESS, 4, 1, MASK, (1, 4, 8, 8), [(4 * MI, 32), (4 * MI + 1, 64)]),
         (FP64, DECOMPRESS, 8, 1, MASK, (1, 1, 4, 4), [(32 * MI, 16), (32 * MI + 1, 32)])]


@pytest.fixture(scope="module")
def decide(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path_factory.mktemp("host") / "brick_rules")
    subprocess.run([hipcc, "--cuda-host-only", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2406_11209_amd", "csrc"),
                    "-I" + os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "host", "brick_rules.hip"), "-o", exe], check=True, capture_output=True)

    def ask(lines):
        out = subprocess.run([exe], input="".join(line + "\n" for line in lines), check=True, capture_output=True, text=True).stdout.split()
        assert len(out) == len(lines)
        return [int(v) for v in out]
    return ask


def test_values_of_a_lane(decide):
    lines, want = [], []
    for work, direction, array, index, mask, block, sizes in TILES:
        for elements, values in sizes:
            lines.append(f"tiles {work} {direction} {array} {index} {mask} {elements} " + " ".join(map(str, block)))
            want.append(values)
    got = decide(lines)
    assert [(line, v) for line, v in zip(lines, got)] == [(line, v) for line, v in zip(lines, want)]
