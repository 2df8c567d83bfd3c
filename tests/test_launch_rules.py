"""Launch rules of the matrix-core kernels, on the CPU, over formats, modes, numbers
of points and samples: where a tile's points are split over a block's waves, the
block has few tiles to take one after another, also in calls of more points than
a launch takes; a block of LLRs, whose slow samples one wave ends, has one."""
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_2011_13695_amd" / "libmdgmi.so"
CUS = 256                       # of the device, or where there is none
ML = (3, 4)
WIDE = (-1, 1, 3)               # shapes of two sample columns per wave
SMALL = 8                       # the 4x4 shape


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not shutil.which("hipcc") or not LIB.exists():
        pytest.skip("hipcc or the built library not available")
    exe = tmp_path_factory.mktemp("launch") / "driver"
    subprocess.run(["hipcc", "-std=c++17", "-O1", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    str(ROOT / "tests" / "sanitize" / "launch_driver.cpp"), "-x", "none", str(LIB),
                    f"-Wl,-rpath,{LIB.parent}", "-o", str(exe)], check=True)

    def ask(forms):
        r = subprocess.run([str(exe)], input="\n".join(" ".join(map(str, f)) for f in forms), capture_output=True,
                           text=True, check=True, timeout=300)
        return [tuple(map(int, line.split())) for line in r.stdout.splitlines()]
    return ask


def forms():
    points = [1, 2, 3, 7, 16, 20, 30, 31, 32, 33, 40, 41, 64, 65, 100, 129, 256, 300]
    samples = [1, 31, 32, 33, 100, 300, 700, 1500, 2049, 5000, 8192, 8193, 12000, 16384, 20000, 100000, 1000003]
    for dim, M in [(1, 1024), (2, 32), (2, 1024), (4, 512), (4, 4096), (8, 32), (8, 512), (8, 2048), (8, 4096)]:
        for split in (0, 1):
            for mode in range(5):
                for n_snr in ([1] if mode in (1, 3) else points):
                    for n in samples:
                        yield dim, M, split, mode, n_snr, n


def per_launch(n_snr):
    launches = -(-n_snr // 32)
    return -(-n_snr // launches)


def test_split_points(rules):
    fs = list(forms())
    split = 0
    for f, (blocks, threads, variant, sp) in zip(fs, rules(fs)):
        if not sp:
            continue
        split += 1
        dim, M, s, mode, n_snr, n = f
        tiles = -(-n // 32)
        assert s == 0 and mode not in ML and M >= 512, f
        assert tiles * per_launch(n_snr) <= 2 * CUS and -(-tiles // blocks) <= (1 if mode == 1 else 3), (f, blocks)
        # both of a CU's blocks fit beside each other: sixteen waves of 128 registers
        assert blocks * per_launch(n_snr) <= CUS * max(16 // (M // 256), 1) or blocks == 1, (f, blocks)
    assert split > 1000


def test_part_blocks_fit(rules):
    """Blocks without work for all their waves fit beside each other: of the bf16
    split's two-column shape (256 registers) one of eight waves per CU, of the
    one-column shapes of eight waves two for GMI of up to four dimensions (122), else
    one. With work for every wave, and LDS for their images, sixteen waves per CU are
    kept in launches of any mode."""
    fs = list(forms())
    seen = 0
    for f, (blocks, threads, variant, sp) in zip(fs, rules(fs)):
        if variant == SMALL or sp:
            continue
        dim, M, s, mode, n_snr, n = f
        waves, points = threads // 64, per_launch(n_snr)
        fit = 8 if variant in WIDE else 16 if waves == 16 or (mode == 0 and dim <= 4) else 12
        tiles = -(-n // (32 * (2 if variant in WIDE else 1)))
        full = -(-tiles // waves)   # blocks whose waves all have a tile
        beside = CUS * max(1, fit // waves) // points
        assert blocks <= max(1, beside, full), (f, blocks, threads)
        image_kib = -(-M // 32) * ((6 * dim + 21) // 16 if s else 1 + (dim == 8))
        if image_kib <= 64 or image_kib > 128:   # two blocks' images fit, or it is read from L2
            assert blocks >= min(full, CUS * (16 // waves) // points), (f, blocks, threads)
        seen += 1
    assert seen > 1000
