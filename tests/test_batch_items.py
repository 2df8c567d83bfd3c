"""Item sizes of a ragged batch's 32 x 32 kind, on the CPU: scheduled onto the CUs
one after another (each to the block that is free first), with an item's time as
measured (tiles of 512 samples, M + 300 points each at 3.2e10 points/s, 8 us more an
item), the plan ends no later than with items of 2^22 pairs, and no later than with
eight items a block."""
import heapq
import random
import shutil
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
LIB = ROOT / "paper_2011_13695_amd" / "libmdgmi.so"
CUS = 256


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not shutil.which("hipcc") or not LIB.exists():
        pytest.skip("hipcc or the built library not available")
    exe = tmp_path_factory.mktemp("batch") / "driver"
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w",
                    str(ROOT / "tests" / "sanitize" / "batch_driver.cpp"), "-x", "none", str(LIB),
                    f"-Wl,-rpath,{LIB.parent}", "-o", str(exe)], check=True)

    def ask(batches):
        text = "\n".join(f"{len(b)} " + " ".join(f"{d} {M} {n}" for d, M, n in b) for b in batches)
        r = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True, timeout=300)
        return [[tuple(map(int, it.split(":"))) for it in line.split()] for line in r.stdout.splitlines()]
    return ask


def span(items):
    free = [0.0] * CUS
    for s, M in items:
        heapq.heappush(free, heapq.heappop(free) + -(-s // 512) * 512 * (M + 300) / 3.2e10 + 8e-6)
    return max(free)


def cut(batch, per):
    return [(min(per(M), n - s), M) for _, M, n in sorted(batch, key=lambda b: -b[1]) for s in range(0, n, per(M))]


def largest(batch):
    return cut(batch, lambda M: max(512, (1 << 22) // M // 512 * 512))


def eight_a_block(batch):
    c = max(400000, min(1 << 22, sum(n * (M + 200) for _, M, n in batch) // (8 * CUS)))
    return cut(batch, lambda M: max(512, c // (M + 200) // 512 * 512))


def test_ends_no_later(plan):
    r = random.Random(7)
    batches = [[(8, 512, 592404)] * 3, [(8, 2048, 50000)] * 8, [(8, 2048, 217357)] * 2, [(8, 1024, 314389)] * 3,
               [(4, 4096, 50000)] * 4, [(4, 1024, 58628)] * 16, [(8, 2048, 100000)], [(8, 512, 1000000)],
               [(8, 512, 1)], [(4, 4096, 512 * 256)], [(4, 4096, 512 * 256 + 1)], [(8, 2048, 10_000_000)] * 16]
    for _ in range(150):
        k = r.choice([1, 1, 2, 3, 8, 16, 40])
        one = (8, r.choice([512, 1024, 2048, 4096]))
        same, n0 = r.random() < 0.5, int(10 ** r.uniform(3, 5.8))
        batches.append([(*(one if same else (8, r.choice([512, 1024, 2048, 4096]))),
                         n0 if same and r.random() < 0.7 else int(10 ** r.uniform(2, 5.5))) for _ in range(k)])
    for b, items in zip(batches, plan(batches)):
        assert sum(s for s, _ in items) == sum(n for _, _, n in b)
        t = span(items)
        assert t <= 1.001 * span(largest(b)) and t <= 1.001 * span(eight_a_block(b)), (len(b), b[:4])
