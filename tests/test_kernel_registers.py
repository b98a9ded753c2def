"""Vector registers that the built kernels spill, from the metadata of the
gfx950 code object in libugks.so (no GPU needed).  A spilled value that a
velocity loop reloads waits for every load issued before it, so a spill there
costs far more than its own bytes."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2412_06546_amd", "libugks.so")
LLVM = "/opt/rocm/llvm/bin"

pytestmark = pytest.mark.skipif(not os.path.exists(os.path.join(LLVM, "llvm-objdump")) or not shutil.which("c++filt"),
                                reason="no ROCm LLVM tools or c++filt")


@pytest.fixture(scope="module")
def spills(tmp_path_factory):
    """Spilled vector registers by demangled kernel name, arguments left out."""
    if not os.path.exists(LIB):
        from paper_2412_06546_amd import build
        build.build(force=False)
    d = str(tmp_path_factory.mktemp("code"))
    shutil.copy(LIB, d)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", "libugks.so"], cwd=d, check=True, capture_output=True)
    code = [f for f in os.listdir(d) if f.endswith("gfx950")]
    assert len(code) == 1
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", code[0]], cwd=d, check=True, capture_output=True,
                           text=True).stdout
    got = re.findall(r"^ +\.name: +(_Z\S+)$.*?\.vgpr_spill_count: (\d+)$", notes, re.M | re.S)
    names = subprocess.run(["c++filt", *(n for n, _ in got)], check=True, capture_output=True,
                           text=True).stdout.split("\n")
    out = {re.sub(r"^void |ugx::|\(.*$", "", n): int(v) for n, (_, v) in zip(names, got)}
    assert len(out) >= 100
    return out


def test_gather_with_prefetch_keeps_its_stencil_in_registers(spills):
    """FP32 and BF16 f: none.  FP64, 2D: 2, or 4 batched (its prefetched stencil
    alone takes 20 registers)."""
    seen = 0
    for name, n in spills.items():
        if not re.match(r"k_sweep(_batch)?_pf<", name):
            continue
        seen += 1
        allowed = 0
        if "<2, double" in name:
            allowed = 4 if "batch" in name else 2
        assert n <= allowed, (name, n)
    assert seen == 24


def test_bricks_spill_nothing(spills):
    got = {k: v for k, v in spills.items() if k.startswith("k_push_brick<")}
    assert len(got) >= 4 and not any(got.values()), got


def test_final_kernels_hold_their_pairs(spills):
    """FP64 sums: up to five pairs a thread nothing is spilled; the last form
    (10,241 velocities and more) spills.  FP32 sums: at most 5 registers of
    scattered BF16 in 2D."""
    got = {k: v for k, v in spills.items() if k.startswith("k_push_final<")}
    assert len(got) == 56
    for name, n in got.items():
        allowed = 5 if name.startswith("k_push_final<2, bf16s, false") else 0
        assert n <= allowed or name.endswith(", 8>"), (name, n)
