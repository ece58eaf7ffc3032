"""Every workgroup of a resident enforcement kernel has to find a place on the chip beside other
kernels, whose waves leave holes: the kernels' registers and LDS, as compiled, leave room for as many
workgroups on a CU as the launch rule counts on, wherever the ones before were put (CPU only)."""
import re
import subprocess

import pytest

from paper_2511_04277_amd import build

REGS, REG_PIECE = 512, 8            # of a SIMD; a workgroup of 512 threads has two waves on each
LDS, LDS_PIECE = 160 * 1024, 1280   # of a CU


def _up(x, piece):
    return -(-x // piece) * piece


def _always_fits(held, size, piece, total):
    """Whether `held` pieces of `size`, put anywhere, leave a hole for one more."""
    return held * size + (held + 1) * (size - piece) < total


def _constant(name):
    text = (build.CSRC / "enforce_kernels.h").read_text()
    return int(re.search(rf"constexpr int {name} = (\d+);", text).group(1))


@pytest.mark.parametrize("source", ["enforce.hip", "batch.hip"])
def test_workgroups_of_a_cu_fit_beside_each_other(source, tmp_path):
    r = subprocess.run([build.HIPCC, *build.COMMON, "-Rpass-analysis=kernel-resource-usage", "--cuda-device-only", "-c",
                        str(build.CSRC / source), "-o", str(tmp_path / "x.o")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    kernels = {}
    for block in r.stderr.split("Function Name: ")[1:]:
        number = {k: int(re.search(rf"{k}[^:]*: (\d+)", block).group(1)) for k in ("VGPRs", "ScratchSize", "LDS Size")}
        kernels[block.split()[0]] = number
    per_cu = _constant("ENF_RES_PER_CU")
    found = 0
    for name, k in kernels.items():
        if "enf_resident" not in name or "init" in name:
            continue
        found += 1
        count = 1 if "wide" in name else per_cu
        regs, lds = _up(k["VGPRs"], REG_PIECE), _up(k["LDS Size"], LDS_PIECE)
        assert k["ScratchSize"] == 0, name  # places in scratch memory are one limit less
        assert 2 * regs <= REGS, name
        for waves in range(2 * count):
            assert _always_fits(waves, regs, REG_PIECE, REGS), (name, waves, regs)
        for groups in range(count):
            assert _always_fits(groups, lds, LDS_PIECE, LDS), (name, groups, lds)
    assert found
    tiles = _constant("ENF_RES_TILES")
    assert tiles * (tiles + 1) // 2 <= per_cu * 256
