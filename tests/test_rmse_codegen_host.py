"""What the compiler makes of the RMSE kernels: registers, scratch and loads
in flight decide their speed, and a rule that suits one width can spill or
serialise another.  Compiles bgmf_rmse.hip for gfx950 (no GPU needed) and
reads the assembly and the resource report.
"""
import os
import re
import subprocess

import pytest

from paper_2304_13724_amd import build as hip_build

SRC = os.path.join(hip_build.PKG, "csrc", "bgmf_rmse.hip")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name with its template arguments: (resources, assembly lines)}"""
    out = str(tmp_path_factory.mktemp("rmse") / "rmse.s")
    flags = [f for f in hip_build.FLAGS if f not in ("-shared",) and not f.startswith("-W")]
    res = subprocess.run(
        [hip_build.HIPCC, *flags, "-I", os.path.join(hip_build.ROOT, "include"),
         "--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage", SRC, "-o", out],
        capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found, cur = {}, None
    for line in res.stderr.splitlines():
        m = re.search(r"remark: .*?(Function Name|VGPRs|ScratchSize \[bytes/lane\]): (\S+)", line)
        if not m:
            continue
        if m.group(1) == "Function Name":
            cur = {}
            found[m.group(2)] = (cur, [])
        else:
            cur[m.group(1).split(" ")[0]] = int(m.group(2))
    with open(out) as f:
        body = None
        for line in f:
            if line.startswith("_Z") and ":" in line and line.split(":")[0] in found:
                body = found[line.split(":")[0]][1]
            elif line.startswith(".Lfunc_end"):
                body = None
            elif body is not None:
                body.append(line.strip())
    named = {}
    for mangled, v in found.items():
        m = re.search(r"(k_rmse_[a-z]+)I([^v]*?)EEv", mangled)
        if m:
            args = re.findall(r"L[ib](\d+)E", m.group(2) + "E")
            named[(m.group(1), *map(int, args))] = v
    assert len(named) >= 32
    return named


def test_no_scratch(kernels):
    for name, (res, _) in kernels.items():
        assert res["ScratchSize"] == 0, (name, res)


def test_heldout_grid_is_resident(kernels):
    """The held-out kernel's fixed grid (1024 workgroups of four waves) is
    four waves on each of 1024 SIMDs: at most 128 registers a lane."""
    coo = [n for n in kernels if n[0] == "k_rmse_coo"]
    assert len(coo) == 8
    for name in coo:
        assert kernels[name][0]["VGPRs"] <= 128, (name, kernels[name][0])
