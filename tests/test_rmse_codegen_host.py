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


def _loads_together(body):
    """Most 16-byte row loads issued with no multiply-add between them."""
    best = now = 0
    for line in body:
        if line.startswith("global_load_dwordx4"):
            now += 1
            best = max(best, now)
        elif line.startswith(("v_fma_f32", "v_fmac_f32")):
            now = 0
    return best


def test_row_loads_are_issued_together(kernels):
    """A wave step's rows (u and v, one slice per lane at k = 16, else four)
    are all requested before the first product, where the kernel fences them;
    the compiler sinks them to their uses otherwise."""
    checked = 0
    for name, (_, body) in kernels.items():
        if name[0] not in ("k_rmse_partial", "k_rmse_stratum"):
            continue
        kp, few = name[1], name[3]
        partial = name[0] == "k_rmse_partial"
        if not ((partial and kp <= 64) or kp == 32 or (kp >= 64 and few)):
            continue
        steps = 8 if kp == 16 else 2 if kp == 32 or few else 1
        want = steps * 2 * (1 if kp == 16 else 4)
        assert _loads_together(body) >= want, (name, _loads_together(body), want)
        checked += 1
    assert checked == 17
