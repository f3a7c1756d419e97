"""Vector registers of the D3Q19 odd step in its flat tiling, the odd step of
cached lattices and of ensembles: a wave of gfx950 takes its share of 512 in
eights, so one register past 72 costs the seventh wave of every SIMD.  The
compiler's own report of the kernel's source is read; nothing runs."""
import os
import re
import subprocess

import pytest

from paper_0707_1581_amd import build

FORMS = [(s, res) for s in (0, 1, 2) for res in ("false", "true")]


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    tmp = tmp_path_factory.mktemp("regs")
    src = tmp / "odd.hip"
    inst = "\n".join(f"template __global__ void lbf::k_step<lbf::D3Q19, {s}, 1, false, 256, {res}>"
                     "(const lbf::LatDesc*, const uint32_t*, uint32_t, uint32_t, lbf::Clock);" for s, res in FORMS)
    src.write_text(f'#include "lbf.h"\n#include "lbf_kernels.h"\n{inst}\n')
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC, *flags, "--cuda-device-only", "-S", "-I", os.path.join(build.ROOT, "include"),
                    "-I", os.path.join(build.HERE, "csrc"), str(src), "-o", str(tmp / "odd.s")], check=True,
                   capture_output=True)
    text = (tmp / "odd.s").read_text()
    out = {}
    for block in text[text.index("amdhsa.kernels:"):].split("  - .agpr_count:")[1:]:
        name = re.search(r"\.name:\s+(\S+)", block).group(1)
        out[name] = int(re.search(r"\.vgpr_count:\s+(\d+)", block).group(1))
    return out


@pytest.mark.parametrize("storage,resident", FORMS)
def test_flat_odd_step_keeps_seven_waves(vgprs, storage, resident):
    key = f"Li{storage}ELi1ELb0ELi256ELb{int(resident == 'true')}E"
    counts = [v for name, v in vgprs.items() if key in name]
    assert len(counts) == 1, sorted(vgprs)
    assert counts[0] <= 72, (storage, resident, counts)
