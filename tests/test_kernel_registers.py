"""What the compiler gives the kernels whose launch counts on it, from the assembly of
the library's own sources."""
import os
import re
import subprocess

import pytest

from paper_2607_04489_amd import build


@pytest.mark.parametrize("source,kernel,threads,per_cu", [("join_direct", "k_probe", 256, 4), ("join_smj", "k_smj_merge", 256, 4)])
def test_probes_fit_the_workgroups_of_their_grid(tmp_path, source, kernel, threads, per_cu):
    """These grids have per_cu workgroups a CU, each with an equal share of the rows: with
    more registers than fit (512 a lane on each of its four SIMDs) the last ones run alone."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    asm = tmp_path / "k.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source + ".hip"), "-o", str(asm)],
                   check=True, capture_output=True)
    meta = asm.read_text().split("amdhsa.kernels:")[1]
    seen = 0
    for k in meta.split("\n  - ")[1:]:
        name = re.search(r"\.name: +(\S+)", k)
        if not name or kernel not in name[1]:
            continue
        seen += 1
        vgprs = int(re.search(r"\.vgpr_count: +(\d+)", k)[1])
        waves = per_cu * threads // 64 // 4
        assert -(-vgprs // 8) * 8 * waves <= 512, (vgprs, k)
        assert int(re.search(r"\.vgpr_spill_count: +(\d+)", k)[1]) == 0
    assert seen == 8
