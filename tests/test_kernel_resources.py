"""What the compiler reports for the engines' kernels: no vector register spilled (a reload is a vector-memory load, and the
wait for it waits for the tile loads in flight), and as many waves per SIMD as each kernel is written for."""
import os
import re
import subprocess

import pytest

from paper_2505_23520_amd import build


@pytest.mark.parametrize("source,waves", [("aa_engine_bf16.hip", 3), ("aa_engine_bf16_pp.hip", 2), ("aa_engine_fp32.hip", 2)])
def test_engines_do_not_spill(tmp_path, source, waves):
    cmd = ["hipcc", *build.FLAGS, *build.EXTRA.get(source, []), "--cuda-device-only", "-S",
           "-Rpass-analysis=kernel-resource-usage", os.path.join(build.CSRC, source), "-o", str(tmp_path / "x.s")]
    report = subprocess.run(cmd, capture_output=True, text=True, check=True).stderr
    names = re.findall(r"Function Name: (\S+)", report)
    spills = [int(x) for x in re.findall(r"VGPRs Spill: (\d+)", report)]
    occupancy = [int(x) for x in re.findall(r"Occupancy \[waves/SIMD\]: (\d+)", report)]
    assert len(names) >= 3 and len(spills) == len(occupancy) == len(names)
    assert not any(spills), dict(zip(names, spills))
    assert min(occupancy) >= waves, dict(zip(names, occupancy))
