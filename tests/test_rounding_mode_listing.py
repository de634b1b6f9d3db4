"""The decoders convert with fp32 rounding toward zero (decode_core.h); nothing else there may round in fp32.  Checked on the
compiler's listing of the averages: an integer quotient is found by an fp32 reciprocal and products of it (CPU only)."""
import os
import re
import subprocess

import pytest

from paper_2204_08211_amd import build as hip_build


@pytest.mark.parametrize("source", ["k_decode.hip", "k_decode_wide.hip"])
def test_no_fp32_reciprocal_in_the_averages(source, tmp_path):
    out = tmp_path / "listing.s"
    subprocess.run([hip_build.HIPCC, "-x", "hip", "-S", "--cuda-device-only", os.path.join(hip_build.CSRC, source), "-o", str(out)] +
                   hip_build.FLAGS, check=True, stderr=subprocess.DEVNULL)
    kernel, found = None, {}
    for line in out.read_text().splitlines():
        m = re.match(r"(_ZN\w+):", line)
        if m:
            kernel = m.group(1)
            found.setdefault(kernel, [])
        elif kernel and re.match(r"\s+v_rcp_(iflag_)?f32", line):
            found[kernel].append(line.strip())
    averages = {k: v for k, v in found.items() if "k_aggregate" in k}
    assert len(averages) >= 3
    assert not any(averages.values()), averages
