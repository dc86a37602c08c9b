"""Every direct-to-LDS copy of the library carries its own M0 write and wait state and takes its address
from vector registers (the assembly block of lds_copy.h), and nothing else in those kernels uses M0."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2605_27081_amd import build as libbuild

SOURCES = [s for s in libbuild.sources() if "copy16_to_lds(" in open(s).read()]


@pytest.mark.parametrize("src", SOURCES, ids=[os.path.basename(s) for s in SOURCES])
def test_copies_stand_alone(src):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        flags = [f for f in libbuild.FLAGS if f != "-fPIC"]
        r = subprocess.run([libbuild.HIPCC, *flags, "-S", "--cuda-device-only", src, "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        text = [l.split(";")[0].strip() for l in open(out)]
    lines = [l for l in text if l and not l.startswith(".") and not l.endswith(":")]
    copies = [i for i, l in enumerate(lines) if l.startswith("global_load_lds")]
    assert copies
    for i in copies:
        assert re.match(r"global_load_lds_dwordx4 v\[\d+:\d+\], off$", lines[i]), lines[i]
        assert lines[i - 1] == "s_nop 0" and re.match(r"s_mov_b32 m0, s\d+$", lines[i - 2]), lines[i - 2:i + 1]
    m0 = [i for i, l in enumerate(lines) if re.search(r"\bm0\b", l)]
    assert all(i + 2 in copies for i in m0)
