"""Kernels whose speed rests on several workgroups of eight wavefronts on a compute unit (two on each of its four SIMDs, which hold 512 vector
registers a lane) use no more registers than that leaves them, and no scratch memory."""
import os
import re
import subprocess
import tempfile

import pytest

from paper_2605_27081_amd import build as libbuild

REGISTERS = {4: 64, 3: 80}       # of a wavefront, with so many workgroups (allocated by eights)


@pytest.mark.parametrize("src,kernels", [
    ("loss.hip", {"loss_partial_kernelILi1ELb1E": 4, "loss_partial_kernelILi2ELb1E": 3}),
    ("loss_grad.hip", {"loss_grad_kernelILi1E": 3}),
    ("trace.hip", {"lru_walk_kernel": 3})])
def test_registers_leave_room(src, kernels):
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        flags = [f for f in libbuild.FLAGS if f != "-fPIC"]
        r = subprocess.run([libbuild.HIPCC, *flags, "-S", "--cuda-device-only", os.path.join(libbuild.CSRC, src), "-o", out], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        text = open(out).read()
    found = re.findall(r"\.amdhsa_kernel (\S+)\n(.*?)\.end_amdhsa_kernel", text, re.S)
    for name, workgroups in kernels.items():
        bodies = [(n, b) for n, b in found if name in n]
        assert bodies, name
        for n, body in bodies:
            assert int(re.search(r"\.amdhsa_next_free_vgpr (\d+)", body).group(1)) <= REGISTERS[workgroups], n
            assert int(re.search(r"\.amdhsa_private_segment_fixed_size (\d+)", body).group(1)) == 0, n
