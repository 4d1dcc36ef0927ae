"""Hand-written selects wait for their masks (host: device assembly of the march).

A select that reads its mask from a pair of scalar registers is due two wait
states after a vector instruction has written the pair.  The compiler counts
them for its own instructions, not for hand-written statements, and may put a
vector write of the mask (a compare, or the reload of a spilled scalar) right in
front of one.  So every hand-written statement with selects opens with the wait.
"""
import os
import re
import subprocess

import pytest

from paper_1601_02012_amd import build as B

KERNELS = """
template __global__ void march_uniform_kernel<{r}, false, uint32_t, kTidal, false, true>(
    const {r}* __restrict__, TraceArgs);
template __global__ void march_uniform_kernel<{r}, true, uint32_t, kMethodA, false, false>(
    const {r}* __restrict__, TraceArgs);
}}
}}
"""


@pytest.mark.parametrize("real", ["float", "double"])
def test_selects_open_with_their_wait(tmp_path, real):
    with open(os.path.join(B.CSRC, "rr_march_uniform.hip")) as f:
        text = f.read()
    text = text[:text.index("__global__ void queue_reset_kernel")] + KERNELS.format(r=real)
    src = tmp_path / "march.hip"
    src.write_text(text)
    out = tmp_path / "march.s"
    flags = [x for x in B.COMMON if x not in ("-fPIC", "-Wall", "-Wno-unused-function")]
    r = subprocess.run([B.HIPCC, *flags, "-I" + B.CSRC, "--cuda-device-only", "-S", "-x", "hip",
                        str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    statements = re.findall(r"#ASMSTART\n(.*?);;#ASMEND", out.read_text(), re.S)
    selects = [s for s in statements if "v_cndmask" in s]
    assert selects
    for s in selects:
        first = s.split("\n")[0].split(";")[0].split()
        assert first[0] == "s_nop" and int(first[1]) >= 1, s
