"""Order of LDS reads, direct loads and barriers in the generated gfx950 code of the library's own kernels (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_attention_ring_has_a_barrier_between_the_first_reads_and_the_first_refill(tmp_path):
    """attn_pipe_d64 loads its first tiles into an LDS ring, waits, reads tile 0 and then refills tile 0's slot: between
    those reads and the first refill every wave must have passed a barrier."""
    out = tmp_path / "attn.s"
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "attn.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    kernels = re.findall(r"^(\S*attn_pipe_d64\S*):[^\n]*\n(.*?)\bs_endpgm\b", out.read_text(), re.S | re.M)
    assert len(kernels) == 4
    for name, body in kernels:
        order = ""
        for line in body.splitlines():
            op = line.split(";")[0].split()
            if op:
                order += "B" if op[0] == "s_barrier" else "L" if op[0].startswith("global_load_lds") else "r" if op[0].startswith("ds_read") else ""
        assert re.match(r"L+Br+B[^L]*L", order), (name, order)
