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


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
@pytest.mark.parametrize("source", [s for s in build.SOURCES if "lds_load" in open(os.path.join(build.CSRC, s)).read()])
def test_every_direct_load_follows_its_own_write_of_m0(source, tmp_path):
    """A direct load takes its LDS address from M0.  Loads written as instructions set M0 themselves, the compiler's are preceded
    by a write of the compiler's: the last write before a load must be of the load's own kind."""
    out = tmp_path / "k.s"
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    inside, last, loads = False, None, 0
    for line in out.read_text().splitlines():
        if line.startswith("_Z"):
            last = None
        if "#ASMSTART" in line or "#ASMEND" in line:
            inside = "#ASMSTART" in line
        op = line.split(";")[0].split()
        if len(op) > 1 and op[0].startswith("s_") and op[1] == "m0,":
            last = inside
        if op and (op[0].startswith("global_load_lds") or (op[0].startswith("buffer_load") and op[-1] == "lds")):
            loads += 1
            assert last is inside, (loads, line)
    assert loads > 0


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
@pytest.mark.parametrize("source,kernels,dwords", [("attn.hip", "attn_wave_d64|attn_pipe_d64", 14), ("tgemm.hip", "tgemm_kernel", 12)])
def test_leading_arguments_come_in_registers(source, kernels, dwords, tmp_path):
    """The kernels whose first requests need only their leading arguments: the code object asks for all of those in scalar registers."""
    out = tmp_path / "k.s"
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True)
    got = re.findall(r"\.amdhsa_kernel (\S*(?:%s)\S*)\n(.*?)\.end_amdhsa_kernel" % kernels, out.read_text(), re.S)
    assert got
    for name, body in got:
        assert int(re.search(r"kernarg_preload_length (\d+)", body)[1]) >= dwords, name
