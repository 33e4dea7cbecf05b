"""Arguments of the GroupNorm kernels in the generated gfx950 code: those of one tensor carry nothing of the form that reads two (a call of few
pixels takes 5 % longer with another line of arguments to fetch; no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2402_19481_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs the compiler")
def test_kernels_of_one_tensor_take_no_second_one(tmp_path):
    out = tmp_path / "gn.s"
    subprocess.run(["hipcc", *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "groupnorm.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    sizes = {}
    for block in re.split(r"^\s+\.amdhsa_kernel ", out.read_text(), flags=re.M)[1:]:
        m = re.match(r"\S*?(gn_stats|gn_apply|gn_group_reg_kernel)I(\S*?)Lb([01])EEEv", block)
        if m:
            size = int(re.search(r"\.amdhsa_kernarg_size (\d+)", block).group(1))
            sizes.setdefault(m.group(1), {}).setdefault(m.group(3), set()).add(size)
    assert set(sizes) == {"gn_stats", "gn_apply", "gn_group_reg_kernel"}
    for name, by_pair in sizes.items():
        one, pair = by_pair["0"], by_pair["1"]
        assert len(one) == 1 and len(pair) == 1, (name, by_pair)
        assert min(pair) - max(one) >= 16, (name, by_pair)      # a pointer, a count and a pointer, beside an empty place
