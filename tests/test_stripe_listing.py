"""Listing of the stripe kernels, built here for gfx950: no GPU."""
import os
import re
import subprocess

from paper_2510_09103_amd.build import CSRC, FLAGS


def test_stripe_kernels_keep_their_values_in_registers(tmp_path):
    """A workgroup of 1024 threads has 128 registers per lane.  At rank class 128 both products of the joint kernel fill them:
    values that are uniform or follow from the thread's number went to scratch (60 bytes per lane, 5 % of the launch's memory
    traffic) unless kept out of them.  Allowed: the 12 bytes of the loop of the thin products, rounded up to whole vectors."""
    out = tmp_path / "k.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *FLAGS, "-S", "--cuda-device-only",
                    os.path.join(CSRC, "k_proj_mfma.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    scratch = {name: int(size) for name, size in
               re.findall(r"^\s*\.amdhsa_kernel (\w*stripe_kernel\w*)\n\s*\.amdhsa_group_segment_fixed_size \d+\n"
                          r"\s*\.amdhsa_private_segment_fixed_size (\d+)", out.read_text(), re.M)}
    assert len(scratch) == 3
    assert all(size <= 16 for size in scratch.values()), scratch
