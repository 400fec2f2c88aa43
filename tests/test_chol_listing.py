"""Listing of the Cholesky kernel, built here for gfx950: no GPU."""
import os
import re
import subprocess

import pytest

from paper_2510_09103_amd.build import CSRC, FLAGS


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    out = tmp_path_factory.mktemp("chol") / "k.s"
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), *FLAGS, "-S", "--cuda-device-only",
                    os.path.join(CSRC, "k_chol.hip"), "-o", str(out)], check=True, stderr=subprocess.DEVNULL)
    return re.search(r"^_Z\w*chol_inv_kernel\w*:(.*?)^\.Lfunc_end", out.read_text(), re.M | re.S).group(1)


def test_pivots_past_the_rank_are_skipped(kernel):
    """The square roots of a diagonal block are one chain; a matrix of small rank pays for its own pivots only, so that a branch stands
    between any two of them."""
    parts = kernel.split("v_rsq_f64")
    assert len(parts) >= 17
    assert all("s_cbranch" in p for p in parts[1:-1])


def test_rows_of_a_diagonal_block_are_handed_to_other_lanes_in_order(kernel):
    """One wave updates a diagonal block in LDS, reads it back a row per lane and writes its inverse over it: other lanes than the
    writing one read what it wrote, without a barrier of the workgroup between.  The source holds both hand-overs in place, which
    leaves two marks in the listing: the block's stores in front of the first, its reads between them, the inverse's stores behind."""
    parts = kernel.split("; wave barrier")
    assert len(parts) == 3
    lds = [re.findall(r"\b(ds_(?:read|write))\w*", p) for p in parts]
    assert lds[0][-1] == "ds_write"
    assert len(lds[1]) >= 8 and set(lds[1]) == {"ds_read"}          # 16 doubles of a row, at most two to a read
    assert lds[2][0] == "ds_write"
