"""Lanes that exchange values through LDS, checked in the assembly of our own build: a lane that
stores a tag byte and reads the byte back expects another lane's store, so every tag store of the
kernel needs a tag read after it. Without a fence between the two the compiler may put the lane's
own value in the read's place, which no result shows as long as the hardware happens to serve the
lanes of one LDS instruction in order."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2608_19677_amd import build as hip_build

# source, kernel, instances, chunks of 64 entries per wavefront (unrolled: a store and a read each)
KERNELS = [("cr_replay.hip", "k_part_scatter_wide", 2, 16), ("cr_plan.hip", "k_wide_scatter", 1, 16)]


@pytest.mark.parametrize("source,kernel,instances,chunks", KERNELS, ids=[k[1] for k in KERNELS])
def test_every_tag_store_has_its_read(source, kernel, instances, chunks, tmp_path):
    if shutil.which(hip_build.HIPCC) is None:
        pytest.skip("no hipcc")
    out = tmp_path / "k.s"
    flags = [f for f in hip_build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hip_build.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(hip_build.CSRC, source), "-o", str(out)],
                   check=True, capture_output=True, timeout=300)
    bodies = re.findall(r"^_Z\S*%s\S*:.*?^\.Lfunc_end" % kernel, out.read_text(), re.S | re.M)
    assert len(bodies) == instances
    for b in bodies:
        count = {op: len(re.findall(r"\b%s\b" % op, b)) for op in ("ds_write_b8", "ds_read_u8")}
        assert count == {"ds_write_b8": chunks, "ds_read_u8": chunks}
