"""The recorded memory traffic of the decoder is reported for the sources it was
counted on only: every file that the decode kernel is compiled from counts."""
import os
import shutil

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_18900_amd", "csrc")


@pytest.mark.parametrize("changed", ["kernels.hip", "lz_device.h", "lz_internal.h"])
def test_every_source_counts(tmp_path, changed):
    import bench
    d = tmp_path / "csrc"
    shutil.copytree(CSRC, d)
    assert bench.decoder_sha(str(d)) == bench.decoder_sha(CSRC)
    with open(d / changed, "a") as f:
        f.write("\n")
    assert bench.decoder_sha(str(d)) != bench.decoder_sha(CSRC)
