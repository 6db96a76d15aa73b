"""The batched kernel's general form (separate stages beside the fused units)."""
import os
import re
import subprocess
import sys

import pytest

from paper_1302_6189_amd import fftrw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("flags", [fftrw.FLAG_LEAVE_PERMUTED, fftrw.FLAG_BATCH_NO_FUSE])
def test_resident_groups_of_the_general_kernel(gpu_lib, flags):
    # the kernel with the separate stages keeps three work-groups (three waves
    # per SIMD) on a compute unit, as the plan's log line says
    import torch
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    code = ("from paper_1302_6189_amd import fftrw\n"
            f"fftrw.Batch([((96, 96, 96), 4)] * 16, flags={flags}).destroy()\n")
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, FFTRW_LOG="1"), capture_output=True,
                       text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    assert int(re.search(r"(\d+) resident groups", r.stderr).group(1)) >= 3 * ncu, r.stderr
