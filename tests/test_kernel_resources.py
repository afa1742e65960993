"""What the compiler reports of the sampling kernels for large batches (tickets, a query per lane): every one of them is bound by the length
of its waves' programs and by the memory, and none may keep values in scratch memory.  Cross-compiled; no GPU."""
import os
import re
import subprocess

import pytest

from paper_2311_17410_amd import build

REPORT = re.compile(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", re.S)


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no compiler")
def test_kernels_with_tickets_use_no_scratch_memory():
    flags = [f for f in build.FLAGS if f != "-shared"]
    runs = [subprocess.Popen([build.HIPCC, *flags, "-x", "hip", "--cuda-device-only", "-c", os.path.join(build.CSRC, src), "-o", os.devnull,
                              "-Rpass-analysis=kernel-resource-usage"], stderr=subprocess.PIPE, text=True)
            for src in ("tns_kernels.hip", "tns_kernels_recent.hip", "tns_kernels_prefix.hip")]
    seen = set()
    for run in runs:
        report = run.communicate(timeout=300)[1]
        assert run.returncode == 0, report[-2000:]
        for name, scratch in REPORT.findall(report):
            kernel = re.search(r"\d+tns_sample_(recent_kernel|prefix_kernelILi1|kernelILi1).*Li1EEEv", name)      # (the last argument: kTickets)
            if kernel:
                seen.add(name)
                assert int(scratch) == 0, f"{name}: {scratch} bytes a lane"
    assert len(seen) == 16, sorted(seen)      # two layouts, two policies, both window ends, both widths of a position
