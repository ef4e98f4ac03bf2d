"""The library allocates no device memory: it imports no HIP call that does
(the caller owns every buffer, include/msm.h).  No GPU needed."""
import subprocess

from paper_1402_7216_amd import msm


def test_library_imports_no_device_allocation():
    msm.lib()
    out = subprocess.run(["nm", "-D", "--undefined-only", msm.LIB_PATH], check=True, capture_output=True, text=True)
    names = [line.split()[-1].split("@")[0] for line in out.stdout.splitlines()]
    assert any(n.startswith("hipLaunch") for n in names)
    assert [n for n in names if n.startswith(("hipMalloc", "hipExtMalloc", "hipFree", "hipMemAlloc", "hipMemPool",
                                              "hipArrayCreate", "hipHostMalloc", "hipHostAlloc"))] == []
