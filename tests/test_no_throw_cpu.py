"""Nothing that may throw stands behind the reductions' C entries: the number
that marks a call's arrivals does not come from std::random_device, whose
constructor and call throw where the system has no entropy source."""
import subprocess

from paper_1412_1127_amd import build


def test_no_random_device():
    names = subprocess.run(["nm", "-D", "-C", "--undefined-only", build.LIB], capture_output=True, text=True, check=True)
    assert "std::" in names.stdout                      # the C++ runtime's names are listed
    assert "random_device" not in names.stdout
