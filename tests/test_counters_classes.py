"""The kernel names that the counter reduction looks for are names of kernels in
the built library (a template argument more would leave a class without a record)."""
import shutil
import subprocess

import pytest

from paper_1303_1377_amd import counters
from tests import test_kernel_registers as built


@pytest.mark.parametrize("cls", list(counters.CLASSES))
def test_prefixes_name_kernels(cls):
    if not shutil.which("c++filt"):
        pytest.skip("no c++filt")
    names = subprocess.run(["c++filt"], input="\n".join(built._kernels()), check=True, capture_output=True, text=True).stdout
    names = names.splitlines()
    for prefix in counters.CLASSES[cls][0]:
        assert any(n.startswith(prefix) for n in names), prefix
