"""What the compiler gives the kernels for gfx950: registers of a lane that do not fit go to scratch memory, which costs every
call, so the kernels that every call runs through have none there, and the others no more than is known of them."""
import os
import re
import subprocess

import pytest

from paper_2507_11941_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc"), reason="needs hipcc")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: bytes of scratch a lane}"""
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    done = subprocess.run(["/opt/rocm/bin/hipcc", *flags, "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", "-o",
                           str(tmp_path_factory.mktemp("resources") / "bpe.o"), *build.SOURCES], capture_output=True, text=True)
    assert done.returncode == 0, done.stderr[-2000:]
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", done.stderr, flags=re.S)
    assert len(found) > 20
    return {name: int(scratch) for name, scratch in found}


def test_no_scratch(kernels):
    """All but the kernels of sixteen waves an item, whose lanes have 128 registers."""
    assert not {name: s for name, s in kernels.items() if s and not re.search("encode_(long|rest)_kernel", name)}
