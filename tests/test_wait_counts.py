"""The counted waits of the big-tile kernels against the operations in the built code (CPU)."""
import os

import pytest

from paper_2607_23099_amd import build
from tests.wait_counts import counted_waits, disassemble

KERNEL = "k_gemm_big"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(build.LIB_DAMOE):
        build.build_damoe()
    code = disassemble(build.LIB_DAMOE, str(tmp_path_factory.mktemp("code")), KERNEL + "I")
    assert len(code) == 4  # GEMM1 / GEMM2, bf16 / fp8
    return code


def test_every_wait_is_covered(kernels):
    loose = []
    for name, code in kernels.items():
        waits = counted_waits(code)
        # 8 instances by token blocks, each with the wait ahead of its K loop and those inside it
        assert len(waits) >= 8 * 3, (name, len(waits))
        loose += [f"{name} {addr:#x}: vmcnt({n}) with {least} operations behind the guarded moves"
                  for addr, n, least in waits if n > least]
    assert not loose, "\n".join(loose)
