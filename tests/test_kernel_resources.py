"""Registers of kernels whose time depends on how many of their waves are resident, as the compiler reports them (no GPU needed)."""
import re
import shutil
import subprocess

import pytest

from paper_2601_22442_amd.build import HIPCC_FLAGS, PKG

FLAGS = [f for f in HIPCC_FLAGS if f not in ("-shared", "-Wall", "-Wextra")]
ADAM = 2
# template arguments: optimizer, bf16 gradients, forward copy (none, fp32, bf16), interleaved EMA vectors, walking
SYNC = [("k_step_sync", (ADAM, bf16, fwd, dil)) for bf16, fwd in ((False, 1), (True, 2), (False, 0)) for dil in (False, True)]
WALKING = [("k_step", (ADAM, bf16, fwd, dil, True)) for bf16, fwd in ((False, 1), (True, 2), (False, 0)) for dil in (False, True)]
# with a delay: by optimizer and interleaving, what the step needs where no factors are given
DELAYED = {("k_step", (opt, False, fwd, dil, False)): limit for (opt, fwd, dil), limit in
           {(ADAM, 1, True): (54, 95), (ADAM, 1, False): (54, 92), (ADAM, 0, True): (54, 92), (1, 0, False): (50, 84), (0, 0, False): (46, 82)}.items()}


def _cxx(kernel):
    name, args = kernel
    return f"am::{name}<{', '.join(str(x).lower() for x in args)}>"


def _mangled(kernel):
    name, args = kernel
    return f"_ZN2am{len(name)}{name}I" + "".join(f"L{'b' if isinstance(x, bool) else 'i'}{int(x)}E" for x in args) + "E"


@pytest.fixture(scope="module")
def resources(tmp_path_factory):
    if shutil.which("hipcc") is None:
        pytest.skip("no hipcc")
    kernels = SYNC + WALKING + list(DELAYED)
    src = tmp_path_factory.mktemp("kernels") / "kernels.hip"
    src.write_text(f'#include "{PKG}/csrc/am_kernels.h"\n' + "".join(f"template __global__ void {_cxx(k)}(const am::StepArgs);\n" for k in kernels))
    out = subprocess.run(["hipcc", *FLAGS, "-c", "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-o", "/dev/null", str(src)],
                         capture_output=True, text=True, check=True).stderr
    found = {}
    for part in out.split("Function Name: ")[1:]:
        found[part.split()[0]] = {k: int(v) for k, v in re.findall(r"remark: .*? (VGPRs|VGPRs Spill|ScratchSize|TotalSGPRs)(?: \[\S+\])?: (\d+)", part)}
    return {k: next(v for name, v in found.items() if name.startswith(_mangled(k))) for k in kernels}


@pytest.mark.parametrize("kernel", SYNC, ids=_cxx)
def test_two_workgroups_of_sixteen_waves_fit(resources, kernel):
    """32 waves on the four SIMDs of a compute unit: eight each, 64 registers of 512."""
    assert resources[kernel]["VGPRs"] <= 64 and resources[kernel]["ScratchSize"] == 0


@pytest.mark.parametrize("kernel", WALKING, ids=_cxx)
def test_the_walking_step_needs_no_scratch(resources, kernel):
    assert resources[kernel]["VGPRs Spill"] == 0 and resources[kernel]["ScratchSize"] == 0


@pytest.mark.parametrize("kernel", DELAYED, ids=_cxx)
def test_a_gradient_factor_takes_no_registers_where_none_is_given(resources, kernel):
    """Held from the operands on, it takes two to four vector registers or two to three scalar ones in every step."""
    vector, scalar = DELAYED[kernel]
    assert resources[kernel]["VGPRs"] <= vector and resources[kernel]["TotalSGPRs"] <= scalar and resources[kernel]["ScratchSize"] == 0
