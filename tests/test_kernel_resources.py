"""The compiler's resource report for the hot kernels (CPU only: hipcc cross-compiles gfx950 without a GPU).

The kernels' waits on their HBM -> LDS rings (fp32: on the registers requested ahead) leave no room in the item loop for a
memory operation the compiler adds on its own: a register spilled to scratch memory, or a variable it leaves in private
memory, brings loads and stores that it answers with a wait for ALL outstanding loads, i.e. one exposed memory
latency per item (measured once: 3 us per launch, with every parity test still green).  So: no scratch, no
spilled vector registers, one wave per SIMD, and the LDS budget of a compute unit kept."""
import os
import re
import shutil
import subprocess

import pytest

import asm_hazards

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """{kernel: (a function that reads a figure of its resource report, its lines of assembly)}"""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "k.s")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "-mllvm", "-amdgpu-mfma-vgpr-form=1", "-Wno-inline-asm",
                          "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2502_15804_amd", "csrc"),
                          "--cuda-device-only", "-S", "-x", "hip", os.path.join(ROOT, "tests", "kernel_resources.hip"),
                          "-o", out, "-Rpass-analysis=kernel-resource-usage"], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    code = dict(asm_hazards.functions(open(out).read()))
    reports = {k.split()[0]: k for k in re.split(r"remark: Function Name: ", res.stderr)[1:]}
    assert set(reports) == set(code)
    figure = lambda report: lambda key: int(re.search(key + r": (\d+)", report).group(1))
    return {name: (figure(report), code[name]) for name, report in reports.items()}


def test_hot_kernel_uses_no_scratch_and_fits_the_lds(compiled):
    hot = {name: k for name, k in compiled.items() if "valu" not in name}
    assert len(hot) == 8
    for name, (val, code) in hot.items():
        assert val(r"ScratchSize \[bytes/lane\]") == 0, name
        assert val("VGPRs Spill") == 0, name
        assert val(r"LDS Size \[bytes/block\]") <= 160 * 1024, name
        assert val(r"Occupancy \[waves/SIMD\]") >= 1, name
        assert not any("scratch_" in t or "buffer_store" in t for t in code), name      # nothing goes to private memory


def test_vector_kernel_has_the_registers_of_a_whole_simd(compiled):
    # with half of them it spills 792 and takes 1.5 to 3 times as long; 351 as built
    (val, _), = (k for name, k in compiled.items() if "valu" in name)
    assert val("VGPRs Spill") <= 400


def test_no_wait_state_is_broken(compiled):
    for name, (_, code) in compiled.items():
        assert asm_hazards.hazards(code) == set(), name


def test_kernels_with_short_pairs_do_not_carry_a_second_set_of_outputs(compiled):
    # what an item starts from is set behind every item, also the last: behind a condition it takes registers of its own (226 instead of 192)
    val, _ = compiled["_ZN6fairkv25fairkv_decode_mfma_kernelILi128ELi8ELb0ELb0ELb1ELb0EEEvNS_10DecodeArgsE"]
    assert val(" VGPRs") <= 200


def test_scalar_registers_of_an_8bit_kernel_with_short_pairs(compiled):
    # spilled ones come back from vector lanes, one instruction each, in front of what needs them: 34 with the end of an item read ahead of its tiles
    val, _ = compiled["_ZN6fairkv25fairkv_decode_mfma_kernelILi64ELi8ELb0ELb1ELb1ELb0EEEvNS_10DecodeArgsE"]
    assert val("SGPRs Spill") <= 14
