"""The inline assembly of the decode kernels keeps the wait states that the compiler does not keep for it (CPU only)."""
import os
import shutil
import subprocess

import pytest

import asm_hazards

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_helpers_hold_behind_a_vector_write_of_their_base(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    out = str(tmp_path / "k.s")
    res = subprocess.run([hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "-Wno-inline-asm", "-I", os.path.join(ROOT, "include"), "-I",
                          os.path.join(ROOT, "paper_2502_15804_amd", "csrc"), "--cuda-device-only", "-S", "-x", "hip",
                          os.path.join(ROOT, "tests", "inline_asm.hip"), "-o", out], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-3000:]
    code = dict(asm_hazards.functions(open(out).read()))
    assert set(code) == {"stores", "small_stores", "loads", "kept_loads", "tile2", "tile4", "argument_lanes", "factor_lanes"}
    for name, lines in code.items():
        assert any("v_readfirstlane" in t for t in lines), name     # the case is there
        assert asm_hazards.hazards(lines) == set(), name


@pytest.mark.parametrize("code,broken", [
    ("v_readlane_b32 s4, v1, 3 / s_nop 3 / global_store_dword v0, v2, s[4:5]", {"s4"}),
    ("v_readlane_b32 s4, v1, 3 / s_nop 4 / global_store_dword v0, v2, s[4:5]", set()),
    ("v_readlane_b32 s4, v1, 3 / s_mov_b64 s[6:7], s[4:5] / global_store_dword v0, v2, s[6:7]", set()),
    ("v_cmp_lt_f32_e64 s[4:5], v1, v2 / s_cbranch_scc0 .L / s_nop 4 / .L: / buffer_load_dword v0, v1, s[4:7], 0 offen", {"s4", "s5"}),
    ("s_mov_b32 m0, s1 / global_load_lds_dwordx4 v0, s[2:3]", {"m0"}),
    ("s_mov_b32 m0, s1 / s_nop 0 / global_load_lds_dwordx4 v0, s[2:3]", set()),
    ("global_store_dwordx4 v0, v[4:7], s[2:3] / s_nop 0 / v_mov_b32_e32 v7, 0", {"v7"}),
    ("global_store_dwordx4 v0, v[4:7], s[2:3] / s_nop 1 / v_mov_b32_e32 v7, 0", set()),
    ("v_readlane_b32 s4, v1, 3 / s_nop 0 / v_writelane_b32 v0, s4, 7", {"s4"}),
    ("v_readlane_b32 s4, v1, 3 / s_nop 1 / v_writelane_b32 v0, s4, 7", set()),
    ("v_readfirstlane_b32 s4, v1 / s_mov_b32 s5, s4 / v_writelane_b32 v0, s5, 7", set()),
    ("v_cmp_lt_f32_e32 vcc, v1, v2 / v_cndmask_b32_e32 v3, v4, v5, vcc", {"svcc"}),
    ("v_add_co_u32 v1, vcc, v2, v3 / s_nop 1 / v_addc_co_u32 v4, vcc, v5, v6, vcc", set()),
    ("v_readlane_b32 s4, v1, 3 / s_nop 2 / v_readlane_b32 s6, v9, s4", {"s4"}),
    ("v_readlane_b32 s4, v1, 3 / s_nop 3 / v_writelane_b32 v9, s8, s4", set()),
    ("v_writelane_b32 v0, s4, 7 / v_readlane_b32 s5, v0, 7", {"v0"}),
    ("v_writelane_b32 v0, s4, 7 / s_nop 0 / v_readlane_b32 s5, v0, 7", set()),
    ("v_mov_b32_e32 v0, v1 / v_readfirstlane_b32 s5, v0", {"v0"}),
])
def test_what_the_search_finds(code, broken):
    assert {r for _, r in asm_hazards.hazards(code.split(" / ") + ["s_endpgm"])} == broken
