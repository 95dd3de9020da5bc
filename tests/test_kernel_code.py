"""What the built render kernels' code must look like for the speed their
comments state, read back from the gfx950 code objects in libsqn.so."""
import os
import re
import subprocess

import pytest

from paper_2204_02585_amd import build
from tests.test_build_guard import LLVM, device_code_objects

pytestmark = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="ROCm llvm tools missing")

TYPE = {"f16": "DF16_", "f32": "f"}


def _kernel(sigma, uvw, D, lanes, skip=True, ndc=False):
    """Mangled name of render_kernel<sigma, uvw, D, no statistics, lanes, skip, Eq. 4, ndc>."""
    types = TYPE[sigma] + TYPE[uvw]      # both are builtin types: no substitution
    return (f"_ZN3sqn12_GLOBAL__N_113render_kernelI{types}Li{D}ELb0ELi{lanes}ELb{int(skip)}ELb0ELb{int(ndc)}"
            "EEEvNS_12RenderParamsE")


@pytest.fixture(scope="module")
def render_object(tmp_path_factory):
    """Path of the code object that holds the render kernels."""
    assert os.path.exists(build.LIB_PATH), "build the library first"
    tmp = tmp_path_factory.mktemp("code")
    for k, (_, blob) in enumerate(device_code_objects(build.LIB_PATH, str(tmp))):
        if b"render_kernel_hybrid" in blob:
            path = tmp / f"render{k}.o"
            path.write_bytes(blob)
            return str(path)
    raise AssertionError("no code object holds the render kernels")


def _disassemble(path, name):
    asm = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--mcpu=gfx950", f"--disassemble-symbols={name}", path],
                         check=True, capture_output=True, text=True).stdout
    assert f"<{name}>:" in asm, f"{name} is not in the library"
    return asm


def _gathers_before_wait(asm):
    """For every queue entry read (ds_read_b128) the 16-byte loads issued
    after it before the first wait for a load."""
    out = []
    for part in asm.split("ds_read_b128")[1:]:
        head = re.split(r"s_waitcnt [^\n]*vmcnt", part)[0]
        out.append(head.count("global_load_dwordx4"))
    return out


@pytest.mark.parametrize("sigma", ["f16", "f32"])
@pytest.mark.parametrize("uvw,D,ndc", [("f32", 8, False), ("f16", 16, False), ("f16", 16, True)])
def test_eight_lane_drains_gather_at_once(render_object, sigma, uvw, D, ndc):
    """Every round of a drain (four unrolled in a full one, and the loops of
    the partial ones) issues its three records' six 16-byte loads before
    waiting for the first of them."""
    counts = _gathers_before_wait(_disassemble(render_object, _kernel(sigma, uvw, D, 8, ndc=ndc)))
    rounds = [n for n in counts if n]     # the other reads are of the ray setup
    assert len(rounds) >= 5 and min(rounds) >= 6, counts


def _resources(path):
    """{kernel name: (VGPRs, bytes of scratch per lane)} from the code object's
    metadata."""
    notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", path], check=True, capture_output=True,
                           text=True).stdout
    out = {}
    for entry in notes.split("- .agpr_count:")[1:]:
        value = lambda key: re.search(rf"\.{key}:\s+(\S+)", entry).group(1)
        out[value("name")] = (int(value("vgpr_count")), int(value("private_segment_fixed_size")))
    return out


def test_marches_that_lost_to_spills_spill_nothing(render_object):
    """binary32 sigma beside binary16 uvw at D = 8: the one-lane march in NDC and
    the hybrid launch keep their 72 registers (7 waves per SIMD) without
    scratch."""
    found = _resources(render_object)
    hybrid = "_ZN3sqn12_GLOBAL__N_120render_kernel_hybridIfDF16_Li8ELb0EEEvNS_12RenderParamsE"
    for name in (_kernel("f32", "f16", 8, 1, ndc=True), hybrid):
        vgprs, scratch = found[name]
        assert vgprs <= 72 and scratch == 0, (name, vgprs, scratch)


def test_opacity_keeps_no_constant_in_a_register(render_object):
    """One register more across the march costs these a wave per SIMD (two
    lanes, binary16 sigma and binary32 uvw: 80 of 80) or a spill (Eq. 5,
    binary32, D = 8: 96 of 96)."""
    found = _resources(render_object)
    eq5 = "_ZN3sqn12_GLOBAL__N_113render_kernelIffLi8ELb0ELi4ELb1ELb1ELb0EEEvNS_12RenderParamsE"
    for name, most in ((_kernel("f16", "f32", 8, 2), 80), (eq5, 96)):
        vgprs, scratch = found[name]
        assert vgprs <= most and scratch == 0, (name, vgprs, scratch)
