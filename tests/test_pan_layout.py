"""The layout that the forward in panels reads, walked on the host: every row meets its entries in storage order, each while
the panel that holds its column is there, whatever the widths."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    tmp = tmp_path_factory.mktemp("pan")
    (tmp / "hip").mkdir()
    (tmp / "hip" / "hip_vector_types.h").write_text("struct int4 { int x, y, z, w; };\nstruct int2 { int x, y; };\n")
    exe = str(tmp / "walk")
    subprocess.run(["g++", "-std=c++17", "-g", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-I", str(tmp),
                    os.path.join(ROOT, "tests", "host_pan_layout.cpp"),
                    os.path.join(ROOT, "paper_2104_11805_amd", "csrc", "sdnn_setup.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("widths", [(16385, 63, 33000, 1023), (70, 16384, 16448, 5), (3, 49153, 24577, 40), (1, 1, 16400, 20000)])
def test_rows_meet_their_entries_in_order(walk, widths):
    env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
    out = subprocess.run([walk, *map(str, widths)], capture_output=True, text=True, env=env)
    assert out.returncode == 0 and "pan layout: ok" in out.stdout, out.stdout + out.stderr


def test_compiler_stays_out_of_the_registers_of_the_sums(tmp_path):
    """k_fwd_pan keeps its sums in v64 .. v127, which the compiler is told nothing of: outside the inline assembly its code names
    none of them, and it spills nothing."""
    import re

    from paper_2104_11805_amd import build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    asm = tmp_path / "sdnn.s"
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-pthread")]
    subprocess.run([hipcc, *flags, "--cuda-device-only", "-S", "-o", str(asm), os.path.join(build.CSRC, "sdnn.hip")], check=True)
    text = asm.read_text()
    bodies = re.findall(r"^_Z9k_fwd_panILi[01]ELb[01]EEv10PanForward:.*?s_endpgm", text, re.S | re.M)
    assert len(bodies) == 3
    for body in bodies:
        outside = re.sub(r";;#ASMSTART.*?;;#ASMEND", "", body, flags=re.S)
        named = [int(n) for m in re.findall(r"\bv(\d+)\b|\bv\[(\d+):(\d+)\]", outside) for n in m if n]
        assert named and max(named) < 64, max(named)
        assert "scratch_" not in outside and "accvgpr" not in outside
        assert "v[64:65]" in body
    assert re.findall(r"k_fwd_panILi[01]ELb[01]EEv10PanForward\.num_vgpr, (\d+)", text) == ["128"] * 3
