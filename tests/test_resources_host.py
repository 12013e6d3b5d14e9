"""What the kernels' machine code holds of the chip, checked without a GPU.

Scratch memory of the built kernels, from the metadata of libauv.so (a kernel that keeps values in
memory between the steps of a loop waits for them there, behind its own stores); and that the
sources' assembly names the special register it writes, which the compiler uses too."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2512_13359_amd", "libauv.so")
LLVM = "/opt/rocm/llvm/bin"
KERNEL = re.compile(r"\.name: +(_ZN3auv\S+)\n(?:(?!\.name: +_ZN3auv).)*?\.private_segment_fixed_size: +(\d+)", re.S)


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    """{kernel's mangled name: bytes of scratch memory per lane}"""
    if not (os.path.exists(LIB) and os.path.exists(os.path.join(LLVM, "llvm-objdump"))):
        pytest.skip("needs the built library and the ROCm LLVM tools")
    tool = lambda name, *a, **k: subprocess.run([os.path.join(LLVM, name), *a], check=True, capture_output=True, text=True, **k).stdout
    d = tmp_path_factory.mktemp("code")
    shutil.copy(LIB, d / "libauv.so")
    tool("llvm-objdump", "--offloading", "libauv.so", cwd=d)
    out = {}
    for f in sorted(d.iterdir()):
        if "amdgcn" in f.name:
            out.update({n: int(b) for n, b in KERNEL.findall(tool("llvm-readelf", "--notes", str(f)))})
    return out


@pytest.mark.parametrize("kernel, forms", [("k_env_quad", 4), ("k_policy_rollout", 24)])
def test_no_scratch(scratch, kernel, forms):
    found = {n: b for n, b in scratch.items() if kernel in n}
    assert len(found) == forms
    assert not any(found.values()), {n: b for n, b in found.items() if b}


def test_assembly_names_m0():
    found = 0
    for path in glob.glob(os.path.join(ROOT, "paper_2512_13359_amd", "csrc", "*.h*")):
        for stmt in re.findall(r"\basm\b[^;]*;", open(path).read()):
            if re.search(r"s_mov_b32 m0\b", stmt):
                found += 1
                assert '"m0"' in stmt, (path, stmt)
    assert found == 1
