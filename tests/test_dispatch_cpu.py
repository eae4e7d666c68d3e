"""How calls are laid out on the GPU and which kernel takes them, checked on
the host: the placement functions and dispatch rules are compiled into a small
driver (and, for the rules, linked with the built library), which no GPU is
needed for."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

from paper_2509_01190_amd import _build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
DRIVER = os.path.join(ROOT, "tests", "host", "dispatch_driver.cpp")


@pytest.mark.skipif(not os.path.exists(_build.HIPCC) or not os.path.exists(DRIVER),
                    reason="ROCm compilers or the driver's source not there")
def test_placement_and_dispatch_rules():
    tmp = tempfile.mkdtemp(prefix="zsa_dispatch_")
    try:
        exe = os.path.join(tmp, "dispatch_driver")
        lib = os.path.dirname(_build.LIB_PATH)
        subprocess.run([_build.HIPCC, "-x", "hip", "--cuda-host-only", f"--offload-arch={_build.ARCH}", "-O2",
                        "-std=c++17", "-c", DRIVER, "-o", exe + ".o"],
                       check=True, capture_output=True, text=True, timeout=300)
        subprocess.run([_build.HIPCC, exe + ".o", _build.LIB_PATH, f"-Wl,-rpath,{lib}", "-o", exe],
                       check=True, capture_output=True, text=True, timeout=300)
        r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stdout + r.stderr
        assert r.stdout.startswith("ok "), r.stdout
    finally:
        shutil.rmtree(tmp, ignore_errors=True)


def test_inline_asm_writes_no_unnamed_m0():
    """m0 holds the LDS address of loads to LDS. The compiler cannot see into
    an asm text: one that wrote m0 without naming it could break a use of the
    compiler's own, and it takes no such register as overwritten. So no text
    writes it; it is an operand."""
    csrc = os.path.join(ROOT, "paper_2509_01190_amd", "csrc")
    seen = 0
    for name in sorted(os.listdir(csrc)):
        for text in re.findall(r"\basm\b[^;]*?\(((?:[^;]|\\n)*?)\)\s*;", open(os.path.join(csrc, name)).read()):
            template = "".join(re.findall(r'"((?:[^"\\]|\\.)*)"', text.split(":")[0]))
            assert not re.search(r"\b\w+\s+m0\s*,", template), f"{name}: {template}"
            if "lds" in template:
                seen += 1
                assert '"{m0}"' in text, f"{name}: {template}"
    assert seen >= 2


def test_bench_knows_every_forward_kernel():
    """The profile summaries put each kernel of a forward into its class: a
    kernel they do not know counts as "misc" and its class's figures are
    wrong."""
    import bench
    csrc = os.path.join(ROOT, "paper_2509_01190_amd", "csrc")
    classes = {"k_attn.hip": "attention", "k_score.hip": "score", "k_norm.hip": "norm", "k_gemm.hip": "gemm"}
    seen = 0
    for name, cls in classes.items():
        text = open(os.path.join(csrc, name)).read()
        for kernel in set(re.findall(r"\b([a-z0-9_]+_kernel)\(\s*\n?\s*const [A-Za-z0-9_]+\* __restrict__", text)):
            if kernel == "rope_table_kernel":  # positions, not a product
                continue
            seen += 1
            assert bench.kernel_class(f"void zsa::(anonymous namespace)::{kernel}<64, 2>(int)") == cls, kernel
    assert seen >= 12
