"""The plans of 3x3 convolutions with the filter in registers, and which calls get them (host only)."""
import os
import re
import shutil

import pytest

from test_sanitizers import CSRC, ENV, ROOT, SAN, _run


def test_plans_read_and_write_what_they_should(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("hipcc not found")
    decls = re.findall(r"VariantList (variants_\w+)\(\);", open(os.path.join(CSRC, "ucl_variants.h")).read())
    stub = tmp_path / "variants.cpp"         # (tables of tile kernels are empty; the plans only ask whether their kernel is there)
    stub.write_text('#include "ucl_variants.h"\nnamespace ucl {\nstatic const VariantDesc kHeld[1] = {};\n' +
                    "".join(f"VariantList {d}() {{ return {{{'kHeld, 1' if 'held' in d else 'nullptr, 0'}}}; }}\n" for d in decls) + "}\n")
    exe = str(tmp_path / "conv_held_plans")
    san = ["-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined", "-Xarch_host", "-fno-sanitize-recover=undefined"]
    _run([hipcc, "--offload-arch=gfx950", "-O1", "-g", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-command-line-argument", "-x", "hip", *san, "-I", CSRC, "-I", os.path.join(ROOT, "include"),
          os.path.join(CSRC, "ucl_transpose.hip"), str(stub), os.path.join(SAN, "conv_held_driver.cpp"), "-o", exe], cwd=str(tmp_path))
    r = _run([exe], env=ENV)
    assert "held plans: ok" in r.stdout and "ERROR: AddressSanitizer" not in r.stderr and "runtime error" not in r.stderr
