"""The plans of 3x3 convolutions with the filter in registers, and which calls get them (host only)."""
import math
import os
import random
import re
import shutil

import pytest

import paper_2603_29010_amd as ucl

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


def runs_on(op, n, H, W, C, Ko, stride=1, residual=False, dt="bf16"):
    chain = [] if op == "dgrad" else [("bias", 0, dt), ("relu",)]
    if residual:
        chain.insert(1 if chain else 0, ("aux_load", 0, dt, 0, 0, 1.0))
    return ucl.ucl_unnamed_kernel(f"conv2d_{op}", dt, dt, conv=(n, H, W, C, Ko, 3, 3, 1, 1, stride, stride, 1, 1), epi=ucl.Epilogue(chain))


# (microseconds in a graph: tile kernel, filter in registers)
@pytest.mark.parametrize("layer,residual,tile,held", [(("fprop", 17, 56, 56, 128, 128), False, 21.8, 33.3), (("fprop", 15, 64, 64, 128, 128), False, 23.5, 37.9),
                                                      (("fprop", 4, 81, 81, 128, 64), False, 11.6, 18.3), (("fprop", 12, 195, 195, 64, 32), False, 65.2, 98.8),
                                                      (("fprop", 16, 57, 57, 128, 128), True, 24.9, 33.6), (("fprop", 2, 181, 181, 64, 8), True, 12.8, 19.0),
                                                      (("fprop", 27, 103, 103, 72, 24), False, 56.8, 81.0), (("fprop", 24, 116, 15, 256, 128), False, 32.7, 46.2),
                                                      (("fprop", 17, 120, 120, 64, 64, 2), False, 16.0, 21.0), (("dgrad", 8, 109, 109, 64, 128), False, 29.3, 38.9),
                                                      (("dgrad", 13, 198, 198, 32, 64), False, 78.7, 106.5), (("dgrad", 52, 91, 91, 8, 96), False, 87.7, 135.5)])
def test_layers_that_tile_kernels_run_faster_stay_there(layer, residual, tile, held):
    assert tile < held and runs_on(*layer, residual=residual) is None


@pytest.mark.parametrize("layer,residual,tile,held", [(("fprop", 32, 56, 56, 64, 128), True, 27.8, 20.2), (("fprop", 32, 56, 56, 64, 64), True, 24.2, 12.3),
                                                      (("fprop", 32, 28, 28, 128, 128), True, 16.3, 12.9), (("fprop", 4, 14, 14, 256, 256), True, 11.1, 7.9),
                                                      (("dgrad", 32, 28, 28, 128, 128), False, 14.9, 12.6), (("dgrad", 32, 14, 14, 256, 256), False, 27.5, 18.9),
                                                      (("dgrad", 4, 14, 14, 256, 256), False, 17.0, 8.1), (("dgrad", 1, 56, 56, 64, 64), False, 10.5, 6.3)])
def test_layers_that_gain_are_taken(layer, residual, tile, held):
    assert held < tile and runs_on(*layer, residual=residual) == "conv_held"


def test_every_tile_kernel_that_such_a_layer_can_get_has_a_price():
    text = open(os.path.join(CSRC, "ucl_costs.h")).read()
    rows = {tuple(int(v) for v in m) for m in re.findall(r"\{(\d+), +(\d+), +(\d+), (\d+), (\d+), (\d+), +(\d+), \d+, ", text.split("kConvRows[] = {")[1].split("};")[0])}
    rng, seen = random.Random(3), set()
    size = lambda lo, hi, step=1: max(step, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step)  # noqa: E731
    for _ in range(6000):
        op, H, W = rng.choice(("fprop", "fprop", "dgrad")), size(1, 400), size(1, 400)
        C, Ko, stride = size(8, 1024, 8), size(8, 1024, 8), 1 if op == "dgrad" else rng.choice((1, 2))
        if rng.random() < .4:
            W, C, Ko = min(W, 58), rng.choice((64, 128, C)), rng.choice((64, 128, Ko))
        t = ucl.ucl_select_tuning(f"conv2d_{op}", "bf16", "bf16", conv=(size(1, 64), H, W, C, Ko, 3, 3, 1, 1, stride, stride, 1, 1))
        if op == "fprop" and C > 256:          # (more channels than are served)
            continue
        seen.add((2 if op == "fprop" else 3, t["tile_m"], t["tile_n"], t["tile_k"], t["stages"], t["k_groups"], 0 if t["iterator"] != 2 else C if op == "fprop" else Ko))
    assert len(seen) > 12 and seen <= rows, seen - rows
