"""The launch rules (csrc/launch.h), asked through a small driver, and what the compiler made of the kernels they
launch, read from the built library's metadata.  No GPU."""
import os
import re
import shutil
import struct
import subprocess
from collections import namedtuple

import pytest

import paper_1912_09268_amd as M

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1912_09268_amd", "csrc")
READELF = shutil.which("llvm-readelf") or "/opt/rocm/llvm/bin/llvm-readelf"
KINDS = ["pack", "reduce", "update", "reduce_update", "pipeline", "direct"]
DTYPES = ["f32", "bf16", "f16"]
CU_LDS, LDS_GRAIN = 160 << 10, 1280
Kernel = namedtuple("Kernel", "few kind half P form lds vgprs")
Shape = namedtuple("Shape", "tiles_per_wg units grid xcd_contiguous run_log2 may_be_few form wgs_per_cu")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("launch") / "driver")
    r = subprocess.run(["g++", "-std=c++17", "-Wall", "-Wno-unused-function", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                        os.path.join(ROOT, "tests", "launch_shape_driver.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr

    def ask(lines):
        r = subprocess.run([exe], input="\n".join(lines), capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        out = [tuple(int(x) for x in line.split()) for line in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out
    return ask


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Every kernel of the built library: the code objects in it are bundles of (offset, size, target)."""
    data, found, at = open(M.library_path(), "rb").read(), [], 0
    part = str(tmp_path_factory.mktemp("kernels") / "code")
    while (at := data.find(b"__CLANG_OFFLOAD_BUNDLE__", at)) >= 0:
        (n,), pos = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            target = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" not in target or size == 0:
                continue
            with open(part, "wb") as f:
                f.write(data[at + offset:at + offset + size])
            notes = subprocess.run([READELF, "--notes", part], capture_output=True, text=True, check=True).stdout
            for text in notes.split("\n  - .a")[1:]:
                m = re.search(r"\.name:\s+\S*mgwfbp_(few|stream)_kernelILi(\d)E(\w+?)Li(\d+)ELi(n?\d)E", text)
                field = lambda key: int(re.search(r"\.%s:\s+(\d+)" % key, text).group(1))  # noqa: E731
                assert field("private_segment_fixed_size") == 0, "spills"
                found.append(Kernel(m.group(1) == "few", int(m.group(2)), m.group(3) != "f", int(m.group(4)),
                                    int(m.group(5).replace("n", "-")), field("group_segment_fixed_size"), field("vgpr_count")))
        at += 24
    assert len(found) > 100
    return found


def test_caps_hold_for_every_kernel(ask, kernels):
    """At most the workgroups asked for fit into a compute unit with the LDS the kernel really has, and as many as the
    grain of 1280 bytes allows."""
    caps = list(range(2, 32))
    answers = iter(ask([f"lds {k.kind} {int(k.few)} {k.form} {n}" for k in kernels for n in caps]))
    for k in kernels:
        for n in caps:
            own, extra = next(answers)
            assert own <= k.lds <= own + 64, k
            grains = -(-(k.lds + extra) // LDS_GRAIN)
            assert CU_LDS // (grains * LDS_GRAIN) <= n, (k, n)
            assert CU_LDS // ((grains - 1) * LDS_GRAIN) > n or n == 2, (k, n)


def test_sixteen_bit_pipeline_of_single_tiles_keeps_its_wave_slots(kernels):
    """Single tiles of 16-bit gradients run uncapped because they need every wavefront a compute unit can hold: eight per
    SIMD (512 registers, granted in eights), six with the addresses of 16 workers, and no LDS for joined steps."""
    single = [k for k in kernels if KINDS[k.kind] == "pipeline" and k.half and k.form == 1]
    assert len(single) == 20
    for k in single:
        assert 512 // (-(-k.vgprs // 8) * 8) >= (6 if k.P == 16 else 8), k
        assert k.lds <= (0 if k.few else 1296), k
