"""Registers and scratch memory of the kernels that the default launches take, from the code objects in libtlb.so.

A kernel whose registers do not suffice keeps values in scratch memory, which goes through the caches like any other
memory.  The limits are what the kernels below were measured with; every other default step kernel has none.
"""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1511_02155_amd", "libtlb.so")

# bytes per lane.  The two-step sweep is held to two wavefronts per SIMD (256 registers); of the D3Q19 kernels those
# of five components in FP64 hold 95 populations and as many stencil sums in one wavefront's 512.
SCRATCH = {
    "k_pair2d<double, false, 3, 2>": 52, "k_batch_pair2d<double>": 52, "k_pair2d<double, true, 3, 2>": 108,
    "k_pair2d<float, true, 3, 2>": 56,
    "k_step3d<double, 64, 4, 0, false, 5>": 96, "k_step3d<double, 64, 4, 0, true, 5>": 68,
    "k_step3d<double, 32, 8, 0, true, 5>": 52, "k_step3d<double, 0, 0, 0, true, 5>": 84,
}


def _kernels(blob):
    """Metadata of the kernels of every AMDGPU code object in the file."""
    at = blob.find(b"\x7fELF")
    while at >= 0:
        if struct.unpack_from("<H", blob, at + 18)[0] == 224:  # EM_AMDGPU
            phoff, = struct.unpack_from("<Q", blob, at + 32)
            size, count = struct.unpack_from("<HH", blob, at + 54)
            for i in range(count):
                kind, _, off, _, _, length = struct.unpack_from("<IIQQQQ", blob, at + phoff + i * size)
                if kind != 4:  # PT_NOTE
                    continue
                p = at + off
                while p < at + off + length:
                    nn, nd, t = struct.unpack_from("<III", blob, p)
                    d = p + 12 + (nn + 3) // 4 * 4
                    if t == 32 and blob[p + 12:p + 18] == b"AMDGPU":
                        yield from msgpack.unpackb(blob[d:d + nd], strict_map_key=False)["amdhsa.kernels"]
                    p = d + (nd + 3) // 4 * 4
        at = blob.find(b"\x7fELF", at + 4)


@pytest.fixture(scope="module")
def kernels():
    found = list(_kernels(open(LIB, "rb").read()))
    assert found
    names = subprocess.run(["c++filt"], input="\n".join(k[".name"] for k in found), capture_output=True, text=True,
                           check=True).stdout.split("\n")
    short = (re.sub(r"^void |tlb::|\(anonymous namespace\)::", "", n).split("(")[0].strip() for n in names)
    return dict(zip(short, found))


def _is_default(name):
    """Step kernels of the default launches (see default_launch and launch_steps in tlb_api.hip)."""
    a = [x.strip() for x in name[name.find("<") + 1:-1].split(",")]
    if name.startswith(("k_tile2d<", "k_pair2d<", "k_batch_pair2d<")):
        return True
    if name.startswith("k_step3d<"):
        nc, variant = int(a[5]), int(a[3])
        return variant == ((2 if nc <= 4 else 1) if a[0] == "float" else (0 if nc > 3 else 1))
    return False


def test_scratch_of_the_default_step_kernels(kernels):
    seen = set()
    for name, k in kernels.items():
        if not _is_default(name):
            continue
        key = re.sub(r", (true|false)>$", ">", name) if name.startswith("k_step3d") else name  # both store policies
        seen.add(key)
        assert k[".private_segment_fixed_size"] <= SCRATCH.get(key, 0), (name, k[".private_segment_fixed_size"])
    assert set(SCRATCH) <= seen and len(seen) > 60
