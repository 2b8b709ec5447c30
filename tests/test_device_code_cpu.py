"""What the built device code must not contain, and that the build sees it. (A vector 64-bit shift
whose amount is the last register of a wave's allocation gives wrong bits, so no kernel shifts 64
bits by a register.)
"""

import glob
import os
import subprocess

from paper_2307_03017_amd import build, hsgd


def test_no_kernel_shifts_64_bits_by_a_register():
    hsgd.lib()                                 # says so if the library has not been built
    assert build.register_shifts(build.LIB) == []


def test_such_a_shift_is_seen(tmp_path):
    """One kernel with a lane's bit of a mask as the compiler makes it, one with a wave's."""
    src, obj = tmp_path / "shift.hip", tmp_path / "shift.o"
    src.write_text("""#include <hip/hip_runtime.h>
__global__ void by_lane(unsigned long long* p) { p[threadIdx.x] = 1ull << (p[threadIdx.x] & 63); }
__global__ void by_wave(unsigned long long* p, int n) { p[threadIdx.x] <<= n & 63; }
""")
    subprocess.run([build.HIPCC, *build.DEVICE_FLAGS, "-c", str(src), "-o", str(obj)], check=True,
                   stderr=subprocess.DEVNULL)
    found = build.register_shifts(str(obj))
    assert len(found) == 1 and "by_lane" in found[0] and "v_lshlrev_b64" in found[0]


def test_a_wave_hands_over_lds_by_the_fence():
    """The builtin barrier of a wave orders no memory: the compiler may move another lane's loads
    before it. It stands in wave_lds_fence alone, between the fence and the clobber that do."""
    uses = []
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*"))):
        lines = open(path).read().splitlines()
        uses += [(os.path.basename(path), lines[i - 1].strip(), lines[i + 1].strip())
                 for i, line in enumerate(lines) if "__builtin_amdgcn_wave_barrier" in line]
    assert uses == [("hsgd_device.h", '__builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");',
                     'asm volatile("" ::: "memory");')]
