"""The search's grid comes from the occupancy of the kernel that is launched: of its row
width, of its cap and of its number of binned axes.  The host side runs against stand-ins
for HIP (fake_hip.c), in a process of its own."""

import os
import subprocess
import sys


from test_mapped_result import HERE, LIB

CALLER = r"""
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before the library: its symbols come first
lib = ctypes.CDLL(sys.argv[2])
class Config(ctypes.Structure):
    _fields_ = [("dims", ctypes.c_int32 * 4)] + [(k, ctypes.c_int32) for k in ("axes", "cell_div", "grid_mult", "flags")]
name = lambda k: ctypes.string_at((ctypes.c_char * 256).in_dll(fake, k)).decode()
room = ctypes.create_string_buffer(1 << 21)
at = (ctypes.addressof(room) + 255) // 256 * 256
p, i64, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_float
for d in (3, 8, 12, 16, 24, 32, 48, 64):
    for K in (8, 64):
        for axes, div in ((0, 0), (3, 0), (3, 2)):
            config, count = Config(axes=axes, cell_div=div), i64(0)
            lib.frnn_build(p(at), i64(10), d, f32(0.1), K, p(at), ctypes.c_size_t(1 << 20), p(at), p(at), i64(100),
                           ctypes.byref(count), ctypes.byref(config), None, None)
            print(name("fake_asked"), name("fake_searched"), flush=True)
"""


def test_the_launched_kernel_is_asked(tmp_path):
    fake = str(tmp_path / "libfake_hip.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", os.path.join(HERE, "fake_hip.c"),
                    "-o", fake], check=True)
    out = subprocess.run([sys.executable, "-c", CALLER, fake, LIB], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stderr
    lines = [line.split() for line in out.stdout.split("\n") if line]
    assert len(lines) == 48 and len({searched for _, searched in lines}) == 30
    # (A kernel is asked for once, before its first launch.)
    seen = set()
    for asked, searched in lines:
        assert asked == searched or searched in seen, (asked, searched)
        seen.add(searched)
