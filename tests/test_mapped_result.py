"""The pinned memory that a thread's synchronous calls get their results in serves every
device: it is portable, and the kernels of a call are given the current device's address
of it.  The host side runs against stand-ins for HIP (fake_hip.c), in a process of its own.
"""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(ROOT, "paper_2202_06929_amd", "libfrnn.so")

CALLER = r"""
import ctypes, struct, sys
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before the library: its symbols come first
entry, map_fails = sys.argv[3], int(sys.argv[4])
var = lambda name: ctypes.c_int.in_dll(fake, name)
name = b"k_cc_label" if entry == "components" else b"k_placeILi4E"
ctypes.memmove(ctypes.addressof((ctypes.c_char * 64).in_dll(fake, "fake_kernel")), name, len(name))
lib = ctypes.CDLL(sys.argv[2])
var("fake_arg").value = 4 if entry == "components" else 26
var("fake_map_fails").value = map_fails
room = ctypes.create_string_buffer(1 << 21)
at = (ctypes.addressof(room) + 255) // 256 * 256
p, i64, f32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_float
for k, device in enumerate((0, 1, 1, 0, 2)):
    var("fake_device").value = device
    count = i64(-1)
    answer = struct.pack("<qq", 40 + k, 0) + bytes(112)
    ctypes.memmove(ctypes.addressof((ctypes.c_char * 128).in_dll(fake, "fake_result")), answer, 128)
    if entry == "components":
        st = lib.frnn_components(p(at), p(at), i64(3), i64(100), None, f32(0), p(at), ctypes.c_size_t(1 << 20), p(at),
                                 ctypes.byref(count), None)
    else:
        st = lib.frnn_build(p(at), i64(10), 3, f32(0.1), 8, p(at), ctypes.c_size_t(1 << 20), p(at), p(at), i64(100),
                            ctypes.byref(count), None, None, None)
    print(device, st, count.value, flush=True)
print(ctypes.c_uint.in_dll(fake, "fake_flags").value, var("fake_copies").value)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    out = tmp_path_factory.mktemp("fake") / "libfake_hip.so"
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-Werror", "-fPIC", "-shared", os.path.join(HERE, "fake_hip.c"),
                    "-o", str(out)], check=True)
    return str(out)


@pytest.mark.parametrize("map_fails", [0, 1])
@pytest.mark.parametrize("entry", ["components", "build"])
def test_a_thread_that_changes_devices(fake, entry, map_fails):
    out = subprocess.run([sys.executable, "-c", CALLER, fake, LIB, entry, str(map_fails)], capture_output=True, text=True,
                         timeout=120)
    assert out.returncode == 0, out.stderr
    lines = [line.split() for line in out.stdout.split("\n") if line]
    for k, (line, device) in enumerate(zip(lines, (0, 1, 1, 0, 2))):
        assert line == [str(device), "0", str(40 + k)], out.stdout
    flags, copies = (int(v) for v in lines[-1])
    assert flags & 1, "portable"  # hipHostMallocPortable
    assert copies == (5 if map_fails else 0)
