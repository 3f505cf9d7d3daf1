"""deft_plan_upload against a stand-in for the HIP runtime (tests/fake_hip), so on the CPU: what it does where the device has
failed, and by which way an image goes.  Each test is a process of its own, since the library keeps its staging slots."""

import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PREAMBLE = """
import ctypes, sys
fake_lib = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before libdeft.so: its functions are found first
names = ("device stream_device pointer_device pointer_type capturing event_error launches copies events_recorded").split()
class Fake(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in names]
fake = Fake.in_dll(fake_lib, "fake")
import numpy as np
from paper_2404_00242_amd import binding
lib = binding.load_library()
EHIP, FAILED, STREAM = -4, 719, 0x1000
def forest(n):
    lens = np.arange(1, n + 1, dtype=np.int32) % 31 + 1
    begins = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int32)
    return binding.deft_plan(begins, lens, np.full(n, -1, np.int32), np.arange(n, dtype=np.int32), int(lens.sum()), 32,
                             binding.DEFT_SPLIT_NODE), begins
plan, begins = forest(20)
size = plan.device_bytes(4, 4)
buf = np.zeros(size + 16, np.uint8)
image = buf[-buf.ctypes.data % 16:][:size]
def upload(stream=STREAM):
    return lib.deft_plan_upload(plan.handle, 4, 4, ctypes.c_void_p(image.ctypes.data), ctypes.c_size_t(size), ctypes.c_void_p(stream))
def arrived():
    return (image[: 4 * len(begins)].view(np.int32) == begins).all()
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "fake_hip", "fake_hip.cpp"), "-o", so], check=True)
    return so


def run(fake, body):
    p = subprocess.run([sys.executable, "-c", PREAMBLE + body, fake], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT,
                       text=True, timeout=60)
    assert p.returncode == 0, p.stdout[-3000:]


needs_gxx = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"), reason="needs g++ and HIP headers")


@needs_gxx
def test_device_failure_is_reported_by_the_upload_that_needs_the_slot(fake):
    # the fetches of the first eight never end: the device has failed, and the runtime says so when it is asked
    run(fake, """
for _ in range(8):
    assert upload() == 0
fake.event_error = FAILED
for _ in range(3):
    assert upload() == EHIP
assert b"staging slot" in lib.deft_last_hip_error()
""")


@needs_gxx
@pytest.mark.parametrize("pointer,stream,kernel", [
    ((0, "Device"), 0, True),
    ((0, "Device"), None, True),    # the null stream, which is the current device's
    ((0, "Host"), 0, False),        # a copy reaches any memory
    ((1, "Device"), 0, False),
    ((1, "Device"), None, False),
    ((1, "Device"), 1, False),      # and goes into streams of other devices than the current one
    ((0, "Device"), 1, False),
])
def test_image_goes_by_a_kernel_only_into_memory_and_streams_of_the_current_device(fake, pointer, stream, kernel):
    run(fake, f"""
fake.pointer_device, fake.pointer_type = {pointer[0]}, {dict(Host=1, Device=2)[pointer[1]]}
fake.stream_device = {stream or 0}
for i in range(1, 20):
    image[:] = 0
    assert upload({'None' if stream is None else 'STREAM'}) == 0
    assert (fake.launches, fake.copies) == ({'i, 0' if kernel else '0, i'})
    assert arrived() != {kernel}  # (kernels are not run here)
""")


@needs_gxx
def test_captured_upload_uses_no_staging_slot(fake):
    # a replay would read the slot when it holds another image, and no event in a graph says when a slot is free
    run(fake, """
ACTIVE = 1
fake.capturing = ACTIVE
for _ in range(20):
    assert upload() == 0
assert (fake.copies, fake.events_recorded) == (0, 0) and fake.launches % 20 == 0 and fake.launches > 0
fake.pointer_device = 1
assert upload() == EHIP and b"captured" in lib.deft_last_hip_error()
fake.capturing = fake.pointer_device = fake.launches = 0
assert upload() == 0 and fake.launches == 1
""")
