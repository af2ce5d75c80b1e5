"""Kernels that may take more than 64 KiB of LDS are told so on every device an index is created on, and a device that refuses
is reported.  The runtime's two calls are stood in for by a small C library in a process of its own: no GPU is needed."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
int stand_in_device = 0, stand_in_calls[4] = {0, 0, 0, 0}, stand_in_refuse = 0;
int hipGetDevice(int *d) { *d = stand_in_device; return 0; }
int hipFuncSetAttribute(const void *f, int what, int value) {
  ++stand_in_calls[stand_in_device];
  return stand_in_refuse ? 1 : 0;  /* hipErrorInvalidValue */
}
"""

PROGRAM = r"""
import ctypes as C, sys
stand_in = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # in front of the runtime for every library loaded from here on
from paper_2408_02937_amd import rtams
L = rtams.lib()
cfg = rtams.Config(d=32, nlist=64, metric=0, block_vecs=64, rearrange_threshold=0, n_resources=1, max_batch=16, max_k=10, max_nprobe=8,
                   max_add_batch=1024)
cfg.pool_bytes = L.rtams_pool_bytes_for(C.byref(cfg), 16)
cfg.scratch_bytes = L.rtams_scratch_bytes_for(C.byref(cfg), 1024)
device, refuse = C.c_int.in_dll(stand_in, "stand_in_device"), C.c_int.in_dll(stand_in, "stand_in_refuse")
calls = (C.c_int * 4).in_dll(stand_in, "stand_in_calls")
cfg.d_pool = cfg.d_scratch = 4096  # never read: there is no device behind the runtime
h = C.c_void_p()
def create():
    rc = L.rtams_create(C.byref(cfg), C.byref(h))
    assert rc == rtams.EHIP and not h.value, rc  # (at the latest where the control data is cleared)
    return L.rtams_last_error().decode()
for d in (0, 1, 0, 1):
    device.value = d
    create()
assert calls[0] == calls[1] >= 22, list(calls)  # 4 contractions, 16 scans, the bound and the scan over codes: once on each device
device.value, refuse.value = 2, 1
assert "allow_large_lds" in create()
assert calls[2] == 1
refuse.value = 0
assert "allow_large_lds" not in create() and calls[2] == 1 + calls[0], list(calls)
print("ok")
"""


def test_every_device_is_told_of_large_workgroups(tmp_path):
    src, lib, prog = tmp_path / "stand_in.c", tmp_path / "libstand_in.so", tmp_path / "program.py"
    src.write_text(STAND_IN)
    prog.write_text(PROGRAM)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    env = {**os.environ, "PYTHONPATH": ROOT, "HIP_VISIBLE_DEVICES": "-1"}
    r = subprocess.run([sys.executable, str(prog), str(lib)], env=env, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr
