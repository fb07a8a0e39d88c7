"""What the library does when the runtime refuses a launch or a kernel's LDS: the host code on a recording stand-in for the HIP
runtime (fake_hip.c), in a child process without torch.  No device, nothing runs."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as C, json, sys
fake_path, lib_path, jobs = sys.argv[1], sys.argv[2], json.loads(sys.argv[3])
fake = C.CDLL(fake_path, mode=C.RTLD_GLOBAL)
fake.fake_launched.restype = C.c_char_p
fake.fake_threads.restype = C.c_double
lib = C.CDLL(lib_path)
V, Z = C.c_void_p, C.c_size_t
big = Z(1 << 50)
W, L, R, state = V(1 << 20), V(2 << 20), V(3 << 20), V(4 << 20)      # never dereferenced by host code

class Adam(C.Structure):
    _fields_ = [(k, C.c_float) for k in ("lr", "b1", "b2", "eps")]
class Cayley(C.Structure):
    _fields_ = [(k, C.c_float) for k in ("lr", "beta", "eps", "q")] + [("s", C.c_int32), ("grad_scale", C.c_float)]
adam, cayley = Adam(1e-4, 0.9, 0.999, 1e-8), Cayley(0.5, 0.9, 1e-8, 0.5, 2, 1.0)

def call(name, cfg):
    p = C.byref(cfg)
    views = lambda n, skip: C.byref((V * n)(*[None if i in skip else (7 << 20) + 4096 * i for i in range(n)]))
    if name == "calib_init": return lib.lq_calib_init(p, L, R, state, big, None)
    if name == "calib_unpack": return lib.lq_calib_unpack(p, state, views(9, ()), None)
    if name == "calib_step": return lib.lq_calib_step(p, W, state, big, C.c_int32(1), C.byref(adam), None, None)
    if name == "rot_step": return lib.lq_rot_step(p, L, R, state, big, C.byref(cayley), None, None)
    if name == "rot_apply": return lib.lq_rot_apply(p, L, R, state, V(5 << 20), V(6 << 20), None)
    if name == "pack": return lib.lq_pack_weights(p, W, L, R, state, big, None)

out = []
for name, cfg_hex, failing_launch, failing_attrs, device in jobs:
    cfg = C.create_string_buffer(bytes.fromhex(cfg_hex))
    fake.fake_reset(failing_launch, failing_attrs, device)
    st = call(name, cfg)
    n = fake.fake_launches()
    out.append([st, [fake.fake_launched(i).decode() for i in range(n)], fake.fake_attrs(), [fake.fake_threads(i) for i in range(n)]])
print(json.dumps(out))
"""
DEVICE_ERROR = 6


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    from paper_2604_18117_amd import binding as lq
    fake = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-Wall", "-Werror", os.path.join(ROOT, "tests", "fake_hip.c"), "-o", fake], check=True)

    def go(jobs):
        jobs = [(n, bytes(lq.make_config(*c[:3], c[3], *c[4:])).hex(), fl, fa, dev) for n, c, fl, fa, dev in jobs]
        r = subprocess.run([sys.executable, "-c", CHILD, fake, os.path.join(ROOT, "paper_2604_18117_amd", "liblq.so"), json.dumps(jobs)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)
    return go


CFG = {"int": (512, 256, 64, "int", 64, 8, 8), "int128": (512, 256, 128, "int", 128, 4, 8), "mx": (512, 256, 128, "mx", 32, 8, 8),
       "mxb": (512, 256, 96, "mxb", 32, 8, 8), "mxb6": (512, 256, 64, "mxb", 32, 6, 6), "mxi": (512, 256, 128, "mxi", 32, 8, 8)}


@pytest.mark.parametrize("call", ["calib_step", "rot_step", "pack"])
@pytest.mark.parametrize("cfg", list(CFG))
def test_nothing_is_launched_after_a_failed_launch(run, call, cfg):
    """An update from gradient parts that were never written would spoil the caller's state behind an error status; a pack call that failed
    must not reach its last launch, which writes the blob's header."""
    (st, names, _, _), = run([(call, CFG[cfg], -1, 0, 0)])
    assert st == 0 and len(names) >= 2
    for k, (st, got, _, _) in enumerate(run([(call, CFG[cfg], k, 0, 0) for k in range(len(names))])):
        assert st == DEVICE_ERROR and got == names[:k + 1], (k, got)
    assert call != "pack" or "pack_residual_kernel" in names[-1]


@pytest.mark.parametrize("call,cfg", [("calib_step", "int"), ("calib_step", "mx"), ("rot_step", "int"), ("rot_step", "mxi"), ("rot_apply", "mxi")])
def test_a_refused_lds_request_fails_the_call_and_is_repeated(run, call, cfg):
    ok, = run([(call, CFG[cfg], -1, 0, 0)])
    kernels = ok[2]                                 # kernels that ask, each once
    assert ok[0] == 0 and kernels >= 1
    refused, again, third, past, past2 = run([(call, CFG[cfg], -1, 1, 0), (call, CFG[cfg], -1, 0, 0), (call, CFG[cfg], -1, 0, 0),
                                              (call, CFG[cfg], -1, 0, 64), (call, CFG[cfg], -1, 0, 64)])
    assert refused[0] == DEVICE_ERROR and len(refused[1]) < len(ok[1])
    assert again[0] == 0 and again[1] == ok[1] and again[2] == kernels
    assert third[0] == 0 and third[2] == 0          # granted: not asked for again
    assert past[0] == past2[0] == 0 and past[2] == past2[2] == kernels  # a device without an entry of its own asks every time


@pytest.mark.parametrize("call", ["calib_init", "calib_step", "calib_unpack", "rot_step", "rot_apply", "pack"])
def test_launches_stay_below_two_to_the_32_threads(run, call):
    """Layers whose matrices fill a third of the device's memory: a launch of 2^32 threads or more is refused by the runtime."""
    cfgs = [(131072, 131072, 128, "int", 128, 8, 8), (131072, 131072, 64, "mxi", 32, 8, 8), (1 << 21, 8192, 16, "int", 64, 8, 8),
            (8192, 1 << 21, 32, "mxb", 32, 8, 8)]
    for st, names, _, threads in run([(call, c, -1, 0, 0) for c in cfgs]):
        assert st == 0 and names and max(threads) < 2.0 ** 32, list(zip(names, threads))
