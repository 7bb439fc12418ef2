"""The library's host code on a stand-in HIP runtime (hip_standin.cpp): handles
on host memory whose kernels are never run.  For scripts that a test runs in a
process of their own (run)."""
import ctypes as C
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))


def build(folder):
    lib = os.path.join(str(folder), "libhip_standin.so")
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-std=c++17", "-w", "-I",
                           "/opt/rocm/include", "-o", lib, os.path.join(HERE, "hip_standin.cpp")])
    return lib


def run(lib, code, timeout=300):
    """The script `code` in a Python of its own, whose library calls the
    stand-in: loaded first, with its names global, they come before those of
    the runtime that the library is linked with."""
    env = dict(os.environ, HIP_STANDIN=lib, PYTHONPATH=HERE + os.pathsep + ROOT)
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True,
                       timeout=timeout)
    assert r.returncode == 0, (r.stdout + r.stderr)[-1500:]
    return r.stdout


_standin = None


def standin():
    global _standin
    if _standin is None:
        _standin = C.CDLL(os.environ["HIP_STANDIN"], mode=C.RTLD_GLOBAL)
        _standin.standin_launches.restype = C.c_long
    return _standin


def faults():
    """What the library did that it must not, since the last call."""
    buf = C.create_string_buffer(4096)
    return buf.value.decode() if standin().standin_faults(buf, 4096) else ""


class Handle:
    """A handle over boxes of (nx, ny, nz, walls) on host memory."""

    def __init__(self, shapes, storage=0, stream=None, **params):
        standin()
        import paper_2309_07801_amd as pkg
        self.pkg, self.L = pkg, pkg.lib()
        d = dict(rho0_r=1.0, rho0_b=0.1, alpha_r=0.9, alpha_b=8.0 / 27.0, nu_r=0.1, nu_b=0.1,
                 sigma=0.01, beta=0.7)
        d.update(params)
        prm = [pkg.box_params(nx=x, ny=y, nz=z, walls=w, **d) for x, y, z, w in shapes]
        pop, aux, total = pkg.query_sizes(prm, storage)
        self.mem = [C.create_string_buffer(n) for n in (pop, pop, aux, total * 4, total * 4,
                                                        total * 12)]
        arr = (pkg.BoxParams * len(prm))(*prm)
        self.h = C.c_void_p()
        self.stream = stream
        self.ok(self.L.cglbm_init(C.byref(self.h), len(prm), arr, storage,
                                  *[C.addressof(m) for m in self.mem], C.c_uint64(0),
                                  C.c_double(0.0), stream))

    def ok(self, rc):
        assert rc == 0, self.L.cglbm_last_error()

    def call(self, name, *args, stream=True):
        self.ok(getattr(self.L, "cglbm_" + name)(self.h, *args, *([self.stream] if stream else [])))

    def close(self):
        self.L.cglbm_destroy(self.h)

