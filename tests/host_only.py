"""The library's host side on a machine without a GPU: libgwg.so with a stand-in
for the HIP runtime (helpers/fake_hip.cpp) preloaded, in a process of its own.
Device memory is a budget, kernels are log lines."""
import ctypes as C
import json
import os
import shutil
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_so = None


def _fake():
    global _so
    if _so is None:
        d = tempfile.mkdtemp()
        _so = os.path.join(d, "fake_hip.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I/opt/rocm/include",
                        "-I" + os.path.join(ROOT, "paper_2601_04370_amd", "csrc"), "-o", _so,
                        os.path.join(ROOT, "tests", "helpers", "fake_hip.cpp"), "-ldl"], check=True)
        import atexit
        atexit.register(shutil.rmtree, d, True)
    return _so


def run(body):
    """Run `body` (Python source; `h` is a Host, `out` a dict) and return out."""
    code = f"import sys, json; sys.path.insert(0, {ROOT!r})\nfrom tests.host_only import Host\nh = Host(); out = {{}}\n{body}\nprint('@' + json.dumps(out))"
    env = {**os.environ, "LD_PRELOAD": " ".join(x for x in (_fake(), os.environ.get("LD_PRELOAD")) if x)}
    r = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return json.loads([x for x in r.stdout.splitlines() if x.startswith("@")][-1][1:])


class Host:
    """In the child: one context, made-up device pointers, the stand-in's controls."""

    def __init__(self):
        from paper_2601_04370_amd import gwg
        import inputs
        self.gwg, self.inputs = gwg, inputs
        self.lib = gwg.load_library()
        self.fake = C.CDLL(None)
        self.fake.fake_log.restype = self.fake.fake_sizes.restype = self.fake.fake_asked.restype = C.c_char_p
        self.fake.fake_used.restype = C.c_size_t
        self.fake.fake_memory.argtypes, self.fake.fake_refuse.argtypes = [C.c_size_t], [C.c_size_t] * 2
        self.fake.fake_costs.argtypes = [C.c_double] * 3
        self.h = C.c_void_p()
        assert self.lib.gwg_create(C.byref(self.h), 0) == 0
        self.ptr = 4096                                      # stands for the caller's device arrays

    def scene(self, name="diff_1200", omega=None, fov=None, **kw):
        import numpy as np
        w = self.inputs.small_variant(name, **kw)
        inp = self.inputs.make_inputs(w)
        if fov is not None:
            inp["fov"] = np.asarray(fov, np.float64)
        return self.gwg.SceneSpec.from_workload(w, inp, omega=omega)

    def forward(self, sc, grad=False, memo=False, table=False, precision=0):
        g = self.gwg
        m, s, p, st, r = sc.structs()
        st.thk_nm = self.ptr
        eb = g.Eyebox(self.ptr, self.ptr, None, 24)
        flags = (g.GWG_FWD_GRAD if grad else 0) | (g.GWG_FWD_MEMO if memo else 0) | (g.GWG_FWD_TABLE if table else 0)
        return self.lib.gwg_trace_forward(self.h, C.byref(s), C.byref(p), C.byref(m), C.byref(st), C.byref(r), 1, 0,
                                          precision, flags, C.byref(eb), None, 1, None, None)

    def tmm(self, n_layers, silver, n, precision=0):
        import numpy as np
        g = self.gwg
        lam = np.array([450.0, 550.0, 650.0])
        n_re = np.tile([1.52, 1.46, 2.35, 0.12], (3, 1))
        n_im = np.tile([0.0, 0.0, 0.0, 3.3 if silver else 0.0], (3, 1))
        mat = (1 + np.arange(n_layers) % (3 if silver else 2)).astype(np.uint8)
        st = g.Stack(n_layers, self.ptr, g._np_ptr(mat, g._u8p), 0, 0)
        mt = g.Materials(*n_re.shape, *(g._np_ptr(x, g._dp) for x in (lam, n_re, n_im)))
        return self.lib.gwg_tmm_rt(self.h, C.byref(st), C.byref(mt), n, self.ptr, self.ptr, precision, self.ptr, None)

    def backward(self, stride=1):
        return self.lib.gwg_trace_backward(self.h, self.ptr, self.ptr, stride, None, None)

    def omega(self):
        return self.lib.gwg_omega_gradient(self.h, self.ptr, self.ptr, self.ptr, None)

    def autotune(self, sc, grad=False, memo=False):
        g = self.gwg
        m, s, p, st, r = sc.structs()
        st.thk_nm = self.ptr
        t = g.Tuning()
        rc = self.lib.gwg_autotune(self.h, C.byref(s), C.byref(p), C.byref(m), C.byref(st), C.byref(r), 1, 0,
                                   (g.GWG_FWD_GRAD if grad else 0) | (g.GWG_FWD_MEMO if memo else 0), None, C.byref(t), None)
        return rc, {k: getattr(t, k) for k, _ in g.Tuning._fields_}

    def tuning(self, **kw):
        t = self.gwg.Tuning(**kw)
        assert self.lib.gwg_set_tuning(self.h, C.byref(t)) == 0

    def kept(self):
        v = C.c_int32(0)
        assert self.lib.gwg_forward_kept_entries(self.h, C.byref(v)) == 0
        return v.value

    def error(self):
        return self.lib.gwg_last_error(self.h).decode()

    def log(self, clear=True):
        """Launches since the last call: [kernel, blocks, threads, {fields}], and "wait" lines."""
        lines = self.fake.fake_log().decode().splitlines()
        if clear:
            self.fake.fake_clear()
        rows = []
        for x in lines:
            f = x.split()
            if f[0] == "wait":
                rows.append(["wait", 0, 0, {}])
            else:
                rows.append([f[0], int(f[1]), int(f[2]), dict(k.split("=") for k in f[3:])])
        return rows

    def sizes(self):
        """Allocations asked for since the log was last cleared, bytes."""
        return [int(x) for x in self.fake.fake_sizes().split()]

    def asked(self):
        """Kernels whose occupancy was asked for."""
        return self.fake.fake_asked().decode().split()

    def kernels(self, name, clear=True):
        return [x for x in self.log(clear) if name in x[0]]
