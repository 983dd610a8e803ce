"""libtr.so on a model of the HIP runtime (hip_model.cpp), for tests of the
library's host side where there is no GPU.  load() replaces the runtime for the
whole process, so each test runs in a process of its own (run)."""
import ctypes as C
import os
import subprocess
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
SRC = os.path.join(HERE, "hip_model.cpp")
LIB = os.path.join(HERE, "libhip_model.so")


def build():
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < os.path.getmtime(SRC):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-o", tmp, SRC, "-lpthread"])
        os.replace(tmp, LIB)


def run(module, test):
    """Run the module's function of that name in a new process."""
    build()
    code = "import sys; sys.path[:0] = [%r, %r]; import hip_model, %s as m; m.%s(*hip_model.load())" % (
        ROOT, os.path.join(ROOT, "tests"), module, test)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, "exit %d\n%s%s" % (r.returncode, r.stdout[-2000:], r.stderr[-4000:])


def load():
    """The model and the package, whose library then binds to the model."""
    model = C.CDLL(LIB, mode=C.RTLD_GLOBAL)
    for f, res in (("model_used", C.c_size_t), ("model_races", C.c_long), ("model_launches", C.c_long),
                   ("model_bad_waits", C.c_long), ("model_misuse", C.c_long), ("model_frees", C.c_long),
                   ("model_mallocs", C.c_long), ("model_staged_changed", C.c_long), ("model_pending", C.c_long)):
        getattr(model, f).restype = res
    model.model_capacity.argtypes = [C.c_int, C.c_size_t]
    model.model_radius.argtypes = [C.c_double]
    model.model_capture.argtypes = [C.c_void_p, C.c_int]
    torch = sys.modules["torch"] = types.ModuleType("torch")  # (the binding loads it first)
    torch.cuda = types.SimpleNamespace(is_available=lambda: True,
                                       current_stream=lambda: types.SimpleNamespace(cuda_stream=None))
    import paper_0801_1500_amd as tr
    tr.lib()
    return model, tr


def launches(model):
    """Launches so far as (kernel, grid, block)."""
    out, buf = [], C.create_string_buffer(4096)
    while model.model_log(len(out), buf, len(buf)) >= 0:
        name, g, b = buf.value.decode().rsplit(" ", 2)
        out.append((name, int(g), int(b)))
    return out
