"""The library on a stand-in HIP runtime (hip_stand_in.c): its host code runs, its launches are only
recorded.  Each test runs in a process of its own, since the library binds to the runtime it finds."""
import ctypes as C
import functools
import os
import subprocess
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class StandIn:
    def __init__(self, lib_path):
        self.lib = C.CDLL(lib_path, mode=C.RTLD_GLOBAL)
        sys.modules.setdefault("torch", types.ModuleType("torch"))   # only its runtime would be wanted
        sys.path.insert(0, ROOT)
        import paper_2506_17506_amd as vl
        self.vl = vl
        self.launches = []   # (kernel, grid, block, LDS bytes, stream, arguments as words)
        kind = C.CFUNCTYPE(None, C.c_char_p, C.c_uint32, C.c_uint32, C.c_uint32, C.c_uint32, C.c_size_t, C.c_void_p, C.POINTER(C.c_void_p))

        def on_launch(name, gx, gy, gz, bx, lds, stream, args):
            self.on_launch(name.decode(), (gx, gy, gz), bx, lds, stream, args)
        self._keep = kind(on_launch)
        vl.load()
        self.lib.stand_in_on_launch(self._keep)

    def on_launch(self, name, grid, block, lds, stream, args):
        """kernels are told apart by the part of their mangled name"""
        words = []
        if "k_summarize" in name:   # its fourth and sixth arguments
            words = [C.cast(args[k], C.POINTER(C.c_uint64))[0] for k in (3, 5)]
        elif "k_walk" in name:       # its job table
            words = [C.cast(args[1], C.POINTER(C.c_uint64))[0]]
        self.launches.append((name, grid, block, lds, stream, words))

    def fail_allocation(self, after, more=0):
        self.lib.stand_in_fail(after, more)

    def counts(self):
        out = (C.c_uint64 * 6)()
        self.lib.stand_in_counts(out)
        return dict(zip(("mallocs", "frees", "uploads", "stream_waits", "device_waits", "largest"), out))


def in_own_process(test):
    """runs test(stand_in) of the module in a fresh interpreter"""
    @functools.wraps(test)
    def outer(tmp_path):
        so = str(tmp_path / "hip_stand_in.so")
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, os.path.join(HERE, "hip_stand_in.c")], check=True)
        code = (f"import sys; sys.path.insert(0, {HERE!r}); import stand_in; s = stand_in.StandIn({so!r}); "
                f"import {test.__module__.split('.')[-1]} as m; m.{test.__name__}.inner(s); print('passed')")
        r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0 and "passed" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
    del outer.__wrapped__   # (its argument is not a fixture)
    outer.inner = test
    return outer
