"""Host tests of the library's launches and workspace layout, without a GPU.

``scenario(module, name)`` runs ``module.name(Fake(...))`` in a fresh interpreter in
which the library is bound to tests/fake_hip.cpp instead of the HIP runtime.
"""
import ctypes as C
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


class Fake:
    def __init__(self, path):
        self.rt = C.CDLL(path, mode=C.RTLD_GLOBAL)
        self.rt.fake_name.restype = C.c_char_p
        self.rt.fake_blocks.restype = self.rt.fake_lds.restype = C.c_longlong
        self.rt.fake_memory_hash.restype = C.c_uint64
        from paper_2504_16446_amd import _lib
        self.lib = _lib.lib()
        self._keep = []

    def buffer(self, nbytes):
        """Zeroed memory, 256-byte aligned."""
        raw = C.create_string_buffer(nbytes + 256)
        self._keep.append(raw)
        return C.c_void_p((C.addressof(raw) + 255) & ~255)

    def create(self, og, model="trilinear", precision=0):
        from helpers import geometry_struct
        g, h = geometry_struct(og, precision), C.c_void_p()
        self._keep.append(og)
        self.ok("tt_create", C.byref(g), C.byref(h))
        self.ok("tt_set_projector", h, int(model == "joseph"))
        return h

    def ok(self, name, *args):
        rc = getattr(self.lib, name)(*args)
        assert rc >= 0, (name, rc, self.lib.tt_last_error())
        return rc

    def workspace(self, h, batch):
        n = self.ok("tt_workspace_bytes", h, batch)
        self.ok("tt_set_workspace", h, self.buffer(n), n)
        return n

    def sizes(self, h):
        out = (C.c_int64 * 8)()
        self.ok("tt_sizes", h, out)
        return list(out)

    def launches(self, call, *args):
        """Return code of a library call and the kernels that it launched: (name, blocks, LDS bytes)."""
        self.rt.fake_reset()
        rc = getattr(self.lib, call)(*args)
        n = self.rt.fake_launches()
        return rc, [(self.rt.fake_name(i).decode(), self.rt.fake_blocks(i), self.rt.fake_lds(i)) for i in range(n)]


_built = None


def scenario(module, name, *args):
    global _built
    if _built is None:
        _built = os.path.join(tempfile.mkdtemp(), "libfake_hip.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.cpp"), "-o", _built],
                       check=True)
    code = (f"import sys, json; sys.path[:0] = [{ROOT!r}, {HERE!r}]; import fake_hip; F = fake_hip.Fake({_built!r}); "
            f"import {module} as M; print('RESULT', json.dumps(M.{name}(F, *json.loads(sys.argv[1]))))")
    r = subprocess.run([sys.executable, "-c", code, json.dumps(args)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.split("RESULT ", 1)[1])
