"""The library on a recording stand-in of the HIP runtime (hip_stub.cpp): its host
side, validation, plans, workspace sizes and launches, without a GPU.  A process of
its own loads the stand-in before the library; `python host_stub.py` of a snippet
is what `run()` starts."""
import ctypes as C
import os
import subprocess
import sys
import types

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
FAKE = 4096  # a device address: nothing dereferences it


def run(snippet, tmp_path):
    """Runs `snippet` in a process whose library uses the stand-in; `h` is this module."""
    so = os.path.join(str(tmp_path), "hip_stub.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    os.path.join(HERE, "hip_stub.cpp"), "-o", so], check=True)
    r = subprocess.run([sys.executable, os.path.abspath(__file__), so, snippet], capture_output=True, text=True,
                       cwd=ROOT, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]
    return r.stdout


def config(hidden, nq, ffn, vocab=151936, fuse=5, layers=1, dtype=1, nkv=8, head_dim=128):
    import paper_2605_29707_amd.binding as bd
    return bd.domino_config(hidden=hidden, n_layers=layers, n_q_heads=nq, n_kv_heads=nkv, head_dim=head_dim, ffn=ffn,
                            vocab=vocab, block=16, gru_hidden=1024, rank=256, mask_token_id=vocab - 1, rms_eps=1e-6,
                            rope_theta=1e6, dtype=dtype, ctx_fuse_layers=fuse)


SHAPES = {"4b": (2560, 32, 9728), "8b": (4096, 32, 12288), "32b": (5120, 64, 25600)}


class Model:
    def __init__(self, cfg):
        import paper_2605_29707_amd.binding as bd
        self.lib, self.h = bd.load(), C.c_void_p()
        arr = C.cast((C.c_void_p * cfg.n_layers)(*[FAKE] * cfg.n_layers), C.POINTER(C.c_void_p))
        w = bd.domino_weights(**{n: (arr if t is bd._PP else FAKE) for n, t in bd.domino_weights._fields_})
        st = self.lib.domino_model_create(C.byref(cfg), C.byref(w), C.byref(self.h))
        assert st == 0, bd.last_error()

    def ws(self, batch, max_ctx, max_new, branch=1):
        return self.lib.domino_workspace_bytes(self.h, batch, max_ctx, max_new, branch)

    def train_ws(self, batch, max_ctx, max_new):
        return self.lib.domino_train_workspace_bytes(self.h, batch, max_ctx, max_new)

    def step(self, batch, max_ctx, n_new, nbytes, branch=1, stream=0):
        return self.lib.domino_draft_step(self.h, batch, FAKE, FAKE, FAKE, FAKE, max_ctx, FAKE if n_new else None, n_new,
                                          branch, None, FAKE, FAKE, None, FAKE, nbytes, stream)

    def train(self, batch, max_ctx, n_new, nbytes, stream=0):
        return self.lib.domino_train_forward(self.h, batch, FAKE, FAKE, FAKE, FAKE, max_ctx, FAKE if n_new else None,
                                             n_new, FAKE, 0.5, 15.0, FAKE, None, None, FAKE, nbytes, stream)

    def paths(self):
        v = C.c_uint32(0)
        assert self.lib.domino_debug_last_paths(self.h, C.byref(v)) == 0
        return v.value


def _main():
    global stub, log
    so, snippet = sys.argv[1:]
    sys.path.insert(0, ROOT)
    stub = C.CDLL(so, mode=C.RTLD_GLOBAL)
    stub.stub_log.restype = C.c_char_p
    stub.stub_fail.argtypes = [C.c_char_p, C.c_int]
    stub.stub_capture.argtypes = [C.c_void_p, C.c_int]

    def log():
        """The calls recorded since the last log(), as lists of words."""
        out = [line.split() for line in stub.stub_log().decode().splitlines()]
        stub.stub_clear()
        return out

    h = types.SimpleNamespace(**globals())
    h.stub, h.log = stub, log
    exec(snippet, {"h": h, "C": C})


if __name__ == "__main__":
    _main()
