"""An engine whose HIP runtime is hip_stub.c: what the library's host side does - states, copies, which kernels it launches -
without a GPU.  Only for a process of its own (the stub's symbols are global): tests run scripts through run_script."""
import ctypes as C
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

OPS = ("launch", "copy", "sync", "record", "wait", "stream_create", "event_create")


class GemmArgs(C.Structure):
    """The beginning of a GEMM launch's argument: what it fetches ahead (the next launch's matrix, its workgroups and column
    groups), its operands and sizes; S shares of K."""
    _fields_ = [("nx_base", C.c_void_p), ("nx_nwg", C.c_int), ("nx_ncg", C.c_int), ("nx_span", C.c_int), ("nx_block_bytes", C.c_longlong),
                ("nx_split_bytes", C.c_longlong), ("nx_narrow_nb", C.c_int), ("nx_Z", C.c_int), ("nx_nblk", C.c_int), ("nx_pairs", C.c_int),
                ("kv_fetch_bytes", C.c_int), ("W", C.c_void_p), ("Xhi", C.c_void_p), ("Xlo", C.c_void_p), ("part", C.c_void_p),
                ("counters", C.c_void_p), ("N", C.c_int), ("KS", C.c_int), ("S", C.c_int), ("rows_total", C.c_int)]


def run_script(tmp_path, text):
    """Runs the script in a process without torch; returns what it prints."""
    lib = os.path.join(str(tmp_path), "libhipstub.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", lib, os.path.join(HERE, "hip_stub.c")], check=True)
    head = f"import sys\nsys.path[:0] = [{ROOT!r}, {HERE!r}]\nfrom host_engine import *\nHostEngine.open({lib!r})\n"
    res = subprocess.run([sys.executable, "-c", head + text], capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert res.returncode == 0, res.stdout + res.stderr
    return res.stdout


class HostEngine:
    """Caller's buffers in host memory and a context over them."""
    stub = lib = None

    @classmethod
    def open(cls, stub_path):
        cls.stub = C.CDLL(stub_path, mode=C.RTLD_GLOBAL)
        cls.stub.stub_launch.restype = C.c_char_p
        cls.stub.stub_launch_arg.restype = C.POINTER(GemmArgs)
        from paper_2512_15176_amd import binding
        cls.binding, cls.lib = binding, binding.load_library()

    def __init__(self, target, drafter, max_batch, max_seq, max_k=32):
        import mmap
        b = self.binding
        self.max_batch = max_batch
        p = b.init_params(target, drafter, max_batch, max_seq, max_k, target.vocab - 1)
        s = b.query_sizes(p)
        buf = lambda n: mmap.mmap(-1, int(n))   # noqa: E731  (pages come when they are touched)
        self._mem = [buf(n) for n in (*s.weights, *s.kv, s.workspace)]
        at = [C.addressof(C.c_char.from_buffer(m)) for m in self._mem]
        bufs = b.Buffers((C.c_void_p * 2)(*at[:2]), (C.c_void_p * 2)(*at[2:4]), at[4])
        self.ctx = C.c_void_p()
        rc = self.lib.deer_init_models(C.byref(p), C.byref(bufs), C.byref(s), C.byref(self.ctx))
        assert rc == 0, self.lib.deer_last_error(None)
        self._draft = (C.c_int32 * (max_batch * 32))()

    def prefill(self, prompts):
        ids = [t for p in prompts for t in p]
        return self.lib.deer_prefill(self.ctx, len(prompts), (C.c_int32 * len(ids))(*ids), (C.c_int32 * len(prompts))(*map(len, prompts)))

    def set_prefilled(self, lens, last):
        return self.lib.deer_set_prefilled(self.ctx, len(lens), (C.c_int32 * len(lens))(*lens), (C.c_int32 * len(last))(*last))

    def draft_block(self, k, T=0.0):
        return self.lib.deer_draft_block(self.ctx, k, T, 0, self._draft)

    def verify_block(self, k, T=0.0):
        return self.lib.deer_verify_block(self.ctx, k, T, self._draft)

    def launches(self):
        """(kernel name without its arguments, grid) of what was launched since the last stub_reset."""
        out = []
        for i in range(self.stub.stub_launches()):
            g = (C.c_uint32 * 3)()
            out.append((self.stub.stub_launch(i, g).decode(), tuple(g)))
        return out

    def gemms(self):
        """(kernel name, grid, arguments) of the GEMM launches among them."""
        return [(n, g, self.stub.stub_launch_arg(i).contents) for i, (n, g) in enumerate(self.launches()) if "8GemmArgs" in n]

    def ops(self):
        """(kind, stream, what) in the order of the calls since the last stub_reset: kernels (with the residual rows of the
        pass they begin, else None), copies to the device (with their destination), waits of the host, events recorded and
        waited for on a stream."""
        out = []
        for i in range(self.stub.stub_ops()):
            stream, what = C.c_void_p(), C.c_void_p()
            kind = OPS[self.stub.stub_op(i, C.byref(stream), C.byref(what))]
            out.append((kind, stream.value, what.value))
        return out
