"""What a call of the library launches, without a GPU: the built library on the stand-ins of launch_recorder.cpp, in a
process of its own.  Pointers are made-up addresses that nothing reads."""
import ctypes
import json
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2310_12109_amd", "libmonarch.so")
DTYPES = {"f32": 0, "bf16": 1, "f16": 2}
GAP = 1 << 38   # between made-up tensors, more than any of them holds


def build(folder):
    so = os.path.join(folder, "launch_recorder.so")
    # (the name under which the library looks for rocBLAS: it finds this object, already loaded)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-Wl,-soname,librocblas.so", os.path.join(HERE, "launch_recorder.cpp"),
                    "-o", so, "-lpthread"], check=True)
    return so


def record(so, script):
    """Runs `script` (Python source; it finds Calls as `calls` and leaves its answer in `result`) and returns the answer."""
    out = subprocess.run([sys.executable, __file__, so], input=script, capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-4000:]
    return json.loads(out.stdout.splitlines()[-1])


def plain(mangled):
    at, name = 3, ""                       # _ZN <length><name> ... [I <arguments> E] E
    while mangled[at].isdigit():
        digits = re.match(r"\d+", mangled[at:]).group()
        at += len(digits) + int(digits)
        name = mangled[at - int(digits):at]
    arguments = mangled[at:].split("EEv")[0] + "E" if mangled[at] == "I" else ""
    return " ".join([name] + re.findall(r"L[ib](\d+)E", arguments))


class Calls:
    def __init__(self, so):
        self.rec = ctypes.CDLL(so, mode=ctypes.RTLD_GLOBAL)
        self.rec.recorder_line.restype = ctypes.c_char_p
        self.rec.recorder_built.restype = ctypes.c_char_p
        self.lib = ctypes.CDLL(LIB)
        self.lib.monarch_last_error.restype = ctypes.c_char_p
        self.lib.monarch_hyena_heads_layer_workspace_bytes.restype = ctypes.c_size_t

    def compute_units(self, n):
        self.rec.recorder_compute_units(n)

    def built(self):
        """Every kernel of the library, as kernels() names them."""
        return [plain(self.rec.recorder_built(i).decode()) for i in range(self.rec.recorder_built_count())]

    def log(self):
        lines = [self.rec.recorder_line(i).decode().split("\t") for i in range(self.rec.recorder_count())]
        self.rec.recorder_reset()
        return lines

    def kernels(self):
        """The kernels launched since the last look: name and whole-number (or truth) template arguments, as in "conv256_bf16_kernel 1 1 0"."""
        return [plain(line[1]) for line in self.log() if line[0] == "kernel"]

    def conv(self, B, H, n, klen, factors, dtype="bf16", causal=0, gates=3, static=False, stream=0):
        nfft = 1
        for f in factors:
            nfft *= f
        u, k, g_in, g_out, y, ws = (ctypes.c_void_p(GAP * i) for i in range(1, 7))
        args = [u, k, g_in if gates & 1 else None, g_out if gates & 2 else None, y, B, H, n, klen, nfft,
                (ctypes.c_int * len(factors))(*factors), len(factors), causal, DTYPES[dtype]]
        if static:
            rc = self.lib.monarch_causal_conv_static(*args, ctypes.c_void_p(stream))
        else:
            rc = self.lib.monarch_causal_conv(*args, ws, ctypes.c_size_t(GAP), ctypes.c_void_p(stream))
        assert rc == 0, (self.lib.monarch_last_error(), B, H, n, klen, factors, dtype)
        return self.kernels()

    def fft(self, rows, factors, dtype="bf16", real=1, inverse=0):
        nfft = 1
        for f in factors:
            nfft *= f
        call = self.lib.monarch_ifft if inverse else self.lib.monarch_fft
        rc = call(ctypes.c_void_p(GAP), ctypes.c_void_p(2 * GAP), ctypes.c_int64(rows), nfft, (ctypes.c_int * len(factors))(*factors), len(factors),
                  real, DTYPES[dtype], ctypes.c_void_p(3 * GAP), ctypes.c_size_t(GAP - 1), None)
        assert rc == 0, (self.lib.monarch_last_error(), rows, factors, dtype)
        return self.kernels()

    def hyena(self, B, n, d, taps, klen, factors, head_dim, dtype, base=GAP, gap=GAP, stream=0):
        nfft = 1
        for f in factors:
            nfft *= f
        fs = (ctypes.c_int * len(factors))(*factors)
        ws_bytes = self.lib.monarch_hyena_heads_layer_workspace_bytes(B, n, d, klen, nfft, fs, len(factors), head_dim, DTYPES[dtype])
        p = [ctypes.c_void_p(base + gap * i) for i in range(9)]   # u, W_in, b_in, k_short, k_long, W_out, b_out, y, ws
        rc = self.lib.monarch_hyena_heads_layer(*p[:8], B, n, d, taps, klen, nfft, fs, len(factors), 1, head_dim, DTYPES[dtype], p[8],
                                                ctypes.c_size_t(ws_bytes), ctypes.c_void_p(stream))
        assert rc == 0, self.lib.monarch_last_error()
        return ws_bytes


if __name__ == "__main__":
    scope = {"calls": Calls(sys.argv[1]), "GAP": GAP}
    exec(compile(sys.stdin.read(), "script", "exec"), scope)
    print(json.dumps(scope["result"]))
