"""What the library enqueues for a call, without a GPU: a stand-in for the HIP runtime notes the launches and can refuse a request.

`record(calls, ...)` runs the calls in a process of its own, in which the stand-in is loaded before the library (one gfx950 device
with 256 CUs; "device memory" is host memory that nothing reads), and returns [{"rc", "launches": [{"kernel", "grid", "block"}]}]."""
import ctypes
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2405_05329_amd", "libkvra.so")

STAND_IN = r"""
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <dlfcn.h>
struct Dim { unsigned x, y, z; };
struct Launch { char name[512]; unsigned grid[3], block[3]; };
static Launch launches[64];
static int n_launches, n_attributes, n_mallocs;
static int refuse_launch, refuse_attribute, refuse_malloc;   // the how-manieth is refused (0: none)
extern "C" {
void recorder_reset(int launch, int attribute, int malloc_) {
  n_launches = n_attributes = n_mallocs = 0;
  refuse_launch = launch; refuse_attribute = attribute; refuse_malloc = malloc_;
}
int recorder_count() { return n_launches; }
const Launch* recorder_launch(int i) { return launches + i; }

int hipLaunchKernel(const void* f, Dim grid, Dim block, void**, size_t, void*) {
  if (n_launches + 1 == refuse_launch || n_launches == 64) return 1;
  Launch& l = launches[n_launches++];
  Dl_info info;
  const char* const symbol = dladdr(f, &info) && info.dli_saddr == f && info.dli_sname ? info.dli_sname : "?";
  int status = 0;
  char* const text = abi::__cxa_demangle(symbol, nullptr, nullptr, &status);
  strncpy(l.name, text ? text : symbol, sizeof(l.name) - 1);
  free(text);
  l.grid[0] = grid.x; l.grid[1] = grid.y; l.grid[2] = grid.z;
  l.block[0] = block.x; l.block[1] = block.y; l.block[2] = block.z;
  return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return ++n_attributes == refuse_attribute ? 1 : 0; }
int hipMalloc(void** p, size_t bytes) { return ++n_mallocs == refuse_malloc ? 2 : (*p = malloc(bytes)) ? 0 : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipMemset(void*, int, size_t) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipStreamGetDevice(void*, int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }   // (the number of CUs is the only one asked for)
int hipStreamIsCapturing(void*, int* status) { *status = 0; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void**, const void*) { return 1; }
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, Dim*, Dim*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
"""


def linear(m, n, k, mode="plain"):
    return {"fn": "linear", "m": m, "n": n, "k": k, "mode": mode}


def layer(hidden, ffn, H, Hkv, d, prefix, m, rope_base=10000.0):
    return {"fn": "layer", "hidden": hidden, "ffn": ffn, "H": H, "Hkv": Hkv, "d": d, "prefix": prefix, "m": m, "rope_base": rope_base}


_stand_in = {}


def _built():
    if not _stand_in:
        tmp = _stand_in["folder"] = tempfile.TemporaryDirectory()   # goes with the process
        src, _stand_in["so"] = os.path.join(tmp.name, "stand_in.cpp"), os.path.join(tmp.name, "stand_in.so")
        with open(src, "w") as f:
            f.write(STAND_IN)
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", src, "-o", _stand_in["so"], "-ldl"], check=True)
    return _stand_in["so"]


def record(calls, refuse_launch=0, refuse_attribute=0, refuse_malloc=0):
    job = {"so": _built(), "calls": calls, "refuse": [refuse_launch, refuse_attribute, refuse_malloc]}
    r = subprocess.run([sys.executable, os.path.abspath(__file__)], input=json.dumps(job), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout)


def _serve():
    job = json.load(sys.stdin)
    i64, i32, f32, vp = ctypes.c_int64, ctypes.c_int, ctypes.c_float, ctypes.c_void_p
    rec = ctypes.CDLL(job["so"], mode=ctypes.RTLD_GLOBAL)
    lib = ctypes.CDLL(LIB)

    class Launch(ctypes.Structure):
        _fields_ = [("name", ctypes.c_char * 512), ("grid", ctypes.c_uint * 3), ("block", ctypes.c_uint * 3)]

    class Layer(ctypes.Structure):
        _fields_ = [(n, i32) for n in ("hidden", "ffn", "H", "Hkv", "d")] + \
                   [(n, f32) for n in ("eps", "rope_base", "scale")] + [("w%d" % i, vp) for i in range(7)]

    rec.recorder_launch.restype = ctypes.POINTER(Launch)
    lib.kvra_linear.argtypes = [vp] * 5 + [i64] * 3 + [vp]
    lib.kvra_layer_chunk.argtypes = [ctypes.POINTER(Layer)] + [vp] * 4 + [i64] * 3 + [vp, i64, vp]
    P, out = 1 << 20, []   # (addresses are never read)
    for c in job["calls"]:
        rec.recorder_reset(*job["refuse"])
        if c["fn"] == "linear":
            rc = lib.kvra_linear(P, P, P if c["mode"] == "swiglu" else None, P if c["mode"] == "residual" else None, P,
                                 c["m"], c["n"], c["k"], None)
        else:
            lay = Layer(c["hidden"], c["ffn"], c["H"], c["Hkv"], c["d"], 1e-6, c["rope_base"], c["d"] ** -0.5, *[P] * 7)
            rc = lib.kvra_layer_chunk(lay, P, P, P, P, c["prefix"], c["m"], c["prefix"] + c["m"], P, 1 << 40, None)
        launches = []
        for i in range(rec.recorder_count()):
            la = rec.recorder_launch(i).contents
            launches.append({"kernel": la.name.decode(), "grid": list(la.grid), "block": list(la.block)})
        out.append({"rc": rc, "launches": launches})
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _serve()
