"""Records what libptq would launch, without a GPU: a child process loads the library on top of a small stand-in for the HIP
runtime that notes every launch (kernel, grid, selected arguments) instead of executing it.  For host-side tests of
dispatch rules and of what the host does when a runtime call fails.

    record([("ptq_hessian_accumulate", [PTR, 4096, ...])], read={"hessian_bf16_big": {"chunk": (5, "i")}})

An argument is an int (passed as 64 bits) or a float; pointers are aligned numbers that nothing reads.
"""
from __future__ import annotations

import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2601_19675_amd", "libptq.so")
PTR = 1 << 20   # aligned, never read

_SHIM = r"""
#include <stddef.h>
#include <stdint.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static struct { const void* host; const char* name; } kernels[4096];
static int count;
static const char* failing = "";
static void (*on_launch)(const char*, unsigned, unsigned, unsigned, void**);
void recorder_set(void (*f)(const char*, unsigned, unsigned, unsigned, void**), const char* fail) { on_launch = f; failing = fail; }
static const char* name_of(const void* host) {
  for (int i = 0; i < count; ++i) if (kernels[i].host == host) return kernels[i].name;
  return "";
}
static dim3 grid_, block_; static size_t lds_; static void* stream_; static void* module;
void** __hipRegisterFatBinary(const void* d) { return &module; }
void __hipUnregisterFatBinary(void** m) {}
void __hipRegisterVar() {}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned n, void* a, void* b, void* c, void* d, int* e) {
  if (count < 4096) { kernels[count].host = host; kernels[count++].name = name; }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { grid_ = g; block_ = b; lds_ = s; stream_ = st; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = grid_; *b = block_; *s = lds_; *st = stream_; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t s, void* st) { on_launch(name_of(f), g.x, g.y, g.z, args); return 0; }
int hipLaunchCooperativeKernel(const void* f, dim3 g, dim3 b, void** args, unsigned s, void* st) { on_launch(name_of(f), g.x, g.y, g.z, args); return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return *failing && strstr(name_of(f), failing) ? 1 : 0; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = &module; return 0; }
int hipEventRecord(void* e, void* s) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = &module; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t s) { *n = 1; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned f) { *s = &module; return 0; }
int hipStreamWaitEvent(void* s, void* e, unsigned f) { return 0; }
"""


def record(calls, read=None, failing=""):
    """[(status, [{"kernel", "grid", **arguments}])] for every (function, arguments).  `read`: arguments to note,
    {part of a kernel's name: {key: (position, "i" for 32 bits or "q" for 64[, bytes into a struct argument])}}; `failing`: part of a kernel's name whose
    hipFuncSetAttribute fails."""
    if not os.path.exists(LIB):
        sys.path.insert(0, ROOT)
        from paper_2601_19675_amd import build
        build.build(verbose=False)
    with tempfile.TemporaryDirectory() as tmp:
        src, shim = os.path.join(tmp, "shim.c"), os.path.join(tmp, "shim.so")
        with open(src, "w") as f:
            f.write(_SHIM)
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", "-o", shim, src], check=True)
        job = json.dumps(dict(shim=shim, calls=calls, read=read or {}, failing=failing))
        r = subprocess.run([sys.executable, os.path.abspath(__file__)], input=job, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return json.loads(r.stdout)


def _child():
    import ctypes as c
    job = json.load(sys.stdin)
    shim = c.CDLL(job["shim"], mode=c.RTLD_GLOBAL)   # before the library: its symbols come first
    lib = c.CDLL(LIB)
    launches = []

    def on_launch(name, x, y, z, args):
        entry = dict(kernel=name.decode(), grid=[x, y, z])
        for part, wanted in job["read"].items():
            if part in entry["kernel"]:
                for key, (at, kind, *into) in wanted.items():
                    entry[key] = c.cast(args[at] + sum(into), c.POINTER(c.c_int32 if kind == "i" else c.c_int64))[0]
        launches.append(entry)

    callback = c.CFUNCTYPE(None, c.c_char_p, c.c_uint, c.c_uint, c.c_uint, c.POINTER(c.c_void_p))(on_launch)
    fail = job["failing"].encode()
    shim.recorder_set(callback, fail)
    out = []
    for name, args in job["calls"]:
        launches.clear()
        rc = getattr(lib, name)(*[c.c_double(a) if isinstance(a, float) else c.c_int64(a) for a in args])
        out.append((rc, list(launches)))
    print(json.dumps(out))


if __name__ == "__main__":
    _child()
