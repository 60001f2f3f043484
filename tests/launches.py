"""What the library's host code launches, seen without a device: the HIP runtime's entry points that libtao.so calls are
answered by a small library of the test's own, which keeps each launch's kernel, grid, block and arguments."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RECORDER = r"""
#include <string.h>
typedef struct { unsigned x, y, z; } dim;
typedef struct { const char* kernel; unsigned grid, block; unsigned char bytes[4][256]; } launch;
static const void* known[4096]; static const char* names[4096]; static int kernels;
static dim next_grid, next_block; static unsigned long next_lds; static void* next_stream;
launch launches[256]; int nlaunches;
char watched_kernel[64];                                 /* of the kernels with this in their name: */
int watched[4] = {-1, -1, -1, -1}, watched_bytes[4];     /* which arguments are kept, and their sizes */
int cus = 256;
void** __hipRegisterFatBinary(const void* data) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void** h) {}
void __hipRegisterFunction(void** h, const void* host, char* device, const char* name, unsigned t, void* a, void* b, void* c, void* d, int* w) {
    known[kernels] = host; names[kernels++] = name;
}
void __hipRegisterVar(void** h, void* var, char* host, char* device, int ext, unsigned long size, int constant, int global) {}
int __hipPushCallConfiguration(dim g, dim b, unsigned long lds, void* st) { next_grid = g; next_block = b; next_lds = lds; next_stream = st; return 0; }
int __hipPopCallConfiguration(dim* g, dim* b, unsigned long* lds, void** st) { *g = next_grid; *b = next_block; *lds = next_lds; *st = next_stream; return 0; }
int hipLaunchKernel(const void* f, dim g, dim b, void** args, unsigned long lds, void* st) {
    launch* l = launches + nlaunches++ % 256;
    l->kernel = "";
    for (int i = 0; i < kernels; ++i) if (known[i] == f) l->kernel = names[i];
    l->grid = g.x; l->block = b.x;
    for (int i = 0; i < 4 && strstr(l->kernel, watched_kernel); ++i) if (watched[i] >= 0) memcpy(l->bytes[i], args[watched[i]], watched_bytes[i]);
    return 0;
}
int hipDeviceGetAttribute(int* v, int a, int dev) { *v = cus; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { return 1; }
int hipMemcpyAsync(void* d, const void* s, unsigned long n, int k, void* st) { return 1; }
int hipStreamSynchronize(void* st) { return 1; }
"""

DRIVER = r"""
import ctypes, json, subprocess, sys, types
sys.modules["torch"] = types.ModuleType("torch")            # (it would bring the real runtime, and find this one's entry points)
class Launch(ctypes.Structure):
    _fields_ = [("kernel", ctypes.c_char_p), ("grid", ctypes.c_uint), ("block", ctypes.c_uint), ("bytes", (ctypes.c_ubyte * 256) * 4)]
recorder = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)       # (found before the runtime's own)
import paper_2510_16028_amd as tao
lib = tao.lib()
_count = ctypes.c_int.in_dll(recorder, "nlaunches")
_launches = (Launch * 256).in_dll(recorder, "launches")
plain = {}
def watch(kernel, *arguments):
    # of the next launches of this kernel: the arguments (place, type) to keep
    (ctypes.c_char * 64).in_dll(recorder, "watched_kernel").value = kernel.encode()
    recorder.kept = [t for _, t in arguments]
    for i in range(4):
        at, t = arguments[i] if i < len(arguments) else (-1, ctypes.c_char)
        (ctypes.c_int * 4).in_dll(recorder, "watched")[i] = at
        (ctypes.c_int * 4).in_dll(recorder, "watched_bytes")[i] = ctypes.sizeof(t)
def launched():
    # (kernel, grid, block, arguments) since the last question
    assert _count.value <= 256
    out = [(l.kernel.decode(), l.grid, l.block, [t.from_buffer_copy(bytes(l.bytes[i][:ctypes.sizeof(t)])) for i, t in enumerate(recorder.kept)])
           for l in _launches[:_count.value]]
    _count.value = 0
    for l in out:
        if l[0] not in plain:
            n = subprocess.run(["c++filt", l[0]], capture_output=True, text=True, check=True).stdout
            plain[l[0]] = n.replace("(anonymous namespace)::", "").replace("tao::", "").replace("void ", "").split(">(")[0].split("(")[0]
    return [(plain[l[0]],) + l[1:] for l in out]
def address(n):
    # stands for device memory, which nothing here reads
    return ctypes.c_void_p(n)
watch("")
"""


def run(body, tmp_path):
    """What `body`, Python that calls `lib` and asks `launched()`, leaves in `result` (through JSON)."""
    src, so = os.path.join(str(tmp_path), "recorder.c"), os.path.join(str(tmp_path), "librecorder.so")
    with open(src, "w") as f:
        f.write(RECORDER)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", src, "-o", so], check=True)
    code = DRIVER + body + "\nprint(json.dumps(result))\n"
    out = subprocess.run([sys.executable, "-c", code, so], cwd=ROOT, check=True, capture_output=True, text=True).stdout
    return json.loads(out.splitlines()[-1])
