"""What the library would launch, without a GPU: a subprocess in which a few functions of the HIP runtime are replaced by ones
that write down each launch and refuse a grid that the hardware's launch packet cannot hold (2^32 threads or more in a
dimension).  The pointers that the calls are given are never followed."""
import json
import os
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r'''
#include <stddef.h>
typedef struct { unsigned x, y, z; } dim3;
static dim3 grid, block;
static size_t shared;
static void *stream;
static int last;
static unsigned log_[64][6];
static const void *kernel_[64];
static unsigned shared_[64];
static int count;
void launched(int at, const void *f, void **args) __attribute__((weak));   /* of `also` */
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, void *s) { grid = g; block = b; shared = sh; stream = s; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, void **s) { *g = grid; *b = block; *sh = shared; *s = stream; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t sh, void *s)
{
    const unsigned long long limit = 1ull << 32;
    if ((unsigned long long)g.x * b.x >= limit || (unsigned long long)g.y * b.y >= limit || (unsigned long long)g.z * b.z >= limit ||
        (unsigned long long)b.x * b.y * b.z > 1024 || !g.x || !g.y || !g.z)
        return last = 9;   /* hipErrorInvalidConfiguration */
    if (count < 64) {
        const unsigned v[6] = {g.x, g.y, g.z, b.x, b.y, b.z};
        for (int i = 0; i < 6; ++i) log_[count][i] = v[i];
        kernel_[count] = f;
        shared_[count] = (unsigned)sh;
        if (launched) launched(count, f, args);
    }
    ++count;
    return 0;
}
int hipGetLastError(void) { const int e = last; last = 0; return e; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int recorded(unsigned *out)
{
    const int n = count < 64 ? count : 64;
    for (int i = 0; i < n; ++i) for (int k = 0; k < 6; ++k) out[i * 6 + k] = log_[i][k];
    count = 0;
    return n;
}
'''

PRELUDE = r'''
import ctypes as C, json, sys
rec = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)      # ahead of the HIP runtime in the order in which symbols are found
sys.path.insert(0, sys.argv[2])
import paper_2111_11124_amd as M
L = M.lib()
P = 0x10000                                        # an aligned address
def launches():
    out = (C.c_uint * (64 * 6))()
    n = rec.recorded(out)
    return [tuple(out[i * 6:i * 6 + 6]) for i in range(n)]
def kernels():
    """(name, template arguments as they are mangled, workgroups, threads of one, dynamic LDS) per launch, with NAMES"""
    import math, re
    rec.recorded_kernel.restype = C.c_char_p
    names = [(rec.recorded_kernel(i).decode(), rec.recorded_shared(i)) for i in range(64)]
    return [(*parts(mangled), math.prod(k[:3]), math.prod(k[3:]), lds) for k, (mangled, lds) in zip(launches(), names)]
def parts(mangled):
    import re
    n = re.match(r"_ZN4mesa(\d+)", mangled)
    at = n.end() + int(n.group(1))
    return mangled[n.end():at], mangled[at + 1:mangled.index("EEv", at)] if mangled[at] == "I" else ""
def all_kernels():
    """(name, template arguments) of every kernel in the library, with NAMES"""
    rec.known_kernel.restype = C.c_char_p
    out = []
    while rec.known_kernel(len(out)): out.append(rec.known_kernel(len(out)).decode())
    return [parts(m) for m in out]
def report(x): print("REPORT " + json.dumps(x))
'''


# for `also`: the kernels' names, which the library hands to the runtime as it is loaded (kept from it here: nothing is launched)
NAMES = r'''
#include <stdlib.h>
#include <string.h>
static struct { const void *f; char *name; } *known;
static int known_n;
void __hipRegisterFunction(void **modules, const void *f, char *device, const char *name, unsigned limit, void *a, void *b, void *c, void *d, int *e)
{
    if (strncmp(name, "_ZN4mesa", 8)) return;
    known = realloc(known, (known_n + 1) * sizeof(*known));
    known[known_n].f = f;
    known[known_n++].name = strdup(name);
}
const char *recorded_kernel(int i)
{
    for (int k = 0; k < known_n; ++k) if (known[k].f == kernel_[i]) return known[k].name;
    return "";
}
unsigned recorded_shared(int i) { return shared_[i]; }
const char *known_kernel(int i) { return i < known_n ? known[i].name : 0; }
'''

# for `also`: the device and its scratch array, for calls that ask the runtime where the library's own array lies
ONE_DEVICE = r'''
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { *p = (void *)0x100000; return 0; }
'''


def run(body, also=""):
    """What `body` hands to report(), run after PRELUDE; `also`: further functions of the runtime, in C."""
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "recorder.so")
        open(os.path.join(d, "recorder.c"), "w").write(SOURCE + also)
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", os.path.join(d, "recorder.c"), "-o", so], check=True)
        out = subprocess.run([sys.executable, "-c", PRELUDE + body, so, ROOT], capture_output=True, text=True, timeout=600)
        assert out.returncode == 0, out.stderr[-3000:]
        return json.loads([l for l in out.stdout.splitlines() if l.startswith("REPORT ")][-1][7:])
