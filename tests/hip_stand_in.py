"""A stand-in for the HIP calls that the library's host code makes in a save or
a launch, for tests of that code on the CPU.  Loaded with RTLD_GLOBAL before
the library (in a child process of its own), its functions are found before
the HIP runtime's: copies are done at once and counted, events are always
ready, and launches are noted and not made."""
import os
import shutil
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dims;
static int copies, launches;
static unsigned shape[64][4]; /* grid x, y, z and threads of the launches noted */
int stand_in_copies(void) { const int n = copies; copies = 0; return n; }
int stand_in_launches(unsigned *out)
{
    const int n = launches;
    memcpy(out, shape, sizeof shape);
    launches = 0;
    return n;
}
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *stream)
{
    (void)kind;
    (void)stream;
    memcpy(dst, src, n);
    ++copies; /* the saver copies under its lock */
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned flags)
{
    (void)flags;
    *p = aligned_alloc(4096, (n + 4095) / 4096 * 4096);
    return *p ? 0 : 2;
}
int hipHostFree(void *p) { free(p); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; *e = &copies; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *stream) { (void)e; (void)stream; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipGetLastError(void) { return 0; }
/* a launch: <<<>>> pushes its configuration, the kernel's stub takes it back and launches */
static struct { dims grid, block; size_t lds; void *stream; } pushed;
int __hipPushCallConfiguration(dims grid, dims block, size_t lds, void *stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dims *grid, dims *block, size_t *lds, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *f, dims grid, dims block, void **args, size_t lds, void *stream)
{
    (void)f;
    (void)args;
    (void)lds;
    (void)stream;
    if (launches < 64) {
        unsigned *s = shape[launches++];
        s[0] = grid.x; s[1] = grid.y; s[2] = grid.z; s[3] = block.x * block.y * block.z;
    }
    return 0;
}
"""

# the start of a child's program: `stand_in`, `ss` (the binding), `launches()`
PRELUDE = r"""
import ctypes, json, sys
stand_in = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import numpy as np
from paper_2509_24626_amd import binding as ss
def launches():
    out = np.zeros((64, 4), np.uint32)
    return out[:stand_in.stand_in_launches(out.ctypes.data_as(ctypes.c_void_p))].tolist()
"""


def build(folder):
    """Compiles the stand-in into `folder`; its path, or None without gcc."""
    cc = shutil.which("gcc")
    if cc is None:
        return None
    src, lib = os.path.join(str(folder), "hip.c"), os.path.join(str(folder), "hip.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    subprocess.run([cc, "-std=c11", "-O1", "-shared", "-fPIC", "-Wall", "-Werror", src, "-o", lib], check=True)
    return lib


def run(lib, program, *args):
    """The last line that `program` (after PRELUDE) prints, in a child process."""
    r = subprocess.run([sys.executable, "-c", PRELUDE + program, lib, *args], cwd=ROOT, capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout.splitlines()[-1]
