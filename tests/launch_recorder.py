"""Host paths of the library without a GPU: a small shared object takes the place of the HIP
runtime's calls (it is loaded with global symbols before the library, in a process of its own)
and writes down every kernel launch as (kernel, grid, workgroup, LDS bytes) instead of making
it.  Pointers are passed through untouched, so any numbers do for device memory."""
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
static struct { const void *host; char name[160]; } known[4096];
static int n_known;
static struct { int kernel; dim3_t grid, block; size_t lds; } log_[65536];
static int n_log;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void *cfg_stream;
static void (*on_copy)(void);

void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g)
{ (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned tl, void *a, void *b,
                           void *c, void *d, int *w)
{
    (void)m; (void)dev; (void)tl; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (n_known < 4096 && !strncmp(name, "_ZN2rd", 6)) { known[n_known].host = host; strncpy(known[n_known].name, name, 159); ++n_known; }
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void *s)
{ cfg_grid = g; cfg_block = b; cfg_lds = lds; cfg_stream = s; return 0; }
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *lds, void **s)
{ *g = cfg_grid; *b = cfg_block; *lds = cfg_lds; *s = cfg_stream; return 0; }
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t lds, void *s)
{
    int k = 0;
    (void)args; (void)s;
    while (k < n_known && known[k].host != f) ++k;
    if (n_log < 65536) {
        log_[n_log].kernel = k; log_[n_log].grid = g; log_[n_log].block = b; log_[n_log].lds = lds;
        ++n_log;
    }
    return 0;
}
int hipGetLastError(void) { return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipMemcpyAsync(void *d, const void *h, size_t n, int k, void *s)
{ (void)d; (void)h; (void)n; (void)k; (void)s; if (on_copy) on_copy(); return 0; }

void rec_on_copy(void (*f)(void)) { on_copy = f; }
void rec_clear(void) { n_log = 0; }
int rec_count(void) { return n_log; }
const char *rec_name(int i) { return log_[i].kernel < n_known ? known[log_[i].kernel].name : "?"; }
void rec_shape(int i, unsigned *v)
{
    v[0] = log_[i].grid.x; v[1] = log_[i].grid.y; v[2] = log_[i].grid.z;
    v[3] = log_[i].block.x; v[4] = (unsigned)log_[i].lds;
}
"""

PRELUDE = """
import ctypes, os, sys
sys.path.insert(0, {root!r})
rec = ctypes.CDLL({shim!r}, mode=ctypes.RTLD_GLOBAL)
rec.rec_name.restype = ctypes.c_char_p
import paper_2008_11486_amd as rd
L = rd.lib()
COPY = ctypes.CFUNCTYPE(None)

def launches():
    out = []
    for i in range(rec.rec_count()):
        v = (ctypes.c_uint * 5)()
        rec.rec_shape(i, v)
        out.append((rec.rec_name(i).decode(),) + tuple(v))
    rec.rec_clear()
    return out

def count(log, part):
    return sum(part in k[0] for k in log)
"""


def run(tmp_path, body):
    """body, Python source, after the prelude above in a fresh process; raises if it fails."""
    src, shim = os.path.join(str(tmp_path), "shim.c"), os.path.join(str(tmp_path), "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", shim, src], check=True)
    code = PRELUDE.format(root=ROOT, shim=shim) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
