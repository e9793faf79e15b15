"""A stand-in for the HIP runtime: the library's host code runs on it in a child process without a GPU.  Kernels are launched nowhere; their
names and grids are kept, memory is counted against a limit, and a launch can be made to fail.  Device memory is 16 bytes an allocation, so
nothing may look behind a pointer."""
import json
import os
import subprocess
import sys

import paper_2505_11564_amd as hf

RUNTIME = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3;
static const void* fn[1024]; static const char* fn_name[1024]; static int n_fn;
static dim3 c_grid, c_block; static size_t c_shm; static void* c_st;
static int last_error, fail_at; static char fail_name[64];
static size_t used, limit = (size_t)1 << 60, total = (size_t)1 << 60, free_said;
static struct { void* p; size_t n; } held[4096]; static int n_held;
static char* text; static size_t text_n, text_cap;
static void say(const char* a, const char* b, size_t x, size_t y) {
  char line[512];
  int k = snprintf(line, sizeof line, "%s %s %zu %zu\n", a, b, x, y);
  if (text_n + k + 1 > text_cap) { text_cap = 2 * (text_cap + k + 4096); text = realloc(text, text_cap); }
  memcpy(text + text_n, line, k + 1);
  text_n += k;
}
/* for the test */
const char* standin_log(void) { return text ? text : ""; }
void standin_clear(void) { text_n = 0; if (text) text[0] = 0; }
void standin_limit(size_t n) { limit = total = n; }
size_t standin_used(void) { return used; }
/* what is free by its own account, until 0 is said: a program beside this one may take it in between */
void standin_free(size_t n) { free_said = n; }
/* the nth launch from now of a kernel whose name has `name` in it fails */
void standin_fail(const char* name, int nth) { strncpy(fail_name, name, 63); fail_at = nth; }

void** __hipRegisterFatBinary(const void* d) { static void* h; return &h; }
void __hipUnregisterFatBinary(void** m) {}
void __hipRegisterVar(void** m, void* v, char* h, char* d, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void** m, const void* host, char* dev, const char* name, unsigned lim, void* a, void* b, void* c, void* d, int* w) {
  if (n_fn < 1024) { fn[n_fn] = host; fn_name[n_fn++] = name; }
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void* st) { c_grid = g; c_block = b; c_shm = s; c_st = st; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** st) { *g = c_grid; *b = c_block; *s = c_shm; *st = c_st; return 0; }
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t s, void* st) {
  const char* name = "?";
  for (int i = 0; i < n_fn; ++i) if (fn[i] == f) name = fn_name[i];
  if (fail_at > 0 && strstr(name, fail_name) && --fail_at == 0) { last_error = 719; say("failed", name, g.x, g.y); return last_error; }
  say("launch", name, g.x, g.y * (size_t)g.z);
  return 0;
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
const char* hipGetErrorString(int e) { return "stand-in error"; }
int hipSetDevice(int d) { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }
int hipMemGetInfo(size_t* f, size_t* t) { *f = free_said ? free_said : limit - used; *t = total; return 0; }
int hipMalloc(void** p, size_t n) {
  if (used + n > limit || n_held == 4096) { last_error = 2; say("refused", "-", n, used); return 2; }
  *p = aligned_alloc(256, 256);
  held[n_held].p = *p; held[n_held++].n = n; used += n;
  say("malloc", "-", n, used);
  return 0;
}
int hipFree(void* p) {
  for (int i = 0; i < n_held; ++i) if (held[i].p == p) { used -= held[i].n; say("free", "-", held[i].n, used); held[i] = held[--n_held]; break; }
  free(p);
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned f) { *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { return 0; }
int hipMemcpy2DAsync(void* d, size_t dp, const void* s, size_t sp, size_t w, size_t h, int k, void* st) { return 0; }
int hipStreamSynchronize(void* st) { return 0; }
int hipDeviceSynchronize(void) { return 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { *e = malloc(1); return 0; }
int hipEventDestroy(void* e) { free(e); return 0; }
int hipEventRecord(void* e, void* st) { return 0; }
int hipEventSynchronize(void* e) { return 0; }
int hipGetSymbolAddress(void** p, const void* s) { *p = 0; return 1; }
"""

CHILD = r"""
import ctypes as C, json, sys
S = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the real runtime in the order of symbols
L = C.CDLL(sys.argv[2])
S.standin_log.restype = C.c_char_p
S.standin_limit.argtypes = S.standin_free.argtypes = [C.c_size_t]
S.standin_used.restype = C.c_size_t
S.standin_fail.argtypes = [C.c_char_p, C.c_int]
vp, i32 = C.c_void_p, C.c_int32
L.hf_create.argtypes = [vp, i32, i32, i32, C.POINTER(vp)]
L.hf_destroy.argtypes = [vp]
L.hf_last_error.argtypes, L.hf_last_error.restype = [vp], C.c_char_p
L.hf_workspace_bytes.argtypes, L.hf_workspace_bytes.restype = [vp], C.c_int64
L.hf_num_params.argtypes, L.hf_num_params.restype = [vp], C.c_int64
L.hf_hvp.argtypes = [vp, vp, vp, vp, i32, i32, vp, vp, vp, vp]
L.hf_hvp_accumulate.argtypes = [vp, vp, vp, vp, i32, i32, i32, vp, vp, vp, vp]
L.hf_hessian_column.argtypes = [vp, vp, vp, vp, i32, i32, C.c_int64, vp, vp, vp]
def create(desc, batch, max_m=0):
    d = C.create_string_buffer(bytes.fromhex(desc))
    c = vp()
    rc = L.hf_create(C.addressof(d), 0, batch, max_m, C.byref(c))
    return rc, c
P, X, Y, V, OUT = (0x10000 * (i + 1) for i in range(5))  # parameters, tokens, labels, direction, result
def hvp(c, batch, seq):
    # HF_EINVAL with "no valid label" is a product that was enqueued to its end: the count of labels that it reads back stays zero here
    return L.hf_hvp(c, P, X, Y, batch, seq, V, OUT, None, None), L.hf_last_error(c).decode()
def log():
    out = [l.split() for l in S.standin_log().decode().split("\n")[:-1]]
    S.standin_clear()
    return out
"""

ENQUEUED = [-1, "no valid label in the batch"]


def run(tmp_path, script, **given):
    """Runs `script` behind CHILD with the names `given`; returns what it prints as JSON with show()."""
    src, lib = tmp_path / "standin.c", tmp_path / "standin.so"
    if not lib.exists():
        src.write_text(RUNTIME)
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    code = CHILD + "def show(x): print('SHOW' + json.dumps(x), flush=True)\n" + "globals().update(json.loads(sys.argv[3]))\n" + script
    r = subprocess.run([sys.executable, "-c", code, str(lib), hf.binding.LIB_PATH, json.dumps(given)], capture_output=True, text=True,
                       timeout=300, cwd=os.path.dirname(hf.binding.LIB_PATH))
    assert r.returncode == 0, r.stderr[-2000:]
    return [json.loads(l[4:]) for l in r.stdout.split("\n") if l.startswith("SHOW")][-1]


def desc(model, dtype="bf16", basis="f32"):
    return bytes(hf.make_desc(model, dtype, basis)).hex()


def kernels(log):
    """(name, x, y * z) of the launches of a log, in order."""
    return [(l[1], int(l[2]), int(l[3])) for l in log if l[0] == "launch"]
