"""What a context asks of the HIP runtime for its pinned result slots, on a stand-in runtime without a GPU (the seven calls that
creating and destroying a context makes): the memory is coherent, since the host reads what kernels stored there after waiting
for an event only; contexts beyond the shared block's 64 slots pin their own and give it back."""
import os
import subprocess
import sys

import paper_2505_11564_amd as hf
import synth_inputs as si

RUNTIME = r"""
#include <stdio.h>
#include <stdlib.h>
int hipSetDevice(int d) { return 0; }
int hipGetLastError(void) { return 0; }
int hipMalloc(void** p, size_t n) { *p = malloc(16); return 0; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t n, unsigned flags) { *p = malloc(n); printf("pin %u\n", flags); fflush(stdout); return 0; }
int hipHostFree(void* p) { free(p); printf("unpin\n"); fflush(stdout); return 0; }
"""

CHILD = r"""
import ctypes as C, sys
C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)  # ahead of the real runtime in the order of symbols
L = C.CDLL(sys.argv[2])
L.hf_create.argtypes = [C.c_void_p, C.c_int32, C.c_int32, C.c_int32, C.POINTER(C.c_void_p)]
L.hf_destroy.argtypes = [C.c_void_p]
desc = C.create_string_buffer(bytes.fromhex(sys.argv[3]))
def create():
    c = C.c_void_p()
    assert L.hf_create(C.addressof(desc), 0, 4, 3, C.byref(c)) == 0
    return c
held = [create() for _ in range(65)]   # one more than the shared block has slots
L.hf_destroy(held.pop())               # its own memory
L.hf_destroy(held.pop(5))              # a slot
held.append(create())                  # which serves again
"""


def test_result_slots_are_coherent_and_given_back(tmp_path):
    src, lib = tmp_path / "runtime.c", tmp_path / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-o", str(lib), str(src)], check=True)
    desc = bytes(hf.make_desc(si.CONFIGS["mlp_tiny"]["model"])).hex()
    r = subprocess.run([sys.executable, "-c", CHILD, str(lib), hf.binding.LIB_PATH, desc], capture_output=True, text=True,
                       timeout=120, cwd=os.path.dirname(hf.binding.LIB_PATH))
    assert r.returncode == 0, r.stderr[-2000:]
    lines = r.stdout.split("\n")[:-1]
    pins = [int(x.split()[1]) for x in lines if x.startswith("pin ")]
    assert [x.split()[0] for x in lines] == ["pin", "pin", "unpin"]   # the block, the 65th context's own, and that one back
    coherent = 0x40000000  # hipHostMallocCoherent
    assert pins and all(f == 0 or f & coherent for f in pins)  # 0: the default, which is coherent
