"""The library's calls with the kernel launches stubbed out: host tests see which kernels a call launches, with no GPU and no pointer
followed."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = """
#include <stddef.h>
typedef struct { unsigned x, y, z; } grid3;
static struct { const void* f; const char* name; } known[4096];
static int n_known, n_launched;
static const char* launched[4096];
void __hipRegisterFunction(void** module, const void* f, char* stub, const char* name, unsigned limit, void* t, void* b, void* bd, void* gd, int* size) {
  if (n_known < 4096) { known[n_known].f = f; known[n_known++].name = name; }
}
int __hipPushCallConfiguration(grid3 g, grid3 b, size_t lds, void* stream) { return 0; }
int __hipPopCallConfiguration(grid3* g, grid3* b, size_t* lds, void** stream) { return 0; }
int hipLaunchKernel(const void* f, grid3 g, grid3 b, void** args, size_t lds, void* stream) {
  int i = 0;
  while (i < n_known && known[i].f != f) ++i;
  if (n_launched < 4096) launched[n_launched++] = i < n_known ? known[i].name : "?";
  return 0;
}
int stub_launched(void) { int n = n_launched; n_launched = 0; return n; }
const char* stub_name(int i) { return launched[i]; }
int hipFuncSetAttribute(const void* f, int attribute, int value) { return 0; }
int hipGetLastError(void) { return 0; }
"""

PROLOGUE = """
import ctypes, random, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # before the library, whose references then go to it
stub.stub_name.restype = ctypes.c_char_p
from paper_2401_10652_amd import binding as B, inputs as I
L = B.lib()
X, Y, W = 1 << 40, 1 << 41, 1 << 42                           # "device" addresses

def kernels():
    return [stub.stub_name(i).decode() for i in range(stub.stub_launched())]
"""


def build(folder):
    source, lib = os.path.join(folder, "stub.c"), os.path.join(folder, "stub.so")
    with open(source, "w") as f:
        f.write(SOURCE)
    subprocess.run(["cc", "-shared", "-fPIC", "-o", lib, source], check=True)
    return lib


def run(lib, code):
    """`code` in a process of its own, behind PROLOGUE."""
    r = subprocess.run([sys.executable, "-c", PROLOGUE + code, lib], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout
