"""The kernels a library call enqueues, listed on the CPU.

A child process puts stand-ins for the HIP runtime's launch entry points
(compiled here with g++) before the runtime in the symbol search order, loads
libeat.so and makes calls with fake addresses that nothing reads.  The
stand-ins note each kernel's demangled name and its grid and launch nothing, so
the list shows what the host code decided.
"""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#include <cxxabi.h>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
struct D3 { uint32_t x, y, z; };
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static std::string& log_() { static std::string s; return s; }
static struct { D3 g, b; size_t shmem; void* stream; } cfg;
static int token;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h = &token; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    names()[f] = st == 0 && d ? d : name;
    free(d);
}
int __hipPushCallConfiguration(D3 g, D3 b, size_t shmem, void* stream) { cfg = {g, b, shmem, stream}; return 0; }
int __hipPopCallConfiguration(D3* g, D3* b, size_t* shmem, void** stream) {
    *g = cfg.g; *b = cfg.b; *shmem = cfg.shmem; *stream = cfg.stream;
    return 0;
}
int hipLaunchKernel(const void* f, D3 g, D3 b, void**, size_t, void*) {
    char at[96];
    snprintf(at, sizeof at, "\t%u\t%u\t%u\t%u\n", g.x, g.y, g.z, b.x * b.y * b.z);
    log_() += names()[f] + at;
    return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int attr, int) { *v = attr == stub_xccs_attr ? 8 : 256; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 1; return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(uintptr_t{1} << 20); return 0; }
int hipEventRecord(void*, void*) { return 0; }
const char* stub_take() { static std::string out; out.swap(log_()); log_().clear(); return out.c_str(); }
}
"""

CHILD = r"""
import ctypes as C, json, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)        # first in the search order
sys.path.insert(0, sys.argv[2])
from paper_2609_33614_amd import _lib as L
stub.stub_take.restype = C.c_char_p
F = 1 << 20
out = []
for call in json.load(sys.stdin):
    kind = call.pop("kind")
    T = call.pop("T")
    if kind == "ppl":
        n = L.eat_ppl_workspace_size(T, call["d"], call["V"])
        L.eat_ppl_trend(F, T, call["d"], F, call["V"], F, F, F, F, F, None, F, n, stream=0)
    else:
        p = L.eat_params_default(**call)
        h = L.eat_create(p, T)
        ws = F if p.d_shared else None
        acc = L.accounts(F, F, F)
        n = L.eat_workspace_size(h, T)
        if kind == "forward":
            L.eat_moe_forward(h, F, T, F, F, F, F, ws, ws, ws, acc, None, F, None, F, F, n, stream=0)
        elif kind == "noalloc":
            L.eat_moe_forward_noalloc(h, F, T, F, F, F, F, ws, ws, ws, acc, None, F, None, F, stream=0)
        elif kind == "stack":
            arr = L.stack_layers([L.eat_stack_layer_t(h, F, F, F, F, ws, ws, ws, F, acc)] * 2)
            n = L.eat_stack_workspace_size(arr, 2, T)
            L.eat_stack_forward(arr, 2, F, T, None, 1e-6, F, None, None, F, n, stream=0)
        L.eat_destroy(h)
    rows = [l.split("\t") for l in stub.stub_take().decode().splitlines()]
    out.append({"bytes": n, "kernels": [[r[0], [int(v) for v in r[1:]]] for r in rows]})
print("LAUNCHES " + json.dumps(out))
"""


def list_launches(tmp_path, calls):
    """For each call -- {"kind": "forward" | "noalloc" | "stack", "T": tokens,
    **eat_params_default overrides} or {"kind": "ppl", "T": sequences, "d", "V"} --
    its workspace bytes and its kernels [name, [grid x, y, z, threads]] in
    launch order."""
    hdr = open("/opt/rocm/include/hip/hip_runtime_api.h").read()
    src, probe, lib = (str(tmp_path / n) for n in ("stub.cpp", "probe.cpp", "libstub.so"))
    assert "hipDeviceAttributeNumberOfXccs" in hdr
    open(probe, "w").write("#include <hip/hip_runtime_api.h>\n#include <cstdio>\n"
                           "int main() { printf(\"%d\", (int)hipDeviceAttributeNumberOfXccs); }\n")
    subprocess.run(["g++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", probe, "-o", probe + ".x"], check=True)
    xccs = subprocess.run([probe + ".x"], check=True, capture_output=True, text=True).stdout
    open(src, "w").write(STUB.replace("stub_xccs_attr", xccs))
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", src, "-o", lib], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, lib, ROOT], input=json.dumps(calls), capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    line = [l for l in r.stdout.splitlines() if l.startswith("LAUNCHES ")]
    assert len(line) == 1, r.stdout[-2000:]
    return json.loads(line[0][len("LAUNCHES "):])
