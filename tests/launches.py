"""Which kernels a call of the library launches, found without a GPU: the library runs in a process of its own on a HIP runtime
that only writes down what it is asked to do.  Pointers are never followed (their alignment is looked at)."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RUNTIME = r"""
#include <cxxabi.h>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
struct dim3 { unsigned x, y, z; };
static std::map<const void *, std::string> names;
static std::string log_;
static int refuse_ = 0;
static dim3 grid_, block_;
static size_t shmem_;
static void *stream_;
extern "C" {
void *__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void *) {}
void __hipRegisterVar(void *, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void *, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    int st;
    char *d = abi::__cxa_demangle(device, nullptr, nullptr, &st);
    names[host] = st == 0 ? d : device;
    std::free(d);
}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void *st) { grid_ = g; block_ = b; shmem_ = s; stream_ = st; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *s, void **st) { *g = grid_; *b = block_; *s = shmem_; *st = stream_; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, void *)
{
    char t[128];
    std::snprintf(t, sizeof t, "\t%u\t%u\t%u\t%u\n", g.x, g.y, g.z, b.x);
    log_ += names[f] + t;
    return 0;
}
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = (void *)0x7000; return 0; }
int hipMallocAsync(void **p, size_t n, void *)
{
    if (refuse_) return 2;
    log_ += "alloc\t" + std::to_string(n) + "\n";
    *p = (void *)0x9000;
    return 0;
}
int hipFreeAsync(void *, void *) { return 0; }
const char *launches() { return log_.c_str(); }
void forget() { log_.clear(); }
void refuse(int on) { refuse_ = on; }
}
"""
CHILD = r"""
import ctypes, json, sys
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rt.launches.restype = ctypes.c_char_p
lib = ctypes.CDLL(sys.argv[2])
out = []
for name, args, refuse in json.load(sys.stdin):
    rt.forget()
    rt.refuse(refuse)
    status = getattr(lib, name)(*[ctypes.c_int64(a) for a in args])
    out.append((status, rt.launches().decode().splitlines()))
json.dump(out, sys.stdout)
"""


def build(folder):
    src, so = os.path.join(folder, "runtime.cpp"), os.path.join(folder, "runtime.so")
    with open(src, "w") as f:
        f.write(RUNTIME)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", src, "-o", so])
    return so


def trace(runtime, calls):
    """calls: (function, integer arguments, whether the memory pool refuses).  Returns per call its status and a list of
    (kernel name, template arguments, grid, threads), or ("alloc", bytes) for scratch memory."""
    lib = os.path.join(ROOT, "paper_2310_10537_amd", "libmx.so")
    r = subprocess.run([sys.executable, "-c", CHILD, runtime, lib], input=json.dumps(calls), capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    out = []
    for status, lines in json.loads(r.stdout):
        seen = []
        for line in lines:
            name, *numbers = line.split("\t")
            if name == "alloc":
                seen.append(("alloc", int(numbers[0])))
                continue
            head = name.replace("(anonymous namespace)::", "").split("(")[0].removeprefix("void ").split("<", 1)
            args = tuple(a.strip() for a in head[1].rstrip(">").split(",")) if len(head) > 1 else ()
            g = tuple(int(v) for v in numbers)
            seen.append((head[0].split("::")[-1], args, g[:3], g[3]))
        out.append((status, seen))
    return out
