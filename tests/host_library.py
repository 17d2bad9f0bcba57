"""The library's host code on a runtime that records launches instead of making them: every call's
dispatch (which kernels, how many launches, their grids and LDS) can be checked without a GPU.

All sources are compiled for the host only and linked with the few runtime entry points they use;
pointers are never followed, so any address serves as device memory."""
import ctypes
import os
import re
import subprocess
from collections import namedtuple
from concurrent.futures import ThreadPoolExecutor

from paper_2511_15369_amd import build as lib_build

RUNTIME = r"""
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <map>
#include <string>
#include <vector>
struct dim3 { uint32_t x, y, z; };
struct Launch { std::string name; uint32_t grid, block; size_t lds; uint32_t first_word; };
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static std::vector<Launch> launches;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    int status = 0;
    char *s = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    names()[host] = s ? s : name;
    free(s);
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3, dim3, size_t, void *) { return 0; }
int __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, void **) { return 0; }
int hipGetLastError() { return 0; }
int hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t lds, void *)
{
    uint32_t word;
    memcpy(&word, args[0], 4);
    launches.push_back({names()[kernel], grid.x, block.x, lds, word});
    return 0;
}
void recorded_clear() { launches.clear(); }
int recorded_count() { return (int)launches.size(); }
const char *recorded(int i, uint32_t *grid, uint32_t *block, uint64_t *lds, uint32_t *first_word)
{
    const Launch &l = launches[i];
    *grid = l.grid; *block = l.block; *lds = l.lds; *first_word = l.first_word;
    return l.name.c_str();
}
}
"""

# (problems: how many a batch's table holds, which its arguments begin with; 1 where the kernel takes one problem's)
Launch = namedtuple("Launch", "kernel arguments grid block lds first_word problems")


def build(folder, replaced=None):
    """The recording library as a ctypes object.  `replaced`: {source file: text compiled in its place}."""
    replaced = replaced or {}
    runtime = os.path.join(folder, "runtime.cpp")
    with open(runtime, "w") as f:
        f.write(RUNTIME)

    def one(src):
        path = os.path.join(lib_build.CSRC, src)
        if src in replaced:
            path = os.path.join(folder, src)
            with open(path, "w") as f:
                f.write(replaced[src])
        obj = os.path.join(folder, src + ".o")
        # (an index past the end of an array traps)
        subprocess.check_call(["hipcc", "-x", "hip", "-c", "--cuda-host-only", "--offload-arch=gfx950", "-O1", "-std=c++17", "-fPIC",
                               "-I" + lib_build.CSRC, "-Xarch_host", "-fsanitize=bounds", "-Xarch_host", "-fsanitize-trap=bounds",
                               path, "-o", obj], stderr=subprocess.DEVNULL)
        return obj

    # (the debug hooks launch kernels and copy memory themselves)
    sources = [s for s in lib_build.SOURCES if s != "debug_hooks.hip"]
    with ThreadPoolExecutor(max_workers=8) as ex:
        objs = list(ex.map(one, sources))
    lib = os.path.join(folder, "libiptq_recording.so")
    # the device code that each object would register: there is none
    symbols = subprocess.check_output(["nm", "-u"] + objs, text=True).split()
    absent = ["-Wl,--defsym=%s=0" % s for s in symbols if s.startswith("__hip_fatbin")]
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", runtime] + objs + absent + ["-o", lib])
    so = ctypes.CDLL(lib)
    so.recorded.restype = ctypes.c_char_p
    return so


def launches(so, call):
    """The launches that `call()` makes (it returns the library's code, which must be 0)."""
    so.recorded_clear()
    assert call() == 0
    out = []
    for i in range(so.recorded_count()):
        grid, block, word, lds = ctypes.c_uint32(), ctypes.c_uint32(), ctypes.c_uint32(), ctypes.c_uint64()
        name = so.recorded(i, ctypes.byref(grid), ctypes.byref(block), ctypes.byref(lds), ctypes.byref(word)).decode()
        m = re.search(r"iptq::(\w+)(?:<([^>]*)>)?", name)
        args = tuple(int(a) if a.lstrip("-").isdigit() else a for a in re.split(r",\s*", m.group(2))) if m.group(2) else ()
        table = "batch" in m.group(1) or any("Batch" in a for a in args if isinstance(a, str))
        out.append(Launch(m.group(1), args, grid.value, block.value, lds.value, word.value, word.value if table else 1))
    return out
