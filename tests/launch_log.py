"""Which kernels a call of the C ABI enqueues, read on the host: a small library that takes the place of hipLaunchKernel notes each launch
by the name its kernel was registered with, and enqueues nothing (or forwards to the runtime up to a launch that it lets fail).

As a program, `python launch_log.py SHIM LIBRARY` reads JSON lines {entry, G, K, N, S, A, C, workspace} from its input and prints for each
the return code and the launches' mangled names; pointers are made up and never followed."""
import ctypes
import json
import os
import re
import subprocess
import sys

SHIM = r"""
#include <dlfcn.h>
#include <cstddef>
#include <cstdint>
#include <map>
#include <string>
struct dim { uint32_t x, y, z; };
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> n; return n; }
static std::string log_;
static int fail_at = -1, forward = 0, count = 0;
static void *real(const char *name) {
    static void *lib = dlopen("libamdhip64.so.7", RTLD_NOW | RTLD_LOCAL);
    return lib ? dlsym(lib, name) : nullptr;
}
extern "C" {
void launch_log_start(int fail, int fwd) { log_.clear(); count = 0; fail_at = fail; forward = fwd; }
const char *launch_log() { return log_.c_str(); }
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid,
                           void *block, void *grid, int *size) {
    names()[host] = name;
    typedef void (*F)(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *);
    if (F f = reinterpret_cast<F>(real("__hipRegisterFunction"))) f(modules, host, device, name, limit, tid, bid, block, grid, size);
}
int hipLaunchKernel(const void *host, dim grid, dim block, void **args, size_t lds, void *stream) {
    log_ += names()[host] + "\n";
    if (count++ == fail_at) return 1;                         // hipErrorInvalidValue
    typedef int (*F)(const void *, dim, dim, void **, size_t, void *);
    return forward ? reinterpret_cast<F>(real("hipLaunchKernel"))(host, grid, block, args, lds, stream) : 0;
}
int hipFuncSetAttribute(const void *host, int attribute, int value) {
    typedef int (*F)(const void *, int, int);
    return forward ? reinterpret_cast<F>(real("hipFuncSetAttribute"))(host, attribute, value) : 0;
}
}
"""


def build_shim(folder):
    from paper_2109_09868_amd import build

    src, out = os.path.join(folder, "launch_log.cpp"), os.path.join(folder, "liblaunch_log.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run([build.host_compiler(), "-O1", "-std=c++17", "-fPIC", "-shared", src, "-o", out, "-ldl"], check=True)
    return out


def library_path():
    from paper_2109_09868_amd import binding

    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.LIB_PATH


def launches(folder, calls):
    """[(return code, [mangled kernel name, ..]), ..] for calls {entry, G, K, N, S, A, C, workspace}."""
    r = subprocess.run([sys.executable, os.path.abspath(__file__), build_shim(str(folder)), library_path()], text=True,
                       input="".join(json.dumps(c) + "\n" for c in calls), capture_output=True, timeout=100)
    assert r.returncode == 0, r.stderr
    got = [json.loads(line) for line in r.stdout.splitlines()]
    assert len(got) == len(calls)
    return [(rc, names) for rc, names in got]


def pairs_tile(name):
    """(MT, TQ, S, mode, Algorithm 1) of a decode_byzantine_pairs_kernel, else None."""
    m = re.search(r"decode_byzantine_pairs_kernelILi(\d+)ELi(\d+)ELi(\d+)ELNS_8PairModeE(\d)ELb(\d)E", name)
    return tuple(int(v) for v in m.groups()) if m else None


def open_library(shim, path):
    """(library whose launches go through the shim, shim); before anything else has loaded the library."""
    log = ctypes.CDLL(shim, mode=ctypes.RTLD_GLOBAL)
    log.launch_log.restype = ctypes.c_char_p
    lib = ctypes.CDLL(path)
    dp = ctypes.POINTER(ctypes.c_double)
    i, q, p = ctypes.c_int, ctypes.c_int64, ctypes.c_void_p
    lib.approxifer_chebyshev_nodes.argtypes = [i, i, dp, dp]
    lib.approxifer_workspace_bytes.argtypes = [q, i, i, i, i, q]
    lib.approxifer_workspace_bytes.restype = ctypes.c_size_t
    for name in ("approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"):
        getattr(lib, name).argtypes = [p, p, p, p, p, q, i, i, i, i, q, dp, dp, i, p, ctypes.c_size_t, p]
    lib.approxifer_decode_byzantine_static.argtypes = [p, p, p, p, p, q, i, i, i, i, q, dp, dp, i, p]
    return lib, log


def _main():
    lib, log = open_library(sys.argv[1], sys.argv[2])
    at = ctypes.c_void_p(1 << 20)
    for line in sys.stdin:
        c = json.loads(line)
        K, N = c["K"], c["N"]
        alpha, beta = (ctypes.c_double * K)(), (ctypes.c_double * N)()
        lib.approxifer_chebyshev_nodes(K, N, alpha, beta)
        need = lib.approxifer_workspace_bytes(c["G"], K, N, c["S"], c["A"], c["C"]) if c["workspace"] else 0
        log.launch_log_start(-1, 0)
        scratch = () if c["entry"].endswith("_static") else (at if need else None, need)
        rc = getattr(lib, c["entry"])(at, at, at, at, at, c["G"], K, N, c["S"], c["A"], c["C"], alpha, beta, 1, *scratch, None)
        print(json.dumps([rc, log.launch_log().decode().split()]))


if __name__ == "__main__":
    _main()
