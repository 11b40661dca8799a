"""Host programs that call the built library with HIP entry points of their own: nothing is launched, allocated or waited
for, and every stream that is created, destroyed or enqueued on and the name of every launched kernel is written down."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1801_04928_amd")

PROLOGUE = r"""
#include "lf.h"
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <string>
#include <vector>
typedef void* stream_t;
struct dim3 { unsigned x, y, z; };
static std::set<stream_t> used, live;
static int created;                                  // streams, events and pinned blocks
static void* pinned;                                 // the last of these
static bool no_pinned_memory;
static void* pinned_word;                            // the last that the device asked for
static bool capturing;
static uintptr_t next_handle = 0x1000;
static int caller_1, caller_2, caller_3;
static stream_t launch_stream;
static std::vector<std::string> launched;            // names of the kernels, in order
static std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> m; return m; }
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* p; return &p; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    kernels()[f] = name;
}
int __hipPushCallConfiguration(dim3, dim3, size_t, stream_t s) { launch_stream = s; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, stream_t* s) {
    *grid = *block = dim3{1, 1, 1}; *lds = 0; *s = launch_stream; return 0;
}
int hipStreamCreateWithFlags(stream_t* s, unsigned) { ++created; *s = (stream_t)(next_handle += 16); live.insert(*s); return 0; }
int hipStreamDestroy(stream_t s) { return live.erase(s) ? 0 : 1; }
int hipEventCreateWithFlags(void** e, unsigned) { ++created; *e = (void*)(next_handle += 16); return 0; }
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, stream_t s) { used.insert(s); return 0; }
int hipStreamWaitEvent(stream_t s, void*, unsigned) { used.insert(s); return 0; }
int hipStreamIsCapturing(stream_t, int* status) { *status = capturing ? 1 : 0; return 0; }
int hipStreamSynchronize(stream_t) { return 0; }
int hipLaunchKernel(const void* f, dim3, dim3, void**, size_t, stream_t s) {
    used.insert(s);
    launched.push_back(kernels()[f]);
    return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, stream_t s) { used.insert(s); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)0x100000; return 0; }
int hipHostMalloc(void** p, size_t n, unsigned) { if (no_pinned_memory) return 2; ++created; *p = pinned = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = pinned_word = h; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 0; return 0; }
}
static int failures;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); ++failures; } } while (0)
// A net of these widths; nothing reads or writes its buffers, which are addresses only.
static lf_net* make(const std::vector<int>& n, int B, lf_dtype dt, lf_sched sched) {
    const int L = (int)n.size();
    uintptr_t next = 0x100000000;
    auto buffer = [&]() { return (void*)(next += 0x100000000); };
    lf_net* net = nullptr;
    const size_t bytes = lf_workspace_bytes_widths(L, n.data(), B, dt);
    CHECK(lf_create_widths(&net, L, n.data(), B, dt, LF_COST_QUADRATIC, buffer(), bytes) == LF_OK);
    std::vector<const void*> w, b;
    std::vector<float*> gw, gb;
    for (int i = 0; i < L - 1; ++i) {
        w.push_back(buffer()); b.push_back(buffer());
        gw.push_back((float*)buffer()); gb.push_back((float*)buffer());
    }
    CHECK(lf_set_params(net, w.data(), b.data()) == LF_OK);
    CHECK(lf_set_grad_buffers(net, gw.data(), gb.data()) == LF_OK);
    CHECK(lf_set_schedule(net, sched) == LF_OK);
    return net;
}
static void* const some_input = (void*)0x1000000;
"""


def build(directory, main):
    """The program of this main function; a path."""
    src, exe = os.path.join(str(directory), "program.cpp"), os.path.join(str(directory), "program")
    with open(src, "w") as f:
        f.write(PROLOGUE + main)
    # (the executable's symbols come before the runtime's)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", exe, src,
                    os.path.join(LIB_DIR, "liblf.so"), f"-Wl,-rpath,{LIB_DIR}", "-Wl,--allow-shlib-undefined"], check=True)
    return exe


def run(exe, *args, **env):
    """Output of the program; the library's tuning overrides are those of `env` alone."""
    base = {n: v for n, v in os.environ.items() if not n.startswith("LF_")}
    out = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, env={**base, **env}, timeout=120)
    assert out.returncode == 0, out.stdout[-3000:] + out.stderr[-3000:]
    return out.stdout
