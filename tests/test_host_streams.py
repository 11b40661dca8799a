"""Which streams a pass uses, from the HIP calls the library makes: a host program loads the built library with HIP
entry points of its own, which do nothing but write down every stream that is created, destroyed or enqueued on.  Two
handles have no worker stream in common (one whose caller's stream is held up cannot hold up the other), a pass that
has run once with its k creates nothing when it runs again (also where that second pass is being captured), and a
handle destroys what it has created."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1801_04928_amd")

PROGRAM = r"""
#include "lf.h"
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>
typedef void* stream_t;
struct dim3 { unsigned x, y, z; };
static std::set<stream_t> used, live;
static int created;                                  // streams, events and pinned blocks
static bool capturing;
static uintptr_t next_handle = 0x1000;
static int caller_1, caller_2;
static stream_t launch_stream;
extern "C" {
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
int hipLaunchKernel(const void*, dim3, dim3, void**, size_t, stream_t s) { used.insert(s); return 0; }
int hipMemcpyAsync(void*, const void*, size_t, int, stream_t s) { used.insert(s); return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "error"; }
int hipGetSymbolAddress(void**, const void*) { return 1; }
int hipHostMalloc(void** p, size_t n, unsigned) { ++created; *p = calloc(1, n); return 0; }
int hipHostFree(void* p) { free(p); return 0; }
int hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 0; return 0; }
}
static const int L = 6;
static int failures;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); ++failures; } } while (0)
static lf_net* make(int N, int B, lf_dtype dt) {
    const size_t bytes = lf_workspace_bytes(L, N, B, dt);
    lf_net* net = nullptr;
    CHECK(lf_create(&net, L, N, B, dt, LF_COST_QUADRATIC, aligned_alloc(256, (bytes + 255) / 256 * 256), bytes) == LF_OK);
    const void* w[L - 1]; const void* b[L - 1]; float* gw[L - 1]; float* gb[L - 1];
    for (int i = 0; i < L - 1; ++i) {
        gw[i] = (float*)aligned_alloc(256, (size_t)4 * N * N); w[i] = gw[i];
        gb[i] = (float*)aligned_alloc(256, (size_t)4 * N); b[i] = gb[i];
    }
    CHECK(lf_set_params(net, w, b) == LF_OK);
    CHECK(lf_set_grad_buffers(net, gw, gb) == LF_OK);
    CHECK(lf_set_schedule(net, LF_SCHED_STREAMS) == LF_OK);
    return net;
}
static std::set<stream_t> pass(lf_net* net, int k, void* stream) {
    static void* data = aligned_alloc(256, 1 << 20);
    used.clear();
    CHECK(lf_forward(net, data, stream) == LF_OK);
    CHECK(lf_backward_leapfrog(net, data, k, stream) == LF_OK);
    return used;
}
int main(int argc, char** argv) {
    const int B = std::atoi(argv[1]), k = std::atoi(argv[3]);
    const lf_dtype dt = argv[2][0] == 'b' ? LF_BF16 : LF_F32;
    const size_t workers = (size_t)std::atoi(argv[4]);
    lf_net* a = make(64, B, dt);
    lf_net* b = make(64, B, dt);
    const std::set<stream_t> first = pass(a, k, &caller_1), other = pass(b, k, &caller_2);
    CHECK(first.size() == 1 + workers && other.size() == 1 + workers);
    for (stream_t s : first) CHECK(!other.count(s));
    // the same pass again, and recorded into a graph: launches, event records and event waits only
    const int before = created;
    CHECK(pass(a, k, &caller_1) == first);
    CHECK(created == before);
    capturing = true;
    const std::set<stream_t> captured = pass(a, k, &caller_1);
    capturing = false;
    CHECK(created == before);
    for (stream_t s : captured) CHECK(!other.count(s));
    lf_destroy(a);
    for (stream_t s : other) CHECK(s == &caller_2 || live.count(s));
    CHECK(pass(b, k, &caller_2) == other);
    lf_destroy(b);
    CHECK(live.empty());
    std::printf("%d failures\n", failures);
    return failures != 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("streams")
    src, exe = tmp / "streams.cpp", tmp / "streams"
    # (the registration of the device code stays the runtime's)
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-rdynamic", "-I", os.path.join(ROOT, "include"), "-o", str(exe), str(src),
                    os.path.join(LIB_DIR, "liblf.so"), f"-Wl,-rpath,{LIB_DIR}", "-Wl,--allow-shlib-undefined"], check=True)
    return str(exe)


@pytest.mark.parametrize("B,dtype,k,workers", [
    (1, "f32", 1, 0),      # the sequential pass: the caller's stream alone
    (1, "f32", 3, 3),      # single sample: a stream per worker
    (20, "f32", 4, 1),     # minibatches: the plan's one stream for all workers,
    (20, "bf16", 2, 1),
])
def test_handles_share_no_stream_and_a_repeated_pass_creates_nothing(program, B, dtype, k, workers):
    env = {n: v for n, v in os.environ.items() if not n.startswith("LF_")}
    out = subprocess.run([program, str(B), dtype, str(k), str(workers)], capture_output=True, text=True, env=env, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr


def test_wide_bf16_nets_share_no_worker_stream_either(program):
    """(the plan with two worker streams, which the widths of this test would not take by themselves)"""
    env = {n: v for n, v in os.environ.items() if not n.startswith("LF_")}
    out = subprocess.run([program, "20", "bf16", "4", "2"], capture_output=True, text=True, env={**env, "LF_GEMM_BIG": "1"},
                         timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
