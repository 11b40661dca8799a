"""Which streams a pass uses, from the HIP calls the library makes.  Two handles have no worker stream in common (one whose
caller's stream is held up cannot hold up the other), a pass that has run once with its k creates nothing when it runs
again (also where that second pass is being captured), and a handle destroys what it has created."""
import pytest

from tests import host_hip

MAIN = r"""
static std::set<stream_t> pass(lf_net* net, int k, void* stream) {
    used.clear();
    CHECK(lf_forward(net, some_input, stream) == LF_OK);
    CHECK(lf_backward_leapfrog(net, some_input, k, stream) == LF_OK);
    return used;
}
int main(int argc, char** argv) {
    const int B = std::atoi(argv[1]), k = std::atoi(argv[3]);
    const lf_dtype dt = argv[2][0] == 'b' ? LF_BF16 : LF_F32;
    const size_t workers = (size_t)std::atoi(argv[4]);
    lf_net* a = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
    lf_net* b = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
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
    return host_hip.build(tmp_path_factory.mktemp("streams"), MAIN)


@pytest.mark.parametrize("B,dtype,k,workers,env", [
    (1, "f32", 1, 0, {}),      # the sequential pass: the caller's stream alone
    (1, "f32", 3, 3, {}),      # single sample: a stream per worker
    (20, "f32", 4, 1, {}),     # minibatches: the plan's one stream for all workers,
    (20, "bf16", 2, 1, {}),
    (20, "bf16", 4, 2, {"LF_GEMM_BIG": "1"}),      # or the two of wide bf16 nets
])
def test_handles_share_no_stream_and_a_repeated_pass_creates_nothing(program, B, dtype, k, workers, env):
    host_hip.run(program, B, dtype, k, workers, **env)
