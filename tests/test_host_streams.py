"""Which streams a pass uses, from the HIP calls the library makes.  Handles on different streams of the caller's have no
worker stream in common (one whose stream is held up cannot hold up the other); handles on one stream share theirs; a
pass that has run once with its k creates nothing when it runs again, also on another stream or while that stream is being
captured; and the last of the handles that use a stream destroys it."""
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
    // on another stream, its own workers; and none of any other net's
    const std::set<stream_t> away = pass(a, k, &caller_3);
    CHECK(created == before && away.size() == 1 + workers);
    for (stream_t s : away) CHECK(!other.count(s) && !first.count(s));
    capturing = true;
    CHECK(pass(a, k, &caller_3) == away);
    capturing = false;
    CHECK(created == before);
    // a third net on the stream of the first: the same workers; it keeps them when the first goes
    lf_net* c = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
    CHECK(pass(c, k, &caller_1) == first);
    lf_destroy(a);
    for (stream_t s : away) CHECK(s == &caller_3 || !live.count(s));
    for (stream_t s : first) CHECK(s == &caller_1 || live.count(s));
    CHECK(pass(c, k, &caller_1) == first);
    lf_destroy(c);
    for (stream_t s : first) CHECK(!live.count(s));
    for (stream_t s : other) CHECK(s == &caller_2 || live.count(s));
    CHECK(pass(b, k, &caller_2) == other);
    lf_destroy(b);
    CHECK(live.empty());
    // nets with different numbers of workers on one stream: each uses as many as it wants, whoever comes first
    for (int i = 0; i < 2; ++i) {
        lf_net* many = make(std::vector<int>(6, 64), 1, LF_F32, LF_SCHED_STREAMS);
        lf_net* few = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
        std::set<stream_t> wide, narrow;
        if (i == 0) wide = pass(many, 5, &caller_1);
        narrow = pass(few, k, &caller_1);
        if (i == 1) wide = pass(many, 5, &caller_1);
        CHECK(wide.size() == 6 && narrow.size() == 1 + workers);
        for (stream_t s : narrow) CHECK(wide.count(s));
        CHECK(pass(few, k, &caller_1) == narrow);
        lf_destroy(many);
        lf_destroy(few);
        CHECK(live.empty());
    }
    // the per-thread stream is another stream in every thread, and a first pass may be a captured one: own workers
    for (int i = 0; i < 2; ++i) {
        void* const caller = i == 0 ? (void*)2 : (void*)&caller_1;
        capturing = i == 1;
        lf_net* d = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
        lf_net* e = make(std::vector<int>(6, 64), B, dt, LF_SCHED_STREAMS);
        const std::set<stream_t> one = pass(d, k, caller), two = pass(e, k, caller);
        capturing = false;
        for (stream_t s : one) CHECK(s == caller || !two.count(s));
        const int now = created;
        CHECK(pass(d, k, caller) == one);
        CHECK(created == now);
        lf_destroy(d);
        lf_destroy(e);
        CHECK(live.empty());
    }
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
def test_handles_on_different_streams_share_none_and_a_repeated_pass_creates_nothing(program, B, dtype, k, workers, env):
    host_hip.run(program, B, dtype, k, workers, **env)
