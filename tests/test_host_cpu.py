"""What the library's host side does around its launches - waits, bounds, copies -, on the CPU with a HIP runtime that only keeps a record."""
from tests.host_check import run_program

WAITS = r"""
// Draft blocks, scoring and prompts wait for the whole device and ask it for the lengths before their first launch: also when the
// object's earlier work went to the same stream (its inputs and outputs may be in use on others, and a handle does not name a
// stream for good: hipStreamPerThread is one handle for many, a destroyed stream's handle is given out again)
int main() {
    Small s;
    void* const streams[] = {nullptr, (void*)0x1000, (void*)2};
    for (void* st : streams)
        for (int what = 0; what < 3; ++what)
            for (int rep = 0; rep < 3; ++rep) {
                s.lengths(8);
                if (rep > 0) s.step(s.GAMMA, st);
                if (rep > 1) sj_kv_rewind(s.kv, std::vector<int32_t>(2, 8).data(), std::vector<int32_t>(2, 1).data(), st);
                calls.clear();
                const int rc = what == 0 ? s.draft(3, 1, st) : what == 1 ? s.score(3, st) : s.prefill(1, 9, st);
                const int wait = first("hipDeviceSynchronize"), ask = first("hipMemcpy", wait + 1), launch = first("launch");
                CHECK(!rc && wait >= 0 && wait < ask && ask < launch, "call %d, stream %p, rep %d: rc %d, wait %d, lengths %d, launch %d", what, st, rep, rc, wait, ask, launch);
            }
    std::printf("%d failures\n", failures);
}
"""


def test_calls_that_ask_for_lengths_wait_for_the_device(tmp_path):
    out = run_program(tmp_path, WAITS)
    assert out.splitlines()[-1] == "0 failures", out


FETCH = r"""
// Results are read behind the whole device, not behind the object's own calls: a graph that the caller captured runs them again on any
// stream, without the library knowing.  It may also write results without the mirror in host memory, so an object with captured calls is
// read by copies.
int main() {
    Small s;
    std::vector<float> p(s.BATCH * s.GAMMA), h(s.BATCH * (s.GAMMA + 1) * s.D);
    auto fetch = [&](bool small, bool copies, const char* what) {
        calls.clear();
        const int rc = small ? sj_debug_fetch(s.kv, SJ_DBG_P_AT_DRAFT, p.data(), p.size() * 4) : sj_debug_fetch(s.kv, SJ_DBG_HIDDEN, h.data(), h.size() * 4);
        const int wait = first("hipDeviceSynchronize"), copy = first("hipMemcpy");
        CHECK(!rc && wait >= 0 && (copies ? copy > wait : copy < 0), "%s: rc %d, wait %d, copy %d", what, rc, wait, copy);
    };
    s.score(3, nullptr);
    s.head(s.GAMMA, nullptr);
    fetch(false, true, "hidden states");
    fetch(true, true, "first fetch");
    s.head(s.GAMMA, nullptr);
    fetch(true, false, "mirrored");
    fetch(false, true, "hidden states of a mirrored call");
    s.head(s.GAMMA, CAPTURING);
    fetch(true, true, "a captured call");
    s.head(s.GAMMA, nullptr);
    fetch(true, true, "a later call of an object with captured calls");
    std::printf("%d failures\n", failures);
}
"""


def test_fetches_wait_for_the_device_and_see_captured_calls(tmp_path):
    out = run_program(tmp_path, FETCH)
    assert out.splitlines()[-1] == "0 failures", out


BOUND = r"""
// A call that fails after some of its launches has moved the lengths on the device.  Verification steps go by the host's upper bound: it
// counts what was queued, so the next step that the bound refuses asks the device instead of writing past the capacity.
int main() {
    struct { const char* call; int nth; const char* what; } fails[] = {
        {"hipGraphInstantiate", 2, "draft block, last token's layers"}, {"hipGraphLaunch", 3, "draft block, third step"},
        {"hipStreamSynchronize", 1, "prompt, after its first chunk"}, {"hipGraphLaunch", 1, "verification step"}};
    for (int i = 0; i < 4; ++i) {
        Small s;
        s.lengths(57);
        fail_next(fails[i].call, fails[i].nth);
        const int rc = i == 2 ? s.prefill(0, 7, nullptr) : i == 3 ? s.step(s.GAMMA, nullptr) : s.draft(4, 1, nullptr);
        CHECK(rc == SJ_EHIP, "%s: rc %d", fails[i].what, rc);
        calls.clear();
        s.step(s.GAMMA, nullptr);                     // 57 + 5 positions fit, 57 + what was queued + 5 do not
        CHECK(first("hipMemcpy") >= 0 && first("hipMemcpy") < first("launch"), "%s: the next step did not ask for the lengths", fails[i].what);
    }
    std::printf("%d failures\n", failures);
}
"""


def test_the_bound_counts_what_a_failed_call_queued(tmp_path):
    out = run_program(tmp_path, BOUND)
    assert out.splitlines()[-1] == "0 failures", out


FREE = r"""
// No call throws: giving an object's host memory back works where there is no memory left for the library's own lists.
#include <new>
static bool no_memory = false;
void* operator new(size_t n) {
    void* p = no_memory ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
int main() {
    Small s;
    std::vector<float> p(s.BATCH * s.GAMMA);
    std::vector<sj_kv*> objects;
    const int32_t cap[s.BATCH] = {64, 64};
    for (int i = 0; i < 12; ++i) {
        sj_kv* kv = nullptr;
        CHECK(!sj_kv_create(s.m, s.BATCH, cap, &kv), "create %d", i);
        std::swap(kv, s.kv);
        s.head(s.GAMMA, nullptr);
        CHECK(!sj_debug_fetch(s.kv, SJ_DBG_P_AT_DRAFT, p.data(), p.size() * 4), "fetch %d", i);
        std::swap(kv, s.kv);
        objects.push_back(kv);
    }
    calls.clear();
    calls.reserve(4096);
    for (sj_kv* kv : objects) {
        bool threw = false;
        quiet = no_memory = true;
        try { sj_kv_free(kv); } catch (...) { threw = true; }
        quiet = no_memory = false;
        CHECK(!threw, "sj_kv_free threw");
    }
    calls.clear();
    for (int i = 0; i < 9; ++i) {                            // eight blocks wait for the next objects, the others went back
        sj_kv* kv = nullptr;
        CHECK(!sj_kv_create(s.m, s.BATCH, cap, &kv), "create again %d", i);
        std::swap(kv, s.kv);
        s.head(s.GAMMA, nullptr);
        calls.clear();
        sj_debug_fetch(s.kv, SJ_DBG_P_AT_DRAFT, p.data(), p.size() * 4);
        CHECK((first("hipHostMalloc") >= 0) == (i == 8), "block %d", i);
        std::swap(kv, s.kv);
    }
    std::printf("%d failures\n", failures);
}
"""


def test_host_memory_goes_back_without_throwing(tmp_path):
    out = run_program(tmp_path, FREE)
    assert out.splitlines()[-1] == "0 failures", out
