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
