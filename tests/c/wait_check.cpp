// wait_until (csrc/msao_wait.h) with a clock, a word and a stream that this
// program plays: used by tests/test_wait_cpu.py.
#include <cstdio>

#include "msao_wait.h"

using msao::StreamState;

static int bad = 0;

// The word is set at set_ms (never if negative); the stream is busy until
// drain_ms (never drained if negative) and fails at fail_ms (never if negative).
static void check(const char* what, double set_ms, double drain_ms, double fail_ms, bool want, double from_ms, double to_ms)
{
    double t = 0.0;
    int queries = 0;
    const bool got = msao::wait_until([&] { return set_ms >= 0.0 && t >= set_ms; },
                                      [&] {
                                          ++queries;
                                          if (fail_ms >= 0.0 && t >= fail_ms) return StreamState::failed;
                                          return drain_ms >= 0.0 && t >= drain_ms ? StreamState::drained : StreamState::busy;
                                      },
                                      [&] { return t += 0.25; });
    const bool ok = got == want && t >= from_ms && t <= to_ms && queries <= 1 + (int)(t / msao::kWaitQueryMs);
    printf("%s %s: returned %d at %.1f ms after %d queries\n", ok ? "ok" : "FAIL", what, (int)got, t, queries);
    if (!ok) bad = 1;
}

int main()
{
    check("word already set", 0.0, -1, -1, true, 0, 0);
    check("word before the first query", 5.0, -1, -1, true, 5, 6);
    check("word after an hour of a busy stream", 3.6e6, -1, -1, true, 3.6e6, 3.6e6 + 1);
    check("device fails", -1, -1, 500.0, false, 500, 520);
    check("device fails from the start", -1, -1, 0.0, false, 0, 20);
    check("stream drained without the word", -1, 100.0, -1, false, 100 + msao::kWaitDrainedMs, 130 + msao::kWaitDrainedMs);
    check("another stream under the handle, word later", 2000.0, 100.0, -1, true, 2000, 2001);
    check("word set as the device fails", 500.0, -1, 500.0, true, 500, 520);
    return bad;
}
