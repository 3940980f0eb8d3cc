// msao_wait.h -- the host's wait for a word that a kernel writes into pinned
// memory. Host code only, without HIP, so that it can be tested on the CPU.
#ifndef MSAO_WAIT_H
#define MSAO_WAIT_H

#include <chrono>
#include <thread>

namespace msao {

enum class StreamState { busy, drained, failed };

// Until ready() holds: a spin, then yields, and every kWaitQueryMs the state of
// the kernel's stream. False if that has failed, or has had nothing left to
// run for kWaitDrainedMs without the word (a stream that was destroyed counts
// as drained: its handle may since be another's, so one look at it is not
// enough). As long as the stream is busy there is no limit, as for an event.
constexpr double kWaitQueryMs = 10.0, kWaitDrainedMs = 5000.0;

template <typename Ready, typename State, typename NowMs>
bool wait_until(Ready&& ready, State&& state, NowMs&& now)
{
    for (int spin = 0; spin < 4096; ++spin)
        if (ready()) return true;
    double next = now() + kWaitQueryMs, drained_since = -1.0;
    for (;;) {
        if (ready()) return true;
        const double t = now();
        if (t < next) {
            std::this_thread::yield();
            continue;
        }
        next = t + kWaitQueryMs;
        switch (state()) {
        case StreamState::busy: drained_since = -1.0; break;
        case StreamState::failed: return ready();
        case StreamState::drained:
            if (drained_since < 0.0) drained_since = t;
            else if (t - drained_since >= kWaitDrainedMs) return ready();
            break;
        }
    }
}

inline double wait_now_ms()
{
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now().time_since_epoch()).count();
}

}  // namespace msao

#endif
