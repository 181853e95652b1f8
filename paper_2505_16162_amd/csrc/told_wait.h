// How the host waits for a pass's own word: plain code, no HIP.
#pragma once
#include <chrono>
#include <thread>

namespace ks {

// A look takes tens of nanoseconds. For TOLD_TIGHT_US the host does nothing else; a pass that lasts longer (a verification of a 40-block
// 13B-shaped model: 5.2 ms) is looked for as long as it lasts, but other threads may have the core between two looks.
constexpr long long TOLD_TIGHT_US = 2000;
// Every so often the stream is asked whether it has ended: one that has ended or failed without the word will never write it. A question
// costs about a microsecond and may put a marker on the stream.
constexpr long long TOLD_ASK_US = 5000;

// look(): is the word there? ended(): has the stream ended or failed? now_us(): a clock; rest(yield): between two looks. Returns whether the word came.
template <typename Look, typename Ended, typename Now, typename Rest>
inline bool told_wait(Look look, Ended ended, Now now_us, Rest rest) {
    const long long begin = now_us();
    long long ask = begin + TOLD_ASK_US;
    bool yield = false;
    for (int n = 1;; ++n) {
        if (look()) return true;
        if ((n & 63) == 0 || yield) {
            const long long now = now_us();
            yield = now - begin >= TOLD_TIGHT_US;
            if (now >= ask) {
                if (ended()) return look();        // what the stream wrote is there when it has ended
                ask = now + TOLD_ASK_US;
            }
        }
        rest(yield);
    }
}

template <typename Look, typename Ended> inline bool told_wait(Look look, Ended ended) {
    return told_wait(look, ended,
                     [] { return (long long)std::chrono::duration_cast<std::chrono::microseconds>(std::chrono::steady_clock::now().time_since_epoch()).count(); },
                     [](bool yield) {
                         if (yield) { std::this_thread::yield(); return; }
#if defined(__x86_64__)
                         __builtin_ia32_pause();
#endif
                     });
}

}  // namespace ks
